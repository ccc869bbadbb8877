// Mapping of the workgroups of a launch over (point, slot) items to the XCDs, and the points that one launch
// holds.  Plain C++ (no HIP) so that a host test can check it; constexpr functions are usable in device code.
//
// Workgroups are dispatched round-robin over the XCDs, so blockIdx % 8 names the XCD and its L2.  Where the
// points fill the XCDs evenly, all slots of a point run on one XCD (point = 8 (block / 8 / slots) + block % 8).
// Where the last group of 8 points would leave more XCDs idle than an eighth of the batch, every XCD takes a
// contiguous eighth of the item list instead: one point of 103 slots by point ran on one XCD only (windows and
// projection 24.8 us, spread 9.6 us).
#pragma once

#include <stddef.h>

constexpr int XCD_COUNT = 8;

constexpr bool xcd_by_point(int points) {
  const int pad = (XCD_COUNT - points % XCD_COUNT) % XCD_COUNT;
  return XCD_COUNT * pad <= points;
}
constexpr unsigned xcd_blocks(int points, int slots) {
  if (xcd_by_point(points)) return (unsigned)((size_t)(points + XCD_COUNT - 1) / XCD_COUNT * XCD_COUNT * slots);
  return (unsigned)(((size_t)points * slots + XCD_COUNT - 1) / XCD_COUNT * XCD_COUNT);
}
// the item of block blk; point >= points: none.  (One division for both orders: two of them cost 1% of the
// windows kernel, a workgroup of which lives for one item.)
constexpr void xcd_item(int blk, int points, int slots, int* point, int* slot) {
  const int xcd = blk % XCD_COUNT, rest = blk / XCD_COUNT;
  const bool by_point = xcd_by_point(points);
  const int per = (points * slots + XCD_COUNT - 1) / XCD_COUNT;  // items of an XCD, not by point
  const int item = by_point ? rest : xcd * per + rest;
  const int p = item / slots;
  *slot = item - p * slots;
  *point = by_point ? p * XCD_COUNT + xcd : p;
}

// The most points whose launch of `slots` workgroups of `threads` threads each stays below the 2^32 threads
// that a grid dimension holds: larger batches run as several launches.  (A multiple of 8 where there are that
// many, so that xcd_blocks does not round up past the limit.)
constexpr int points_per_launch(int slots, int threads) {
  const size_t blocks = (((size_t)1 << 32) - 1) / threads / XCD_COUNT * XCD_COUNT;
  size_t n = blocks / slots;
  if (n >= (size_t)XCD_COUNT) n = n / XCD_COUNT * XCD_COUNT;
  if (n < 1) n = 1;
  return n > 0x7ffffff8 ? 0x7ffffff8 : (int)n;
}
