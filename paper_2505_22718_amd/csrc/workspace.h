// Points that the chunked workspace of a plan holds.  Plain C++ (no HIP) so that a host test can check it.
//
// The paths that run through the workspace take the points in chunks, and a point's results do not depend on
// its chunk (the gradients not by a bit, C of growth not beyond rounding): larger chunks only fill the chip
// better.  So a plan needs `base` points of V rows (what its multipole chunks are sized for) and takes more as
// long as half of the device's free memory is left to others.
#pragma once

#include <stddef.h>

struct workspace_request {
  size_t vbuf_point;    // bytes of V rows per point, shared by the paths
  size_t growth_point;  // bytes of the growth product's own operands per point
  int base;             // points of V rows that the plan needs
  int adjoint;          // points that the adjoint would like to run at once
  int growth;           // points that the growth product would like to run at once (0: none)
};
struct workspace_points {
  int vbuf, adjoint, growth;
};

// The points to ask for with free_bytes free: never below base (and one point of growth, if it is wanted).
constexpr workspace_points workspace_fit(const workspace_request& r, size_t free_bytes) {
  const size_t budget = free_bytes / 2;
  const size_t need = (size_t)r.base * r.vbuf_point;
  size_t g = 0;
  if (r.growth > 0) {
    g = budget / (r.vbuf_point + r.growth_point);  // more points than base: rows and operands
    if (g < (size_t)r.base) g = budget > need ? (budget - need) / r.growth_point : 0;
    if (g > (size_t)r.base && g * (r.vbuf_point + r.growth_point) > budget) g = r.base;
    if (g > (size_t)r.growth) g = r.growth;
    if (g < 1) g = 1;
  }
  const size_t rows = g > (size_t)r.base ? g : (size_t)r.base;
  const size_t left = budget > g * r.growth_point ? budget - g * r.growth_point : 0;
  size_t a = left / r.vbuf_point;
  if (a > (size_t)r.adjoint) a = r.adjoint;
  if (a < (size_t)r.base) a = r.base;
  return {(int)(a > rows ? a : rows), (int)a, (int)g};
}
