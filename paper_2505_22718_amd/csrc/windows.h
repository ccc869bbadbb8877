// The coefficients of one FP32 window, shared by the projection and the adjoints.
#pragma once

#include "common.h"
#include "internal.h"

// Shape of a kernel of 16 wavefronts that keeps the rows of NT tracers per wavefront in registers and passes
// them through LDS in slabs of k, double-buffered in the space of the transforms' scratch.  PAD: floats after a
// slab row; TILES: 16 x 16 result tiles summed over the wavefronts at the end (0: none).  bytes: with the
// twiddles before it.
template <int M, int NT, int PAD, int TILES> struct slab_shape {
  static constexpr int RL = M / SWIFTCL_WAVE;
  static constexpr int SE = NT == 2 ? (RL >= 4 ? RL / 4 : 1) : RL / 2;  // register pairs per slab
  static constexpr int NS = RL / SE;                                    // slabs
  static constexpr int SW = 2 * SWIFTCL_WAVE * SE;                      // k nodes per slab
  static constexpr int SP = SW + PAD;                                   // row stride
  static constexpr size_t bytes() {
    size_t n = (size_t)16 * fft_lds_size(M, 4) * 8;
    if ((size_t)2 * 16 * NT * SP * 4 > n) n = (size_t)2 * 16 * NT * SP * 4;
    if ((size_t)16 * TILES * 1024 > n) n = (size_t)16 * TILES * 1024;
    return n + (size_t)2 * M * 8;
  }
};

// d_n conjugated of one window: c_n U_l(n) and the RSD and magnification terms of a clustering tracer,
// which share its prefactor and k scale
template <int M, int EXTRA>
__device__ __forceinline__ void window_coeffs(const plan_dev& P, const swiftcl_inputs& in, int b, int t, int kind,
                                              int ei, int band, int lane, float2 (&v)[M / SWIFTCL_WAVE]) {
  typedef float R;
  constexpr int RL = M / SWIFTCL_WAVE;
  const size_t row = (((size_t)b * P.max_tracers + t) * P.n_bands + band) * M;
  const C2<R>* ch = (const C2<R>*)P.chat + row;
  const C2<R>* Ur = (const C2<R>*)P.U + ((size_t)kind * P.n_ell + ei) * M;
#pragma unroll
  for (int e = 0; e < RL; ++e) {
    const int n = lane + SWIFTCL_WAVE * e;
    v[e] = cconj(cmul(ch[n], Ur[n]));
  }
  if ((EXTRA & 1) && kind == SWIFTCL_CLUSTERING) {
    const C2<R>* chr = (const C2<R>*)P.chat_r + row;
    const C2<R>* URr = (const C2<R>*)P.UR + (size_t)ei * M;
#pragma unroll
    for (int e = 0; e < RL; ++e) {
      const int n = lane + SWIFTCL_WAVE * e;
      v[e] = cadd(v[e], cconj(cmul(chr[n], URr[n])));
    }
  }
  if ((EXTRA & 2) && in.mag && kind == SWIFTCL_CLUSTERING) {
    // l(l+1) U at the bias b - 2
    const C2<R>* chm = (const C2<R>*)P.chat_mu + row;
    const C2<R>* Umr = (const C2<R>*)P.Umu + (size_t)ei * M;
#pragma unroll
    for (int e = 0; e < RL; ++e) {
      const int n = lane + SWIFTCL_WAVE * e;
      v[e] = cadd(v[e], cconj(cmul(chm[n], Umr[n])));
    }
  }
}
