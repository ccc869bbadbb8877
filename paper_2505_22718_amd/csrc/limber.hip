// The Limber limit (paper Sec. 2.6, eq. Limber): j_l(k chi) acts as a delta function at
// k = (l + 1/2) / chi, so for every multipole
//   C_l^{ij} = int dchi / chi^2 g_i(chi) g_j(chi) P((l + 1/2) / chi),   g = c(l, k) f,
// with c = 1 for clustering, F(l) / k^2 = F(l) chi^2 / (l + 1/2)^2 for lensing and l(l+1) chi^2 /
// (l + 1/2)^2 for CMB lensing (Sec. 2.4).  The integral
// runs on the log-chi nodes of the FFTLog path (dchi = chi dln chi), with the same edge weights:
//   C_l^{ij} = Delta sum_m w_m g_i(chi_m) g_j(chi_m) P((l + 1/2) / chi_m) / chi_m,
// P by the natural cubic spline of ln P in ln k (zero outside the k nodes).  The kernels come from
// the assembly (band 0 samples, untilted), so this is a cheap branch for high multipoles and a
// check of the FFTLog windows where the Limber error O(1/l) is small.
#include "common.h"
#include "geometry.h"
#include "internal.h"

namespace {

__device__ __forceinline__ int clamp_l(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// ln P and its natural-spline moments in ln k: one block per point.
__global__ __launch_bounds__(512) void k_limber_pk(plan_dev P, swiftcl_inputs in) {
  extern __shared__ double sh[];
  const int b = blockIdx.x, nk = P.n_k;
  double* y = sh;
  double* Mo = sh + nk;
  bool bad = false;
  for (int j = threadIdx.x; j < nk; j += blockDim.x) {
    const double v = in.pk[(size_t)b * nk + j];
    bad |= !(v > 0.0) || !isfinite(v);
    y[j] = log(fmax(v, 1e-300));
  }
  if (bad) atomicOr(P.flags, FLAG_NONFINITE);
  __syncthreads();
  __shared__ double scan[block_scan_doubles(1, 512)];
  const double* const ys[1] = {y};
  double* const ms[1] = {Mo};
  block_spline<1>(ys, P.lu_k, nk, ms, scan);
  for (int j = threadIdx.x; j < nk; j += blockDim.x) {
    P.lnp[((size_t)b * 2) * nk + j] = y[j];
    P.lnp[((size_t)b * 2 + 1) * nk + j] = Mo[j];
  }
}

// One block of LB_LG wavefronts per (point, group of LB_LG multipole slots), wavefront w = slot w of
// the group.  Per chunk of chi nodes the block stages H_t(m) = w_m f_t(chi_m) [chi_m^2 for the
// lensing kinds] in LDS once for the whole group (it does not depend on the multipole; w_m f_t is the
// band-0 kernel sample without its tilt; the CMB-lensing sample of the last node, which carries the
// linear-end weight, is brought to w_m; the node factors of each kind are formed once per node, the
// FP64 divisions once per kind instead of once per tracer), and every wavefront its weights
// s_l(m) = Delta P(nu_l / chi_m) / (chi_m w_m).  The pair sums are then the Gram matrix
// sum_m H_i(m) [s_l(m) H_j(m)] on the 16x16x4 MFMA, four nodes per lane and load (both operands take
// the nodes in the same order).  The factor c(l) / nu^2 (F(l) or l(l+1)) per lensing-kind tracer of
// the pair is applied at the end.  Bound by the FP64 exp and spline of the weights and the MFMA
// issue (vector issue 44% of the cycles, matrix cores 22%): 177 us for 256 points x 15 tracers x 103
// multipoles (445 nodes); with one thread per tracer pair on VALU (120 of 256 threads at work) the
// kernel took 290 us.
constexpr int LB_LG = 8;     // multipole slots per block
constexpr int LB_CH = 256;   // chi nodes per LDS chunk
constexpr int LB_HS = LB_CH + 4;  // row stride of H: the 16 rows x 4 node groups of a load on distinct banks

template <typename R> struct lmfma;
template <> struct lmfma<float> {
  typedef float type __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane / 16) + r; }
  static __device__ __forceinline__ type step(float a, float b, type c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <> struct lmfma<double> {
  typedef double type __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int row(int lane, int r) { return lane / 16 + 4 * r; }
  static __device__ __forceinline__ type step(double a, double b, type c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// TWO: a second 16-row tracer tile (more than 16 tracers)
template <typename R, bool TWO>
__global__ __launch_bounds__(LB_LG * SWIFTCL_WAVE) void k_limber(plan_dev P, swiftcl_inputs in, R* __restrict__ Cout, int b0,
                                                                   int nbp) {
  extern __shared__ __align__(16) unsigned char smem[];
  using acc_t = typename lmfma<R>::type;
  constexpr int ROWS = TWO ? 32 : 16;
  const int T = P.max_tracers, Lm = P.max_ell, N = P.N, nb = P.n_bands, nk = P.n_k;
  double* sc = (double*)smem;                   // [kind][LB_CH] H / g of every node
  R* H = (R*)(sc + SWIFTCL_NKINDS * LB_CH);     // [ROWS][LB_HS]
  R* s = H + (size_t)ROWS * LB_HS;              // [LB_LG][LB_CH]
  __shared__ int kinds[ROWS];
  const int ngrp = (Lm + LB_LG - 1) / LB_LG;
  const int bl = blockIdx.x / ngrp, l0 = (blockIdx.x % ngrp) * LB_LG;
  if (bl >= nbp) return;
  const int b = b0 + bl;
  const int tid = threadIdx.x, nth = LB_LG * SWIFTCL_WAVE;
  const int wave = __builtin_amdgcn_readfirstlane(tid / SWIFTCL_WAVE), lane = tid % SWIFTCL_WAVE;
  const int npair = T * (T + 1) / 2;
  const int Tb = clamp_l(in.n_tracers[b], 0, T);
  const int Lb = clamp_l(in.n_ell[b], 0, Lm);
  // slots of the group past the point's multipoles: zeros
  for (int e = tid; e < LB_LG * npair; e += nth) {
    const int l = l0 + e / npair;
    if (l < Lm && l >= Lb) Cout[((size_t)b * Lm + l) * npair + e % npair] = (R)0;
  }
  if (l0 >= Lb) return;
  const int li = l0 + wave;
  const bool active = li < Lb;
  int ei = 0;
  if (active) {
    ei = in.ell_idx[(size_t)b * Lm + li];
    if (ei < 0 || ei >= P.n_ell) {
      if (lane == 0) atomicOr(P.flags, FLAG_BAD_INDEX);
      ei = 0;
    }
  }
  const double nu = P.ell_v[ei] + 0.5, lnu = log(nu);
  if (tid < ROWS) kinds[tid] = tid < Tb ? tracer_kind(in, T, b, tid) : 0;
  const double* pt = P.pt + (size_t)b * PT_STRIDE;
  const double lchi0 = log(pt[PT_CHI0]), theta = pt[PT_THETA];
  const int m0 = P.m0, m1 = (int)pt[PT_M1];
  const double* lnp = P.lnp + (size_t)b * 2 * nk;
  const double* lnk = P.lnk;
  const double* lkih = P.lu_k + 3 * (size_t)nk;
  R* sw = s + wave * LB_CH;
  const int r = lane & 15, q = lane >> 4;
  acc_t a00 = {0, 0, 0, 0}, a01 = {0, 0, 0, 0}, a11 = {0, 0, 0, 0};
  for (int mc = m0; mc <= m1; mc += LB_CH) {
    const int cnt = m1 - mc + 1 < LB_CH ? m1 - mc + 1 : LB_CH;
    const int cntp = (cnt + 15) & ~15;
    __syncthreads();  // the previous chunk's readers are done (and kinds is written)
    for (int e = tid; e < SWIFTCL_NKINDS * LB_CH; e += nth) {
      const int kind = e / LB_CH, idx = e % LB_CH, m = mc + idx;
      double f = 0.0;
      if (idx < cnt) {
        f = 1.0 / P.ebm[((size_t)kind * nb) * N + m];
        if (kind != SWIFTCL_CLUSTERING) {
          const double chi = exp(lchi0 + (double)m * P.delta);
          f *= chi * chi;
        }
        if (kind == SWIFTCL_CMB_LENSING && m == m1 && m1 > m0) f *= (0.5 + theta) / (0.5 + 0.5 * theta);
      }
      sc[e] = f;
    }
    if (active)
      for (int idx = lane; idx < cntp; idx += SWIFTCL_WAVE) {
        const int m = mc + idx;
        double sv = 0.0;
        if (m <= m1) {
          const double lchi = lchi0 + (double)m * P.delta;
          const double w = m == m0 ? 0.5 : (m == m1 ? 0.5 + theta : 1.0);
          const double x = lnu - lchi;  // ln k of the Limber node
          if (x >= lnk[0] && x <= lnk[nk - 1]) {
            const int iv = clamp_l((int)floor((x - lnk[0]) / P.delta), 0, nk - 2);
            const double lv = spline_at(lnk, lkih, lnp, lnp + nk, iv, x, nullptr);
            sv = P.delta * exp(lv - lchi) / w;
          }
        }
        sw[idx] = (R)sv;
      }
    __syncthreads();
    for (int t = wave; t < ROWS; t += LB_LG) {
      const R* g = (const R*)P.g + (((size_t)b * T + t) * nb) * N + mc;
      const double* f = sc + kinds[t] * LB_CH;
      for (int idx = lane; idx < cntp; idx += SWIFTCL_WAVE)
        H[(size_t)t * LB_HS + idx] = (t < Tb && idx < cnt) ? (R)((double)g[idx] * f[idx]) : (R)0;
    }
    __syncthreads();
    if (!active) continue;
    for (int k0 = 0; k0 < cntp; k0 += 16) {
      const R* sp = sw + k0 + 4 * q;
      const R* hp = H + (size_t)r * LB_HS + k0 + 4 * q;
      R h0[4], h1[4], sv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sv[j] = sp[j];
        h0[j] = hp[j];
        if constexpr (TWO) h1[j] = hp[16 * LB_HS + j];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a00 = lmfma<R>::step(h0[j], h0[j] * sv[j], a00);
        if constexpr (TWO) {
          const R hs = h1[j] * sv[j];
          a01 = lmfma<R>::step(h0[j], hs, a01);
          a11 = lmfma<R>::step(h1[j], hs, a11);
        }
      }
    }
  }
  __syncthreads();
  if (!active) return;
  const double inu2 = 1.0 / (nu * nu);
  R* c = Cout + ((size_t)b * Lm + li) * npair;
  // entry (i, j) of the Gram matrix, i <= j < T
  auto store = [&](int i, int j, R v) {
    if (i > j || j >= T) return;
    R out = (R)0;
    if (j < Tb) {
      double f = (double)v;
      if (kinds[i]) f *= P.fell[(size_t)kinds[i] * P.n_ell + ei] * inu2;
      if (kinds[j]) f *= P.fell[(size_t)kinds[j] * P.n_ell + ei] * inu2;
      out = (R)f;
    }
    c[i * T - i * (i - 1) / 2 + (j - i)] = out;
  };
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = lmfma<R>::row(lane, e);
    store(i, r, a00[e]);
    if constexpr (TWO) {
      store(i, 16 + r, a01[e]);
      store(16 + i, 16 + r, a11[e]);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Adjoint of the Limber rule.  With H_t(m) and s_l(m) as above and a_t = c_t(l) / nu^2 (1 for
// clustering), C_l^{ij} = a_i a_j sum_m H_i H_j s_l, so for L = sum_l sum_{ij} G_ij C_l^{ij} (G the
// symmetrised cotangent) and Q_t = sum_j G_tj a_j H_j:
//   dL/dH_t(m)      = sum_l 2 a_t s_l(m) Q_t(m)
//   dL/dln P(k_lm)  = s_l(m) sum_t a_t H_t(m) Q_t(m)        (s is P at the node's Limber k)
// The second goes through the spline of ln P (value weights of each node, then the moments'
// adjoint), the first through H = g / e^{-b m Delta} [chi^2] back to the kernel-sample cotangents
// dg, from which the FFTLog adjoint's chain rule (k_bwd_tracer, k_bwd_point) gives db, dn(z), dD.
// ---------------------------------------------------------------------------------------------

__global__ void k_limber_zero(plan_dev P, swiftcl_inputs in) {
  const size_t n = (size_t)in.batch * 2 * P.n_k;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    P.lim_acc[i] = 0.0;
}

// One block of 8 wavefronts per (point, 64 chi nodes of the support), FP64: wavefront (tile w % 4,
// half w / 4) takes 16 nodes and every other group of four multipoles, so no barrier stands inside
// the multipole loop.  Q = G (a H) is one 16x16 MFMA product per multipole and 16-row tracer tile:
// lane (c, q) feeds the rows of G from dC itself (A) and a_j H_j of node c, j = 4 s + q (B, H in
// registers); the accumulator holds Q_t of the same tracers t = q + 4 s, so dH and the ln P
// cotangent are formed in place.  The FP64 exp, log and spline of the weights s_l run on 64 lanes at
// once, lane (c, q) for the group's multipole q and node c.  The ln P cotangents go to LDS (FP64
// atomics; the nodes of one multipole fall on distinct intervals) and once per block to the point's
// global rows.  The two halves' dH meet in LDS; the block writes the dg rows of its nodes (band 0; the
// other bands 0; nodes outside the support are never read).  567 us for 256 points x 15
// tracers x 103 multipoles (445 nodes), bound by latency at four wavefronts per SIMD (vector issue 33% of the
// cycles, matrix cores 14%, LDS 5% without bank conflicts, 0.3 TB/s; 12 B of scratch per lane); with Q formed
// by two threads per node from LDS and two barriers per multipole it took 3530 us.
constexpr int LB_BN = 64;  // chi nodes per block of the adjoint

template <typename R, int NT>  // NT: 16-row tracer tiles
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 4 : 2))) void k_limber_bwd(plan_dev P, swiftcl_inputs in, const R* __restrict__ dC, int b0, int nbp) {
  extern __shared__ __align__(16) unsigned char smem[];
  typedef double v4 __attribute__((ext_vector_type(4)));
  const int T = P.max_tracers, Lm = P.max_ell, N = P.N, nb = P.n_bands, nk = P.n_k;
  double* comb = (double*)smem;                // [4 tiles][NT][4][64]
  double* dy = comb + 4 * NT * 4 * SWIFTCL_WAVE;  // [nk]
  double* dM = dy + nk;                        // [nk]
  const int nch = (N - P.m0 + LB_BN - 1) / LB_BN;
  const int bl = blockIdx.x / nch, mc = P.m0 + (blockIdx.x % nch) * LB_BN;
  if (bl >= nbp) return;
  const int b = b0 + bl;
  const double* pt = P.pt + (size_t)b * PT_STRIDE;
  const double lchi0 = log(pt[PT_CHI0]), theta = pt[PT_THETA];
  const int m0 = P.m0, m1 = (int)pt[PT_M1];
  if (mc > m1) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / SWIFTCL_WAVE), lane = tid % SWIFTCL_WAVE;
  const int tile = wave & 3, half = wave >> 2;
  const int c = lane & 15, q = lane >> 4;
  const int Tb = clamp_l(in.n_tracers[b], 0, T);
  const int Lb = clamp_l(in.n_ell[b], 0, Lm);
  const int npair = T * (T + 1) / 2;
  for (int j = tid; j < nk; j += blockDim.x) dy[j] = dM[j] = 0.0;
  const int m = mc + 16 * tile + c;  // this lane's node
  const bool mok = m <= m1;
  const double lchi = lchi0 + (double)m * P.delta;
  const double w = m == m0 ? 0.5 : (m == m1 ? 0.5 + theta : 1.0);
  // H / g and dg / dH of node m for tracer kind `kind`
  auto node_factor = [&](int kind) {
    double f = 1.0 / P.ebm[((size_t)kind * nb) * N + m];
    if (kind != SWIFTCL_CLUSTERING) {
      const double chi = exp(lchi);
      f *= chi * chi;
    }
    if (kind == SWIFTCL_CMB_LENSING && m == m1 && m1 > m0) f *= (0.5 + theta) / (0.5 + 0.5 * theta);
    return f;
  };
  double H[4 * NT];  // H_t(m), t = q + 4 s
  int kd[4 * NT];    // kind of tracer t (clustering past the point's tracers)
#pragma unroll
  for (int s = 0; s < 4 * NT; ++s) {
    const int t = q + 4 * s;
    kd[s] = t < Tb ? tracer_kind(in, T, b, t) : 0;
    H[s] = (t < Tb && mok) ? (double)((const R*)P.g)[(((size_t)b * T + t) * nb) * N + m] * node_factor(kd[s]) : 0.0;
  }
  // packed index of G[row][4 s + q], row = 16 i + c: -1 outside the point's tracers
  int gp[NT][4 * NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int s = 0; s < 4 * NT; ++s) {
      const int row = 16 * i + c, j = q + 4 * s;
      const int lo = row < j ? row : j, hi = row < j ? j : row;
      gp[i][s] = hi < Tb ? lo * T - lo * (lo - 1) / 2 + (hi - lo) : -1;
    }
  const double* lnp = P.lnp + (size_t)b * 2 * nk;
  const double* lnk = P.lnk;
  const double* lkih = P.lu_k + 3 * (size_t)nk;
  double dH[4 * NT];
#pragma unroll
  for (int s = 0; s < 4 * NT; ++s) dH[s] = 0.0;
  __syncthreads();
  for (int lg = 4 * half; lg < Lb; lg += 8) {
    // lane (c, q): multipole lg + q
    const int lq = lg + q;
    int ei = 0;
    if (lq < Lb) {
      ei = in.ell_idx[(size_t)b * Lm + lq];
      if (ei < 0 || ei >= P.n_ell) {
        if (c == 0) atomicOr(P.flags, FLAG_BAD_INDEX);
        ei = 0;
      }
    }
    const double nu = P.ell_v[ei] + 0.5, inu2 = 1.0 / (nu * nu);
    const double al = P.fell[(size_t)SWIFTCL_LENSING * P.n_ell + ei] * inu2;
    const double ac = P.fell[(size_t)SWIFTCL_CMB_LENSING * P.n_ell + ei] * inu2;
    double sv = 0.0, wa = 0.0, wb = 0.0, wc = 0.0, wd = 0.0;
    int iv = 0;
    if (lq < Lb && mok) {
      const double x = log(nu) - lchi;
      if (x >= lnk[0] && x <= lnk[nk - 1]) {
        iv = clamp_l((int)floor((x - lnk[0]) / P.delta), 0, nk - 2);
        const spline_w wt(lnk, lkih, iv, x);
        const double lv = wt.wa * lnp[iv] + wt.wb * lnp[iv + 1] + wt.wc * lnp[nk + iv] + wt.wd * lnp[nk + iv + 1];
        sv = P.delta * exp(lv - lchi) / w;
        wa = wt.wa;
        wb = wt.wb;
        wc = wt.wc;
        wd = wt.wd;
      }
    }
    double apq = 0.0;
#pragma unroll(NT == 1 ? 4 : 1)
    for (int i4 = 0; i4 < 4; ++i4) {
      const int li = lg + i4;
      if (li >= Lb) break;
      const double sl = __shfl(sv, 16 * i4 + c), all = __shfl(al, 16 * i4), acl = __shfl(ac, 16 * i4);
      const R* g = dC + ((size_t)b * Lm + li) * npair;
      double a[4 * NT];
#pragma unroll
      for (int s = 0; s < 4 * NT; ++s)
        a[s] = kd[s] == SWIFTCL_CLUSTERING ? 1.0 : (kd[s] == SWIFTCL_LENSING ? all : acl);
      double ap = 0.0;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        v4 Q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4 * NT; ++s) {
          double gv = gp[i][s] >= 0 ? (double)g[gp[i][s]] : 0.0;
          if (16 * i + c != q + 4 * s) gv *= 0.5;
          Q = __builtin_amdgcn_mfma_f64_16x16x4f64(gv, a[s] * H[s], Q, 0, 0, 0);
        }
        // Q[e] = Q_t of tracer t = 16 i + q + 4 e at node c
        if (sl != 0.0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const double v = a[4 * i + e] * Q[e];
            dH[4 * i + e] += 2.0 * sl * v;
            ap += H[4 * i + e] * v;
          }
        }
      }
      ap += __shfl_xor(ap, 16);
      ap += __shfl_xor(ap, 32);
      if (q == i4) apq = ap;
    }
    if (sv != 0.0) {
      const double d = apq * sv;
      unsafeAtomicAdd(&dy[iv], wa * d);
      unsafeAtomicAdd(&dy[iv + 1], wb * d);
      unsafeAtomicAdd(&dM[iv], wc * d);
      unsafeAtomicAdd(&dM[iv + 1], wd * d);
    }
  }
  double* cb = comb + (size_t)tile * NT * 4 * SWIFTCL_WAVE;
  if (half == 1)
#pragma unroll
    for (int s = 0; s < 4 * NT; ++s) cb[s * SWIFTCL_WAVE + lane] = dH[s];
  __syncthreads();
  if (half == 0 && mok) {
    R* dg = (R*)P.dg;
#pragma unroll
    for (int s = 0; s < 4 * NT; ++s) {
      const int t = q + 4 * s;
      if (t >= T) continue;
      const double v = t < Tb ? (dH[s] + cb[s * SWIFTCL_WAVE + lane]) * node_factor(kd[s]) : 0.0;
      for (int bi = 0; bi < nb; ++bi) dg[(((size_t)b * T + t) * nb + bi) * N + m] = (R)(bi == 0 ? v : 0.0);
    }
  }
  for (int j = tid; j < nk; j += blockDim.x) {
    if (dy[j] != 0.0) atomicAdd(&P.lim_acc[((size_t)b * 2) * nk + j], dy[j]);
    if (dM[j] != 0.0) atomicAdd(&P.lim_acc[((size_t)b * 2 + 1) * nk + j], dM[j]);
  }
}

// dL/dP per point: the moments' cotangents through the spline solve, then ln P -> P.
__global__ __launch_bounds__(512) void k_limber_bwd_pk(plan_dev P, swiftcl_inputs in, double* dpk) {
  extern __shared__ double sh[];
  __shared__ double scan[block_scan_doubles(1, 512)];
  const int b = blockIdx.x, nk = P.n_k;
  double* dy = sh;
  double* dM = sh + nk;
  for (int j = threadIdx.x; j < nk; j += blockDim.x) {
    dy[j] = P.lim_acc[((size_t)b * 2) * nk + j];
    dM[j] = P.lim_acc[((size_t)b * 2 + 1) * nk + j];
  }
  block_spline_adjoint(dy, dM, P.lu_k, nk, scan);
  for (int j = threadIdx.x; j < nk; j += blockDim.x) {
    const double v = in.pk[(size_t)b * nk + j];
    // ln P is taken of max(P, 1e-300): no gradient below that floor
    dpk[(size_t)b * nk + j] = v > 1e-300 ? dy[j] / v : 0.0;
  }
}

}  // namespace

size_t limber_bwd_lds_bytes(const plan_dev& p) {
  return sizeof(double) * ((size_t)4 * (p.max_tracers > 16 ? 2 : 1) * 4 * SWIFTCL_WAVE + 2 * (size_t)p.n_k);
}

size_t limber_lds_bytes(const plan_dev& p) {
  const size_t rs = p.precision == SWIFTCL_FP64 ? 8 : 4;
  return sizeof(double) * SWIFTCL_NKINDS * LB_CH +
         rs * ((size_t)(p.max_tracers > 16 ? 32 : 16) * LB_HS + (size_t)LB_LG * LB_CH);
}

static hipError_t launch_limber_pk(const plan_dev& p, const swiftcl_inputs* in, hipStream_t s) {
  hipLaunchKernelGGL(k_limber_pk, dim3(in->batch), dim3(512), sizeof(double) * 2 * (size_t)p.n_k, s, p, *in);
  return hipGetLastError();
}

hipError_t launch_limber(const plan_dev& p, const swiftcl_inputs* in, void* C, hipStream_t s) {
  hipError_t e = launch_limber_pk(p, in, s);
  if (e != hipSuccess) return e;
  const int ngrp = (p.max_ell + LB_LG - 1) / LB_LG, most = points_per_launch(ngrp, LB_LG * SWIFTCL_WAVE);
  const size_t lds = limber_lds_bytes(p);
  if (p.precision == SWIFTCL_FP64 && p.max_tracers > 16) return hipErrorNotSupported;  // (no such plan is built)
  for (int b0 = 0; b0 < in->batch; b0 += most) {
    const int nbp = in->batch - b0 < most ? in->batch - b0 : most;
    const dim3 grid((unsigned)((size_t)nbp * ngrp)), blk(LB_LG * SWIFTCL_WAVE);
    if (p.precision == SWIFTCL_FP64)
      hipLaunchKernelGGL((k_limber<double, false>), grid, blk, lds, s, p, *in, (double*)C, b0, nbp);
    else if (p.max_tracers > 16)
      hipLaunchKernelGGL((k_limber<float, true>), grid, blk, lds, s, p, *in, (float*)C, b0, nbp);
    else
      hipLaunchKernelGGL((k_limber<float, false>), grid, blk, lds, s, p, *in, (float*)C, b0, nbp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_limber_backward(const plan_dev& p, const swiftcl_inputs* in, const void* dC, double* dpk,
                                  double* dbias, double* dnz, double* dD, hipStream_t s) {
  hipError_t e = launch_limber_pk(p, in, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_limber_zero, dim3(256), dim3(256), 0, s, p, *in);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int nch = (p.N - p.m0 + LB_BN - 1) / LB_BN, most = points_per_launch(nch, 512);
  const size_t lds = limber_bwd_lds_bytes(p);
  if (p.precision == SWIFTCL_FP64 && p.max_tracers > 16) return hipErrorNotSupported;
  for (int b0 = 0; b0 < in->batch; b0 += most) {
    const int nbp = in->batch - b0 < most ? in->batch - b0 : most;
    const dim3 grid((unsigned)((size_t)nbp * nch));
    if (p.precision == SWIFTCL_FP64)
      hipLaunchKernelGGL((k_limber_bwd<double, 1>), grid, dim3(512), lds, s, p, *in, (const double*)dC, b0, nbp);
    else if (p.max_tracers > 16)
      hipLaunchKernelGGL((k_limber_bwd<float, 2>), grid, dim3(512), lds, s, p, *in, (const float*)dC, b0, nbp);
    else
      hipLaunchKernelGGL((k_limber_bwd<float, 1>), grid, dim3(512), lds, s, p, *in, (const float*)dC, b0, nbp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (dpk) {
    hipLaunchKernelGGL(k_limber_bwd_pk, dim3(in->batch), dim3(512), sizeof(double) * 2 * (size_t)p.n_k, s, p, *in,
                       dpk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return launch_bwd_chain(p, in, dbias, dnz, dD, s);
}
