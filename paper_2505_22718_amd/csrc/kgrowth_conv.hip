// Scale-dependent growth D(k, z) (paper Sec. 3.2).  The power spectrum factorises as
// P(k, z_fid) D(k, z(chi)) D(k, z(chi')), so the FFTLog coefficients of f(chi) D(k, chi) depend on k.
// The growth is given at N_interp nodes kappa_a, uniform in ln k from k_min to k_max, and continued
// to every k node by the natural cubic spline in ln k.  The coefficients are linear in the growth, so
// the spline may act on the growth itself instead of on every tracer's coefficients, and the n-sum of
// the window collapses into a sum over the chi nodes of the support (m0 <= m <= m1, about 0.43 N):
//   W_l(k_j) = c(l) k_j^{-1-b} [k_j^-2 for lensing] sum_m K_l(j + m) g_m D_j(m),
//   K_l(s)   = chi_0^{-b} / N Re sum_{n<N/2} h_n U_l(n) phase_n e^{-2 pi i n s / N}   (h_0 = 1, else 2).
// K_l is periodic in s with period N and shared by the point's tracers of one kind: one FP64 inverse
// real transform per (point, kind, multipole).  The tilt of band beta relative to band 0,
// (k_0 e^{s Delta})^{-(b_beta - b_0)}, is a function of s = j + m alone, so it is folded into K_l and
// the multipoles of all bands share the rows of one product: per (point, kind)
//   [multipoles x s] . [s x (tracer, k node)],  right operand g_t(s - j) D_j(s - j),
// as three bf16 parts per operand on the 16x16x32 bf16 MFMA, writing sqrt(s) W to the workspace for the
// projection kernel.
//
// (kgrowth.hip has the same windows through the node coefficients, which the gradients use.)
//
// Stages per chunk of points:
//   k_kc_dz       per (point, node): D(kappa_a, z) splined in z and sampled on the chi nodes (FP64)
//   k_kc_dk       per (point, chi node): the moments of the natural spline along ln k (FP64)
//   k_kc_dj       D_j(m) of every k node, and the kernel samples, in the operand layout of the product
//   k_kc_bessel   the rows K_l of every (point, kind, multipole) (FP64 transforms)
//   k_kc_windows  the product, one workgroup per (point, 4 NC (tracer, 16 k nodes) tiles, 112 multipoles)
//   k_contract    C = V V^T per (point, multipole) from the workspace (forward.hip)
#include <type_traits>

#include "common.h"
#include "geometry.h"
#include "internal.h"

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any 4-byte address

namespace {

__device__ __forceinline__ int clamp_i(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Growth at the nodes: one workgroup per (point, node); its spline moments in LDS [n_zg].
__global__ __launch_bounds__(256) void k_kc_dz(plan_dev P, swiftcl_inputs in, const double* __restrict__ Dkz, int b0,
                                               int nbp) {
  extern __shared__ double Mo[];
  __shared__ double scan[block_scan_doubles(1, 256)];
  const int nzg = P.n_zg, A = P.n_interp, N = P.N, NS = P.kc_ns;
  const int bl = blockIdx.x / A, a = blockIdx.x % A;
  if (bl >= nbp) return;
  const int b = b0 + bl;
  const double* y = Dkz + ((size_t)b * A + a) * nzg;
  bool bad = false;
  for (int i = threadIdx.x; i < nzg; i += blockDim.x) bad |= !isfinite(y[i]);
  if (bad) atomicOr(P.flags, FLAG_NONFINITE);
  const double* const ys[1] = {y};
  double* const ms[1] = {Mo};
  block_spline<1>(ys, P.lu_geom, nzg, ms, scan);
  const int m0 = P.m0, m1 = (int)P.pt[(size_t)b * PT_STRIDE + PT_M1];
  const double* zgih = P.lu_geom + 3 * (size_t)nzg;
  double* out = P.kc_dn + ((size_t)bl * A + a) * NS;
  for (int m = m0 + threadIdx.x; m <= m1; m += blockDim.x) {
    const int ig = P.node_i[(size_t)b * 3 * N + m];
    out[m - m0] = spline_w(P.z_geom, zgih, ig, P.node_f[(size_t)b * 4 * N + m]).at(y, Mo, ig);
  }
}

// Moments along ln k: one thread per (point, chi node), the system
//   M_{a-1} + 4 M_a + M_{a+1} = 6/h^2 (D_{a+1} - 2 D_a + D_{a-1}),  M_0 = M_{A-1} = 0,
// by the two Thomas sweeps (1/pivots in kc_ip).  A serial chain over the nodes, bound by load latency:
// KC_SEG nodes are loaded together, one segment ahead of the chain.
constexpr int KC_SEG = 16;

__global__ __launch_bounds__(64) void k_kc_dk(plan_dev P, int b0, int nbp, double s6) {
  const int A = P.n_interp, NS = P.kc_ns;
  const int bl = blockIdx.y, x = blockIdx.x * blockDim.x + threadIdx.x;
  if (bl >= nbp) return;
  const int ns = (int)P.pt[(size_t)(b0 + bl) * PT_STRIDE + PT_M1] - P.m0 + 1;
  if (x >= ns) return;
  const double* c = P.kc_dn + (size_t)bl * A * NS + x;
  double* mo = P.kc_dm + (size_t)bl * A * NS + x;
  const double* ip = P.kc_ip;
  mo[0] = 0.0;
  mo[(size_t)(A - 1) * NS] = 0.0;
  double cur[KC_SEG], nxt[KC_SEG];
  // the values after nodes a0 .. a0 + KC_SEG - 1
  auto load = [&](int a0) {
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) nxt[i] = c[(size_t)min(a0 + i + 1, A - 1) * NS];
  };
  double cm = c[0], c0 = c[NS], d = 0.0;
  load(1);
  for (int a0 = 1; a0 + 1 < A; a0 += KC_SEG) {
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) cur[i] = nxt[i];
    load(a0 + KC_SEG);
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) {
      const int a = a0 + i;
      if (a + 1 < A) {
        d = (s6 * (cur[i] - 2.0 * c0 + cm) - d) * ip[a];
        cm = c0;
        c0 = cur[i];
        mo[(size_t)a * NS] = d;
      }
    }
  }
  auto loadm = [&](int a1) {
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) nxt[i] = mo[(size_t)max(a1 - i, 0) * NS];
  };
  double mn = 0.0;
  loadm(A - 2);
  for (int a1 = A - 2; a1 >= 1; a1 -= KC_SEG) {
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) cur[i] = nxt[i];
    loadm(a1 - KC_SEG);  // (nodes below this segment: not written by it)
#pragma unroll
    for (int i = 0; i < KC_SEG; ++i) {
      const int a = a1 - i;
      if (a >= 1) {
        mn = cur[i] - ip[a] * mn;
        mo[(size_t)a * NS] = mn;
      }
    }
  }
}

// The right operand's factors, zero outside the support.  Blocks x < NJ: the growth rows
// kc_dt[j][x] = D_j(m0 + x - j % 16) of the 16 k nodes of group x (shifted, so that a lane of the
// product reads the same column for every k node of the group); blocks x >= NJ: the band-0 kernel
// samples of tracer x - NJ, kc_f[t][y] = g_t(m0 + y - 16).
constexpr int KC_J = 16;   // k nodes per column tile
constexpr int KC_PAD = 16; // zeros before the kernel samples

__global__ __launch_bounds__(256) void k_kc_dj(plan_dev P, swiftcl_inputs in, int b0, int nbp) {
  const int A = P.n_interp, NS = P.kc_ns, SP = P.kc_sp, nk = P.n_k, T = P.max_tracers, nb = P.n_bands, N = P.N;
  const int NJ = (nk + KC_J - 1) / KC_J;
  const int bl = blockIdx.y, jg = blockIdx.x;
  if (bl >= nbp) return;
  const int b = b0 + bl, m0 = P.m0;
  const int ns = (int)P.pt[(size_t)b * PT_STRIDE + PT_M1] - m0 + 1;
  if (jg >= NJ) {
    const int t = jg - NJ;
    const float* g = (const float*)P.g + ((size_t)b * T + t) * nb * N;
    float* f = P.kc_f + ((size_t)bl * T + t) * (SP + KC_PAD);
    for (int y = threadIdx.x; y < SP + KC_PAD; y += blockDim.x)
      f[y] = (y >= KC_PAD && y - KC_PAD < ns) ? g[m0 + y - KC_PAD] : 0.f;
    return;
  }
  float* out = P.kc_dt + ((size_t)bl * NJ + jg) * KC_J * SP;
  // (thread i: chi node i of every k node of the group, the node values kept while the interval stays)
  for (int i = threadIdx.x; i < ns; i += blockDim.x) {
    const double* dn = P.kc_dn + (size_t)bl * A * NS + i;
    const double* dm = P.kc_dm + (size_t)bl * A * NS + i;
    double da = 0.0, db = 0.0, ma = 0.0, mb = 0.0;
    int at = -1;
    for (int r = 0; r < KC_J; ++r) {
      const int jc = min(jg * KC_J + r, nk - 1), a = P.kg_ia[jc];
      const double* w = P.kc_w + 4 * (size_t)jc;
      if (a != at) {
        at = a;
        da = dn[(size_t)a * NS];
        db = dn[(size_t)(a + 1) * NS];
        ma = dm[(size_t)a * NS];
        mb = dm[(size_t)(a + 1) * NS];
      }
      out[(size_t)r * SP + r + i] = (float)(w[0] * da + w[1] * db + w[2] * ma + w[3] * mb);
    }
  }
  // zeros before node m0 and after m1, up to the last group of 16 offsets that the product reads
  const int end = (ns + KC_J - 1 + 15) / 16 * 16;
  for (int e = threadIdx.x; e < KC_J * 32; e += blockDim.x) {  // (end - ns < 32)
    const int r = e / 32, x = e % 32;
    if (x < r) out[(size_t)r * SP + x] = 0.f;
    else if (x + ns < end) out[(size_t)r * SP + x + ns] = 0.f;
  }
}

// x as the sum of three bf16, each the nearest to what is left: all 24 bits of x.  (Cutting instead of
// rounding gives every part the sign of x, so that the part products left out have a bias: with both operands
// cut the error of C grew from 2.1e-7 to 3.0e-7, with one of them to 2.4e-7.)
__device__ __forceinline__ void split3(float x, unsigned short (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const __bf16 h = (__bf16)x;
    p[i] = __builtin_bit_cast(unsigned short, h);
    x -= (float)h;
  }
}
// of two values at a time, packed (x0 in the low half)
__device__ __forceinline__ void split3_pair(float x0, float x1, unsigned int (&p)[3]) {
  typedef float v2f __attribute__((ext_vector_type(2)));
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const v2f x = {x0, x1};
    p[i] = __builtin_bit_cast(unsigned int, __builtin_convertvector(x, v2bf));
    if (i < 2) {
      x0 -= __uint_as_float(p[i] << 16);
      x1 -= __uint_as_float(p[i] & 0xffff0000u);
    }
  }
}

// K_l rows: one wavefront per (point, multipole slot, kind), idle for kinds the point has no tracer
// of.  FP64 from the FP64 U table to the row, which holds K_l rounded to FP32 as the sum of three bf16.
// kc_k[point][kind][slot][part][s - m0], s = m0 .. m1 + n_k - 1, zeros after.
template <int M>
__global__ __launch_bounds__(256) void k_kc_bessel(plan_dev P, swiftcl_inputs in, int b0, int nbp) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int N = 2 * M, RL = M / SWIFTCL_WAVE;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / SWIFTCL_WAVE), lane = threadIdx.x % SWIFTCL_WAVE;
  const int T = P.max_tracers, Lm = P.max_ell;
  const int item = blockIdx.x * 4 + wave;
  const int kind = item % SWIFTCL_NKINDS, li = (item / SWIFTCL_NKINDS) % Lm, bl = item / (SWIFTCL_NKINDS * Lm);
  if (bl >= nbp) return;  // whole wavefronts leave; no block barrier below
  const int b = b0 + bl;
  const int Tb = clamp_i(in.n_tracers[b], 0, T);
  if (li >= clamp_i(in.n_ell[b], 0, Lm)) return;
  const int mine = lane < Tb ? tracer_kind(in, T, b, lane) : -1;  // (T <= 32)
  if (!__any(mine == kind)) return;
  int ei = in.ell_idx[(size_t)b * Lm + li];
  if (ei < 0 || ei >= P.n_ell) {
    if (lane == 0) atomicOr(P.flags, FLAG_BAD_INDEX);
    ei = 0;
  }
  const int band = P.ell_band[ei];
  const double* pt = P.pt + (size_t)b * PT_STRIDE;
  const double scale = pt[PT_CHI0B + kind * SWIFTCL_MAX_BANDS + band] / (double)N;
  const double2* U = P.kc_u + ((size_t)kind * P.n_ell + ei) * M;
  const double2* ph = (const double2*)P.phase + (size_t)b * M;
  double2 v[RL];
#pragma unroll
  for (int e = 0; e < RL; ++e) {
    const int n = lane + SWIFTCL_WAVE * e;
    v[e] = cscale(cconj(cmul(U[n], ph[n])), scale);
  }
  wave_c2r<double, M>(v, (double2*)smem + (size_t)wave * fft_lds_size(M, 8), P.kc_tw, lane);
  // v[e] = K(s), K(s + 1) at s = 2 (lane + 64 e): through the scratch, so that every lane then holds eight
  // consecutive entries of the row and stores 16 bytes of each part.  The band tilt advances by e^{-db Delta}.
  double* Kr = (double*)((double2*)smem + (size_t)wave * fft_lds_size(M, 8));
  const int m0 = P.m0, SK = P.kc_sk, last = (int)pt[PT_M1] + P.n_k - 1;
  const double db = P.fftlog_b[kind][band] - P.fftlog_b[kind][0];
  wave_sync();
#pragma unroll
  for (int e = 0; e < RL; ++e) *(double2*)(Kr + 2 * (lane + SWIFTCL_WAVE * e)) = v[e];
  wave_sync();
  const double q1 = exp(-db * P.delta);
  unsigned short* out = P.kc_k + (((size_t)bl * SWIFTCL_NKINDS + kind) * Lm + li) * 3 * SK;
  for (int y = 8 * lane; y < SK; y += 8 * SWIFTCL_WAVE) {
    const int s = m0 + y;
    double f = exp(-db * (log(P.k0) + P.delta * (double)s));
    typedef unsigned short v8us __attribute__((ext_vector_type(8)));
    v8us p0, p1, p2;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      unsigned short part[3];
      split3(s + i <= last ? (float)(Kr[(s + i) & (N - 1)] * f) : 0.f, part);
      p0[i] = part[0];
      p1[i] = part[1];
      p2[i] = part[2];
      f *= q1;
    }
    *(v8us*)(out + y) = p0;
    *(v8us*)(out + SK + y) = p1;
    *(v8us*)(out + 2 * SK + y) = p2;
  }
}

__device__ __forceinline__ unsigned short bf16_rne_kc(float x) {
  const unsigned int u = __float_as_uint(x);
  return (unsigned short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// The product by 4 wavefronts.  A column tile is one tracer and 16 consecutive k nodes; the tiles of
// a (point, kind) are numbered k-group major, so that the 4 NC tiles of a workgroup read nearly the
// same s.  Wave w owns tiles NC w .. NC w + NC - 1 and all of the workgroup's multipoles (<= 7 tiles of
// 16 rows).  The rows K_l go through LDS, 32 offsets s per step, double-buffered (one block barrier per
// step, the next step's rows in flight during this one's MFMAs).  The right operand is formed in
// registers, one product g_t(s - j) D_j(s - j) per value, from eight consecutive entries of the padded
// kernel samples and of the shifted growth row, and split like the rows.
// Both operands are FP32 values as three bf16 each, and six of the nine part products are summed in FP32
// on the 16x16x32 bf16 MFMA, small ones first (the three left out are below 2^-26 of the product): 2.7 times the rate of the f32
// MFMA.  64 points of 15 tracers, 103 multipoles, 1024 k nodes and 442 chi nodes: 0.66 ms (1.01 ms on the f32
// MFMA), the matrix cores busy in 39% of the cycles, the vector unit in 34% (splits, loads), 1.2 TB/s of HBM
// and no bank conflicts: the two units take turns, three wavefronts per SIMD.  The same windows from the node
// coefficients (an n-sum of 1024 terms, its 200-node FFTs and splines) take 5.7 ms.
constexpr int KC_RT = 7;            // 16-row multipole tiles per workgroup
constexpr int KC_SC = 32;           // offsets s per step
typedef unsigned short v8us __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// nrg: row groups of the launch; per point they share its multipole tiles evenly.
template <bool SPLIT, int NC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_kc_windows(plan_dev P, swiftcl_inputs in, int b0, int nbp, int nrg) {
  // [buffer][part][row][32]; the four 16-byte groups of a row are swizzled by the row (bits 1 and 2), so
  // that eight rows' reads of one group fall on distinct banks
  __shared__ __align__(16) unsigned short Ks[2][3][KC_RT * 16][KC_SC];
  constexpr int NT = 4 * NC;  // column tiles per workgroup
  const int T = P.max_tracers, Lm = P.max_ell, nk = P.n_k, nb = P.n_bands;
  const int NJ = (nk + KC_J - 1) / KC_J, SP = P.kc_sp, SK = P.kc_sk;
  // every XCD takes a contiguous eighth of the (point, tile group, row group) list, so that the rows
  // and the growth of the few points it works on stay in its L2 whatever the number of points
  const int per8 = gridDim.x / SWIFTCL_NXCD;
  const int item = (int)(blockIdx.x % SWIFTCL_NXCD) * per8 + (int)(blockIdx.x / SWIFTCL_NXCD);
  const int npt = ((T * NJ + NT - 1) / NT + SWIFTCL_NKINDS - 1) * nrg;  // items per point
  const int bl = item / npt;
  if (bl >= nbp) return;
  const int rg = (item % npt) % nrg;
  int tb = (item % npt) / nrg;  // tile group among all kinds
  const int b = b0 + bl;
  const int Tb = clamp_i(in.n_tracers[b], 0, T);
  const int Lb = clamp_i(in.n_ell[b], 0, Lm);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / SWIFTCL_WAVE), lane = tid % SWIFTCL_WAVE;
  // the kind of this tile group: the kinds' groups follow one another
  const int mine = lane < Tb ? tracer_kind(in, T, b, lane) : -1;
  unsigned int mask = 0;
  int kind = -1;
  for (int kd = 0; kd < SWIFTCL_NKINDS && kind < 0; ++kd) {
    const unsigned int mk = (unsigned int)__ballot(mine == kd);
    const int ng = (__popc(mk) * NJ + NT - 1) / NT;
    if (tb < ng) {
      kind = kd;
      mask = mk;
    } else {
      tb -= ng;
    }
  }
  if (kind < 0) return;
  const int Tk = __popc(mask);
  const int ntile = Tk * NJ, t0 = tb * NT;
  // multipole rows of this row group
  const int tl = (Lb + 15) / 16, per = (tl + nrg - 1) / nrg;
  const int r0 = 16 * per * rg, cnt = min(Lb - r0, 16 * per);
  if (cnt <= 0) return;
  const int nrt = (cnt + 15) / 16;
  const int ns = (int)P.pt[(size_t)b * PT_STRIDE + PT_M1] - P.m0 + 1;
  const int nh = (ns + KC_J - 1 + 15) / 16;  // groups of 16 offsets that reach a tile's support
  const int jg0 = t0 / Tk, jg1 = min(t0 + NT, ntile) - 1;  // (last tile)
  const int nst = (nh + jg1 / Tk - jg0 + 1) / 2;           // steps of 32 offsets
  const int r = lane & 15, q = lane >> 4;
  int jg[NC], tt[NC], hoff[NC];
  // byte offsets of this lane's operands from the point's arrays
  const char* fb = (const char*)(P.kc_f + (size_t)bl * T * (SP + KC_PAD));
  const char* db = (const char*)(P.kc_dt + (size_t)bl * NJ * KC_J * SP);
  unsigned int fo[NC], dof[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int tile = min(t0 + wave * NC + c, ntile - 1);  // (tiles past the end repeat the last one)
    jg[c] = tile / Tk;
    unsigned int mk = mask;
    for (int i = tile % Tk; i > 0; --i) mk &= mk - 1;
    tt[c] = __ffs(mk) - 1;
    hoff[c] = jg[c] - jg0;
    fo[c] = 4u * (unsigned int)(tt[c] * (SP + KC_PAD) + KC_PAD + 8 * (q & 1) - r);
    dof[c] = 4u * (unsigned int)((jg[c] * KC_J + r) * SP + 8 * (q & 1));
  }
  // K rows: 16-byte pieces (part, row, group); a thread takes group tid % 4 of rows tid / 4 and tid / 4 + 64
  // (rows past cnt repeat the last one), every part
  const char* kr = (const char*)(P.kc_k + (((size_t)bl * SWIFTCL_NKINDS + kind) * Lm + r0) * 3 * SK + jg0 * KC_J);
  const int krow = tid >> 2, kgrp = tid & 3;
  v4f acc[KC_RT][NC];
#pragma unroll
  for (int i = 0; i < KC_RT; ++i)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[i][c] = (v4f){0.f, 0.f, 0.f, 0.f};
  // the loop, instantiated for the number of row tiles so that no MFMA sits behind a branch
  auto loop = [&](auto nrt_c) {
    constexpr int NRT = decltype(nrt_c)::value;
    constexpr int NB = (NRT * 16 + 63) / 64;  // blocks of 64 rows
    unsigned int ko[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) ko[i] = 2u * (unsigned int)(min(krow + 64 * i, cnt - 1) * 3 * SK + 8 * kgrp);
    v8us kn[NB][3];
    unsigned short* kl = &Ks[0][0][krow][8 * (kgrp ^ ((krow >> 1) & 3))];
    auto kget = [&](int st) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int part = 0; part < 3; ++part)
          kn[i][part] = *(const v8us*)(kr + (ko[i] + 2u * (unsigned int)(part * SK + KC_SC * st)));
    };
    auto kput = [&](int buf) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int part = 0; part < 3; ++part)
          if (NRT % 4 == 0 || i + 1 < NB || krow + 64 * i < NRT * 16)
            *(v8us*)(kl + ((buf * 3 + part) * KC_RT * 16 + 64 * i) * KC_SC) = kn[i][part];
    };
    kget(0);
    kput(0);
    v4f fn[NC][2], dn[NC][2];
    auto fetch = [&](int st) {  // this lane's eight offsets of step st
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        // (outside the tile's groups: a group inside them, taken times zero)
        const int hh = 2 * st + (q >> 1) - hoff[c], hc = min(max(hh, 0), nh - 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const v4f d = *(const v4f*)(db + (dof[c] + 64u * (unsigned int)hc + 16u * i));
          fn[c][i] = *(const v4fu*)(fb + (fo[c] + 64u * (unsigned int)hc + 16u * i));
          dn[c][i] = hh == hc ? d : (v4f){0.f, 0.f, 0.f, 0.f};
        }
      }
    };
    fetch(0);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
      const int buf = st & 1;
      const bool more = st + 1 < nst;
      if (more) kget(st + 1);
      v8bf bp[3][NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        typedef unsigned int v4ui __attribute__((ext_vector_type(4)));
        v4ui w[3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          unsigned int part[3];
          const int g = e >> 1, o = 2 * (e & 1);
          split3_pair(fn[c][g][o] * dn[c][g][o], fn[c][g][o + 1] * dn[c][g][o + 1], part);
#pragma unroll
          for (int i = 0; i < 3; ++i) w[i][e] = part[i];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) bp[i][c] = __builtin_bit_cast(v8bf, w[i]);
      }
      fetch(st + 1);
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const int at = 8 * (q ^ ((r >> 1) & 3));
        const v8bf ah = *(const v8bf*)&Ks[buf][0][16 * rt + r][at];
        const v8bf am = *(const v8bf*)&Ks[buf][1][16 * rt + r][at];
        const v8bf al = *(const v8bf*)&Ks[buf][2][16 * rt + r][at];
#define SWIFTCL_KC_STEP(A, B)                                                                         \
  for (int c = 0; c < NC; ++c) acc[rt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[c], acc[rt][c], 0, 0, 0)
#pragma unroll
        SWIFTCL_KC_STEP(al, bp[0]);
#pragma unroll
        SWIFTCL_KC_STEP(ah, bp[2]);
#pragma unroll
        SWIFTCL_KC_STEP(am, bp[1]);
#pragma unroll
        SWIFTCL_KC_STEP(am, bp[0]);
#pragma unroll
        SWIFTCL_KC_STEP(ah, bp[1]);
#pragma unroll
        SWIFTCL_KC_STEP(ah, bp[0]);
#undef SWIFTCL_KC_STEP
      }
      if (more) kput(buf ^ 1);
      __syncthreads();
    }
  };
  switch (nrt) {
    case 1: loop(std::integral_constant<int, 1>{}); break;
    case 2: loop(std::integral_constant<int, 2>{}); break;
    case 3: loop(std::integral_constant<int, 3>{}); break;
    case 4: loop(std::integral_constant<int, 4>{}); break;
    case 5: loop(std::integral_constant<int, 5>{}); break;
    case 6: loop(std::integral_constant<int, 6>{}); break;
    default: loop(std::integral_constant<int, 7>{}); break;
  }
  // V = F(l) kscale sqrt(s) W into the workspace rows (point, slot, tracer); F(l) is folded into U and
  // the tilts of the higher bands into K, so the scale is band 0's
  const size_t lo_off = (size_t)P.vchunk * Lm * 32 * nk;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = jg[c] * KC_J + r;
    if (j >= nk || t0 + wave * NC + c >= ntile) continue;
    const float sc = ((const float*)P.kss)[((size_t)b * SWIFTCL_NKINDS + kind) * nb * nk + j];
#pragma unroll
    for (int rt = 0; rt < KC_RT; ++rt) {
      if (rt >= nrt) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * rt + 4 * q + i;
        if (row >= cnt) continue;
        const float x = sc * acc[rt][c][i];
        const size_t o = (((size_t)bl * Lm + r0 + row) * 32 + tt[c]) * nk + j;
        if (SPLIT) {
          const unsigned short hi = bf16_rne_kc(x);
          const unsigned short lo = bf16_rne_kc(x - __uint_as_float((unsigned int)hi << 16));
          ((unsigned short*)P.vbuf)[o] = hi;
          ((unsigned short*)P.vbuf)[lo_off + o] = lo;
        } else {
          ((float*)P.vbuf)[o] = x;
        }
      }
    }
  }
}

// The windows of points [b0, b0 + nbp) into the workspace (see the stages above)
template <int M>
hipError_t launch_kc_rows(const plan_dev& p, const swiftcl_inputs* in, const double* D_kz, int b0, int nbp,
                          hipStream_t s) {
  const int T = p.max_tracers, A = p.n_interp;
  const double h = (double)(p.n_k - 1) * p.delta / (double)(A - 1);
  const int NJ = (p.n_k + KC_J - 1) / KC_J;
  hipLaunchKernelGGL(k_kc_dz, dim3((unsigned)((size_t)nbp * A)), dim3(256), (size_t)p.n_zg * sizeof(double), s, p,
                     *in, D_kz, b0, nbp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_kc_dk, dim3((p.kc_ns + 63) / 64, nbp), dim3(64), 0, s, p, b0, nbp, 6.0 / (h * h));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_kc_dj, dim3(NJ + T, nbp), dim3(256), 0, s, p, *in, b0, nbp);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t rows = (size_t)nbp * p.max_ell * SWIFTCL_NKINDS;
  hipLaunchKernelGGL(k_kc_bessel<M>, dim3((unsigned)((rows + 3) / 4)), dim3(256),
                     4 * (size_t)fft_lds_size(M, 8) * sizeof(double2), s, p, *in, b0, nbp);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // two column tiles per wavefront halve the LDS reads per MFMA; one where the launch would otherwise
  // leave compute units without a workgroup
  const int nrg = ((p.max_ell + 15) / 16 + KC_RT - 1) / KC_RT;
  const bool one = (long)nbp * (T * NJ / 8) * nrg < 2 * p.persist_blocks;
  const int nt = one ? 4 : 8;
  const size_t items = (size_t)nbp * ((T * NJ + nt - 1) / nt + SWIFTCL_NKINDS - 1) * nrg;
  const dim3 gw((unsigned)((items + SWIFTCL_NXCD - 1) / SWIFTCL_NXCD * SWIFTCL_NXCD));
  const bool split = p.precision == SWIFTCL_SPLIT_BF16;
  if (one && split) hipLaunchKernelGGL((k_kc_windows<true, 1>), gw, dim3(256), 0, s, p, *in, b0, nbp, nrg);
  else if (one) hipLaunchKernelGGL((k_kc_windows<false, 1>), gw, dim3(256), 0, s, p, *in, b0, nbp, nrg);
  else if (split) hipLaunchKernelGGL((k_kc_windows<true, 2>), gw, dim3(256), 0, s, p, *in, b0, nbp, nrg);
  else hipLaunchKernelGGL((k_kc_windows<false, 2>), gw, dim3(256), 0, s, p, *in, b0, nbp, nrg);
  return hipGetLastError();
}

// kc_chunk points at a time, in chunks of equal size (no short last one)
template <int M>
hipError_t launch_kc_t(const plan_dev& pd, const swiftcl_inputs* in, const double* D_kz, void* C, hipStream_t s) {
  plan_dev p = pd;
  p.vchunk = p.kc_chunk;
  const int nch = (in->batch + p.vchunk - 1) / p.vchunk, size = (in->batch + nch - 1) / nch;
  for (int b0 = 0; b0 < in->batch; b0 += size) {
    const int nbp = in->batch - b0 < size ? in->batch - b0 : size;
    hipError_t e = launch_kc_rows<M>(p, in, D_kz, b0, nbp, s);
    if (e == hipSuccess) e = launch_contract(p, in, C, b0, nbp, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// the widths of the operand rows for supports up to the whole chi box (a plan's rows are sized once;
// the support of a point is known on the device only)
void kgrowth_conv_sizes(plan_dev& p) {
  p.kc_ns = p.N - p.m0;
  p.kc_sp = (p.kc_ns + KC_J - 1 + KC_SC - 1) / KC_SC * KC_SC + KC_SC;
  p.kc_sk = (p.n_k + KC_J - 1) / KC_J * KC_J + p.kc_sp + KC_SC;
}

size_t kgrowth_conv_bytes(const plan_dev& p) {
  const size_t NJ = (size_t)(p.n_k + KC_J - 1) / KC_J;
  return (size_t)2 * p.n_interp * p.kc_ns * sizeof(double) + NJ * KC_J * p.kc_sp * sizeof(float) +
         (size_t)p.max_tracers * (p.kc_sp + KC_PAD) * sizeof(float) +
         (size_t)SWIFTCL_NKINDS * p.max_ell * 3 * p.kc_sk * sizeof(unsigned short);
}

hipError_t launch_kgrowth_conv(const plan_dev& p, const swiftcl_inputs* in, const double* D_kz, void* C, hipStream_t s) {
  switch (p.M) {
    case 128: return launch_kc_t<128>(p, in, D_kz, C, s);
    case 256: return launch_kc_t<256>(p, in, D_kz, C, s);
    case 512: return launch_kc_t<512>(p, in, D_kz, C, s);
    case 1024: return launch_kc_t<1024>(p, in, D_kz, C, s);
  }
  return hipErrorInvalidValue;
}
