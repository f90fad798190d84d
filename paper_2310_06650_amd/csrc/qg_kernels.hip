// HIP kernels of one solver step for gfx950 (MI355X).
//
// Stage map (one launch each, in stream order):
//   k_forward       per-(t, branch) AC flows and penalties          (Section II-B Ex. 1, 4; II-G)
//                   + base-case DC flows on FP64 MFMA:                 (eqs. (Yb_solve)-(p_flow))
//                     F_t = ISF[:, gen] p_t - ISF load_t - mean_t ISF 1 (uniform slack)
//   k_ctg_rows      per-(t, l, k) outage flows F_l + LODF_lk F_k, their (eqs. (rank_correct),
//                     penalties and reductions, per-(t, k) penalties z_tk, (sfr_pen)-(zctg), (2nd_lin_sys))
//                     per-chunk worst and sum (branch-stacked tile: k_ctg_main
//                     and k_ctg_zred instead; QG_FLAG_CTG_NO_SKIP: k_ctg_test
//                     before it)
//   k_ctg_asm       per-(t, l) dL/dF and dL/dqmax2 (mean + worst-contingency weights)
//                   + per-(t, bus) power balance from bus-sorted endpoint flows
//                     (LDS-staged segmented sums)                      (Ex. 4)
//                   + one block per period: device terms, reserve     (Ex. 2, 3; eq. (nlp_updated))
//                     shortfall
//   k_adjoint       dL/dp_tj (DC part) = sum_l dL/dF_tl (ISF[l][bus(j)] - rowsum_l/N)
//                     on FP64 MFMA, split over the branch dimension      (eqs. (2nd_lin_sys), (correction))
//                   + per-(t, branch) reverse of the AC flows into bus-sorted endpoint slots
//   k_final         per-(t, bus) segmented sums of endpoint adjoints and per-(t, generator)
//                     gradient assembly, then either the gradient or the fused Adam
//                     update with clip (Alg. 3), and the deterministic sum of the terms.
//   k_update        k_adjoint and k_final in one launch, in a small grid's own step
//
// Every reduction has a fixed order (no floating-point atomics), so a step is
// bitwise reproducible run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cfloat>
#include <climits>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "qg_internal.h"

namespace qg {

typedef double v4d __attribute__((ext_vector_type(4)));

struct StepParams {
  double eps, beta, rho_s;
};

struct EvalArgs {
  DevProblem p;
  DevWork w;
  DevPtr<const double> x;
  DevPtr<double> grad, terms_out, m, v;
  EvalMode mode;
  int fuse_adam;
  int nb_br, nb_bus, bus_chunks, nb_gen, nsplit;
  int nLb, nKb, nKc, nLc, tc, lt;
  // period-split tile: branch slices of a map-reduce block (0: branch-stacked
  // tile) and the contingency-block stride of w.rq and w.hot
  int nsl, rqs;
  int ntest;  // blocks of k_ctg_test
  TermOffsets toff;
  // contingencies scored this step (Alg. 2): slot s of the map-reduce holds
  // contingency act_k[s] (the identity when act_k is null), na slots in use,
  // outage factors of the slots in rows of kst entries at lodf_sel;
  // act_slot maps a contingency back to its slot (-1 when not scored)
  DevPtr<const int> act_k, act_slot;
  int na, kst;
  const void* lodf_sel;
  // [nKb][Lp] largest |factor| of a branch over 64 slots (null: test every row)
  DevPtr<const double> lmax;
};

// ---------------------------------------------------------------------------
// small device helpers

__device__ __forceinline__ double soft_relu(double e, double eps) {
  const double m = fmax(e, 0.0);
  return sqrt(m * m + eps * eps);
}

// d sigma/de = max(e,0)/sigma(e), 0 where max(e,0) = 0
__device__ __forceinline__ double soft_relu_d(double e, double eps) {
  const double m = fmax(e, 0.0);
  if (!(m > 0.0)) return 0.0;
  return m / sqrt(m * m + eps * eps);
}

// 1/sqrt(x) for x > 0: the hardware estimate (about 2^-23) refined by one
// third-order step on y^-2 = x: with r = 1 - x y^2, y (1 + r/2 + 3 r^2 / 8) is
// off by 5 r^3 / 16, far below FP64 rounding.  Three instructions fewer than two
// Newton steps, and a shorter chain.
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double r = fma(-x * y, y, 1.0);
  return fma(y * r, fma(0.375, r, 0.5), y);
}

// sigma(e) = sqrt(max(e,0)^2 + eps^2) and d sigma/de = max(e,0)/sigma (0 where
// max(e,0) = 0) from one reciprocal square root, for the per-generator
// penalties: a dependent sqrt and division per term cost more than the
// whole rest of a period block at 18 periods.  Both 0 when eps = 0 and e <= 0.
__device__ __forceinline__ double soft_relu_pair(double e, double eps, double& d) {
  const double m = fmax(e, 0.0);
  const double x = fma(m, m, eps * eps);
  if (!(x > 0.0)) {
    d = 0.0;
    return 0.0;
  }
  const double r = rsqrt_nr(x);
  d = m * r;
  return x * r;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wavefront (all lanes active), returned in every
// lane.  Butterflies inside each row of 16 lanes (quad swaps, half-row and
// row mirrors) give every lane its row sum; row_bcast15 then adds row 0's
// sum into row 1 and row 2's into row 3, and row_bcast31 adds rows 0+1 into
// row 3, so lane 63 holds ((r0 + r1) + (r2 + r3)).
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v += dpp_f64<0x141, 0xF>(v);   // row_half_mirror
  v += dpp_f64<0x140, 0xF>(v);   // row_mirror
  v += dpp_f64<0x142, 0xA>(v);   // row_bcast15 into rows 1 and 3
  v += dpp_f64<0x143, 0xC>(v);   // row_bcast31 into rows 2 and 3
  return readlane_f64(v, 63);
}

// Cross-half exchanges of gfx950: permlane32_swap trades lanes 32..63 of
// its first operand with lanes 0..31 of its second, permlane16_swap the odd
// 16-lane rows of the first with the even rows of the second.  After either,
// the sum of the two results holds, in the lanes whose exchanged bit is 0,
// a summed over the lane pair, and in the others b summed over the pair.
template <int W>
__device__ __forceinline__ double swap_add(double a, double b) {
  const unsigned alo = __double2loint(a), ahi = __double2hiint(a);
  const unsigned blo = __double2loint(b), bhi = __double2hiint(b);
  unsigned xlo, ylo, xhi, yhi;
  if constexpr (W == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
    xlo = l[0]; ylo = l[1]; xhi = h[0]; yhi = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
    xlo = l[0]; ylo = l[1]; xhi = h[0]; yhi = h[1];
  }
  return __hiloint2double((int)xhi, (int)xlo) + __hiloint2double((int)yhi, (int)ylo);
}

// dpp_f64 for patterns that read a lane of the same row for every lane
// (quad permutations, mirrors): no lane keeps its old value, so none is set.
template <int CTRL>
__device__ __forceinline__ double dpp_f64_row(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// Wavefront totals of two per-lane values at once (all lanes active): lanes
// 0..31 return the sum of a over the 64 lanes, lanes 32..63 the sum of b.
// The 32-lane swap leaves a's pair sums in the low half and b's in the high
// half, the 16-lane swap adds the two rows of each half, and four DPP steps
// finish inside each row.
__device__ __forceinline__ double pair_sum(double a, double b) {
  double v = swap_add<32>(a, b);
  v = swap_add<16>(v, v);
  v += dpp_f64_row<0xB1>(v);     // quad_perm [1,0,3,2]
  v += dpp_f64_row<0x4E>(v);     // quad_perm [2,3,0,1]
  v += dpp_f64_row<0x141>(v);    // row_half_mirror
  v += dpp_f64_row<0x140>(v);    // row_mirror
  return v;
}

// Largest value over the 64 lanes of a wavefront (all lanes active), in every
// lane: butterflies inside each row of 16 lanes, then the two cross-row
// exchanges.  NaN inputs are dropped (fmax).
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_f64_row<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmax(v, dpp_f64_row<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmax(v, dpp_f64_row<0x141>(v));  // row_half_mirror
  v = fmax(v, dpp_f64_row<0x140>(v));  // row_mirror
  const unsigned lo = __double2loint(v), hi = __double2hiint(v);
  auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  v = fmax(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
  const unsigned lo2 = __double2loint(v), hi2 = __double2hiint(v);
  l = __builtin_amdgcn_permlane32_swap(lo2, lo2, false, false);
  h = __builtin_amdgcn_permlane32_swap(hi2, hi2, false, false);
  return fmax(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
}

// Read-only view of device memory in the constant address space: loads at
// wavefront-uniform addresses through it become scalar loads into SGPRs.
// Only for data that no kernel of the same launch writes.
typedef __attribute__((address_space(4))) const double cdouble;
__device__ __forceinline__ const cdouble* as_const(const double* q) {
  return (const cdouble*)q;
}

// a * b + c with c wavefront-uniform, read straight from its SGPR pair (one
// VOP3 instruction instead of a copy into VGPRs and an accumulate).
__device__ __forceinline__ double fma_uniform_c(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}
__device__ __forceinline__ float fma_uniform_c(float a, float b, float c) {
  float d;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// ---- FP32 counterparts for the reduced-precision contingency map-reduce

// 1/sqrt(x) for x > 0 in FP32: the hardware estimate and one Newton step.
__device__ __forceinline__ float rsqrt_nr(float x) {
  float y = __builtin_amdgcn_rsqf(x);
  const float r = fmaf(-x * y, y, 1.0f);
  return fmaf(0.5f * y, r, y);
}

__device__ __forceinline__ float readlane_any(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double readlane_any(double v, int lane) { return readlane_f64(v, lane); }
// v with lane `lane` replaced by the wavefront-uniform x
template <typename R>
__device__ __forceinline__ R writelane_any(R v, R x, int lane) {
  return (int)(threadIdx.x & 63) == lane ? x : v;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// FP32 form of pair_sum (the same lane pattern, one register per value).
__device__ __forceinline__ float pair_sum(float a, float b) {
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  float v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  v = __uint_as_float(y[0]) + __uint_as_float(y[1]);
  v += dpp_f32<0xB1>(v);
  v += dpp_f32<0x4E>(v);
  v += dpp_f32<0x141>(v);
  v += dpp_f32<0x140>(v);
  return v;
}

// Outage factor of the stored kind, widened to the arithmetic type.
__device__ __forceinline__ double lodf_load(const double* q, size_t e) { return q[e]; }
__device__ __forceinline__ float lodf_load(const float* q, size_t e) { return q[e]; }
__device__ __forceinline__ float lodf_load(const uint16_t* q, size_t e) {
  return __uint_as_float((unsigned)q[e] << 16);
}
__device__ __forceinline__ double lodf_value(const DevProblem& p, int l, int k) {
  const size_t e = (size_t)l * p.Kp + k;
  if (p.lodf_kind == kLodfF64) return p.lodf[e];
  if (p.lodf_kind == kLodfF32) return (double)p.lodf32[e];
  return (double)lodf_load(p.lodf16, e);
}

// Largest value over the 64 lanes of a wavefront, ties to the smaller index
// (a total order, so the combination order does not matter); every lane gets
// the winner.  Entries with index INT_MAX are empty.
__device__ __forceinline__ bool better(double v2, int i2, double v, int i) {
  if (i2 == INT_MAX) return false;
  if (i == INT_MAX) return true;
  return v2 > v || (v2 == v && i2 < i);
}

template <int CTRL>
__device__ __forceinline__ void argmax_step(double& v, int& i) {
  const double v2 = dpp_f64<CTRL, 0xF>(v);
  const int i2 = __builtin_amdgcn_update_dpp(0, i, CTRL, 0xF, 0xF, false);
  if (better(v2, i2, v, i)) { v = v2; i = i2; }
}

__device__ __forceinline__ void wave_argmax(double& v, int& i) {
  argmax_step<0xB1>(v, i);
  argmax_step<0x4E>(v, i);
  argmax_step<0x141>(v, i);
  argmax_step<0x140>(v, i);
  // every lane of a row holds the row's winner; combine rows 0..3 in order
  double bv = readlane_f64(v, 0);
  int bi = __builtin_amdgcn_readlane(i, 0);
  for (int r = 16; r < 64; r += 16) {
    const double v2 = readlane_f64(v, r);
    const int i2 = __builtin_amdgcn_readlane(i, r);
    if (better(v2, i2, bv, bi)) { bv = v2; bi = i2; }
  }
  v = bv;
  i = bi;
}

// Deterministic block sum of NV values; every thread returns the totals.
// Each wavefront reduces with DPP, then the per-wavefront sums are added in
// wavefront order.  lds holds NV * 16 doubles; ends with a barrier so that
// lds can be reused.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const double ws = wave_sum(v[q]);
    if (lane == 0) lds[q * 16 + wv] = ws;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += lds[q * 16 + w];
    v[q] = s;
  }
  __syncthreads();
}

// Block argmax (ties to the smaller index); lds holds 16 doubles and 16 ints.
__device__ __forceinline__ void block_argmax(double& v, int& i, double* ldsv, int* ldsi) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  wave_argmax(v, i);
  if (lane == 0) { ldsv[wv] = v; ldsi[wv] = i; }
  __syncthreads();
  double bv = ldsv[0];
  int bi = ldsi[0];
  for (int w = 1; w < nw; ++w)
    if (better(ldsv[w], ldsi[w], bv, bi)) { bv = ldsv[w]; bi = ldsi[w]; }
  v = bv;
  i = bi;
  __syncthreads();
}

// sum_{q < n} src[q * stride] in ascending q, with up to U loads in flight.
template <int U>
__device__ __forceinline__ double strided_sum(const double* src, int n, size_t stride) {
  double acc = 0.0;
  for (int q0 = 0; q0 < n; q0 += U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = (q0 + u < n) ? src[(size_t)(q0 + u) * stride] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  return acc;
}

// Homotopy of this step: from the arguments, or from the row of the schedule
// table (eqs. (norm_t)-(step_size), evaluated on the host per iteration) that the
// step counter points at, copied ahead by the previous step (k_ctg_asm) or by
// k_set_step: one load instead of the counter and then the row.
__device__ __forceinline__ StepParams resolve_params(const EvalArgs& a) {
  if (a.mode.schedule == 0) return {a.mode.eps, a.mode.beta, a.mode.rho_s};
  const double* row = a.w.snext;
  return {row[0], row[1], row[2]};
}

// Contribution of one overloaded outage element: with s = sqrt(s2),
// e = s - s_ctg and sigma = sqrt(max(e,0)^2 + eps^2), returns sigma - eps (the
// penalty above its floor), and dC/dP, dC/dqmax2 scaled by kt.
template <typename R>
__device__ __forceinline__ R ctg_overload(R P, R s2, R smx, R eps, R eps2, R kt, R& dP, R& dq) {
  const R rs = rsqrt_nr(s2);
  const R s = s2 * rs;
  const R em = fmax(s - smx, R(0));
  const R w2 = fma(em, em, eps2);
  // w2 = 0 only when eps = 0 and s sits exactly on the rating: sigma = 0
  // there and the one-sided derivative is taken as 0
  const bool pos = w2 > R(0);
  const R rw = rsqrt_nr(pos ? w2 : R(1));
  const R sig = w2 * rw;
  const R gs = pos ? kt * em * rw : R(0);
  dP = gs * P * rs;
  dq = R(0.5) * gs * rs;
  return sig - eps;
}

// ---------------------------------------------------------------------------
// LDS-staged segmented sums over bus-sorted endpoint slots.  The block owns
// buses [i0, i0 + nbus) of one period; their slots are contiguous, so they are
// loaded with coalesced reads in chunks and each thread sums its own segment
// in ascending slot order.

constexpr int kSegChunk = 1024;

// A chunk's slots are all in flight at once; ahead() issues loads of the
// caller's that go out with the first chunk's.
template <class Ahead>
__device__ __forceinline__ void bus_segsum(const Pair* src, const DevProblem& p, int i0,
                                           int nbus, Pair* lds, double (&acc)[2], Ahead ahead) {
  constexpr int U = kSegChunk / kBlock;
  const int tid = threadIdx.x;
  const int* bptr = p.bptr;
  // the ends of the whole range are known without a load to wait for
  const int s_lo = i0 == 0 ? 0 : bptr[i0], s_hi = i0 + nbus == p.N ? p.twoL : bptr[i0 + nbus];
  int a = 0, b = 0;
  if (tid < nbus) { a = bptr[i0 + tid]; b = bptr[i0 + tid + 1]; }
  ahead();
  acc[0] = acc[1] = 0.0;
  for (int c0 = s_lo; c0 < s_hi; c0 += kSegChunk) {
    const int c1 = min(c0 + kSegChunk, s_hi);
    double vx[U], vy[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Pair e = src[min(c0 + u * kBlock + tid, c1 - 1)];
      vx[u] = e.x;
      vy[u] = e.y;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) lds[u * kBlock + tid] = Pair{vx[u], vy[u]};
    __syncthreads();
    const int lo = max(a, c0), hi = min(b, c1);
    for (int s = lo; s < hi; ++s) {
      const Pair e = lds[s - c0];
      acc[0] += e.x;
      acc[1] += e.y;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// FP64 MFMA slab product.  A 256-thread block computes the 16 output columns
// [n0, n0+16) of C = A * B over the reduction range [k0, k1) (multiples of 4)
// for all MT*16 rows; aload(k, row) supplies A[row][k] (zero outside A) and B
// is row-major (ldb).  The range is split over the four wavefronts; operands
// of NB consecutive k-steps are loaded before their MFMAs so that their
// memory latencies overlap.  The partial tiles are summed in LDS in wavefront order.
// v_mfma_f64_16x16x4f64 operands: lane l holds A[l%16][l/16] and
// B[l/16][l%16]; the result D[l/16 + 4r][l%16] sits in register r of lane l.
template <int MT, int NB, class ALoad, class Epi>
__device__ __forceinline__ void mfma_slab(ALoad aload, const double* __restrict__ B, int ldb,
                                          int k0, int k1, int n0, double* lds, Epi epi) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  const int steps = (k1 - k0) >> 2;
  const int s0 = (steps * wv) >> 2, s1 = (steps * (wv + 1)) >> 2;
  v4d acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = v4d{0.0, 0.0, 0.0, 0.0};
  const int kr = lane >> 4, cc = lane & 15;
  int st = s0;
  for (; st + NB <= s1; st += NB) {
    double bb[NB], aa[NB][MT];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int k = k0 + (st + u) * 4 + kr;
      bb[u] = B[(size_t)k * ldb + n0 + cc];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) aa[u][mt] = aload(k, mt * 16 + cc);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(aa[u][mt], bb[u], acc[mt], 0, 0, 0);
  }
  if (st < s1) {
    // the last, partial batch: its loads in flight together as well (the
    // step range is wavefront-uniform, so the guards do not diverge)
    double bb[NB], aa[NB][MT];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const bool in = st + u < s1;
      const int k = k0 + (st + u) * 4 + kr;
      bb[u] = in ? B[(size_t)k * ldb + n0 + cc] : 0.0;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) aa[u][mt] = in ? aload(k, mt * 16 + cc) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
      if (st + u < s1)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(aa[u][mt], bb[u], acc[mt], 0, 0, 0);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) lds[((wv * MT + mt) * 4 + r) * 64 + lane] = acc[mt][r];
  __syncthreads();
  for (int e = tid; e < MT * 256; e += kBlock) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += lds[w * MT * 256 + e];
    const int mt = e >> 8, rem = e & 255, r = rem >> 6, ln = rem & 63;
    const int row = mt * 16 + (ln >> 4) + 4 * r;
    const int col = n0 + (ln & 15);
    epi(row, col, s);
  }
  __syncthreads();
}

// NB: k-steps whose operands are loaded together; more steps in flight
// cost registers (the flow product shares its kernel with the branch and
// period blocks, so it takes 4 with 3-4 row tiles).
template <int NB34, class ALoad, class Epi>
__device__ __forceinline__ void mfma_slab_dispatch(int mtiles, ALoad aload, const double* B,
                                                   int ldb, int k0, int k1, int n0, double* lds,
                                                   Epi epi) {
  switch (mtiles) {
    case 1: mfma_slab<1, 8>(aload, B, ldb, k0, k1, n0, lds, epi); break;
    case 2: mfma_slab<2, 8>(aload, B, ldb, k0, k1, n0, lds, epi); break;
    case 3: mfma_slab<3, NB34>(aload, B, ldb, k0, k1, n0, lds, epi); break;
    default: mfma_slab<4, NB34>(aload, B, ldb, k0, k1, n0, lds, epi); break;
  }
}

// ---------------------------------------------------------------------------
// K1: branch forward, reserve and padding blocks, flow slabs

// Consecutive block indices go to the eight XCDs in turn.  xcd_group(p, n)
// renumbers block p of n so that the blocks of one XCD take one contiguous
// range of the logical order (the first n % 8 ranges one block longer), so
// that neighbouring logical blocks share an L2: the consecutive branches of
// a period store their bus-sorted endpoint slots through it (which merges
// the scattered stores into whole lines), and the blocks that read one
// operand fetch it from memory once per XCD.  Used by the branch blocks of
// the forward and adjoint kernels, the flow-adjoint assembly and the
// adjoint product's slabs.
__device__ __forceinline__ int xcd_group(int p, int n) {
  const int q = n >> 3, rem = n & 7, x = p & 7, i = p >> 3;
  return x * q + min(x, rem) + i;
}

__device__ void branch_forward(const EvalArgs& a, const StepParams& sp, int blk, double* lds) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int T = p.T, L = p.L, N = p.N;
  const int idx = blk * kBlock + threadIdx.x;
  double part[2] = {0.0, 0.0};
  if (idx < T * L) {
    const int t = idx / L, l = idx - t * L;
    const double* V = a.x;
    const double* TH = a.x + (size_t)T * N;
    const int f = p.br_from[l], o = p.br_to[l];
    const double vf = V[(size_t)t * N + f], vt = V[(size_t)t * N + o];
    const double d = TH[(size_t)t * N + f] - TH[(size_t)t * N + o];
    double sn, cs;
    sincos(d, &sn, &cs);
    const double g = p.br_g[l], b = p.br_b[l], bh = p.br_bh[l];
    const double vv = vf * vt;
    const double pf = g * vf * vf + vv * (-g * cs - b * sn);
    const double qf = -(b + bh) * vf * vf + vv * (b * cs - g * sn);
    const double pt = g * vt * vt + vv * (-g * cs + b * sn);
    const double qt = -(b + bh) * vt * vt + vv * (b * cs + g * sn);
    const size_t ep = (size_t)t * p.twoL;
    w.ep[ep + p.slot_fr[l]] = Pair{pf, qf};
    w.ep[ep + p.slot_to[l]] = Pair{pt, qt};
    // thermal penalty on the larger side, Example 1; ties go to the from side,
    // also where only the rounded roots are equal (squares further apart than
    // 2^-50 have different roots).  The root is sqrt's: of an infinite square it is
    // infinite, where x rsqrt_nr(x) is NaN and the penalty would fall to its floor
    const double sf2 = pf * pf + qf * qf, st2 = pt * pt + qt * qt;
    bool use_f = sf2 >= st2;
    if (!use_f && sf2 >= st2 * (1.0 - 0x1p-50)) use_f = sqrt(sf2) >= sqrt(st2);
    const double ss = sqrt(use_f ? sf2 : st2);
    const double eb = ss - p.br_smax[l];
    const double kbr = p.dt[t] * p.c_s * sp.beta;
    double kth, kp = 0.0, kq = 0.0;
    part[0] = kbr * soft_relu_pair(eb, sp.eps, kth);
    kth *= kbr;
    if (ss > 0.0) {
      kp = kth * (use_f ? pf : pt) / ss;
      kq = kth * (use_f ? qf : qt) / ss;
    }
    // angle-difference penalty
    const double ea = fabs(d) - p.ang_max;
    const double kang = p.dt[t] * p.c_ang * sp.beta;
    double ka;
    part[1] = kang * soft_relu_pair(ea, sp.eps, ka);
    const double sgn = d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0);
    const double kd = kang * ka * sgn;
    // reactive part of the contingency flows: max(q_fr^2, q_to^2), ties: from
    const double qf2 = qf * qf, qt2 = qt * qt;
    const bool qfr = qf2 >= qt2;
    const double qm2 = qfr ? qf2 : qt2;
    w.q2[(size_t)t * p.Lp + l] = qm2;
    // radius of the map-reduce's first test: with margins of 2^-40 on s_ctg^2
    // and 2^-50 on the root, fl(P^2 + qmax2) > s_ctg^2 implies |P| > thr
    // under FP64 rounding; -1 (every flow passes) where qmax2 alone comes
    // within the margin of the rating
    const double A = p.ctg_smax2[l] * (1.0 - 0x1p-40) - qm2;
    const double thr = A > 0.0 ? sqrt(A) * (1.0 - 0x1p-50) : -1.0;
    w.thr[(size_t)t * p.Lp + l] = thr;
    const size_t TL = (size_t)T * L, e = (size_t)t * L + l;
    // written once and read once: 49 bytes and four stores a branch, the ends'
    // flows in one scattered 16-byte store each (nine coefficients and four
    // 8-byte stores took 1.6 us more of 14.7 at 2800 branches and 48 periods, and as
    // much in the reverse pass)
    w.bco[e] = Pair{cs, sn};
    w.bco[TL + e] = Pair{kp, kq};
    w.bco[2 * TL + e] = Pair{kd, 2.0 * (qfr ? qf : qt)};
    w.bside[e] = (uint8_t)((use_f ? 0 : kThermalTo) | (qfr ? 0 : kReactiveTo));
  }
  block_sum<2>(part, lds);
  if (threadIdx.x == 0) {
    w.tpart[a.toff.br + blk] = part[0];
    w.tpart[a.toff.ang + blk] = part[1];
  }
}

// One block per period t and slice sl of 256 generators, one thread per
// generator: block-bid cost, no-load, start-up/shut-down and reserve costs
// (Examples 2-3), the penalised device constraints of eq. (nlp_updated) and
// their partials, and the slice's sums of the cost and penalty terms.  The
// next period's terms that depend on this period's p and u are included, so
// each thread writes only its own partials; the reserve shortfall, which
// needs the whole period's reserve, is reserve_pad_block's.  Only the final
// kernel reads what it writes, so it runs in k_ctg_asm's launch, beside the
// contingency reductions: in the forward kernel its registers (the most of
// any block there) held that kernel to four wavefronts per SIMD.
__device__ void period_block(const EvalArgs& a, const StepParams& sp, int t, int sl,
                             double* lds) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int T = p.T, N = p.N, G = p.G, M = p.M;
  const int tid = threadIdx.x;
  const double* xP = a.x + 2 * (size_t)T * N;
  const double* xQ = xP + (size_t)T * G;
  const double* xR = xQ + (size_t)T * G;
  const double* xU = xR + (size_t)T * G;
  const size_t TG = (size_t)T * G;
  const double dtt = p.dt[t];
  const double kpen = sp.rho_s * p.rho * sp.beta * dtt;
  const double eps = sp.eps;
  double acc[2] = {0.0, 0.0};  // dev, pen
  const int j = sl * kBlock + tid;
  if (j < G) {
    const size_t e = (size_t)t * G + j;
    // every load of the generator first, so that their latencies overlap
    const double pj = xP[e], qj = xQ[e], rj = xR[e], uj = xU[e];
    const double pm1 = t > 0 ? xP[e - G] : p.p0[j];
    const double um1 = t > 0 ? xU[e - G] : p.u0[j];
    const bool nxt = t + 1 < T;
    const double p1 = nxt ? xP[e + G] : 0.0, u1 = nxt ? xU[e + G] : 0.0;
    const double pmax = p.pmax[j], pmin = p.pmin[j], qmax = p.qmax[j], qmin = p.qmin[j];
    const double rmax = p.rmax[j], ru = p.ru[j], rd = p.rd[j], rusu = p.rusu[j];
    const double rdsd = p.rdsd[j], con = p.con[j], csu = p.csu[j], csd = p.csd[j];
    const double cr = p.cr[j];
    double sz4[4], cm4[4], pc4[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bool in = m < M;
      sz4[m] = in ? p.seg_size[j * M + m] : 0.0;
      cm4[m] = in ? p.seg_cost[j * M + m] : 0.0;
      pc4[m] = in ? p.pcum[j * M + m] : 0.0;
    }
    // block-bid energy cost, eq. (costs): sum_m c_m max(min(p - Pcum_{m-1}, D_m), 0)
    double cost = 0.0, dcost = 0.0, lo = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (m < M) {
        const double am = pj - lo;
        cost += cm4[m] * fmax(fmin(am, sz4[m]), 0.0);
        if (am > 0.0 && am <= sz4[m]) dcost += cm4[m];
        lo = pc4[m];
      }
    }
    for (int m = 4; m < M; ++m) {
      const double am = pj - lo;
      const double sz = p.seg_size[j * M + m], cm = p.seg_cost[j * M + m];
      cost += cm * fmax(fmin(am, sz), 0.0);
      if (am > 0.0 && am <= sz) dcost += cm;
      lo = p.pcum[j * M + m];
    }
    const double du = uj - um1;
    const double dev = dtt * cost + dtt * con * uj + csu * fmax(du, 0.0) +
                       csd * fmax(-du, 0.0) + dtt * cr * rj;
    double gp = dtt * dcost;
    double gu = dtt * con + (du > 0.0 ? csu : 0.0) - (-du > 0.0 ? csd : 0.0);
    double gr = dtt * cr;
    double gq = 0.0;
    if (nxt) {
      const double du1 = u1 - uj;
      gu -= (du1 > 0.0 ? csu : 0.0) - (-du1 > 0.0 ? csd : 0.0);
    }
    double pen = 0.0, a_, dd;
    a_ = pj + rj - pmax * uj;                             // headroom
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gp += dd; gr += dd; gu -= dd * pmax;
    a_ = pmin * uj - pj;                                  // minimum output
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gu += dd * pmin; gp -= dd;
    a_ = pj - pm1 - dtt * (ru * uj + rusu * (1.0 - uj));  // ramp up
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gp += dd; gu -= dd * dtt * (ru - rusu);
    a_ = pm1 - pj - dtt * (rd * uj + rdsd * (1.0 - uj));  // ramp down
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gp -= dd; gu -= dd * dtt * (rd - rdsd);
    a_ = qj - qmax * uj;                                  // reactive upper
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gq += dd; gu -= dd * qmax;
    a_ = qmin * uj - qj;                                  // reactive lower
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gu += dd * qmin; gq -= dd;
    a_ = rj - rmax * uj;                                  // reserve capability
    pen += soft_relu_pair(a_, eps, dd); dd *= kpen;
    gr += dd; gu -= dd * rmax;
    if (nxt) {  // the next period's ramp constraints depend on p_t
      const double dt1 = p.dt[t + 1];
      const double k1 = sp.rho_s * p.rho * sp.beta * dt1;
      a_ = p1 - pj - dt1 * (ru * u1 + rusu * (1.0 - u1));
      double d1;
      (void)soft_relu_pair(a_, eps, d1);
      gp -= k1 * d1;
      a_ = pj - p1 - dt1 * (rd * u1 + rdsd * (1.0 - u1));
      (void)soft_relu_pair(a_, eps, d1);
      gp += k1 * d1;
    }
    w.gdev[0 * TG + e] = gp;
    w.gdev[1 * TG + e] = gq;
    w.gdev[2 * TG + e] = gr;
    w.gdev[3 * TG + e] = gu;
    acc[0] = dev;
    acc[1] = kpen * pen;
  }
  block_sum<2>(acc, lds);
  if (tid == 0) {
    const int q = t * ((G + kBlock - 1) / kBlock) + sl;
    w.tpart[a.toff.dev + q] = acc[0];
    w.tpart[a.toff.pen + q] = acc[1];
  }
}

// Period t's reserve shortfall penalty and its derivative (eq.
// (nlp_updated)), which every generator's reserve partial needs; and the
// padding of period t that the map-reduce reads: branches past L pass
// every test (q2 = 0, radius -1), outages past K have no flow.
__device__ void reserve_pad_block(const EvalArgs& a, const StepParams& sp, int t, double* lds) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x, T = p.T, G = p.G;
  const double* xR = a.x + 2 * (size_t)T * p.N + 2 * (size_t)T * G;
  double acc[1] = {0.0};
  for (int j = tid; j < G; j += kBlock) acc[0] += xR[(size_t)t * G + j];
  block_sum<1>(acc, lds);
  if (tid == 0) {
    const double short_ = p.rsv_req[t] - acc[0];
    const double krs = p.dt[t] * p.c_rsv * sp.beta;
    w.tpart[a.toff.rsv + t] = krs * soft_relu(short_, sp.eps);
    w.drs[t] = krs * soft_relu_d(short_, sp.eps);
  }
  for (int l = p.L + tid; l < p.Lp; l += kBlock) {
    w.q2[(size_t)t * p.Lp + l] = 0.0;
    w.thr[(size_t)t * p.Lp + l] = -1.0;
  }
  for (int k = p.K + tid; k < p.Kp; k += kBlock) w.Fk[(size_t)t * p.Kp + k] = 0.0;
}

// LDS of an MFMA slab: four wavefronts x up to 4 row tiles x 256 partial
// results.
constexpr int kSlabLds = 4 * 4 * 256;
// LDS of the forward kernel: the flow slab's single row tile (its block sums
// need 32 doubles), so that LDS does not limit its blocks per CU.
constexpr int kFwdLds = 4 * 1 * 256;
static_assert(kFwdLds >= 2 * 16, "LDS carve");

// Base-case DC flows of 16 branches for 16 periods, on FP64 MFMA, with the
// uniform slack folded into the operand: F[t][l] = sum_j p_tj (ISF[l][bus(j)]
// - rowsum_l / N) - c[t][l], where the per-grid constant c holds the loads'
// part (ISF load_t - rowsum_l sum_i load_ti / N).  Also the outaged branches'
// flows.  One block per (16 branches, 16 periods): a single row tile keeps
// eight k-steps of operands in flight (the k-loop's load round trips, not
// the MFMAs, set a slab's time).
__device__ void flow_slab(const EvalArgs& a, int blk, double* smem) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int T = p.T, G = p.G, Lp = p.Lp, Kp = p.Kp, N = p.N;
  const int mtiles = p.Tp / 16;
  // consecutive blocks go to the eight XCDs in turn: the period tiles of a
  // slab take block indices eight apart, so they run on one XCD and its L2
  // fetches the slab's ISF columns once (the last group of fewer than eight
  // slabs spreads them over its own slabs' count)
  const int nsl = Lp / 16, grp = 8 * mtiles;
  const int q = blk / grp, r = blk - q * grp;
  const int ns = min(8, nsl - 8 * q);
  const int slab = 8 * q + r % ns, r0 = (r / ns) * 16;
  const double* xP = a.x + 2 * (size_t)T * N;
  const int n0 = slab * 16;
  double* F = w.F;
  double* Fk = w.Fk;
  const int* kof = p.kof;
  const double* cload = p.cload;
  auto aload = [=](int k, int row) -> double {
    const int t = r0 + row;
    return (t < T && k < G) ? xP[(size_t)t * G + k] : 0.0;
  };
  auto epi = [=](int row, int col, double v) {
    const int t = r0 + row;
    if (t < T) {
      const double f = v - cload[(size_t)t * Lp + col];
      F[(size_t)t * Lp + col] = f;
      const int k = kof[col];
      if (k >= 0) Fk[(size_t)t * Kp + k] = f;
    }
  };
  mfma_slab<1, 8>(aload, p.isf_gT, Lp, 0, p.G4, n0, smem, epi);
}

// Blocks [0, T): the reserve shortfall and the padding of one period each;
// [T, T + nb_br): branch forward; then (Lp / 16) x (Tp / 16) flow slabs.
__device__ __forceinline__ void forward_body(const EvalArgs& a, int b, double* smem) {
  const StepParams sp = resolve_params(a);
  if (b == 0 && threadIdx.x < QG_NCLASS + 3) {
    // the step's parameters for the later kernels, with the row's step sizes and
    // bias corrections (0 and 1 without a schedule); one entry a thread: an
    // array indexed by a loop would live in scratch memory, whose set-up delays
    // the kernel that follows
    double* pb = a.w.params;
    const int c = threadIdx.x;
    const bool sched = a.mode.schedule != 0;
    if (c < QG_NCLASS)
      pb[PB_ALPHA + c] = sched ? a.w.snext[3 + c] : 0.0;
    else if (c == QG_NCLASS)
      pb[PB_EPS] = sp.eps;
    else if (c == QG_NCLASS + 1)
      pb[PB_BETA] = sp.beta;
    else
      pb[PB_RHO] = sp.rho_s;
    if (c < 2) pb[PB_BC1 + c] = sched ? a.w.snext[3 + QG_NCLASS + c] : 1.0;
  }
  if (b < a.p.T)
    reserve_pad_block(a, sp, b, smem);
  else if (b < a.nb_br + a.p.T)
    branch_forward(a, sp, xcd_group(b - a.p.T, a.nb_br), smem);
  else
    flow_slab(a, b - a.nb_br - a.p.T, smem);
}

__global__ __launch_bounds__(kBlock) void k_forward(EvalArgs a) {
  __shared__ double smem[kFwdLds];
  forward_body(a, blockIdx.x, smem);
}

// Per-(t, bus) power balance (Example 4): segmented sums of the bus's
// endpoint flows staged through LDS, minus its generators; multipliers and
// the soft-abs value.
__device__ void bus_balance(const EvalArgs& a, int blk, Pair* smem) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x;
  const int t = blk / a.bus_chunks;
  const int c = blk - t * a.bus_chunks;
  const int i0 = c * kBlock;
  const int nbus = min(kBlock, p.N - i0);
  const double eps = w.params[PB_EPS], beta = w.params[PB_BETA];
  // the bus's loads and its first generator, in flight with the endpoint flows
  const int i = i0 + tid;
  const size_t ti = (size_t)t * p.N + i;
  int g0 = 0, g1 = 0, j0 = -1;
  double ldp = 0.0, ldq = 0.0;
  if (tid < nbus) {
    g0 = p.gptr[i];
    g1 = p.gptr[i + 1];
    ldp = p.load_p[ti];
    ldq = p.load_q[ti];
  }
  double fl[2];
  bus_segsum(w.ep + (size_t)t * p.twoL, p, i0, nbus, smem, fl, [&]() {
    if (g0 < g1) j0 = p.glist[g0];
  });
  double part[1] = {0.0};
  if (tid < nbus) {
    const double* xP = a.x + 2 * (size_t)p.T * p.N;
    const double* xQ = xP + (size_t)p.T * p.G;
    double sp_ = 0.0, sq = 0.0;
    for (int g = g0; g < g1; ++g) {
      const size_t e = (size_t)t * p.G + (g == g0 ? j0 : p.glist[g]);
      sp_ += xP[e];
      sq += xQ[e];
    }
    const double dp = ldp + fl[0] - sp_;
    const double dq = ldq + fl[1] - sq;
    const double kb = p.dt[t] * beta;
    // |.|_eps = sqrt(v^2 + eps^2) and its derivative v / |.|_eps from one
    // reciprocal square root each (0 where both vanish)
    const double xp = fma(dp, dp, eps * eps), xq = fma(dq, dq, eps * eps);
    const double rp = xp > 0.0 ? rsqrt_nr(xp) : 0.0, rq = xq > 0.0 ? rsqrt_nr(xq) : 0.0;
    const double lp = kb * p.c_p * (dp * rp), lq = kb * p.c_q * (dq * rq);
    w.lamp[ti] = lp;
    w.lamq[ti] = lq;
    // the same multipliers per generator of the bus (read by k_final)
    for (int g = g0; g < g1; ++g) {
      const size_t e = (size_t)t * p.G + (g == g0 ? j0 : p.glist[g]);
      w.lamg[e] = lp;
      w.lamqg[e] = lq;
    }
    part[0] = kb * (p.c_p * (xp * rp) + p.c_q * (xq * rq));
  }
  block_sum<1>(part, reinterpret_cast<double*>(smem));
  if (tid == 0) w.tpart[a.toff.bal + blk] = part[0];
}

// ---------------------------------------------------------------------------
// K3: contingency map-reduce over (t, l, k).
//
// A wavefront owns 64 contingencies (one per lane) and BL consecutive
// branches; its BL outage factors stay in registers.  A block stacks WL
// wavefronts along l and covers the periods [t0, t0 + TC) (grid.z splits
// the periods).  The branch quantities F_tl, qmax2_tl and s_ctg^2 are the
// same for every lane, so they are read with scalar loads into SGPRs; the
// flows of the block's 64 outaged branches are staged in LDS.  For each
// period and group of 8 branches every lane forms the post-outage flows
// P = F_tl + LODF_lk F_tk and tests P^2 + qmax2_tl > s_ctg^2 (one compare
// into a ballot per branch).  Only a branch with an overloaded lane
// evaluates soft-ReLUs and sums dP (-> R, d/dF_tl) and dq (-> Q,
// d/dqmax2_tl) over its 64 lanes; the other branches store zero partials.
// z_tk and S_tk (the derivative through F_tk) accumulate in the lane over l
// and are summed over the block's wavefronts in LDS.  The outaged branch
// itself and the padding carry a NaN factor, so they never test overloaded.

// LT: storage type of the outage factors (double, float, or BF16 bits);
// R: arithmetic type (double with FP64 factors, float otherwise).
template <int BL, typename LT>
__global__ __launch_bounds__(512) void k_ctg_main(EvalArgs a, const LT* __restrict__ lodf) {
  static_assert(BL % 8 == 0 && BL <= 32, "branches per wavefront");
  typedef typename std::conditional<std::is_same<LT, double>::value, double, float>::type R;
  constexpr bool kF64 = std::is_same<R, double>::value;
  // LDS: sFk[TC][64] (outaged branches' flows), then per period and
  // wavefront the lanes' z and S: zsh[TC][WL][64], ssh[TC][WL][64]
  extern __shared__ double dyn[];
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int WL = blockDim.x >> 6;
  const int lb = blockIdx.x, kb = blockIdx.y;
  const int T = p.T, Lp = p.Lp, Kp = p.Kp;
  const int TC = a.tc;
  const int t0 = blockIdx.z * TC;
  const int nt = min(TC, T - t0);
  const int k = kb * 64 + lane;  // slot of the lane
  double* sFk = dyn;
  double* zsh = dyn + TC * 64;
  double* ssh = zsh + TC * WL * 64;
  for (int e = threadIdx.x; e < nt * 64; e += blockDim.x) {
    const int tt = e >> 6, s = kb * 64 + (e & 63);
    sFk[e] = w.Fk[(size_t)(t0 + tt) * Kp + (a.act_k ? a.act_k[s] : s)];
  }
  const cdouble* Sc = as_const(p.ctg_smax2);
  const cdouble* Mc = as_const(p.ctg_smax);
  const cdouble* Dc = as_const(p.dt);
  const double beta = w.params[PB_BETA];
  const R eps = (R)w.params[PB_EPS];
  const R eps2 = eps * eps;
  // the block covers a.lt consecutive tiles of WL * BL branches; z and S of
  // each (period, wavefront, lane) accumulate over them in LDS
  for (int it = 0; it < a.lt; ++it) {
    const int lbase = __builtin_amdgcn_readfirstlane((lb * a.lt + it) * BL * WL + wv * BL);
    const bool on = lbase < Lp;
    R lod[BL], smx2[BL];
    // lane e of chunk c holds F, qmax2 and (FP64) the test radius thr of
    // period t0 + e / 8, branch lbase + 8 c + e % 8 (TC * 8 <= 64 entries)
    R fv[BL / 8], qv[BL / 8], hv[BL / 8];
    if (on) {
#pragma unroll
      for (int j = 0; j < BL; ++j) {
        lod[j] = lodf_load(lodf, (size_t)(lbase + j) * a.kst + k);
        smx2[j] = (R)Sc[lbase + j];
      }
      const int et = lane >> 3, eg = lane & 7;
#pragma unroll
      for (int c = 0; c < BL / 8; ++c) {
        fv[c] = R(0);
        qv[c] = R(0);
        hv[c] = R(0);
        if (et < nt) {
          const size_t e = (size_t)(t0 + et) * Lp + lbase + c * 8 + eg;
          fv[c] = (R)w.F[e];
          qv[c] = (R)w.q2[e];
          if constexpr (kF64) hv[c] = w.thr[e];
        }
      }
    }
    if (it == 0) __syncthreads();  // sFk staged
    // R and Q of (period t0 + e / 8, branch lbase + 8 c + e % 8) gather in
    // lane e of racc[c], qacc[c] (zero where nothing is overloaded) and go
    // out once per tile, so the period loop itself stores nothing
    R racc[BL / 8], qacc[BL / 8];
#pragma unroll
    for (int c = 0; c < BL / 8; ++c) {
      racc[c] = R(0);
      qacc[c] = R(0);
    }
    for (int tt = 0; tt < nt; ++tt) {
      const int t = t0 + tt;
      R zacc = R(0), sacc = R(0);
      if (on) {
        const R fk = (R)sFk[tt * 64 + lane];
#pragma unroll
        for (int c = 0; c < BL / 8; ++c) {
          R Fr[8], Qr[8], P[8];
          unsigned rows = 0;
          if constexpr (kF64) {
            // FP64: |P| > thr, which every element of the exact test passes
            // (the radius of k_forward); the exact test follows per branch
#pragma unroll
            for (int g = 0; g < 8; ++g) {
              Fr[g] = readlane_any(fv[c], tt * 8 + g);
              const R Hr = readlane_any(hv[c], tt * 8 + g);
              P[g] = fma_uniform_c(lod[c * 8 + g], fk, Fr[g]);
              if (__builtin_amdgcn_ballot_w64(fabs(P[g]) > Hr)) rows |= 1u << g;
            }
          } else {
#pragma unroll
            for (int g = 0; g < 8; ++g) {
              Fr[g] = readlane_any(fv[c], tt * 8 + g);
              Qr[g] = readlane_any(qv[c], tt * 8 + g);
            }
#pragma unroll
            for (int g = 0; g < 8; ++g) {
              const int j = c * 8 + g;
              P[g] = fma_uniform_c(lod[j], fk, Fr[g]);
              const R s2 = fma_uniform_c(P[g], P[g], Qr[g]);
              if (__builtin_amdgcn_ballot_w64(s2 > smx2[j])) rows |= 1u << g;
            }
          }
          if (rows) {
            const R kt = (R)(Dc[t] * p.c_s * beta);
#pragma unroll
            for (int g = 0; g < 8; ++g) {
              if ((rows >> g) & 1u) {
                const int j = c * 8 + g;
                if constexpr (kF64) Qr[g] = readlane_any(qv[c], tt * 8 + g);
                // the square is formed again (the same fused operation, so
                // the same value) rather than kept across the test of all
                // eight branches: fewer live registers
                const R s2 = fma(P[g], P[g], Qr[g]);
                R dP = R(0), dq = R(0);
                if (s2 > smx2[j]) {
                  zacc += ctg_overload(P[g], s2, (R)Mc[lbase + j], eps, eps2, kt, dP, dq);
                  sacc = fma(lod[j], dP, sacc);
                }
                const R r = pair_sum(dP, dq);  // lane 0: sum of dP, lane 32: of dq
                racc[c] = writelane_any(racc[c], readlane_any(r, 0), tt * 8 + g);
                qacc[c] = writelane_any(qacc[c], readlane_any(r, 32), tt * 8 + g);
              }
            }
          }
        }
      }
      const int zi = (tt * WL + wv) * 64 + lane;
      if (it == 0) {
        zsh[zi] = (double)zacc;
        ssh[zi] = (double)sacc;
      } else {
        zsh[zi] += (double)zacc;
        ssh[zi] += (double)sacc;
      }
    }
    if (on && lane < nt * 8) {
      const size_t o = ((size_t)kb * T + t0 + (lane >> 3)) * Lp + lbase + (lane & 7);
#pragma unroll
      for (int c = 0; c < BL / 8; ++c) {
        w.rpart[o + c * 8] = (double)racc[c];
        w.qpart[o + c * 8] = (double)qacc[c];
      }
    }
  }
  // sum z and S over the block's wavefronts (wavefront order), every
  // (period, contingency) of the block by one thread
  __syncthreads();
  for (int e = threadIdx.x; e < nt * 64; e += blockDim.x) {
    const int tt = e >> 6, kk = e & 63;
    double z = 0.0, s2 = 0.0;
    for (int q = 0; q < WL; ++q) {
      z += zsh[(tt * WL + q) * 64 + kk];
      s2 += ssh[(tt * WL + q) * 64 + kk];
    }
    const size_t o = ((size_t)lb * T + t0 + tt) * Kp + kb * 64 + kk;
    w.zpart[o] = z;
    w.spart[o] = s2;
  }
}

// Row-compacted form of the same map-reduce (the period-split tile, default).
//
// One block covers one period and 64 contingencies (a lane each) over every
// branch, so z_tk and S_tk are complete at its end and the block finishes
// them itself (ctg_finish_z); the branches are split into a.nsl slices, one
// wavefront each, whose z and S are added in slice order.  A slice takes the
// 64-branch groups s, s + nsl, ...  For a group every lane first decides one
// branch l by a bound: |P_tlk| = |F_tl + LODF_lk F_tk| <= |F_tl| + Lm Fm, with
// Lm the largest |LODF_lk| of the row over the block's 64 contingencies (a
// per-grid table, a.lmax) and Fm the largest |F_tk| of its lanes.  When
// |F_tl| (1 + 2^-40) + Lm Fm <= thr_tl (1 - 2^-40) holds in floating point, no
// element of the row passes the test |fl(P)| > thr_tl: the margins cover the
// rounding of the bound, of its comparison and of fl(P) (a few units of
// 2^-53).  NaN in F or thr makes the comparison false (the row is tested).
// Only the rows that the ballot leaves are loaded and tested, four at a time,
// and only rows with a flagged lane evaluate the penalty, two at a time:
// their sums over the lanes (R = sum dP, Q = sum dq) share one reduction
// tree.  R and Q of such rows are stored per contingency block, with one
// 64-bit word of row flags per group; the readers consult the word first.
// Neither the pairing of rows nor the bound changes any sum's order, so
// testing every row (lmax null) gives bitwise the same results, as does a
// block of fewer wavefronts than slices.  ALL: every row was tested by
// k_ctg_test, and the flagged rows come from its words.
//
// FP64 tests |P| > thr_tl with thr_tl from k_forward, a radius a little below
// sqrt(s_ctg^2 - qmax2_tl), so that every element the exact test
// P^2 + qmax2 > s_ctg^2 accepts passes it; the exact test is applied again
// when the row is evaluated.  FP32 arithmetic (FP32 or BF16 factors) tests
// fl(P^2 + qmax2) > s_ctg^2 in FP32 on FP32 roundings of F, qmax2 and s_ctg^2,
// and Lm is the largest stored factor.  There |fl(P)| <= (Lm Fm + |F|)(1 + u)^2
// and the test's left side is at most ((Lm Fm + |F|)^2 + qmax2)(1 + u)^5 (u =
// 2^-24), so a row is passed over when (Lm Fm + |F|)^2 (1 + 2^-18) + qmax2 (1 +
// 2^-18) <= s_ctg^2 (1 - 2^-18), computed in FP64.  FP32 sums of z and S are
// flushed to FP64 at every multiple of eight branches.
//
// What it measured, against a tile of eight branches and four periods per
// wavefront whose half rows (four branches) were skipped together and whose
// z and S went through memory to a reduction kernel (us in the steps of solves a
// fifth under way, map-reduce + reduction before, this kernel now): 2000 buses x 48
// periods 55.6 + 10.0 -> 34, 617 x 18 9.4 + 4.8 -> 7.2, twelve grids of 100-1000 buses
// in a batch 262 + 17 -> 39 (along the benchmark's solves from the flat start 29 and 7.2 in
// the two grids).  There 2.1 % of the rows at 2000 buses are hot, and most
// of them in all 64 lanes (the branch is overloaded before the outage); 3.8 %
// remain after the bound (13 % of half rows did).  At 2000 buses the vector
// instructions bound it (they issue in about three quarters of the SIMD cycles,
// half of them for the hot rows); at 617 buses its chain of four memory round
// trips does.  Slower: the slices' hot rows spread evenly over the wavefronts
// after the test (two more barriers and a lookup: 48 us where it took 36, 10 us
// at 617 buses), one list of undecided rows for four groups with F and thr by
// scalar loads (44 us), R and Q staged in LDS (44 us).

// A hot row (one with a flagged lane): the lane's post-outage flow and factor,
// the branch (-1: none), its qmax2 and rating.
template <typename R>
struct HotRow {
  R P, lod, q2, smx, smx2;
  int l;
};

// Penalty above its floor and derivatives of the row's element in this lane,
// 0 where the exact test fails (NaN factors, flows inside the rating).  FP64:
// dP and dq per unit of kt and kt / 2, which are applied to the sums.
__device__ __forceinline__ bool hot_eval(const HotRow<float>& h, float eps, float eps2, float kt,
                                         float& z, float& dP, float& dq) {
  const float s2 = fma(h.P, h.P, h.q2);
  const bool m = s2 > h.smx2;
  z = ctg_overload(h.P, m ? s2 : 1.0f, h.smx, eps, eps2, kt, dP, dq);
  z = m ? z : 0.0f;
  dP = m ? dP : 0.0f;
  dq = m ? dq : 0.0f;
  return m;
}
__device__ __forceinline__ bool hot_eval(const HotRow<double>& h, double eps, double eps2, double,
                                         double& z, double& dP, double& dq) {
  const double s2 = fma(h.P, h.P, h.q2);
  const bool m = s2 > h.smx2;
  const double rs = rsqrt_nr(m ? s2 : 1.0);
  const double em = fmax(fma(s2, rs, -h.smx), 0.0);
  const double w2 = fma(em, em, eps2);
  // w2 = 0 only when eps = 0 and s sits exactly on the rating
  const bool pos = m && w2 > 0.0;
  const double rw = rsqrt_nr(pos ? w2 : 1.0);
  z = pos ? fma(w2, rw, -eps) : 0.0;
  dq = pos ? em * rw * rs : 0.0;
  dP = pos ? dq * h.P : 0.0;
  return m;
}

// Wavefront totals of two rows' dP and dq at once: lanes 0..15 return the sum
// of pa, lanes 16..31 of pb, 32..47 of qa, 48..63 of qb, each summed over the
// 64 lanes by pair_sum's tree.
__device__ __forceinline__ double quad_sum(double pa, double qa, double pb, double qb) {
  double v = swap_add<16>(swap_add<32>(pa, qa), swap_add<32>(pb, qb));
  v += dpp_f64_row<0xB1>(v);
  v += dpp_f64_row<0x4E>(v);
  v += dpp_f64_row<0x141>(v);
  v += dpp_f64_row<0x140>(v);
  return v;
}
__device__ __forceinline__ float quad_sum(float pa, float qa, float pb, float qb) {
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(pa), __float_as_uint(qa), false,
                                                  false);
  const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(pb), __float_as_uint(qb), false,
                                                  false);
  const float a = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  const float b = __uint_as_float(y[0]) + __uint_as_float(y[1]);
  const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  float v = __uint_as_float(w[0]) + __uint_as_float(w[1]);
  v += dpp_f32<0xB1>(v);
  v += dpp_f32<0x4E>(v);
  v += dpp_f32<0x141>(v);
  v += dpp_f32<0x140>(v);
  return v;
}

// z_tk of the block's 64 slots from their sums over the branches (plus the
// floor (L-1) eps), and the chunk's worst penalty (smallest index on ties)
// and sum; one wavefront, lane = slot.
__device__ __forceinline__ void ctg_finish_z(const EvalArgs& a, int kc, int t, double kt,
                                             double eps, double zs) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int lane = threadIdx.x & 63, s = kc * 64 + lane;
  double z = -DBL_MAX, zsum = 0.0;
  int idx = INT_MAX;
  if (s < a.na) {
    const int k = a.act_k ? a.act_k[s] : s;
    z = kt * ((double)(p.L - 1) * eps + zs);
    w.zval[(size_t)t * p.Kp + k] = z;
    idx = k;
    zsum = z;
  }
  const double tot = wave_sum(zsum);
  wave_argmax(z, idx);
  if (lane == 0) {
    const size_t c = (size_t)t * a.nKc + kc;
    w.zmaxp[c] = z;
    w.zargp[c] = (double)idx;
    w.zsump[c] = tot;
  }
}

// The mean outage-correction derivative of the block's slots.
__device__ __forceinline__ void ctg_finish_s(const EvalArgs& a, int kc, int t, double ss) {
  const int s = kc * 64 + (threadIdx.x & 63);
  if (s < a.na)
    a.w.smean[(size_t)t * a.p.Kp + s] = a.p.ctg_sum ? ss : ss / (double)a.p.K;
}

// LT: storage type of the outage factors; lds: a.nsl x 128 doubles.
template <typename LT, bool ALL>
__device__ __forceinline__ void ctg_rows_body(const EvalArgs& a, int b, double* lds) {
  typedef typename std::conditional<std::is_same<LT, double>::value, double, float>::type R;
  constexpr bool kF64 = std::is_same<R, double>::value;
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const LT* __restrict__ lodf = DevPtr<const LT>(static_cast<const LT*>(a.lodf_sel));
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int T = p.T, L = p.L, Lp = p.Lp, ng = Lp >> 6;
  const int kb = b / T, t = b - kb * T;
  const unsigned k = (unsigned)(kb * 64 + lane);  // slot of the lane
  const double* __restrict__ Ft = w.F + (size_t)t * Lp;
  const double* __restrict__ Ht = (kF64 ? w.thr : w.q2) + (size_t)t * Lp;  // thr, or qmax2
  const double* __restrict__ lmax = ALL ? nullptr : a.lmax + (size_t)kb * Lp;
  // F, thr and the largest factor of a lane's branch in the first group, in
  // flight with the outaged branches' flows; later groups' one group ahead
  double Fn = 0.0, Hn = 0.0, Mn = 0.0;
  uint64_t flags = 0;
  uint64_t* __restrict__ words = w.hot + (size_t)t * ng * a.rqs + kb;
  auto prefetch = [&](int g) {
    if (g < ng) {
      const int l = g * 64 + lane;
      Fn = Ft[l];
      Hn = Ht[l];
      if constexpr (ALL)
        flags = words[(size_t)g * a.rqs];
      else
        Mn = lmax[l];
    }
  };
  prefetch(wv);
  const R fk = (R)w.Fk[(size_t)t * p.Kp + (a.act_k ? a.act_k[k] : (int)k)];
  const double deps = w.params[PB_EPS];
  const double dkt = p.dt[t] * p.c_s * w.params[PB_BETA];
  const R eps = (R)deps, eps2 = eps * eps, kt = (R)dkt;
  const double fkm = wave_max(fabs((double)fk));
  // lane 0 stores R and lane 32 Q of a pair's first row, lanes 16 and 48
  // those of the second
  double* __restrict__ rq = w.rq + ((size_t)t * Lp * a.rqs + kb) * 2 + (lane >> 5);
  const double rqk = !kF64 ? 1.0 : lane < 32 ? dkt : 0.5 * dkt;
  for (int s = wv; s < a.nsl; s += nw) {
    double zacc = 0.0, sacc = 0.0;
    R zt = R(0), st = R(0);  // FP32 only: sums of the current eight branches
    int tile = -1;
    HotRow<R> pend;
    pend.l = -1;
    auto add = [&](const HotRow<R>& h, bool m, R z, R dP) {
      if constexpr (kF64) {
        zacc += z;
        sacc = m ? fma(h.lod, dP, sacc) : sacc;
      } else {
        if ((h.l >> 3) != tile) {
          zacc += (double)zt;
          sacc += (double)st;
          zt = st = R(0);
          tile = h.l >> 3;
        }
        zt += z;
        st = m ? fma(h.lod, dP, st) : st;
      }
    };
    auto flush = [&](const HotRow<R>& h0, const HotRow<R>& h1) {
      R z, p0, q0, p1 = R(0), q1 = R(0);
      const bool m0 = hot_eval(h0, eps, eps2, kt, z, p0, q0);
      add(h0, m0, z, p0);
      if (h1.l >= 0) {
        const bool m1 = hot_eval(h1, eps, eps2, kt, z, p1, q1);
        add(h1, m1, z, p1);
      }
      const R v = quad_sum(p0, q0, p1, q1);
      const int row = (lane & 16) ? h1.l : h0.l;
      if ((lane & 15) == 0 && row >= 0) rq[(size_t)row * a.rqs * 2] = (double)v * rqk;
    };
    if (s != wv) prefetch(s);
    for (int g = s; g < ng; g += a.nsl) {
      const int l = g * 64 + lane;
      const double F = Fn, H = Hn, M = Mn;
      const uint64_t known = flags;
      const double smx = p.ctg_smax[l];
      double q2 = H;
      if constexpr (kF64) q2 = w.q2[(size_t)t * Lp + l];
      prefetch(g + a.nsl);
      bool cold = false;
      if constexpr (ALL) {
        cold = !((known >> lane) & 1);
      } else if constexpr (kF64) {
        const double e = fabs(F) * (1.0 + 0x1p-40) - H * (1.0 - 0x1p-40);
        cold = fma(M, fkm, e) <= 0.0;
      } else {
        const double e = fma(M, fkm, fabs(F));
        cold = (e * e + q2) * (1.0 + 0x1p-18) <= smx * smx * (1.0 - 0x1p-18);
      }
      uint64_t und = __builtin_amdgcn_ballot_w64(l < L && !cold), hot = 0;
      while (und) {
        constexpr int U = 4;
        int r[U];
        R lod[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          r[u] = und ? __builtin_ctzll(und) : -1;
          und &= und - 1;  // 0 stays 0
          if (r[u] >= 0) lod[u] = lodf_load(lodf + (size_t)(g * 64 + r[u]) * a.kst, k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (r[u] < 0) break;
          HotRow<R> h;
          h.P = fma(lod[u], fk, (R)readlane_f64(F, r[u]));
          bool over;
          if constexpr (kF64) {
            over = fabs(h.P) > readlane_f64(H, r[u]);
          } else {
            const double m = readlane_f64(smx, r[u]);
            h.q2 = (R)readlane_f64(H, r[u]);
            h.smx2 = (R)(m * m);
            over = fma(h.P, h.P, h.q2) > h.smx2;
          }
          if (!ALL && __builtin_amdgcn_ballot_w64(over) == 0) continue;
          hot |= (uint64_t)1 << r[u];
          const double m = readlane_f64(smx, r[u]);
          h.smx = (R)m;
          if constexpr (kF64) {
            h.q2 = readlane_f64(q2, r[u]);
            h.smx2 = m * m;
          }
          h.lod = lod[u];
          h.l = g * 64 + r[u];
          if (pend.l < 0) {
            pend = h;
          } else {
            flush(pend, h);
            pend.l = -1;
          }
        }
      }
      if (!ALL && lane == 0) words[(size_t)g * a.rqs] = hot;
    }
    if (pend.l >= 0) {
      HotRow<R> none;
      none.l = -1;
      flush(pend, none);
    }
    lds[s * 128 + lane] = zacc + (double)zt;
    lds[s * 128 + 64 + lane] = sacc + (double)st;
  }
  __syncthreads();
  // z by the first wavefront, S by the second (or the first again)
  for (int half = wv; half < 2; half += nw) {
    double v = 0.0;
    for (int s = 0; s < a.nsl; ++s) v += lds[s * 128 + half * 64 + lane];
    if (half == 0)
      ctg_finish_z(a, kb, t, dkt, deps, v);
    else
      ctg_finish_s(a, kb, t, kF64 ? v * dkt : v);
  }
}

// Blocks (contingency block, period), XCD-grouped: the periods of one
// contingency block read the same factor rows through one L2.
template <typename LT, bool ALL>
__global__ __launch_bounds__(1024) void k_ctg_rows(EvalArgs a) {
  extern __shared__ double dyn[];
  ctg_rows_body<LT, ALL>(a, xcd_group(blockIdx.x, gridDim.x), dyn);
}

// The test of every row, where no bound is to decide any (lmax null): a block tests a
// group of 64 branches against 64 contingencies in several periods and stores the
// group's flags a period.  The factors are turned over through LDS, so that a lane
// holds a branch: it keeps the largest |P| of its row (NaN dropped), an FMA and a
// maximum an element with F_k by v_readlane, and the lanes' tests of that largest flow
// are the word.  With FP32 the test fl(P^2 + qmax2) > s_ctg^2 grows with |P|: the
// largest flow passes it if any does.
// WIDE: each wavefront takes kTestTp periods of its own; otherwise all take the same
// ones and a quarter of the contingencies each, for grids of few blocks or periods
// (2800 branches x 2 periods: a step of 43.0 us, 54.3 in wide blocks).
// Bound by the vector instructions.  With 2800 branches, 2432 contingencies and 48
// periods it takes 68 us (FP32 41), and k_ctg_rows then 21 (17); testing the rows one
// period and four rows at a time in k_ctg_rows took 190 (210).  Slower: F and radius
// by scalar loads and a lane a contingency, a compare and its ballot an element (70;
// FP32 by v_readlane 90).
constexpr int kTestTp = 4;     // periods of a wavefront
constexpr int kTestWaves = 4;  // wavefronts of a block
constexpr int test_periods(bool wide) { return wide ? kTestTp * kTestWaves : kTestTp; }

template <typename LT, bool WIDE>
__device__ __forceinline__ void ctg_test_block(const EvalArgs& a, int q, double* lds) {
  typedef typename std::conditional<std::is_same<LT, double>::value, double, float>::type R;
  constexpr bool kF64 = std::is_same<R, double>::value;
  constexpr int TP = kTestTp, kRow = 65;
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const LT* __restrict__ lodf = DevPtr<const LT>(static_cast<const LT*>(a.lodf_sel));
  const int lane = threadIdx.x & 63, T = p.T, Lp = p.Lp, ng = Lp >> 6;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntc = (T + test_periods(WIDE) - 1) / test_periods(WIDE);
  // period chunks of one tile side by side: they read the same factors
  const int kg = q / ntc, kb = kg / ng, g = kg - kb * ng;
  const int t0 = (q - kg * ntc) * test_periods(WIDE) + (WIDE ? wv * TP : 0);
  const unsigned k = (unsigned)(kb * 64 + lane);  // slot of the lane while loading
  R* tile = reinterpret_cast<R*>(lds);            // [64 branches][kRow]
  const LT* __restrict__ row = lodf + (size_t)(g * 64 + wv * 16) * a.kst;
  R in[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) in[j] = lodf_load(row + (size_t)j * a.kst, k);
  const int l = g * 64 + lane;  // branch of the lane
  const int kc = a.act_k ? a.act_k[k] : (int)k;
  R fk[TP], F[TP], m[TP];
  double H[TP];  // thr, or qmax2
#pragma unroll
  for (int i = 0; i < TP; ++i) {
    const size_t t = min(t0 + i, T - 1);  // periods past the last store nothing
    fk[i] = (R)w.Fk[t * p.Kp + kc];
    F[i] = (R)w.F[t * Lp + l];
    H[i] = (kF64 ? w.thr : w.q2)[t * Lp + l];
    m[i] = R(-1);
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) tile[(wv * 16 + j) * kRow + lane] = in[j];
  __syncthreads();
  const R* mine = tile + lane * kRow;
  const int k0 = WIDE ? 0 : wv * 16, k1 = WIDE ? 64 : k0 + 16;
#pragma unroll 8
  for (int kk = k0; kk < k1; ++kk) {
    const R lod = mine[kk];
#pragma unroll
    for (int i = 0; i < TP; ++i) m[i] = fmax(m[i], fabs(fma(lod, readlane_any(fk[i], kk), F[i])));
  }
  __syncthreads();
  if constexpr (!WIDE) {
    R* part = tile;  // [wavefront][TP][64]
#pragma unroll
    for (int i = 0; i < TP; ++i) part[(wv * TP + i) * 64 + lane] = m[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int u = 0; u < kTestWaves; ++u) m[i] = fmax(m[i], part[(u * TP + i) * 64 + lane]);
    __syncthreads();  // the next tile's factors overwrite them
  }
  float s2 = 0.f;
  if constexpr (!kF64) {
    const double r = p.ctg_smax[l];
    s2 = (float)(r * r);
  }
#pragma unroll
  for (int i = 0; i < TP; ++i) {
    bool over;
    if constexpr (kF64)
      over = m[i] > H[i];
    else
      over = m[i] >= 0.f && fmaf(m[i], m[i], (float)H[i]) > s2;
    const uint64_t word = __builtin_amdgcn_ballot_w64(over);
    if (t0 + i < T && lane == 0 && (WIDE || wv == 0))
      w.hot[((size_t)(t0 + i) * ng + g) * a.rqs + kb] = word;
  }
}

// lds: 64 x 65 factors.
template <typename LT, bool WIDE>
__device__ __forceinline__ void ctg_test_body(const EvalArgs& a, int b, double* lds) {
  const int n = a.nKb * (a.p.Lp >> 6) * ((a.p.T + test_periods(WIDE) - 1) / test_periods(WIDE));
  for (int q = b; q < n; q += a.ntest) ctg_test_block<LT, WIDE>(a, q, lds);
}

template <typename LT, bool WIDE>
__global__ __launch_bounds__(kTestWaves * 64) void k_ctg_test(EvalArgs a) {
  __shared__ double lds[64 * 65 * (std::is_same<LT, double>::value ? 2 : 1) / 2];
  ctg_test_body<LT, WIDE>(a, xcd_group(blockIdx.x, gridDim.x), lds);
}

// ---------------------------------------------------------------------------
// K4 (branch-stacked tile only): per-(t, k) penalties z_tk from the l-block
// partials, the mean outage-correction derivative, and per 64-contingency
// chunk the worst penalty and the sum.  One 64-thread block per (chunk, t).

__global__ __launch_bounds__(64) void k_ctg_zred(EvalArgs a) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int kc = blockIdx.x, t = blockIdx.y;
  const double kt = p.dt[t] * p.c_s * w.params[PB_BETA];
  const size_t o = (size_t)t * p.Kp + kc * 64 + threadIdx.x;
  const size_t stride = (size_t)p.T * p.Kp;
  // the l-block partials in l-block order, 16 of each in flight
  const double zs = strided_sum<16>(w.zpart + o, a.nLb, stride);
  const double ss = strided_sum<16>(w.spart + o, a.nLb, stride);
  ctg_finish_s(a, kc, t, ss);
  ctg_finish_z(a, kc, t, kt, w.params[PB_EPS], zs);
}

// ---------------------------------------------------------------------------
// K5: per-(t, l) adjoint of the flows: dL/dF_tl (transposed, the A operand of
// the adjoint product) and dL/dqmax2_tl, with weight 1/K for every
// contingency plus 1 for the worst of the period (Table 1's two contingency
// rows).  The worst contingency's own column is re-evaluated here; its
// outage-correction term S* = sum_l LODF_lk* dP_tlk* belongs to dL/dF at the
// outaged branch and is applied in k_final as a rank-1 term (per-chunk sums).

// OR of a 64-bit word over the 64 lanes of a wavefront, in every lane.
__device__ __forceinline__ uint64_t wave_or(uint64_t v) {
  unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
#define QG_OR_STEP(CTRL)                                                        \
  lo |= (unsigned)__builtin_amdgcn_mov_dpp((int)lo, CTRL, 0xF, 0xF, false);     \
  hi |= (unsigned)__builtin_amdgcn_mov_dpp((int)hi, CTRL, 0xF, 0xF, false);
  QG_OR_STEP(0xB1)   // quad_perm [1,0,3,2]
  QG_OR_STEP(0x4E)   // quad_perm [2,3,0,1]
  QG_OR_STEP(0x141)  // row_half_mirror
  QG_OR_STEP(0x140)  // row_mirror
#undef QG_OR_STEP
  uint64_t r = 0;
  for (int row = 0; row < 64; row += 16)
    r |= ((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)hi, row) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)lo, row);
  return r;
}

// R and Q of the wavefront's 64 branches (lane = branch l of period t) from
// the map-reduce's per-contingency-block sums.  Few branches hold any, and
// those that do mostly hold one in every block, so each is summed across the
// lanes (lane = contingency block, one 16-byte load each), four branches'
// loads in flight together (eight cost registers and a block per CU: 19.3 us
// against 17.2 in a batch of twelve grids, 7.1 against 6.5 at 617 buses).  mid()
// runs while the first branches' loads are in flight.
// hot: the lane's word of the first 64 contingency blocks (hot_word).
__device__ __forceinline__ uint64_t hot_word(const EvalArgs& a, int t, int g, int c) {
  const int ng = a.p.Lp >> 6;
  return g < ng && c < a.nKb ? a.w.hot[((size_t)t * ng + g) * a.rqs + c] : (uint64_t)0;
}
template <class Mid>
__device__ __forceinline__ void gather_rq(const EvalArgs& a, int t, int g, uint64_t hot, double& r,
                                          double& q, Mid mid) {
  constexpr int U = 4;
  const DevProblem& p = a.p;
  const int lane = threadIdx.x & 63;
  bool first = true;
  for (int c0 = 0; c0 < a.nKb; c0 += 64) {
    const uint64_t word = c0 == 0 ? hot : hot_word(a, t, g, c0 + lane);
    uint64_t any = wave_or(word);
    const double2* src = reinterpret_cast<const double2*>(+a.w.rq) +
                         ((size_t)t * p.Lp + g * 64) * a.rqs + c0 + lane;
    do {
      int row[U];
      double2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        row[u] = any ? __builtin_ctzll(any) : -1;
        any &= any - 1;  // 0 stays 0
        v[u] = double2{0.0, 0.0};
        if (row[u] >= 0 && ((word >> row[u]) & 1)) v[u] = src[(size_t)row[u] * a.rqs];
      }
      if (first) mid();
      first = false;
#pragma unroll
      for (int u = 0; u < U; u += 2) {
        if (row[u] < 0) break;
        const double s = quad_sum(v[u].x, v[u].y, v[u + 1].x, v[u + 1].y);
        const double r0 = readlane_f64(s, 0), r1 = readlane_f64(s, 16);
        const double q0 = readlane_f64(s, 32), q1 = readlane_f64(s, 48);
        if (lane == row[u]) {
          r += r0;
          q += q0;
        }
        if (lane == row[u + 1]) {
          r += r1;
          q += q1;
        }
      }
    } while (any);
  }
}

template <bool SPLIT>
__device__ void ctg_assemble(const EvalArgs& a, int t, int lc, double* red) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x;
  const int T = p.T, L = p.L, K = p.K, Lp = p.Lp, Kp = p.Kp, Tp = p.Tp;
  const double eps = w.params[PB_EPS], beta = w.params[PB_BETA];
  const double kt = p.dt[t] * p.c_s * beta;
  const int l = lc * kBlock + tid;
  const bool hasl = l < L;
  // independent loads first
  double r = 0.0, q = 0.0, Fl = 0.0, q2l = 0.0, sm2 = 0.0, sm = 0.0;
  int kk = -1;
  const size_t o = (size_t)t * Lp + l;
  if (hasl) {
    Fl = w.F[o];
    q2l = w.q2[o];
    sm2 = p.ctg_smax2[l];
    sm = p.ctg_smax[l];
    kk = p.kof[l];
  }
  double sacc[1] = {0.0};
  if (K > 0) {
    // per-chunk worst penalties and sums (chunk c0 + u in lane u), combined by
    // wavefront reductions (the argmax is a total order, the sum has a fixed
    // order) and followed by the worst contingency's factor and flow, all
    // while the k-block partials of R and Q are in flight.  Without
    // contingencies the partials were never written.
    const int lane = tid & 63;
    double zmax = -DBL_MAX, zsum = 0.0;
    int kstar = INT_MAX;
    const size_t ob = (size_t)t * a.nKc;
    double cz = -DBL_MAX, cs = 0.0;
    int ci = INT_MAX;
    if (lane < a.nKc) {
      cz = w.zmaxp[ob + lane];
      ci = (int)w.zargp[ob + lane];
      cs = w.zsump[ob + lane];
    }
    // the outaged branch's own factor is NaN: it never tests overloaded
    double lo = 0.0, fstar = 0.0, sm_k = 0.0;
    auto worst = [&]() {
      for (int c0 = 0; c0 < a.nKc; c0 += 64) {
        if (c0 > 0) {
          const int c = c0 + lane;
          cz = c < a.nKc ? w.zmaxp[ob + c] : -DBL_MAX;
          ci = c < a.nKc ? (int)w.zargp[ob + c] : INT_MAX;
          cs = c < a.nKc ? w.zsump[ob + c] : 0.0;
        }
        wave_argmax(cz, ci);
        const double ssum = wave_sum(cs);
        if (better(cz, ci, zmax, kstar)) { zmax = cz; kstar = ci; }
        zsum += ssum;
      }
      if (!(kstar >= 0 && kstar < K)) kstar = 0;  // NaN penalties: keep every index in range
      fstar = w.Fk[(size_t)t * Kp + kstar];
      if (hasl) {
        lo = lodf_value(p, l, kstar);
        const int sl = kk >= 0 && a.act_slot ? a.act_slot[kk] : kk;
        if (sl >= 0) sm_k = w.smean[(size_t)t * Kp + sl];
      }
    };
    if constexpr (SPLIT) {
      const int g = __builtin_amdgcn_readfirstlane(lc * (kBlock / 64) + (tid >> 6));
      gather_rq(a, t, g, hot_word(a, t, g, lane), r, q, worst);
    } else {
      worst();
      const size_t st = (size_t)T * Lp;
      if (hasl) {
        r = strided_sum<16>(w.rpart + o, a.nKb, st);
        q = strided_sum<16>(w.qpart + o, a.nKb, st);
      }
    }
    // weight of every scored contingency: 1/K for the mean (plus 1 for the
    // period's worst), or 1 for the plain sum
    const double invK = 1.0 / (double)K;
    const double wk = p.ctg_sum ? 1.0 : invK;
    if (hasl) {
      r *= wk;
      q *= wk;
      const double P = fma(lo, fstar, Fl);
      const double s2 = fma(P, P, q2l);
      if (!p.ctg_sum && s2 > sm2) {
        double dP, dq;
        ctg_overload(P, s2, sm, eps, eps * eps, kt, dP, dq);
        r += dP;
        q += dq;
        sacc[0] = lo * dP;
      }
      r += sm_k;
    }
    if (lc == 0 && tid == 0) {
      w.tpart[a.toff.cmax + t] = p.ctg_sum ? 0.0 : zmax;
      // contingencies not scored this step take their no-overload penalty
      const double rest = (double)(K - a.na) * (kt * ((double)(L - 1) * eps));
      w.tpart[a.toff.cmean + t] = (zsum + rest) * wk;
      w.kstar[t] = (double)kstar;
    }
  } else if (lc == 0 && tid == 0) {
    w.tpart[a.toff.cmax + t] = 0.0;
    w.tpart[a.toff.cmean + t] = 0.0;
    w.kstar[t] = 0.0;
  }
  if (l < Lp) {
    w.gfT[(size_t)l * Tp + t] = hasl ? r : 0.0;
    w.qtot[(size_t)t * Lp + l] = hasl ? q : 0.0;
  }
  block_sum<1>(sacc, red);
  if (tid == 0) w.smaxp[(size_t)t * a.nLc + lc] = sacc[0];
}

// Blocks [0, T nsl): the device terms of one period and one slice of 256
// generators each (period_block, with the step's parameters as the forward
// kernel resolved them; nsl slices per period); then nLc T blocks of flow
// adjoints of (period, 256-branch chunk); then the nb_bus power-balance
// blocks, which only need the forward flows.
template <bool SPLIT>
__device__ __forceinline__ void ctg_asm_body(const EvalArgs& a, int b, int nblocks,
                                             Pair* smem) {
  const int T = a.p.T, nasm = a.nLc * T;
  const int nsl = (a.p.G + kBlock - 1) / kBlock, nper = T * nsl;
  // scheduled steps: the next step's schedule row (the counter is advanced
  // by k_final, after this kernel), clamped to the table; a new table comes
  // with k_set_step, which copies its own row
  if (a.mode.schedule && b == nblocks - 1 && threadIdx.x < kSchedStride) {
    const int64_t s1 = min(a.w.step[0] + 1, (int64_t)kSchedCap - 1);
    a.w.snext[threadIdx.x] = a.w.sched[s1 * kSchedStride + threadIdx.x];
  }
  if (b < nper) {
    const StepParams sp{a.w.params[PB_EPS], a.w.params[PB_BETA], a.w.params[PB_RHO]};
    period_block(a, sp, b / nsl, b % nsl, reinterpret_cast<double*>(smem));
  } else if (b < nper + nasm) {
    // XCD-grouped: the blocks of consecutive periods store the transposed
    // flow adjoints gfT[l][t] of the same branches through one L2
    const int g = xcd_group(b - nper, nasm);
    ctg_assemble<SPLIT>(a, g / a.nLc, g % a.nLc, reinterpret_cast<double*>(smem));
  } else {
    bus_balance(a, b - nper - nasm, smem);
  }
}

template <bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_ctg_asm(EvalArgs a) {
  __shared__ Pair smem[kSegChunk];
  ctg_asm_body<SPLIT>(a, blockIdx.x, gridDim.x, smem);
}

// ---------------------------------------------------------------------------
// K6: adjoint DC product + branch reverse

// Adjoints (V, theta) of branch l's two ends in period t, at their bus-sorted
// slots.
__device__ __forceinline__ void branch_reverse(const EvalArgs& a, int t, int l, Pair* ge) {
  // FMAs inside an expression only: across statements the choice would depend on
  // where the function is inlined, and k_update and k_adjoint_b would round
  // differently
#pragma clang fp contract(on)
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int T = p.T, L = p.L, N = p.N;
  const size_t TL = (size_t)T * L, e = (size_t)t * L + l;
  const Pair trig = w.bco[e], kth = w.bco[TL + e], kq = w.bco[2 * TL + e];
  const int side = w.bside[e];
  const double cs = trig.x, sn = trig.y;
  const int f = p.br_from[l], o = p.br_to[l], sf = p.slot_fr[l], so = p.slot_to[l];
  const double vf = a.x[(size_t)t * N + f], vt = a.x[(size_t)t * N + o];
  const double Qc = w.qtot[(size_t)t * p.Lp + l];
  const bool th_to = side & kThermalTo, q_to = side & kReactiveTo;
  const double lpf = w.lamp[(size_t)t * N + f] + (th_to ? 0.0 : kth.x);
  const double lqf =
      w.lamq[(size_t)t * N + f] + (th_to ? 0.0 : kth.y) + Qc * (q_to ? 0.0 : kq.y);
  const double lpt = w.lamp[(size_t)t * N + o] + (th_to ? kth.x : 0.0);
  const double lqt =
      w.lamq[(size_t)t * N + o] + (th_to ? kth.y : 0.0) + Qc * (q_to ? kq.y : 0.0);
  const double g = p.br_g[l], b = p.br_b[l], bh = p.br_bh[l];
  const double A = -g * cs - b * sn;   // p_fr cross coefficient
  const double Bq = b * cs - g * sn;   // q_fr
  const double Ct = -g * cs + b * sn;  // p_to
  const double Dq = b * cs + g * sn;   // q_to
  const double gvf = lpf * (2.0 * g * vf + vt * A) + lqf * (-2.0 * (b + bh) * vf + vt * Bq) +
                     lpt * (vt * Ct) + lqt * (vt * Dq);
  const double gvt = lpf * (vf * A) + lqf * (vf * Bq) + lpt * (2.0 * g * vt + vf * Ct) +
                     lqt * (-2.0 * (b + bh) * vt + vf * Dq);
  const double vv = vf * vt;
  const double gd = kq.x + lpf * vv * (g * sn - b * cs) +
                    lqf * vv * (-b * sn - g * cs) + lpt * vv * (g * sn + b * cs) +
                    lqt * vv * (-b * sn + g * cs);
  ge[sf] = Pair{gvf, gd};
  ge[so] = Pair{gvt, -gd};
}

__device__ void reverse_block(const EvalArgs& a, int blk) {
  const DevProblem& p = a.p;
  const int idx = blk * kBlock + threadIdx.x;
  if (idx >= p.T * p.L) return;
  const int t = idx / p.L;
  branch_reverse(a, t, idx - t * p.L, a.w.epG + (size_t)t * p.twoL);
}

// Branches [k0, k1) of slice sp of the adjoint product's reduction.
__device__ __forceinline__ void adjoint_slice(const EvalArgs& a, int sp, int& k0, int& k1) {
  const int steps = a.p.Lp / 4;
  const int per = (steps + a.nsplit - 1) / a.nsplit;
  k0 = min(steps, sp * per) * 4;
  k1 = min(steps, (sp + 1) * per) * 4;
}

// Blocks [0, nslab * nsplit): the DC part of dL/dp, one 16-generator slab and
// one slice of the branch dimension each (partials summed in k_final); then
// nb_br branch-reverse blocks; then the worst outage's ISF rows.
__device__ __forceinline__ void adjoint_body(const EvalArgs& a, int bx, double* smem) {
  const DevProblem& p = a.p;
  const int nslab = p.G16 / 16;
  if (bx < nslab * a.nsplit) {
    // XCD-grouped: the slabs of one slice, which read the same rows of the
    // flow adjoints, mostly share an L2
    const int g = xcd_group(bx, nslab * a.nsplit);
    const int slab = g % nslab, sp = g / nslab;
    const int n0 = slab * 16;
    int k0, k1;
    adjoint_slice(a, sp, k0, k1);
    const int T = p.T, Tp = p.Tp, G16 = p.G16;
    double* out = a.w.gpdc + (size_t)sp * T * G16;
    const double* gfT = a.w.gfT;
    // rows past T of gfT are never written: they enter as zeros
    auto aload = [=](int k, int row) -> double {
      return row < T ? gfT[(size_t)k * Tp + row] : 0.0;
    };
    auto epi = [=](int row, int col, double v) {
      if (row < T) out[(size_t)row * G16 + col] = v;
    };
    mfma_slab_dispatch<8>(p.Tp / 16, aload, p.isf_ga, G16, k0, k1, n0, smem, epi);
    return;
  }
  const int b = bx - nslab * a.nsplit;
  if (b < a.nb_br) {
    reverse_block(a, xcd_group(b, a.nb_br));
    return;
  }
  // the worst outage's ISF row of each period (generator columns), for the
  // rank-1 outage-correction term that k_final adds to dL/dp
  const int idx = (b - a.nb_br) * kBlock + threadIdx.x;
  if (idx < p.T * p.G16) {
    const int t = idx / p.G16, j = idx - t * p.G16;
    const int bks = p.brk[(int)a.w.kstar[t]];
    a.w.isfk[idx] = p.isf_ga[(size_t)bks * p.G16 + j];
  }
}

__global__ __launch_bounds__(kBlock) void k_adjoint(EvalArgs a) {
  __shared__ double smem[kSlabLds];
  adjoint_body(a, blockIdx.x, smem);
}

// ---------------------------------------------------------------------------
// K7: bus reduce, generator assembly, gradient or fused Adam, terms

struct AdamCtx {
  double b1, b2, eps, bc1, bc2;
  int eps_num;
};

// x, m, v of one variable.  The loads of every variable a thread updates are
// issued before its first store: x, m and v may alias as far as the compiler
// knows, so a load after a store would wait for it.
struct AdamVar {
  double x, m, v;
};
__device__ __forceinline__ AdamVar adam_load(const double* x, const double* m, const double* v,
                                             size_t e) {
  return AdamVar{x[e], m[e], v[e]};
}
__device__ __forceinline__ void adam_store(double* x, double* m, double* v, size_t e,
                                           const AdamVar& s, double g, double lr, double lo,
                                           double hi, const AdamCtx& c) {
#pragma clang fp contract(on)  // as in branch_reverse
  const double mm = c.b1 * s.m + (1.0 - c.b1) * g;
  const double vv = c.b2 * s.v + (1.0 - c.b2) * g * g;
  const double mh = mm / c.bc1;
  const double vh = vv / c.bc2;
  const double num = c.eps_num ? mh + c.eps : mh;
  double xn = s.x - lr * num / (sqrt(vh) + c.eps);
  xn = fmin(fmax(xn, lo), hi);
  m[e] = mm;
  v[e] = vv;
  x[e] = xn;
}
__device__ __forceinline__ void adam_entry(double* x, double* m, double* v, size_t e, double g,
                                           double lr, double lo, double hi, const AdamCtx& c) {
  adam_store(x, m, v, e, adam_load(x, m, v, e), g, lr, lo, hi, c);
}

// Entry idx of q, r or u (cls 1, 2, 3).
__device__ __forceinline__ void final_qru(const EvalArgs& a, const AdamCtx& ac, int cls, int idx) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int t = idx / p.G, j = idx - t * p.G;
  const size_t TG = (size_t)p.T * p.G;
  const size_t e = 2 * (size_t)p.T * p.N + cls * TG + idx;
  double* xm = const_cast<double*>(+a.x);
  AdamVar sv{0.0, 0.0, 0.0};
  if (a.fuse_adam) sv = adam_load(xm, a.m, a.v, e);
  double g = w.gdev[cls * TG + idx], lo = 0.0, hi = 1.0;
  if (cls == 1) {
    lo = p.qmin[j];
    hi = p.qmax[j];
    g -= w.lamqg[idx];
  } else if (cls == 2) {
    hi = p.rmax[j];
    g -= w.drs[t];
  }
  if (a.fuse_adam)
    adam_store(xm, a.m, a.v, e, sv, g, w.params[PB_ALPHA + QG_C_P + cls], lo, hi, ac);
  else if (a.grad)
    a.grad[e] = g;
}

// The deterministic sums of the terms' partials, two of the eight a wavefront
// with all of a lane's loads in flight together (four wavefronts; others only
// pass the barrier), and the step counter.
__device__ __forceinline__ void final_terms(const EvalArgs& a, double* smem) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x, T = p.T, G = p.G;
  if (a.mode.schedule && tid == 255) w.step[0] = w.step[0] + 1;
  const TermOffsets& to = a.toff;
  const int lane = tid & 63, wv = min(tid >> 6, 3);
  const int ndev = T * ((G + kBlock - 1) / kBlock);  // device-term slices
  const int qa = wv == 0 ? QG_T_BR : wv == 1 ? QG_T_DEV : wv == 2 ? QG_T_BAL : QG_T_CTG_MAX;
  const int qb = wv == 0 ? QG_T_ANG : wv == 1 ? QG_T_PEN : wv == 2 ? QG_T_RSV : QG_T_CTG_MEAN;
  const int oa = wv == 0 ? to.br : wv == 1 ? to.dev : wv == 2 ? to.bal : to.cmax;
  const int ob = wv == 0 ? to.ang : wv == 1 ? to.pen : wv == 2 ? to.rsv : to.cmean;
  const int na = wv == 0 ? a.nb_br : wv == 1 ? ndev : wv == 2 ? a.nb_bus : T;
  const int nb = wv == 0 ? a.nb_br : wv == 1 ? ndev : T;
  const double sum = pair_sum(strided_sum<8>(w.tpart + oa + lane, (na - lane + 63) >> 6, 64),
                              strided_sum<8>(w.tpart + ob + lane, (nb - lane + 63) >> 6, 64));
  if (tid < 256 && (lane & 31) == 0) smem[lane == 0 ? qa : qb] = sum;
  __syncthreads();
  if (tid < QG_NTERMS) {
    double tot = smem[0];
    for (int q = 1; q < QG_T_LOADVAL; ++q) tot += smem[q];
    const double o = tid < QG_T_LOADVAL ? smem[tid] : tid == QG_T_LOADVAL ? p.vload : tot - p.vload;
    w.terms[tid] = o;
    if (a.terms_out) a.terms_out[tid] = o;
  }
}

__device__ __forceinline__ AdamCtx adam_ctx(const EvalArgs& a) {
  if (!a.fuse_adam) return AdamCtx{};
  return AdamCtx{a.mode.adam_b1,      a.mode.adam_b2,      a.mode.adam_eps,
                 a.w.params[PB_BC1], a.w.params[PB_BC2], a.mode.eps_in_num};
}

// Blocks [0, nb_bus): voltages and angles of one period's buses; then nb_gen
// blocks for each generator variable p, q, r, u (one variable a thread: four
// chains of Adam's divisions and roots in one thread took longer than every other
// block); then the sum of the terms.
__device__ __forceinline__ void final_body(const EvalArgs& a, int bx, Pair* smem) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x;
  const int T = p.T, N = p.N, G = p.G;
  const AdamCtx ac = adam_ctx(a);
  double* xm = const_cast<double*>(+a.x);
  if (bx < a.nb_bus) {
    const int t = bx / a.bus_chunks;
    const int c = bx - t * a.bus_chunks;
    const int i0 = c * kBlock;
    const int nbus = min(kBlock, N - i0);
    // the bus's Adam state, loaded while the endpoint sums are formed
    const int i = i0 + tid;
    const size_t ev = (size_t)t * N + i, et = (size_t)T * N + ev;
    const bool upd = a.fuse_adam && tid < nbus;
    const AdamVar sv = upd ? adam_load(xm, a.m, a.v, ev) : AdamVar{0.0, 0.0, 0.0};
    const AdamVar st = upd ? adam_load(xm, a.m, a.v, et) : AdamVar{0.0, 0.0, 0.0};
    const double vlo = upd ? p.vmin[i] : 0.0, vhi = upd ? p.vmax[i] : 0.0;
    double gsum[2];
    bus_segsum(w.epG + (size_t)t * p.twoL, p, i0, nbus, smem, gsum, []() {});
    if (tid < nbus) {
      if (a.fuse_adam) {
        adam_store(xm, a.m, a.v, ev, sv, gsum[0], w.params[PB_ALPHA + QG_C_V], vlo, vhi, ac);
        adam_store(xm, a.m, a.v, et, st, gsum[1], w.params[PB_ALPHA + QG_C_TH], -DBL_MAX, DBL_MAX,
                   ac);
      } else if (a.grad) {
        a.grad[ev] = gsum[0];
        a.grad[et] = gsum[1];
      }
    }
    return;
  }
  const int gb = bx - a.nb_bus;
  if (gb < 4 * a.nb_gen) {
    const int cls = gb / a.nb_gen;  // p, q, r, u
    const int idx = (gb - cls * a.nb_gen) * kBlock + tid;
    if (idx >= T * G) return;
    if (cls > 0) {
      final_qru(a, ac, cls, idx);
      return;
    }
    // dL/dp: device partials, balance multiplier, and the DC part: the MFMA
    // split partials plus the worst contingency's rank-1 term
    // S*_t (ISF[br(k*)][bus(j)] - rowsum/N).  Every single load first (the Adam
    // state too), then the partial sums.
    const int t = idx / G, j = idx - t * G;
    const size_t e = 2 * (size_t)T * N + idx;
    AdamVar sv{0.0, 0.0, 0.0};
    if (a.fuse_adam) sv = adam_load(xm, a.m, a.v, e);
    const double gd = w.gdev[idx], lg = w.lamg[idx], isk = w.isfk[(size_t)t * p.G16 + j];
    const double hi = p.pmax[j];
    const double smax = strided_sum<16>(w.smaxp + (size_t)t * a.nLc, a.nLc, 1);
    const double dc = strided_sum<16>(w.gpdc + (size_t)t * p.G16 + j, a.nsplit, (size_t)T * p.G16);
    const double g = gd - lg + fma(smax, isk, dc);
    if (a.fuse_adam)
      adam_store(xm, a.m, a.v, e, sv, g, w.params[PB_ALPHA + QG_C_P], 0.0, hi, ac);
    else if (a.grad)
      a.grad[e] = g;
    return;
  }
  final_terms(a, reinterpret_cast<double*>(smem));
}

__global__ __launch_bounds__(kBlock) void k_final(EvalArgs a) {
  __shared__ Pair smem[kSegChunk];
  final_body(a, blockIdx.x, smem);
}

// ---------------------------------------------------------------------------
// K6 and K7 in one launch, for grids whose step is bound by its launches: a
// period's branches and buses are one block's, so the end adjoints stay in LDS
// and the updates follow a barrier instead of a launch, and one block forms every
// slice of a p slab.  Sums have the order of k_adjoint and k_final: the results are
// bitwise theirs.

// Period t's voltages and angles: the branches' end adjoints to their slots in
// LDS, then each bus's segment in ascending slot order.  Only this block reads
// or writes the period's V and theta in this kernel.
__device__ __forceinline__ void update_period(const EvalArgs& a, const AdamCtx& ac, int t,
                                              Pair* ge) {
  const DevProblem& p = a.p;
  const int N = p.N, tid = threadIdx.x;
  double* xm = const_cast<double*>(+a.x);
  // the first buses' Adam state and segments, in flight with the branches
  const size_t TN = (size_t)p.T * N;
  AdamVar sv{0.0, 0.0, 0.0}, st{0.0, 0.0, 0.0};
  double vlo = 0.0, vhi = 0.0;
  int lo = 0, hi = 0;
  auto fetch = [&](int i) {
    if (i < N) {
      lo = p.bptr[i];
      hi = p.bptr[i + 1];
      if (a.fuse_adam) {
        const size_t ev = (size_t)t * N + i;
        sv = adam_load(xm, a.m, a.v, ev);
        st = adam_load(xm, a.m, a.v, TN + ev);
        vlo = p.vmin[i];
        vhi = p.vmax[i];
      }
    }
  };
  fetch(tid);
  for (int l = tid; l < p.L; l += kUpdateBlock) branch_reverse(a, t, l, ge);
  __syncthreads();
  for (int i = tid; i < N; i += kUpdateBlock) {
    const size_t ev = (size_t)t * N + i, et = TN + ev;
    double sum_v = 0.0, sum_t = 0.0;
    for (int s = lo; s < hi; ++s) {
      const Pair e = ge[s];
      sum_v += e.x;
      sum_t += e.y;
    }
    if (a.fuse_adam) {
      adam_store(xm, a.m, a.v, ev, sv, sum_v, a.w.params[PB_ALPHA + QG_C_V], vlo, vhi, ac);
      adam_store(xm, a.m, a.v, et, st, sum_t, a.w.params[PB_ALPHA + QG_C_TH], -DBL_MAX, DBL_MAX,
                 ac);
    } else if (a.grad) {
      a.grad[ev] = sum_v;
      a.grad[et] = sum_t;
    }
    fetch(i + kUpdateBlock);
  }
}

// p of 16 generators in 16 periods: every slice of the adjoint product, a quarter
// of a slice a wavefront as k_adjoint cuts them, then what k_final does.
__device__ __forceinline__ void update_slab(const EvalArgs& a, const AdamCtx& ac, int blk,
                                            double* smem) {
  const DevProblem& p = a.p;
  const DevWork& w = a.w;
  const int tid = threadIdx.x, lane = tid & 63, T = p.T, Tp = p.Tp, G = p.G, G16 = p.G16;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mtiles = Tp / 16;
  const int n0 = blk / mtiles * 16, r0 = blk % mtiles * 16;
  double* xm = const_cast<double*>(+a.x);
  // everything else of the thread's output first, in flight with the product
  const int j = n0 + (tid & 15), t = r0 + (lane >> 4) + 4 * (tid >> 6);
  const bool out = tid < 256 && t < T && j < G;
  const size_t idx = (size_t)t * G + j, e = 2 * (size_t)T * p.N + idx;
  AdamVar sv{0.0, 0.0, 0.0};
  double gd = 0.0, lg = 0.0, hi = 0.0, smax = 0.0, isk = 0.0;
  if (out) {
    if (a.fuse_adam) sv = adam_load(xm, a.m, a.v, e);
    gd = w.gdev[idx];
    lg = w.lamg[idx];
    hi = p.pmax[j];
    const int bks = p.brk[(int)w.kstar[t]];
    isk = p.isf_ga[(size_t)bks * G16 + j];
    smax = strided_sum<4>(w.smaxp + (size_t)t * a.nLc, a.nLc, 1);
  }
  const int kr = lane >> 4, cc = lane & 15;
  const bool row = r0 + cc < T;  // rows past T of gfT are never written: they enter as zeros
  const double* __restrict__ A = w.gfT + r0 + cc;
  const double* __restrict__ B = p.isf_ga + n0 + cc;
  for (int seg = wv; seg < 4 * a.nsplit; seg += kUpdateBlock / 64) {
    constexpr int NB = 8;
    int k0, k1;
    adjoint_slice(a, seg >> 2, k0, k1);
    const int steps = (k1 - k0) >> 2, q = seg & 3;
    const int s0 = (steps * q) >> 2, s1 = (steps * (q + 1)) >> 2;
    v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
    for (int st = s0; st < s1; st += NB) {
      double bb[NB], aa[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const bool in = st + u < s1;
        const int k = k0 + (st + u) * 4 + kr;
        bb[u] = in ? B[(size_t)k * G16] : 0.0;
        aa[u] = in && row ? A[(size_t)k * Tp] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (st + u < s1) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(aa[u], bb[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) smem[(seg * 4 + r) * 64 + lane] = acc[r];
  }
  __syncthreads();
  if (!out) return;
  double dc = 0.0;
  for (int sp = 0; sp < a.nsplit; ++sp) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) v += smem[(sp * 4 + q) * 256 + tid];
    w.gpdc[((size_t)sp * T + t) * G16 + j] = v;
    dc += v;
  }
  const double g = gd - lg + fma(smax, isk, dc);
  if (a.fuse_adam)
    adam_store(xm, a.m, a.v, e, sv, g, w.params[PB_ALPHA + QG_C_P], 0.0, hi, ac);
  else if (a.grad)
    a.grad[e] = g;
}

// Blocks [0, T): one period's voltages and angles each; then the p slabs, (G16 /
// 16) x (Tp / 16); then the blocks of q, r and u; then the terms.  Every block
// updates entries of x that no other block of the kernel reads.
__global__ __launch_bounds__(kUpdateBlock) void k_update(EvalArgs a) {
  extern __shared__ Pair dyn2[];
  double* smem = reinterpret_cast<double*>(dyn2);
  const DevProblem& p = a.p;
  const AdamCtx ac = adam_ctx(a);
  int bx = blockIdx.x;
  if (bx < p.T) {
    update_period(a, ac, bx, dyn2);
    return;
  }
  bx -= p.T;
  const int nslab = p.G16 / 16 * (p.Tp / 16);
  if (bx < nslab) {
    update_slab(a, ac, bx, smem);
    return;
  }
  bx -= nslab;
  const int TG = p.T * p.G, nb = (TG + kUpdateBlock - 1) / kUpdateBlock;
  if (bx < 3 * nb) {
    const int cls = 1 + bx / nb, idx = (bx - (cls - 1) * nb) * kUpdateBlock + threadIdx.x;
    if (idx < TG) final_qru(a, ac, cls, idx);
    return;
  }
  final_terms(a, smem);
}

// ---------------------------------------------------------------------------
// standalone Adam (qg_adam_step) and helpers

__global__ __launch_bounds__(kBlock) void k_adam(DevProblem p, double* x, double* m, double* v,
                                                 const double* g, double lr0, double lr1,
                                                 double lr2, double lr3, double lr4, double lr5,
                                                 AdamCtx ac) {
  const size_t TN = (size_t)p.T * p.N, TG = (size_t)p.T * p.G;
  const size_t n = 2 * TN + 4 * TG;
  const size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n) return;
  double lr, lo, hi;
  if (e < TN) {
    const int i = (int)(e % p.N);
    lr = lr0; lo = p.vmin[i]; hi = p.vmax[i];
  } else if (e < 2 * TN) {
    lr = lr1; lo = -DBL_MAX; hi = DBL_MAX;
  } else {
    const size_t r = e - 2 * TN;
    const int cls = (int)(r / TG);
    const int j = (int)((r - cls * TG) % p.G);
    switch (cls) {
      case 0: lr = lr2; lo = 0.0; hi = p.pmax[j]; break;
      case 1: lr = lr3; lo = p.qmin[j]; hi = p.qmax[j]; break;
      case 2: lr = lr4; lo = 0.0; hi = p.rmax[j]; break;
      default: lr = lr5; lo = 0.0; hi = 1.0; break;
    }
  }
  adam_entry(x, m, v, e, g[e], lr, lo, hi, ac);
}

__global__ void k_set_step(int64_t* step, int64_t value, const double* sched, double* snext) {
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) step[0] = value;
  if (threadIdx.x < kSchedStride) snext[threadIdx.x] = sched[value * kSchedStride + threadIdx.x];
}

__global__ void k_clear_flag(int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) flag[0] = 0;
}

__global__ __launch_bounds__(kBlock) void k_check_finite(const double* x, size_t n, int* flag) {
  const size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (e < n && !isfinite(x[e])) flag[0] = 1;
}

// ---------------------------------------------------------------------------
// launchers

template <typename LT>
void launch_ctg_main(int bl, dim3 grid, dim3 block, hipStream_t s, const EvalArgs& a,
                     const LT* lodf) {
  // sFk[tc][64] + z and S of every (period, wavefront, lane)
  const size_t lds = (size_t)a.tc * 64 * (1 + 2 * (block.x / 64)) * sizeof(double);
  switch (bl) {
    case 8: hipLaunchKernelGGL((k_ctg_main<8, LT>), grid, block, lds, s, a, lodf); break;
    case 16: hipLaunchKernelGGL((k_ctg_main<16, LT>), grid, block, lds, s, a, lodf); break;
    default: hipLaunchKernelGGL((k_ctg_main<32, LT>), grid, block, lds, s, a, lodf); break;
  }
}

// Blocks of k_ctg_test (which loop past 2^20 of them).
static int test_blocks(const Problem* pr, const EvalArgs& a, bool wide) {
  const int n = test_periods(wide);
  const int64_t tiles = (int64_t)a.nKb * (pr->Lp / 64) * ((pr->T + n - 1) / n);
  return (int)std::min<int64_t>(tiles, 1 << 20);
}
// Blocks that count for its wide form (half its wavefronts have a period), and whether
// they are four a CU.
static int wide_blocks(const Problem* pr, const EvalArgs& a) {
  return pr->T > test_periods(true) / 2 ? test_blocks(pr, a, true) : 0;
}
static bool test_wide(int64_t blocks) { return blocks >= 4 * 256; }

template <typename LT>
void launch_ctg(const Problem* pr, hipStream_t s, const EvalArgs& a, const LT* lodf) {
  const CtgTile& t = pr->tile;
  if (t.split) {
    if (!a.lmax) {
      EvalArgs b = a;
      const bool wide = test_wide(wide_blocks(pr, a));
      b.ntest = test_blocks(pr, a, wide);
      auto test = wide ? k_ctg_test<LT, true> : k_ctg_test<LT, false>;
      hipLaunchKernelGGL(test, dim3(b.ntest), dim3(kTestWaves * 64), 0, s, b);
    }
    auto rows = a.lmax ? k_ctg_rows<LT, false> : k_ctg_rows<LT, true>;
    hipLaunchKernelGGL(rows, dim3(a.nKb * pr->T), dim3(64 * a.nsl),
                       (size_t)a.nsl * 128 * sizeof(double), s, a);
    return;
  }
  launch_ctg_main(t.bl, dim3(pr->nLb, a.nKb, (pr->T + t.tc - 1) / t.tc), dim3(64 * t.wl), s, a,
                  lodf);
}

static EvalArgs make_args(const Problem* pr, const DevWork& w, const double* x, double* grad,
                          double* terms_out, const EvalMode& mode, int fuse_adam, double* m,
                          double* v) {
  EvalArgs a;
  a.p = pr->dp;
  a.w = w;
  a.x = x;
  a.grad = grad;
  a.terms_out = terms_out;
  a.m = m;
  a.v = v;
  a.mode = mode;
  a.fuse_adam = fuse_adam;
  a.nb_br = pr->nb_br;
  a.nb_bus = pr->nb_bus;
  a.bus_chunks = pr->bus_chunks;
  a.nb_gen = pr->nb_gen;
  a.nsplit = pr->nsplit;
  a.nLb = pr->nLb;
  a.nKb = pr->nKb;
  a.nKc = pr->nKc;
  a.nLc = pr->nLc;
  a.tc = pr->tile.tc;
  a.lt = pr->tile.lt;
  a.rqs = pr->nKb_max;
  a.toff = pr->toff;
  const Screen& sc = pr->scr;
  if (mode.screened) {
    a.act_k = sc.act_k;
    a.act_slot = sc.act_slot;
    a.na = sc.n_act;
    a.kst = sc.Ka;
    a.nKb = a.nKc = sc.Ka / kCtgLanes;
    a.lodf_sel = sc.lodf_act;
    a.lmax = pr->dp.lmax ? sc.lmax_act : nullptr;
  } else {
    a.act_k = nullptr;
    a.act_slot = nullptr;
    a.na = pr->K;
    a.kst = pr->Kp;
    const DevProblem& dp = pr->dp;
    a.lodf_sel = dp.lodf_kind == kLodfF64 ? (const void*)dp.lodf
                 : dp.lodf_kind == kLodfF32 ? (const void*)dp.lodf32 : (const void*)dp.lodf16;
    a.lmax = dp.lmax;
  }
  a.nsl = ctg_slices(*pr, a.nKb);
  a.ntest = 0;
  return a;
}

// Blocks of k_ctg_asm: the device-term slices, the flow-adjoint chunks and
// the bus-balance blocks.
static int asm_blocks(const Problem* pr) {
  return pr->T * ((pr->G + kBlock - 1) / kBlock) + pr->nLc * pr->T + pr->nb_bus;
}

// Whether the reverse pass and the update of a problem's own step are one
// kernel.  A launch and the loads it waits for cost 2 to 3 us, but a period's branches
// then come through one CU, at about 48 GB/s from the other XCDs' stores.  A step
// in one kernel and in two takes 16.5 and 18.5 us with 20 branches and 4 periods,
// 21.2 and 24.3 with 183 and 48, 24.2 and 26.4 with 420 and 24, 25.0 and 25.2 with 700
// and 12, 26.6 and 26.2 with 864 and 18, 43.6 and 39.1 with 1680 and 24.  A batch fills the
// chip with its problems and stays with two.
static bool one_update(const Problem* pr) { return pr->L <= kUpdateMaxL; }

// One kernel of the step, in stream order 0..kStages-1.
static void launch_stage(const Problem* pr, const EvalArgs& a, int stage, hipStream_t s) {
  switch (stage) {
    case 0:
      hipLaunchKernelGGL(k_forward, dim3(pr->nb_br + pr->T + pr->Lp / 16 * (pr->Tp / 16)),
                         dim3(kBlock), 0, s, a);
      break;
    case 1:
      if (pr->K > 0) {
        const int kind = pr->dp.lodf_kind;
        if (kind == kLodfF64)
          launch_ctg(pr, s, a, static_cast<const double*>(a.lodf_sel));
        else if (kind == kLodfF32)
          launch_ctg(pr, s, a, static_cast<const float*>(a.lodf_sel));
        else
          launch_ctg(pr, s, a, static_cast<const uint16_t*>(a.lodf_sel));
      }
      break;
    case 2:
      if (pr->K > 0 && a.nsl == 0)  // k_ctg_rows finishes z itself
        hipLaunchKernelGGL(k_ctg_zred, dim3(a.nKc, pr->T), dim3(64), 0, s, a);
      break;
    case 3:
      if (a.nsl > 0)
        hipLaunchKernelGGL(k_ctg_asm<true>, dim3(asm_blocks(pr)), dim3(kBlock), 0,
                           s, a);
      else
        hipLaunchKernelGGL(k_ctg_asm<false>, dim3(asm_blocks(pr)), dim3(kBlock), 0,
                           s, a);
      break;
    case 4:
      if (one_update(pr)) break;  // k_update does both stages' work
      hipLaunchKernelGGL(k_adjoint,
                         dim3(pr->G16 / 16 * pr->nsplit + pr->nb_br +
                              (pr->T * pr->G16 + kBlock - 1) / kBlock),
                         dim3(kBlock), 0,
                         s, a);
      break;
    default:
      if (one_update(pr)) {
        // a period's end adjoints, or a slab's partial tiles
        const size_t lds = sizeof(double) * std::max(4 * (size_t)pr->L, 4 * (size_t)pr->nsplit * 256);
        const int nb = (pr->T * pr->G + kUpdateBlock - 1) / kUpdateBlock;
        hipLaunchKernelGGL(k_update, dim3(pr->T + pr->G16 / 16 * (pr->Tp / 16) + 3 * nb + 1),
                           dim3(kUpdateBlock), lds, s, a);
        break;
      }
      hipLaunchKernelGGL(k_final, dim3(pr->nb_bus + 4 * pr->nb_gen + 1), dim3(kBlock), 0, s,
                         a);
      break;
  }
}

int launch_eval(const Problem* pr, const DevWork& w, const double* x, double* grad,
                double* terms_out, const EvalMode& mode, int fuse_adam, double* m, double* v,
                void* stream, void** events) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const EvalArgs a = make_args(pr, w, x, grad, terms_out, mode, fuse_adam, m, v);
  for (int i = 0; i < kStages; ++i) {
    if (events) (void)hipEventRecord(static_cast<hipEvent_t>(events[i]), s);
    launch_stage(pr, a, i, s);
  }
  if (events) (void)hipEventRecord(static_cast<hipEvent_t>(events[kStages]), s);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched step: the same stages for many independent problems, one launch
// per stage.  A block finds its problem and its block of that problem in the
// stage's table (one scalar load); the kernel arguments of every problem sit
// in the batch buffer.  Each problem's blocks do exactly what they do in a
// launch of its own, so a batched step gives bitwise the points of the
// problems' own steps.

__device__ __forceinline__ void batch_entry(const uint32_t* __restrict__ tab, uint32_t i, int& s,
                                            int& loc) {
  const uint32_t e = tab[i];
  s = (int)(e >> kBatchLocBits);
  loc = (int)(e & ((1u << kBatchLocBits) - 1u));
}

__global__ __launch_bounds__(kBlock) void k_forward_b(const EvalArgs* __restrict__ args,
                                                      const uint32_t* __restrict__ tab) {
  __shared__ double smem[kFwdLds];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  forward_body(args[s], b, smem);
}

// Batched row-compacted map-reduce: each wavefront takes slices of its block's
// (period, contingency block) in turn; the sums are added in slice order, as in
// a launch of the problem's own.
// ALL: a problem of the batch has every row tested.
template <typename LT, bool ALL>
__global__ __launch_bounds__(kCtgSlices * 64) void k_ctg_rows_b(const EvalArgs* __restrict__ args,
                                                                const uint32_t* __restrict__ tab) {
  extern __shared__ double dyn[];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  const EvalArgs& a = args[s];
  b = xcd_group(b, a.nKb * a.p.T);
  if (ALL && !a.lmax)
    ctg_rows_body<LT, true>(a, b, dyn);
  else
    ctg_rows_body<LT, false>(a, b, dyn);
}

template <typename LT, bool WIDE>
__global__ __launch_bounds__(kTestWaves * 64) void k_ctg_test_b(const EvalArgs* __restrict__ args,
                                                                const uint32_t* __restrict__ tab) {
  __shared__ double lds[64 * 65 * (std::is_same<LT, double>::value ? 2 : 1) / 2];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  ctg_test_body<LT, WIDE>(args[s], b, lds);
}

__global__ __launch_bounds__(kBlock) void k_ctg_asm_b(const EvalArgs* __restrict__ args,
                                                      const uint32_t* __restrict__ tab) {
  __shared__ Pair smem[kSegChunk];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  const EvalArgs& a = args[s];
  ctg_asm_body<true>(a, b, a.p.T * ((a.p.G + kBlock - 1) / kBlock) + a.nLc * a.p.T + a.nb_bus,
                     smem);
}

// Four blocks per CU (two registers fewer than the compiler would take): 14.7 us
// against 15.2 for twelve grids; with five it spills, 19.2.
__global__ __launch_bounds__(kBlock, 4) void k_adjoint_b(const EvalArgs* __restrict__ args,
                                                      const uint32_t* __restrict__ tab) {
  __shared__ double smem[kSlabLds];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  adjoint_body(args[s], b, smem);
}

__global__ __launch_bounds__(kBlock) void k_final_b(const EvalArgs* __restrict__ args,
                                                    const uint32_t* __restrict__ tab) {
  __shared__ Pair smem[kSegChunk];
  int s, b;
  batch_entry(tab, blockIdx.x, s, b);
  final_body(args[s], b, smem);
}

// Blocks of each stage of one problem.
static void stage_blocks(const Problem* pr, const EvalArgs& a, int out[kStages]) {
  out[0] = pr->nb_br + pr->T + pr->Lp / 16 * (pr->Tp / 16);
  out[1] = pr->K > 0 ? a.nKb * pr->T : 0;
  out[2] = a.ntest;  // k_ctg_test, before stage 1 (k_ctg_rows finishes z itself)
  out[3] = asm_blocks(pr);
  out[4] = pr->G16 / 16 * pr->nsplit + pr->nb_br + (pr->T * pr->G16 + kBlock - 1) / kBlock;
  out[5] = pr->nb_bus + 4 * pr->nb_gen + 1;
}

static size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

int plan_batch(const Problem* const* prs, const DevWork* ws, int n, const double* const* x,
               double* const* m, double* const* v, const EvalMode& mode, BatchPlan* plan,
               std::vector<unsigned char>* image, std::string* err) {
  BatchPlan P;
  P.n = n;
  std::vector<EvalArgs> args((size_t)n);
  std::vector<std::array<int, kStages>> nb((size_t)n);
  int64_t wide = 0;  // blocks of k_ctg_test's wide form
  for (int i = 0; i < n; ++i) {
    const EvalArgs a = make_args(prs[i], ws[i], x[i], nullptr, nullptr, mode, 1, m[i], v[i]);
    if (prs[i]->K > 0 && !a.lmax) wide += wide_blocks(prs[i], a);
  }
  P.test_wide = test_wide(wide);
  for (int i = 0; i < n; ++i) {
    const Problem* pr = prs[i];
    const CtgTile& t = pr->tile;
    if (pr->K > 0 && !(t.split && t.wl == kBatchWl && t.tc == kBatchTcw)) {
      *err = "problem " + std::to_string(i) +
             ": the batched step needs a period-split tile of 4 wavefronts of 4 periods";
      return 1;
    }
    if (pr->scr.on) {
      *err = "problem " + std::to_string(i) + ": screening is not supported in a batch";
      return 1;
    }
    if (i > 0 && pr->dp.lodf_kind != prs[0]->dp.lodf_kind) {
      *err = "every problem of a batch needs the same storage of the outage factors";
      return 1;
    }
    args[i] = make_args(pr, ws[i], x[i], nullptr, nullptr, mode, 1, m[i], v[i]);
    if (pr->K > 0 && !args[i].lmax) args[i].ntest = test_blocks(pr, args[i], P.test_wide);
    int b[kStages];
    stage_blocks(pr, args[i], b);
    for (int q = 0; q < kStages; ++q) {
      if (b[q] >= (1 << kBatchLocBits)) {
        *err = "problem " + std::to_string(i) + " has too many blocks for a batch";
        return 1;
      }
      nb[i][q] = b[q];
      P.nblk[q] += b[q];
    }
  }
  P.lodf_kind = n > 0 ? prs[0]->dp.lodf_kind : 0;
  size_t o = 0;
  P.off_args = o;
  o = align_up(o + (size_t)n * sizeof(EvalArgs));
  for (int q = 0; q < kStages; ++q) {
    P.off_tab[q] = o;
    o = align_up(o + (size_t)P.nblk[q] * sizeof(uint32_t));
  }
  P.bytes = o;
  if (image) {
    image->assign(P.bytes, 0);
    std::memcpy(image->data() + P.off_args, args.data(), (size_t)n * sizeof(EvalArgs));
    // map-reduce blocks: problems by decreasing work per block (branches)
    std::vector<int> order((size_t)n);
    for (int i = 0; i < n; ++i) order[i] = i;
    auto item_work = [&](int i) { return prs[i]->Lp; };
    std::stable_sort(order.begin(), order.end(),
                     [&](int a2, int b2) { return item_work(a2) > item_work(b2); });
    for (int q = 0; q < kStages; ++q) {
      uint32_t* tab = reinterpret_cast<uint32_t*>(image->data() + P.off_tab[q]);
      size_t k = 0;
      for (int j = 0; j < n; ++j) {
        const int i = q == 1 ? order[j] : j;
        for (int b = 0; b < nb[i][q]; ++b)
          tab[k++] = ((uint32_t)i << kBatchLocBits) | (uint32_t)b;
      }
    }
  }
  for (int i = 0; i < n; ++i) P.nsl = std::max(P.nsl, args[i].nsl);
  // Four wavefronts a block of the map-reduce, more only while the chip (28 a
  // CU) has room for them: a block of few hands its place on sooner, and a small
  // batch needs them to fill the chip.  Twelve grids (4414 blocks): 39 us a step
  // with 3 or 4, 47 with 2, 5 or 8, 56 with 12.
  P.row_waves = 4;
  while (2 * P.row_waves <= kCtgSlices && (int64_t)P.nblk[1] * 2 * P.row_waves <= 28 * 256)
    P.row_waves *= 2;
  *plan = P;
  return 0;
}

int launch_eval_batch(const BatchPlan& P, void* d_buf, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned char* b = static_cast<unsigned char*>(d_buf);
  const EvalArgs* args = reinterpret_cast<const EvalArgs*>(b + P.off_args);
  auto tab = [&](int q) { return reinterpret_cast<const uint32_t*>(b + P.off_tab[q]); };
  hipLaunchKernelGGL(k_forward_b, dim3(P.nblk[0]), dim3(kBlock), 0, s, args, tab(0));
  if (P.nblk[1] > 0) {
    const size_t lds = (size_t)P.nsl * 128 * sizeof(double);
    const dim3 g(P.nblk[1]), blk(P.row_waves * 64);
    auto go = [&](auto test, auto all, auto rows) {
      if (P.nblk[2] > 0)
        hipLaunchKernelGGL(test, dim3(P.nblk[2]), dim3(kTestWaves * 64), 0, s, args, tab(2));
      hipLaunchKernelGGL(P.nblk[2] > 0 ? all : rows, g, blk, lds, s, args, tab(1));
    };
    if (P.lodf_kind == kLodfF64)
      go(P.test_wide ? k_ctg_test_b<double, true> : k_ctg_test_b<double, false>,
         k_ctg_rows_b<double, true>, k_ctg_rows_b<double, false>);
    else if (P.lodf_kind == kLodfF32)
      go(P.test_wide ? k_ctg_test_b<float, true> : k_ctg_test_b<float, false>,
         k_ctg_rows_b<float, true>, k_ctg_rows_b<float, false>);
    else
      go(P.test_wide ? k_ctg_test_b<uint16_t, true> : k_ctg_test_b<uint16_t, false>,
         k_ctg_rows_b<uint16_t, true>, k_ctg_rows_b<uint16_t, false>);
  }
  hipLaunchKernelGGL(k_ctg_asm_b, dim3(P.nblk[3]), dim3(kBlock), 0, s, args, tab(3));
  hipLaunchKernelGGL(k_adjoint_b, dim3(P.nblk[4]), dim3(kBlock), 0, s, args, tab(4));
  hipLaunchKernelGGL(k_final_b, dim3(P.nblk[5]), dim3(kBlock), 0, s, args, tab(5));
  return (int)hipGetLastError();
}

int time_stage(const Problem* pr, const DevWork& w, const double* x, const EvalMode& mode,
               int stage, int reps, void* stream, double* mean_ms) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const EvalArgs a = make_args(pr, w, x, nullptr, nullptr, mode, 0, nullptr, nullptr);
  for (int i = 0; i < kStages; ++i) launch_stage(pr, a, i, s);  // inputs of every stage
  hipEvent_t e0, e1;
  hipError_t err = hipEventCreate(&e0);
  if (err != hipSuccess) return (int)err;
  err = hipEventCreate(&e1);
  if (err != hipSuccess) { (void)hipEventDestroy(e0); return (int)err; }
  launch_stage(pr, a, stage, s);  // warm
  (void)hipEventRecord(e0, s);
  for (int r = 0; r < reps; ++r) launch_stage(pr, a, stage, s);
  (void)hipEventRecord(e1, s);
  err = hipEventSynchronize(e1);
  float ms = 0.f;
  if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (err != hipSuccess) return (int)err;
  *mean_ms = (double)ms / reps;
  return (int)hipGetLastError();
}

int launch_adam(const Problem* pr, double* x, double* m, double* v, const double* g,
                const double lr[QG_NCLASS], double bc1, double bc2, double b1, double b2,
                double eps, int eps_in_num, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  AdamCtx ac{b1, b2, eps, bc1, bc2, eps_in_num};
  const int nb = (int)((pr->n_x + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_adam, dim3(nb), dim3(kBlock), 0, s, pr->dp, x, m, v, g, lr[0], lr[1],
                     lr[2], lr[3], lr[4], lr[5], ac);
  return (int)hipGetLastError();
}

int launch_set_step(const Problem* pr, const DevWork& w, int64_t value, void* stream) {
  (void)pr;
  if (value < 0 || value >= kSchedCap) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_set_step, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                     w.step, value, (const double*)w.sched, w.snext);
  return (int)hipGetLastError();
}

int launch_check_finite(const Problem* pr, const double* x, int* flag, void* stream) {
  const int nb = (int)((pr->n_x + kBlock - 1) / kBlock);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(64), 0, s, flag);
  hipLaunchKernelGGL(k_check_finite, dim3(nb), dim3(kBlock), 0, s, x, (size_t)pr->n_x, flag);
  return (int)hipGetLastError();
}

}  // namespace qg
