// Multilayer perceptron of the learned warm start (qg_mlp.h): FP32 training
// on MFMA (v_mfma_f32_16x16x4f32) and BF16 inference (v_mfma_f32_16x16x32_bf16
// with FP32 accumulation), GELU activations, mean squared error, Adam.
//
// FP32 products of the batch with a weight matrix are one kernel (k_product),
// the weight gradients another (k_dw), which carries the bias gradient and, in a
// training step, the Adam update and the loss; the BF16 products are a third
// (k_gemm_bf16).  Where an output has few tiles grid.z splits the reduction
// dimension: the blocks write raw sums and k_reduce_epi adds the slices in a
// fixed order and applies the layer's epilogue (bias, GELU, GELU derivative, BF16
// rounding); otherwise the product applies it itself.  No floating-point
// atomics: results are bitwise reproducible.
//
// MFMA operand layouts (gfx950): lane l holds A[l%16][KPL*(l/16) + i] and
// B[KPL*(l/16) + i][l%16] for i < KPL (KPL = 1 for FP32, 8 for BF16); the
// 16 x 16 result sits at D[4*(l/16) + r][l%16] in register r of lane l.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>

#include "qg_internal.h"
#include "qg_mlp.h"

namespace qg {
qg_status fail(qg_status s, const std::string& msg);
}

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kT = 64;        // output tile edge
constexpr int kBK = 32;       // reduction depth of a k-step
constexpr int kThreads = 256;
constexpr int kGemm = 512;    // threads of a product's block: wavefronts of 32 x 16 outputs
constexpr int kEl = kT * kBK / kGemm;  // elements of each operand per thread and k-step

enum Epi { kStore = 0, kBiasGelu = 1, kBias = 2, kGeluBwd = 3, kBiasGeluBf16 = 4, kMse = 5 };

__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
// d gelu / dz = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_d(float z) {
  const float phi = 0.39894228040143268f * expf(-0.5f * z * z);
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * phi;
}
// FP32 -> BF16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const unsigned u = __float_as_uint(f);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((unsigned)h << 16); }

// What happens to the sum s of output element e (column n) of a product.
struct EpiArgs {
  int kind;
  const float* bias;       // [N], or null
  const uint16_t* bias16;  // [N] BF16 biases, widened, when bias is null
  float* z;                // kBiasGelu: pre-activation out; kGeluBwd: pre-activation in
  float* out;              // float result
  uint16_t* out16;         // kBiasGeluBf16
  const float* t;          // kMse: targets; out receives d loss / d y
  float inv;               // kMse: 1 / (M N)
  float* loss_part;        // kMse: one partial sum of squares per block
};

// Its column's bias and stored pre-activation are read ahead of the sum.
struct Aux {
  float b, z;
};
__device__ __forceinline__ Aux epi_aux(const EpiArgs& ep, size_t e, int n) {
  return {ep.bias ? ep.bias[n] : ep.bias16 ? from_bf16(ep.bias16[n]) : 0.f,
          ep.kind == kGeluBwd ? ep.z[e] : 0.f};
}
__device__ __forceinline__ void epilogue(const EpiArgs& ep, size_t e, const Aux& x, float s) {
  switch (ep.kind) {
    case kBiasGelu: {
      const float z = s + x.b;
      ep.z[e] = z;
      ep.out[e] = gelu(z);
      break;
    }
    case kBias: ep.out[e] = s + x.b; break;
    case kGeluBwd: ep.out[e] = s * gelu_d(x.z); break;
    case kBiasGeluBf16: ep.out16[e] = to_bf16(gelu(s + x.b)); break;
    default: ep.out[e] = s; break;
  }
}

// Sum of one value per thread of a block of N, by a tree in a fixed order (in
// thread 0); red holds N floats.
template <int N>
__device__ __forceinline__ float block_tree(float v, float* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = N / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  return red[0];
}

// The bytes of a matrix from base on; loads at or past the end return 0.  As a raw
// buffer the address of a load is base + the lane's 32-bit offset; the view of an
// operand moves with the k-step, so that the lanes' offsets are the same in every step
// and the loop needs no address arithmetic.  FAR: for tiles whose rows span more
// than the 4 GiB of such an offset (rows_far), with 64-bit offsets.
template <bool FAR>
struct View {
  typedef unsigned Off;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ View(const void* base, int64_t bytes) {
    const int hi = (int)(bytes >> 32);
    const uint32_t n = hi < 0 ? 0u : hi > 0 ? 0xFFFFFFFFu : (uint32_t)bytes;
    r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)n, 0x00020000);
  }
  __device__ __forceinline__ float f32(Off o) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
  }
  __device__ __forceinline__ v4f f32x4(Off o) const {
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
  }
  __device__ __forceinline__ unsigned u32(Off o) const {
    return __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
  }
  __device__ __forceinline__ unsigned u16(Off o) const {
    return __builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0);
  }
};
template <>
struct View<true> {
  typedef uint64_t Off;
  const char* base;
  int64_t bytes;
  __device__ __forceinline__ View(const void* b, int64_t n)
      : base(static_cast<const char*>(b)), bytes(n) {}
  template <typename T>
  __device__ __forceinline__ T get(Off o) const {
    return (int64_t)(o + sizeof(T)) <= bytes ? *reinterpret_cast<const T*>(base + o) : T(0);
  }
  __device__ __forceinline__ float f32(Off o) const { return get<float>(o); }
  __device__ __forceinline__ v4f f32x4(Off o) const {
    return v4f{f32(o), f32(o + 4), f32(o + 8), f32(o + 12)};
  }
  __device__ __forceinline__ unsigned u32(Off o) const { return get<unsigned>(o); }
  __device__ __forceinline__ unsigned u16(Off o) const { return get<uint16_t>(o); }
};
// View of the k-step at k0 of an operand X[r][k] (rows of ld elements, r from
// r0 of R, k contiguous) or X[k][r] (k < ke; ROWK).
template <bool ROWK, bool FAR, typename T>
__device__ __forceinline__ View<FAR> operand(const T* X, int ld, int R, int r0, int k0, int ke) {
  const int64_t at = ROWK ? (int64_t)k0 * ld + r0 : (int64_t)r0 * ld + k0;
  return View<FAR>(X + at, ((ROWK ? (int64_t)ke * ld : (int64_t)R * ld) - at) * (int64_t)sizeof(T));
}
// Whether a tile of rows rows of ld elements of 4 bytes (less is on the safe side)
// has offsets past 32 bits.
inline bool rows_far(int rows, int ld) { return (int64_t)rows * ld > (int64_t)1 << 30; }

// FP32 tile product with the reduction over the operands' rows: acc = the
// 64 x 64 tile at (m0, n0) of A^T B, A [K][M] and B [K][N], over the range [kb, ke).
// The operands of the next kDepth 32-deep k-steps are in flight in registers
// while the current one is multiplied from one of two LDS buffers (one barrier
// per k-step: a buffer is refilled only after every wavefront has passed the
// barrier that follows its last use).  Past the end of the reduction both
// operands read zeros; rows and columns past the matrix only reach outputs that
// are not stored.
constexpr int kDepth = 2;
// Both operands sit in LDS with k contiguous: lane l takes k = 8 (l/16) .. + 7 of
// its row in two 16-byte reads, and the q-th of the k-step's eight MFMAs
// multiplies everyone's q-th element (which k a lane multiplies when does not
// matter as long as A and B agree).  Rows are kPitch floats apart: 16-byte
// aligned, and 16 rows cover every bank once.
constexpr int kPitch = kBK + 4;
struct alignas(16) TileLds {
  float a[2][kT][kPitch];  // [m][k]
  float b[2][kT][kPitch];  // [n][k]
};

template <bool FAR>
struct Tile {
  typedef typename View<FAR>::Off Off;
  float ra[kDepth][kEl], rb[kDepth][kEl];
  Off oa[kEl], ob[kEl];  // byte offsets in the operands' views
  // element e of a k-step's operand: row (or column) e % 64, k = e / 64
  __device__ __forceinline__ void load(int d, const View<FAR>& va, const View<FAR>& vb) {
#pragma unroll
    for (int q = 0; q < kEl; ++q) ra[d][q] = va.f32(oa[q]);
#pragma unroll
    for (int q = 0; q < kEl; ++q) rb[d][q] = vb.f32(ob[q]);
  }
  __device__ __forceinline__ void put(int d, TileLds& s, int buf) {
#pragma unroll
    for (int q = 0; q < kEl; ++q) {
      const int e = threadIdx.x + q * kGemm;
      s.a[buf][e & 63][e >> 6] = ra[d][q];
      s.b[buf][e & 63][e >> 6] = rb[d][q];
    }
  }
  // ahead(): called once the first k-steps' loads are issued; step(buf): after the
  // barrier of every k-step with its LDS buffer, before its products
  template <class Ahead, class Step>
  __device__ __forceinline__ void run(const float* __restrict__ A, int lda,
                                      const float* __restrict__ B, int ldb, int M, int N, int kb,
                                      int ke, int m0, int n0, TileLds& s, v4f (&acc)[2],
                                      Ahead ahead, Step step) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = (wv >> 2) * 32, wn = (wv & 3) * 16;
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kEl; ++q) {
      const int e = threadIdx.x + q * kGemm;
      oa[q] = ((Off)(e >> 6) * lda + (e & 63)) * 4u;
      ob[q] = ((Off)(e >> 6) * ldb + (e & 63)) * 4u;
    }
    auto fetch = [&](int d, int k0) {
      load(d, operand<true, FAR>(A, lda, M, m0, k0, ke), operand<true, FAR>(B, ldb, N, n0, k0, ke));
    };
#pragma unroll
    for (int d = 0; d < kDepth; ++d) fetch(d, kb + d * kBK);
    ahead();
    __builtin_amdgcn_sched_barrier(0);
    // the loads stay ahead of the products, and a k-step's LDS reads ahead of
    // its first product (a wavefront or two per SIMD do not hide them)
    auto step1 = [&](int d, int buf, int k0) {
      put(d, s, buf);
      __syncthreads();
      fetch(d, k0 + kDepth * kBK);
      step(buf);
      v4f a[2][2], b[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = lane & 15, k = 8 * (lane >> 4) + 4 * h;
#pragma unroll
        for (int i = 0; i < 2; ++i)
          a[i][h] = *reinterpret_cast<const v4f*>(&s.a[buf][wm + i * 16 + r][k]);
        b[h] = *reinterpret_cast<const v4f*>(&s.b[buf][wn + r][k]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][q >> 2][q & 3], b[q >> 2][q & 3],
                                                        acc[i], 0, 0, 0);
    };
    // whole rounds of kDepth k-steps (zeros past the end): a way out between
    // two of them would let the compiler move the loads behind it
    static_assert(kDepth == 2, "one LDS buffer per k-step of a round");
    int k0 = kb;
    auto round = [&]() {
#pragma unroll
      for (int d = 0; d < kDepth; ++d, k0 += kBK) step1(d, d, k0);
    };
    round();  // apart from the loop: its waits do not count ahead()'s loads
    while (k0 < ke) round();
  }
};

// f(row, col, value) for the thread's 8 elements of a 64 x 64 tile at (m0, n0)
// that lie inside the matrix.
template <class F>
__device__ __forceinline__ void tile_elements(const v4f (&acc)[2], int m0, int n0, int M, int N,
                                              F f) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = (wv >> 2) * 32, wn = (wv & 3) * 16;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + wm + i * 16 + 4 * (lane >> 4) + r, col = n0 + wn + (lane & 15);
      if (row < M && col < N) f(row, col, acc[i][r]);
    }
}

// C = A op(B) for a product whose operands are read once or nearly so (batch
// rows against a weight matrix): A [M][K] row-major, op(B) = B [K][N] (TB = 0) or
// B [N][K] transposed (TB = 1).  A block of four wavefronts (eight where MI = 1)
// computes a tile of 16 MI x 64 outputs; its wavefronts take the 16-deep steps of
// the block's reduction slice in turn, each holding the whole tile, and are
// added through LDS at the end in a fixed order.  The main loop has no LDS and
// no barrier: a lane's 16-byte loads are MFMA operands as they stand (the q-th
// MFMA of a step takes the q-th of a lane's four k, and with TB = 0 the j-th
// column block is the j-th column of each lane's four), and DEPTH steps are in
// flight in registers.
// Rows of any dword alignment will do.  Past the end of the slice A is
// masked and B reads zeros (TB = 0) or is masked; rows and columns past the
// matrix only reach outputs that are not stored.
// split: raw sums to C + z M N, otherwise the epilogue at once.
//
// At 64 rows bound by the weights' first read from HBM: 512 x 29412 (60 MB) with
// the loss and dY takes 32 us, 2.3 TB/s (a streaming sum of 60 MB that no cache
// holds takes 28); staged through LDS, in two slices, then added up and compared by
// kernels of their own it took 67.  Its transposed product takes 26 us (32
// through LDS).  More steps in flight (DEPTH 3, 4 at MI = 4) were 10 % slower.
constexpr int kStep = 16;
// Steps of one accumulation chain: 32 of the reduction, added to a wavefront's sum
// at its end.  With one chain per wavefront (64 at 512 deep) the outputs of
// 600 -> 3 x 512 -> 600 at 64 rows are off by 3.4e-7, with this by 2.7e-7, and
// a pass takes 26.6 us where it took 26.4, at 1024 rows 54.9 where it took 50.1.
constexpr int kChain = 2;
constexpr int waves_of(int mi) { return mi == 1 ? 8 : 4; }
constexpr int kCPitch = kT + 4;
template <int DEPTH, int MI, int TB, bool FAR>
__global__ __launch_bounds__(waves_of(MI) * 64) void k_product(const float* __restrict__ A, int lda,
                                                         const float* __restrict__ B, int ldb,
                                                         float* __restrict__ C, int M, int N, int K,
                                                         int kslice, int split, EpiArgs ep) {
  constexpr int kWaves = waves_of(MI);
  constexpr bool kOne = DEPTH == 1 || (MI == 1 && DEPTH <= kChain);  // a wavefront's steps: one chain
  __shared__ alignas(16) float s[kWaves][16 * MI][kCPitch];
  const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.y * 16 * MI, n0 = blockIdx.x * kT;
  const int kb = blockIdx.z * kslice, ke = min(K, kb + kslice);
  v4f acc[MI][4], done[MI][4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = done[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  v4f a[DEPTH][MI], b[DEPTH][4];
  typedef typename View<FAR>::Off Off;
  Off oa[MI], ob[4];  // byte offsets in the operands' views
#pragma unroll
  for (int i = 0; i < MI; ++i) oa[i] = ((Off)(16 * i + r) * lda + 4 * kq) * 4u;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    ob[j] = (TB ? (Off)(16 * j + r) * ldb + 4 * kq : (Off)(4 * kq + j) * ldb + 4 * r) * 4u;
  auto fetch = [&](int d, int k0) {
    const View<FAR> va = operand<false, FAR>(A, lda, M, m0, k0, ke);
    const View<FAR> vb = operand<TB == 0, FAR>(B, ldb, N, n0, k0, ke);
#pragma unroll
    for (int j = 0; j < 4; ++j) b[d][j] = vb.f32x4(ob[j]);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[d][i] = va.f32x4(oa[i]);
  };
  int k0 = kb + wv * kStep;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) fetch(d, k0 + d * kWaves * kStep);
  // whole rounds of DEPTH steps (zeros past the end): a way out between two of
  // them would let the compiler move the loads behind it
  do {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d, k0 += kWaves * kStep) {
      if (k0 + kStep > ke) {
        const int left = ke - k0 - 4 * kq;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q >= left) {
#pragma unroll
            for (int i = 0; i < MI; ++i) a[d][i][q] = 0.f;
            if (TB) {
#pragma unroll
              for (int j = 0; j < 4; ++j) b[d][j][q] = 0.f;
            }
          }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                a[d][i][q], TB ? b[d][j][q] : b[d][q][j], acc[i][j], 0, 0, 0);
      fetch(d, k0 + DEPTH * kWaves * kStep);
      if (!kOne && d % kChain == kChain - 1) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            done[i][j] += acc[i][j];
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  } while (k0 - wv * kStep < ke);
  if (kOne) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) done[i][j] = acc[i][j];
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float* row = s[wv][16 * i + 4 * kq + q];
      if (TB) {
#pragma unroll
        for (int j = 0; j < 4; ++j) row[16 * j + r] = done[i][j][q];
      } else {
        *reinterpret_cast<v4f*>(row + 4 * r) =
            v4f{done[i][0][q], done[i][1][q], done[i][2][q], done[i][3][q]};
      }
    }
  __syncthreads();
  const int n = n0 + lane;
  float sq = 0.f;
  if (n < N) {
    // rows wv, wv + kWaves, ... of the tile; the bodies are kept apart and small: a
    // launch meets a cold instruction cache
    const size_t e0 = (size_t)m0 * N + n;
    const int rows = min(16 * MI, M - m0);
    auto sum = [&](int i) {
      float v = s[0][i][lane];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += s[w][i][lane];
      return v;
    };
    if (split) {
      float* Cz = C + (size_t)blockIdx.z * M * N + e0;
#pragma unroll 4
      for (int i = wv; i < rows; i += kWaves) Cz[(size_t)i * N] = sum(i);
    } else if (ep.kind == kMse) {
      const float bn = ep.bias[n];
#pragma unroll
      for (int q = 0; q < 16 * MI / kWaves; ++q) {
        const int i = wv + kWaves * q;
        if (i < rows) {
          const float d = (sum(i) + bn) - ep.t[e0 + (size_t)i * N];
          ep.out[e0 + (size_t)i * N] = 2.f * d * ep.inv;
          sq += d * d;
        }
      }
    } else {
#pragma unroll 1
      for (int i = wv; i < rows; i += kWaves) {
        const size_t e = e0 + (size_t)i * N;
        epilogue(ep, e, epi_aux(ep, e, n), sum(i));
      }
    }
  }
  if (!split && ep.kind == kMse) {
    __syncthreads();  // the partial tiles' LDS becomes the tree's
    const float tot = block_tree<kWaves * 64>(sq, &s[0][0][0]);
    if (threadIdx.x == 0) ep.loss_part[blockIdx.y * gridDim.x + blockIdx.x] = tot;
  }
}

// Adam's constants of one step (beta1 0.9, beta2 0.999, eps 1e-8).
struct AdamArgs {
  float lr, bc1, bc2;
};
__device__ __forceinline__ void adam_f32(float* __restrict__ p, float* __restrict__ m,
                                         float* __restrict__ v, size_t e, float ge,
                                         const AdamArgs& c) {
  const float mm = 0.9f * m[e] + 0.1f * ge;
  const float vv = 0.999f * v[e] + 0.001f * ge * ge;
  m[e] = mm;
  v[e] = vv;
  p[e] -= c.lr * (mm / c.bc1) / (sqrtf(vv / c.bc2) + 1e-8f);
}

// The block's tile (x, y), such that each XCD takes a contiguous run of tiles of
// a row of the grid: blocks go to the 8 XCDs in turn.
__device__ __forceinline__ int2 xcd_tile() {
  const unsigned n = gridDim.x * gridDim.y, l = blockIdx.y * gridDim.x + blockIdx.x;
  const unsigned x = l & 7, t = x * (n >> 3) + min(x, n & 7) + (l >> 3);
  return {(int)(t % gridDim.x), (int)(t / gridDim.x)};
}

// Sums of a weight gradient's chains, of eight terms each but the last.
constexpr int kDwLevels = 4;
constexpr int kDwShort = 8 * kBK;  // longest batch for which one sum is enough

// Weight and bias gradient of one layer, dW [M = fan_in][N = n_out] = in^T dZ
// and db = column sums of dZ [K = batch][N], and with ADAM the update of the
// layer's weights, biases and moments from them at once: the update needs 28
// bytes per weight and would otherwise read the gradient again in a pass of
// its own.  A block's tile goes through LDS so that a wavefront's accesses to
// the parameters, the moments and the gradient are whole rows of 64.  The
// column sums are formed by the blocks of the first row of tiles from the
// staged operand, each column's rows in eight interleaved parts that are then
// added in order.
// Chains of one k-step (32 rows) are added up eight at a time, those sums eight at
// a time, and so on: with longer chains, or all of them in one sum, the rounding
// error grows with the batch (65536 rows of 40 -> 2 x 32 -> 40: 2.3e-7 of the gradient
// with chains of 256 in one sum).
// Bound by memory: at a batch of 64 the 15.1 M weights of 512 x 29412 (421 MB)
// take 104 us, 4.1 TB/s (89 us with the product left out), the 5.7 M of
// 11124 x 512 take 38; as products, column sums and a pass of updates these were
// 32.7 + 15.8 + 101 us for the whole network.  Stores past the caches (read
// again only in the next step) and neighbouring tiles on one XCD (rows are
// not line-aligned, so neighbours share lines) give 4 and 3 us of it.  One kernel is
// the faster at every batch and number of tiles: with sliced products and passes of
// their own 11124 -> 3 x 512 -> 29412 takes 283 us a step at 64 rows against 264,
// 600 -> 3 x 512 -> 600 2597 us at 8192 rows against 1500; and one tile a layer walked
// by one block, 40 -> 2 x 32 -> 40 11.5 ms at 65,536 rows with slices, 6.6 here, 64 -> 16 ->
// 8 7.3 and 4.4.
struct DwArgs {
  float *gw, *gb;                        // gradients out
  float *pw, *mw, *vw, *pb, *mb, *vb;    // ADAM: parameters and moments
  AdamArgs adam;
  // ADAM or not, block (0, 0) with loss != null: *loss = inv sum loss_part
  const float* loss_part;
  int n_loss;
  float inv;
  float* loss;
};

template <bool ADAM, int kLevels, bool FAR>
__global__ __launch_bounds__(kGemm, 4) void k_dw(const float* __restrict__ in, int fan_in,
                                                 const float* __restrict__ dZ, int n_out, int batch,
                                                 DwArgs w) {
  __shared__ union alignas(16) {
    TileLds t;
    float c[kT][kT + 1];
    float red[kGemm];
  } s;
  const int2 t = xcd_tile();
  const int m0 = t.y * kT, n0 = t.x * kT;
  const int c = threadIdx.x & 63, q8 = threadIdx.x >> 6;
  const bool first = t.y == 0;
  float cs = 0.f;  // this eighth's part of column n0 + c
  constexpr int R = kT * kT / kGemm;  // elements per thread
  const int n = n0 + c;
  const int rows = n < n_out ? min(kT, fan_in - m0) : 0;
  const size_t e0 = (size_t)m0 * n_out + n;
  // parameters and moments, in flight while the product is formed: loads return
  // in order, so the operands', which come from L2, go first.  Unconditional (past
  // the matrix they read zeros or the next row, and are not used): a wait
  // behind a load that may not have been issued waits for all.  104 us where it
  // was 107 with these loads first.
  float p[R], m[R], v[R];
  auto params = [&]() {
    if constexpr (ADAM) {
      const auto vp = operand<true, FAR>(w.pw, n_out, n_out, n0, m0, fan_in);
      const auto vm = operand<true, FAR>(w.mw, n_out, n_out, n0, m0, fan_in);
      const auto vv = operand<true, FAR>(w.vw, n_out, n_out, n0, m0, fan_in);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const typename View<FAR>::Off o =
            ((typename View<FAR>::Off)(q8 + 8 * i) * n_out + c) * 4u;
        p[i] = vp.f32(o);
        m[i] = vm.f32(o);
        v[i] = vv.f32(o);
      }
    }
  };
  Tile<FAR> tile;
  v4f acc[2], sum[kLevels][2];
#pragma unroll
  for (int j = 0; j < kLevels; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) sum[j][i] = v4f{0.f, 0.f, 0.f, 0.f};
  int chains = 0;  // in the sums
  tile.run(in, fan_in, dZ, n_out, fan_in, n_out, 0, batch, m0, n0, s.t, acc, params, [&](int buf) {
    if (first)
      for (int k = q8; k < kBK; k += 8) cs += s.t.b[buf][c][k];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      sum[0][i] += acc[i];
      acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 1, n = 8; j < kLevels; ++j, n *= 8)
      if (chains > 0 && chains % n == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          sum[j][i] += sum[j - 1][i];
          sum[j - 1][i] = v4f{0.f, 0.f, 0.f, 0.f};
        }
      }
    ++chains;
  });
#pragma unroll
  for (int j = 0; j < kLevels; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i] += sum[j][i];
  __syncthreads();
  tile_elements(acc, 0, 0, kT, kT, [&](int row, int col, float v) { s.c[row][col] = v; });
  __syncthreads();
  if constexpr (ADAM) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int row = q8 + 8 * i;
      if (row < rows) {
        const size_t e = e0 + (size_t)row * n_out;
        const float ge = s.c[row][c];
        const float mm = 0.9f * m[i] + 0.1f * ge;
        const float vv = 0.999f * v[i] + 0.001f * ge * ge;
        __builtin_nontemporal_store(ge, &w.gw[e]);
        __builtin_nontemporal_store(mm, &w.mw[e]);
        __builtin_nontemporal_store(vv, &w.vw[e]);
        __builtin_nontemporal_store(
            p[i] - w.adam.lr * (mm / w.adam.bc1) / (sqrtf(vv / w.adam.bc2) + 1e-8f), &w.pw[e]);
      }
    }
  } else {
    for (int row = q8; row < rows; row += 8) w.gw[e0 + (size_t)row * n_out] = s.c[row][c];
  }
  if (!first) return;
  __syncthreads();
  s.red[threadIdx.x] = cs;
  __syncthreads();
  if (q8 == 0 && n < n_out) {
    float g = s.red[c];
    for (int q = 1; q < 8; ++q) g += s.red[q * 64 + c];
    w.gb[n] = g;
    if constexpr (ADAM) adam_f32(w.pb, w.mb, w.vb, (size_t)n, g, w.adam);
  }
  if (t.x == 0 && w.loss) {
    float part = 0.f;
    for (int i = threadIdx.x; i < w.n_loss; i += kGemm) part += w.loss_part[i];
    __syncthreads();
    const float tot = block_tree<kGemm>(part, s.red);
    if (threadIdx.x == 0) *w.loss = tot * w.inv;
  }
}

// BF16 operands (A32: A in FP32, rounded as it is staged), row-major A [M][K]
// and B [K][N], FP32 sums; pipelined like the FP32 tile with DEPTH k-steps in
// flight.
// APAIR, PAIR: two neighbouring elements of A, B per load (their rows' length and
// base even).  Every output's products are added in the order of one accumulator
// per slice.  CHAIN: one launch keeps the sums of slices that were not launched,
// chains of chain k-steps added as k_reduce_epi adds slices; 1: up to eight, in
// order; 2: sixteen of one or two k-steps, c and c + 8 first.
// Bound by the weights' first read: at 64 rows 512 x 29412 (30 MB) with
// its biases takes 14.3 us and 11124 x 512 12.5; the whole forward pass of
// 11124 -> 3 x 512 -> 29412 takes 41 us, and 83 with conversions, copies and an
// unpipelined loop.
template <int DEPTH, bool A32, bool APAIR, bool PAIR, int CHAIN, bool FAR>
__global__ __launch_bounds__(kGemm) void k_gemm_bf16(const void* __restrict__ Av, int lda,
                                                       const uint16_t* __restrict__ B, int ldb,
                                                       float* __restrict__ C, int M, int N, int K,
                                                       int kslice, int split, int chain,
                                                       EpiArgs ep) {
  __shared__ alignas(16) uint16_t As[2][kT][kBK + 8];  // [m][k], 16-byte rows of 8 k
  __shared__ alignas(16) uint16_t Bs[2][kT][kBK + 4];  // [n][k] (transposed), 8-byte halves
  const float* __restrict__ Af = static_cast<const float*>(Av);
  const uint16_t* __restrict__ Ah = static_cast<const uint16_t*>(Av);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m0 = blockIdx.y * kT, n0 = blockIdx.x * kT;
  const int kb = blockIdx.z * kslice, ke = min(K, kb + kslice);
  const int wm = (wv >> 2) * 32, wn = (wv & 3) * 16;
  const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
  v4f acc[2] = {zero, zero}, part[2] = {zero, zero}, done[2] = {zero, zero};
  // A: FP32 element by element, BF16 in pairs of k where its rows are even;
  // B: pairs (n, n + 1) of one k
  float rf[DEPTH][kEl];
  unsigned ra[DEPTH][kEl / 2], rb[DEPTH][kEl / 2];
  typedef typename View<FAR>::Off Off;
  Off oa[kEl], ob[kEl / 2];
#pragma unroll
  for (int q = 0; q < kEl; ++q) {
    const int e = tid + q * kGemm;
    oa[q] = A32 ? ((Off)(e >> 5) * lda + (e & 31)) * 4u : ((Off)(e >> 4) * lda + 2 * (e & 15)) * 2u;
    if (q < kEl / 2) ob[q] = ((Off)(e >> 5) * ldb + 2 * (e & 31)) * 2u;
  }
  auto pair = [](const View<FAR>& v, Off o, bool whole) -> unsigned {
    return whole ? v.u32(o) : v.u16(o) | v.u16(o + 2) << 16;
  };
  auto load = [&](int d, int k0) {
    if constexpr (A32) {
      const View<FAR> va = operand<false, FAR>(Af, lda, M, m0, k0, ke);
#pragma unroll
      for (int q = 0; q < kEl; ++q) rf[d][q] = va.f32(oa[q]);
    } else {
      const View<FAR> va = operand<false, FAR>(Ah, lda, M, m0, k0, ke);
#pragma unroll
      for (int q = 0; q < kEl / 2; ++q) ra[d][q] = pair(va, oa[q], APAIR);
    }
    const View<FAR> vb = operand<true, FAR>(B, ldb, N, n0, k0, ke);
#pragma unroll
    for (int q = 0; q < kEl / 2; ++q) rb[d][q] = pair(vb, ob[q], PAIR);
  };
  auto put = [&](int d, int buf, int left) {
    if constexpr (A32) {
#pragma unroll
      for (int q = 0; q < kEl; ++q) {
        const int e = tid + q * kGemm;
        As[buf][e >> 5][e & 31] = (e & 31) < left ? to_bf16(rf[d][q]) : (uint16_t)0;
      }
    } else {
#pragma unroll
      for (int q = 0; q < kEl / 2; ++q) {
        const int e = tid + q * kGemm, k = 2 * (e & 15);
        const unsigned v = k + 1 < left ? ra[d][q] : k < left ? ra[d][q] & 0xFFFFu : 0u;
        *reinterpret_cast<unsigned*>(&As[buf][e >> 4][k]) = v;
      }
    }
#pragma unroll
    for (int q = 0; q < kEl / 2; ++q) {
      const int e = tid + q * kGemm;
      const int k = e >> 5, n = 2 * (e & 31);
      Bs[buf][n][k] = (uint16_t)rb[d][q];
      Bs[buf][n + 1][k] = (uint16_t)(rb[d][q] >> 16);
    }
  };
  // k of the n-th k-step: in order, or the chains' in pairs c, c + 8; past the last
  // one nothing but zeros
  const int steps = CHAIN == 2 ? 16 * chain : (ke - kb + kBK - 1) / kBK;
  auto at = [&](int n) {
    if (CHAIN != 2) return kb + n * kBK;
    const int c = n >> (chain - 1);
    return n < steps ? (n + ((c & 1) * 8 + (c >> 1) - c) * chain) * kBK : ke;
  };
  if (steps > 0) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, at(d));
  }
  int left = chain, c = 0;
  auto step1 = [&](int d, int buf, int n) {
    put(d, buf, ke - at(n));
    __syncthreads();
    load(d, at(n + DEPTH));
    v8bf a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a[i] = __builtin_bit_cast(
          v8bf, *reinterpret_cast<const uint4*>(&As[buf][wm + i * 16 + (lane & 15)][8 * (lane >> 4)]));
    const uint16_t* src = &Bs[buf][wn + (lane & 15)][8 * (lane >> 4)];
    const uint2 lo = *reinterpret_cast<const uint2*>(src);
    const uint2 hi = *reinterpret_cast<const uint2*>(src + 4);
    const v8bf b = __builtin_bit_cast(v8bf, uint4{lo.x, lo.y, hi.x, hi.y});
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i], 0, 0, 0);
    if (CHAIN > 0 && --left == 0) {
      left = chain;
      const bool hold = CHAIN == 2 && (c++ & 1) == 0;  // the pair's first
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (CHAIN == 2) {
          part[i] = hold ? acc[i] : part[i] + acc[i];
          if (!hold) done[i] += part[i];
        } else {
          done[i] += acc[i];
        }
        acc[i] = zero;
      }
    }
  };
  // whole rounds of DEPTH k-steps, as in the FP32 tile
  int buf = 0;
  for (int n = 0; n < steps;) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d, ++n, buf ^= 1) step1(d, buf, n);
  }
  if (CHAIN > 0) {  // with what is left of a chain that the reduction's end cuts short
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i] += done[i];
  }
  if (split) {
    float* Cz = C + (size_t)blockIdx.z * M * N;
    tile_elements(acc, m0, n0, M, N,
                  [&](int row, int col, float v) { Cz[(size_t)row * N + col] = v; });
    return;
  }
  // the two kinds' bodies are kept apart: a launch meets a cold instruction cache
  if (ep.kind == kBias) {
    const int n = n0 + wn + (lane & 15);
    const float b = n < N ? from_bf16(ep.bias16[n]) : 0.f;
    tile_elements(acc, m0, n0, M, N,
                  [&](int row, int col, float v) { ep.out[(size_t)row * N + col] = v + b; });
    return;
  }
  tile_elements(acc, m0, n0, M, N, [&](int row, int col, float v) {
    const size_t e = (size_t)row * N + col;
    epilogue(ep, e, epi_aux(ep, e, col), v);
  });
}

// out = epilogue(sum over slices of P[s][m][n]) for an M x N matrix (ld N).
// The slices of 32 elements are summed by 8 groups of threads (group g takes
// slices g, g + 8, ..., U loads in flight), the group sums then added in
// group order: a fixed order.
template <int U>
__global__ __launch_bounds__(kThreads) void k_reduce_epi(const float* __restrict__ P, int slices,
                                                         int M, int N, EpiArgs ep) {
  __shared__ float red[8][33];
  const size_t MN = (size_t)M * N;
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  for (size_t e0 = (size_t)blockIdx.x * 32; e0 < MN; e0 += (size_t)gridDim.x * 32) {
    const size_t e = e0 + c, ec = e < MN ? e : MN - 1;
    Aux x{0.f, 0.f};
    if (g == 0) x = epi_aux(ep, ec, (int)(ec % N));
    float part = 0.f;
    for (int q0 = g; q0 < slices; q0 += 8 * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = P[(size_t)min(q0 + 8 * u, slices - 1) * MN + ec];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q0 + 8 * u < slices) part += v[u];
    }
    red[g][c] = part;
    __syncthreads();
    if (g == 0 && e < MN) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) s += red[q][c];
      epilogue(ep, e, x, s);
    }
    __syncthreads();  // red is refilled by the next round
  }
}

// dY = 2 (Y - T) / (M N); per-block partial sums of (Y - T)^2
__global__ __launch_bounds__(kThreads) void k_mse(const float* __restrict__ Y,
                                                  const float* __restrict__ T, size_t n, float inv,
                                                  float* __restrict__ dY, float* __restrict__ part) {
  __shared__ float red[kThreads];
  float acc = 0.f;
  for (size_t e = (size_t)blockIdx.x * kThreads + threadIdx.x; e < n;
       e += (size_t)gridDim.x * kThreads) {
    const float d = Y[e] - T[e];
    dY[e] = 2.f * d * inv;
    acc += d * d;
  }
  const float tot = block_tree<kThreads>(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kThreads) void k_to_bf16(const float* __restrict__ x, size_t n,
                                                      uint16_t* __restrict__ y) {
  for (size_t e = (size_t)blockIdx.x * kThreads + threadIdx.x; e < n;
       e += (size_t)gridDim.x * kThreads)
    y[e] = to_bf16(x[e]);
}

// ---------------------------------------------------------------------------
// host side

constexpr int kLossBlocks = 256;  // blocks of k_mse
constexpr int kOneSlice = 512;    // most blocks of a product in tiles of 16 rows

struct Ws {
  float* z[QG_MLP_MAX_DEPTH];  // pre-activations [B][width]
  float* h[QG_MLP_MAX_DEPTH];  // activations [B][width]
  float* y;                    // [B][d_out]
  float* dy;                   // [B][d_out]
  float* da;                   // [B][width]
  float* dz;                   // [B][width]
  float* part;                 // product slices
  float* loss_part;            // [loss_parts]
  uint16_t* a16[2];            // BF16 activations [B][width]
  int loss_parts;              // at most: blocks of k_mse, or of the output layer's product
  size_t part_floats;
  size_t total;
};

constexpr int kMaxSlices = 128;

bool valid(const qg_mlp_desc* d) {
  return d && d->d_in > 0 && d->width > 0 && d->d_out > 0 && d->depth >= 1 &&
         d->depth <= QG_MLP_MAX_DEPTH;
}

size_t al(size_t v) { return (v + 63) / 64 * 64; }

void layout(const qg_mlp_desc* d, qg_mlp_layout* L) {
  int64_t o = 0;
  int64_t fan_in = d->d_in;
  for (int i = 0; i <= d->depth; ++i) {
    const int64_t out = (i == d->depth) ? d->d_out : d->width;
    L->w_off[i] = o;
    o = (int64_t)al((size_t)(o + fan_in * out));
    L->b_off[i] = o;
    o = (int64_t)al((size_t)(o + out));
    fan_in = d->width;
  }
  for (int i = d->depth + 1; i <= QG_MLP_MAX_DEPTH; ++i) L->w_off[i] = L->b_off[i] = -1;
  L->n_params = o;
}

int tiles_of(int M, int N) { return ((M + kT - 1) / kT) * ((N + kT - 1) / kT); }

// Slices of a deep FP32 product: about one block per CU, each slice at least 64
// deep.  With that (32 slices of 64 x 512 over 29412 and 11124, 8 tiles) a training
// step of 11124 -> 3 x 512 -> 29412 at 64 rows takes 252 us, with half as many 268, with
// twice as many 264 (more sums to write, fewer rows of the weights in each).
int slices_f32(int M, int N, int K) {
  const int tiles = tiles_of(M, N);
  if (tiles >= 64 && K <= 512) return 1;  // no second kernel: 5.8 against 4.6 + 4.8 us (7353 x 200)
  int s = 1;
  while (s < kMaxSlices && tiles * s < 256 && K / (s * 2) >= 2 * kBK) s *= 2;
  return s;
}

// Slices of a BF16 product.  The hidden layers' sums are rounded to BF16, so
// their slices are part of the result: about four blocks per CU, each slice at
// least 32 deep.
int slices_bf16(int M, int N, int K) {
  const int tiles = tiles_of(M, N);
  int s = 1;
  while (s < kMaxSlices && tiles * s < 1024 && K / (s * 2) >= 32) s *= 2;
  return s;
}

Ws carve(const qg_mlp_desc* d, int B, void* base) {
  Ws w;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = (o + bytes + 255) / 256 * 256;
    return base ? static_cast<unsigned char*>(base) + at : nullptr;
  };
  const size_t BW = (size_t)B * d->width, BO = (size_t)B * d->d_out;
  for (int i = 0; i < d->depth; ++i) {
    w.z[i] = reinterpret_cast<float*>(take(BW * 4));
    w.h[i] = reinterpret_cast<float*>(take(BW * 4));
  }
  w.y = reinterpret_cast<float*>(take(BO * 4));
  w.dy = reinterpret_cast<float*>(take(BO * 4));
  w.da = reinterpret_cast<float*>(take(BW * 4));
  w.dz = reinterpret_cast<float*>(take(BW * 4));
  // the largest sliced product: B x width outputs with up to kMaxSlices
  // slices, or one B x d_out slice
  w.part_floats = std::max((size_t)kMaxSlices * BW, BO);
  w.part = reinterpret_cast<float*>(take(w.part_floats * 4));
  w.loss_parts = std::max(std::max(kLossBlocks, kOneSlice), tiles_of(B, d->d_out));
  w.loss_part = reinterpret_cast<float*>(take((size_t)w.loss_parts * 4));
  w.a16[0] = reinterpret_cast<uint16_t*>(take(BW * 2));
  w.a16[1] = reinterpret_cast<uint16_t*>(take(BW * 2));
  w.total = o;
  return w;
}

int grid1(size_t n) { return (int)std::min<size_t>(4096, (n + kThreads - 1) / kThreads); }
// k_reduce_epi: 32 elements a block and round
int grid_red(size_t n) { return (int)std::min<size_t>(4096, (n + 31) / 32); }

int fit_slices(int sl, int M, int N, const Ws& w) {
  while (sl > 1 && (size_t)sl * M * N > w.part_floats) sl /= 2;
  return sl;
}

// How k_product computes an M x N product over K: tiles of 16 mi rows, at most
// sl slices.  A product that is not deep and has few tiles is cut into tiles of 16
// rows, read with eight wavefronts a block, instead of slices: the second kernel
// costs more than the weights' repeated reads from L2.  One forward pass of
// 600 -> 3 x 512 -> 600 at 64 rows takes 26.1 us in this way, 31.0 in slices; of
// 1400 -> 2 x 256 -> 3300 17.3, in slices 26.7.  With more blocks than kOneSlice the
// repeated reads win (29412 outputs: 86.0 us a pass against 53.1).  The transposed
// product reads 64 bytes of each of the weights' rows at a time, which a few
// blocks do slowly over a long reduction: 600 -> 3 x 512 -> 600 trains in 83.6 us with
// the limit at 256, in 90.5 with 512 (1400 -> 2 x 256 -> 3300 in 61.4 with 128, 256 or
// 512).
struct Plan {
  int mi, sl;
  bool far;
};
Plan plan_f32(int tb, int M, int N, int K, const Ws& w) {
  // A has rows of K; op(B) is read in 64 rows of K or 16 of N
  if (rows_far(kT, K) || (!tb && rows_far(kStep, N)))
    return {4, fit_slices(slices_f32(M, N, K), M, N, w), true};
  const int64_t t16 = (int64_t)((M + 15) / 16) * ((N + kT - 1) / kT);
  if (K <= (tb ? 256 : 1024) && t16 <= kOneSlice) return {1, 1, false};
  return {M <= 16 ? 1 : M <= 32 ? 2 : 4, fit_slices(slices_f32(M, N, K), M, N, w), false};
}
int blocks_of(const Plan& p, int M, int N) {
  return ((M + 16 * p.mi - 1) / (16 * p.mi)) * ((N + kT - 1) / kT);
}

// The slices' sums of an M x N product in w.part through the epilogue, with the
// loads that a group has: eight for eight slices (seven of them for nothing) took 27 us
// where one takes 14 (300 x 2048).
void reduce_epi(hipStream_t s, const Ws& w, int slices, int M, int N, const EpiArgs& ep) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid_red((size_t)M * N)), dim3(kThreads), 0, s, w.part, slices,
                       M, N, ep);
  };
  if (slices <= 8) go(k_reduce_epi<1>);
  else if (slices <= 16) go(k_reduce_epi<2>);
  else if (slices <= 32) go(k_reduce_epi<4>);
  else go(k_reduce_epi<8>);
}

// A op(B) with epilogue as planned; slices go through ws.part
hipError_t product(hipStream_t s, int tb, const float* A, int lda, const float* B, int ldb, int M,
                   int N, int K, const Plan& p, const EpiArgs& ep, const Ws& w) {
  const int kRound = waves_of(p.mi) * kStep;
  const int kslice = ((K + p.sl - 1) / p.sl + kRound - 1) / kRound * kRound;
  const int sl = (K + kslice - 1) / kslice;
  const int split = sl > 1;
  const dim3 grid((N + kT - 1) / kT, (M + 16 * p.mi - 1) / (16 * p.mi), sl);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(waves_of(p.mi) * 64), 0, s, A, lda, B, ldb, w.part, M, N,
                       K, kslice, split, ep);
  };
  auto rows = [&](auto t) {
    constexpr int T = decltype(t)::value;
    const int steps = kslice / kRound;  // of a wavefront
    if (p.far) {
      go(k_product<2, 4, T, true>);
    } else if (p.mi == 1) {
      if (steps == 1) go(k_product<1, 1, T, false>);
      else if (steps == 2) go(k_product<2, 1, T, false>);
      else go(k_product<4, 1, T, false>);
    } else if (p.mi == 2) {
      if (steps == 1) go(k_product<1, 2, T, false>);
      else go(k_product<2, 2, T, false>);
    } else {
      if (steps == 1) go(k_product<1, 4, T, false>);
      else go(k_product<2, 4, T, false>);
    }
  };
  if (tb) rows(std::integral_constant<int, 1>{});
  else rows(std::integral_constant<int, 0>{});
  if (split) reduce_epi(s, w, sl, M, N, ep);
  return hipGetLastError();
}

// A B with BF16 operands (a32: A in FP32) and the sums of sl slices; whole: in one
// launch all the same (K <= 1024, BF16 A).
hipError_t product16(hipStream_t s, const void* A, bool a32, int lda, const uint16_t* B, int M,
                     int N, int K, int sl, bool whole, const EpiArgs& ep, const Ws& w) {
  int kslice = ((K + sl - 1) / sl + kBK - 1) / kBK * kBK;
  const int chain = kslice / kBK, chains = whole ? sl : 1;
  if (chains > 1) {
    kslice *= chains;  // the whole reduction
    sl = 1;
  }
  const int split = sl > 1;
  const dim3 grid((N + kT - 1) / kT, (M + kT - 1) / kT, sl);
  const bool pair = N % 2 == 0 && (reinterpret_cast<uintptr_t>(B) & 3u) == 0;
  const bool apair = lda % 2 == 0;  // A is the workspace's
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kGemm), 0, s, A, lda, B, N, w.part, M, N, K, kslice,
                       split, chain, ep);
  };
  auto depth = [&](auto d, auto ch) {
    constexpr int D = decltype(d)::value, C = decltype(ch)::value;
    if (C == 0 && a32 && pair) go(k_gemm_bf16<D, true, false, true, 0, false>);
    else if (C == 0 && a32) go(k_gemm_bf16<D, true, false, false, 0, false>);
    else if (apair && pair) go(k_gemm_bf16<D, false, true, true, C, false>);
    else if (apair) go(k_gemm_bf16<D, false, true, false, C, false>);
    else if (pair) go(k_gemm_bf16<D, false, false, true, C, false>);
    else go(k_gemm_bf16<D, false, false, false, C, false>);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  const int steps = kslice / kBK;
  // as many k-steps in flight as a slice has, two in longer ones (with three a pass
  // of 11124 -> 2048 -> 3000 at 2048 rows takes 489 us, with two 456; with two in slices
  // of three that of 11124 -> 3 x 512 -> 29412 at 64 rows takes 42.5, with three 42.3)
  if (rows_far(kT, K) || rows_far(kBK, N)) {
    if (chains > 8) go(k_gemm_bf16<2, false, false, false, 2, true>);
    else if (chains > 1) go(k_gemm_bf16<2, false, false, false, 1, true>);
    else if (a32) go(k_gemm_bf16<2, true, false, false, 0, true>);
    else go(k_gemm_bf16<2, false, false, false, 0, true>);
  } else if (chains > 8) depth(I2{}, I2{});
  else if (chains > 1) depth(I2{}, I1{});
  else if (steps == 1) depth(I1{}, I0{});
  else if (steps == 3) depth(I3{}, I0{});
  else depth(I2{}, I0{});
  if (split) reduce_epi(s, w, sl, M, N, ep);
  return hipGetLastError();
}

bool al256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

qg_status check_common(const qg_mlp_desc* d, int batch, const void* ws) {
  if (!valid(d)) return qg::fail(QG_ERR_ARG, "bad network description");
  if (batch < 1) return qg::fail(QG_ERR_ARG, "batch must be >= 1");
  if (!ws || !al256(ws)) return qg::fail(QG_ERR_ARG, "workspace must be non-null and 256-byte aligned");
  return QG_OK;
}

qg_status dev_fail(hipError_t e, const char* where) {
  return qg::fail(QG_ERR_DEVICE, std::string(where) + ": " + hipGetErrorString(e));
}

// forward in FP32, activations kept for the reverse pass; the output layer's
// product ends in out (with its bias, an epilogue of kind kBias or kMse)
hipError_t forward(hipStream_t s, const qg_mlp_desc* d, const qg_mlp_layout& L, const float* P,
                   const float* x, int B, EpiArgs out, const Plan& out_plan, const Ws& w) {
  const float* in = x;
  int fan_in = d->d_in;
  for (int i = 0; i < d->depth; ++i) {
    EpiArgs ep{};
    ep.kind = kBiasGelu;
    ep.bias = P + L.b_off[i];
    ep.z = w.z[i];
    ep.out = w.h[i];
    hipError_t e = product(s, 0, in, fan_in, P + L.w_off[i], d->width, B, d->width, fan_in,
                           plan_f32(0, B, d->width, fan_in, w), ep, w);
    if (e != hipSuccess) return e;
    in = w.h[i];
    fan_in = d->width;
  }
  out.bias = P + L.b_off[d->depth];
  return product(s, 0, in, fan_in, P + L.w_off[d->depth], d->d_out, B, d->d_out, fan_in,
                 out_plan, out, w);
}

// Adam's state of a training step.
struct Update {
  float *p, *m, *v;
  AdamArgs adam;
};

// Loss, gradient and (u non-null) the update; null buffers checked before.
hipError_t grad_step(hipStream_t s, const qg_mlp_desc* d, const qg_mlp_layout& L, const float* P,
                     const float* x, const float* t, int B, float* grad, float* loss,
                     const Update* u, const Ws& w) {
  const int D = d->depth, W = d->width;
  const size_t BO = (size_t)B * d->d_out;
  const float inv = 1.0f / (float)BO;
  const Plan op = plan_f32(0, B, d->d_out, W, w);
  const bool one = op.sl == 1;  // the output layer's product ends in dY and the loss
  EpiArgs out{};
  out.kind = one ? kMse : kBias;
  out.out = one ? w.dy : w.y;
  out.t = t;
  out.inv = inv;
  out.loss_part = w.loss_part;
  hipError_t e = forward(s, d, L, P, x, B, out, op, w);
  if (e != hipSuccess) return e;
  int n_loss = blocks_of(op, B, d->d_out);
  if (!one) {
    n_loss = kLossBlocks;
    hipLaunchKernelGGL(k_mse, dim3(kLossBlocks), dim3(kThreads), 0, s, w.y, t, BO, inv, w.dy,
                       w.loss_part);
  }
  // output layer: dW_out = h_D^T dY, db_out = colsum dY, dh_D = dY W_out^T
  const float* dcur = w.dy;  // gradient at the current layer's output
  int n_out = d->d_out;
  for (int i = D; i >= 0; --i) {
    const float* in = (i == 0) ? x : w.h[i - 1];
    const int fan_in = (i == 0) ? d->d_in : W;
    float* dst = (dcur == w.dz) ? w.da : w.dz;
    if (i > 0) {
      // dz_{i-1} = (dcur W_i^T) * gelu'(z_{i-1}), W_i is [fan_in][n_out]; before
      // the layer's update
      EpiArgs ep{};
      ep.kind = kGeluBwd;
      ep.z = w.z[i - 1];
      ep.out = dst;
      e = product(s, 1, dcur, n_out, P + L.w_off[i], n_out, B, fan_in, n_out,
                  plan_f32(1, B, fan_in, n_out, w), ep, w);
      if (e != hipSuccess) return e;
    }
    const size_t wo = (size_t)L.w_off[i], bo = (size_t)L.b_off[i];
    DwArgs a{};
    a.gw = grad + wo;
    a.gb = grad + bo;
    if (i == D) {
      a.loss_part = w.loss_part;
      a.n_loss = n_loss;
      a.inv = inv;
      a.loss = loss;
    }
    const dim3 grid((n_out + kT - 1) / kT, (fan_in + kT - 1) / kT);
    if (u) {
      a.pw = u->p + wo; a.mw = u->m + wo; a.vw = u->v + wo;
      a.pb = u->p + bo; a.mb = u->m + bo; a.vb = u->v + bo;
      a.adam = u->adam;
    }
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(kGemm), 0, s, in, fan_in, dcur, n_out, B, a);
    };
    const bool far = rows_far(kBK, fan_in) || rows_far(kT, n_out);
    if (u && far) go(k_dw<true, kDwLevels, true>);
    else if (far) go(k_dw<false, kDwLevels, true>);
    else if (u && B <= kDwShort) go(k_dw<true, 1, false>);
    else if (u) go(k_dw<true, kDwLevels, false>);
    else if (B <= kDwShort) go(k_dw<false, 1, false>);
    else go(k_dw<false, kDwLevels, false>);
    dcur = dst;
    n_out = W;
  }
  return hipGetLastError();
}

}  // namespace

extern "C" {

qg_status qg_mlp_sizes(const qg_mlp_desc* desc, int32_t max_batch, qg_mlp_layout* lay,
                       size_t* workspace_bytes) {
  if (!valid(desc)) return qg::fail(QG_ERR_ARG, "bad network description");
  if (max_batch < 1 || !lay || !workspace_bytes) return qg::fail(QG_ERR_ARG, "bad arguments");
  layout(desc, lay);
  *workspace_bytes = carve(desc, max_batch, nullptr).total;
  return QG_OK;
}

qg_status qg_mlp_forward(const qg_mlp_desc* desc, const float* d_params, const float* d_x,
                         int32_t batch, float* d_y, void* d_ws, void* stream) {
  qg_status st = check_common(desc, batch, d_ws);
  if (st != QG_OK) return st;
  if (!d_params || !d_x || !d_y) return qg::fail(QG_ERR_ARG, "null buffer");
  qg_mlp_layout L;
  layout(desc, &L);
  const Ws w = carve(desc, batch, d_ws);
  hipStream_t s = static_cast<hipStream_t>(stream);
  EpiArgs out{};
  out.kind = kBias;
  out.out = d_y;
  hipError_t e = forward(s, desc, L, d_params, d_x, batch, out,
                         plan_f32(0, batch, desc->d_out, desc->width, w), w);
  return e == hipSuccess ? QG_OK : dev_fail(e, "mlp forward");
}

qg_status qg_mlp_grad(const qg_mlp_desc* desc, const float* d_params, const float* d_x,
                      const float* d_t, int32_t batch, float* d_grad, float* d_loss, void* d_ws,
                      void* stream) {
  qg_status st = check_common(desc, batch, d_ws);
  if (st != QG_OK) return st;
  if (!d_params || !d_x || !d_t || !d_grad || !d_loss) return qg::fail(QG_ERR_ARG, "null buffer");
  qg_mlp_layout L;
  layout(desc, &L);
  const Ws w = carve(desc, batch, d_ws);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = grad_step(s, desc, L, d_params, d_x, d_t, batch, d_grad, d_loss, nullptr, w);
  return e == hipSuccess ? QG_OK : dev_fail(e, "mlp reverse");
}

qg_status qg_mlp_train_step(const qg_mlp_desc* desc, float* d_params, float* d_m, float* d_v,
                            float* d_grad, const float* d_x, const float* d_t, int32_t batch,
                            int64_t iter, float lr, float* d_loss, void* d_ws, void* stream) {
  if (!d_m || !d_v || iter < 1 || !(lr > 0.f)) return qg::fail(QG_ERR_ARG, "bad Adam arguments");
  qg_status st = check_common(desc, batch, d_ws);
  if (st != QG_OK) return st;
  if (!d_params || !d_x || !d_t || !d_grad || !d_loss) return qg::fail(QG_ERR_ARG, "null buffer");
  qg_mlp_layout L;
  layout(desc, &L);
  const Ws w = carve(desc, batch, d_ws);
  const float bc1 = 1.0f - std::pow(0.9f, (float)iter);
  const float bc2 = 1.0f - std::pow(0.999f, (float)iter);
  const Update u{d_params, d_m, d_v, AdamArgs{lr, bc1, bc2}};
  hipError_t e = grad_step(static_cast<hipStream_t>(stream), desc, L, d_params, d_x, d_t, batch,
                           d_grad, d_loss, &u, w);
  return e == hipSuccess ? QG_OK : dev_fail(e, "mlp training step");
}

qg_status qg_mlp_to_bf16(const qg_mlp_desc* desc, const float* d_params, uint16_t* d_params16,
                         void* stream) {
  if (!valid(desc) || !d_params || !d_params16) return qg::fail(QG_ERR_ARG, "bad arguments");
  qg_mlp_layout L;
  layout(desc, &L);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_to_bf16, dim3(grid1((size_t)L.n_params)), dim3(kThreads), 0, s, d_params,
                     (size_t)L.n_params, d_params16);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? QG_OK : dev_fail(e, "bf16 conversion");
}

qg_status qg_mlp_forward_bf16(const qg_mlp_desc* desc, const uint16_t* d_params16,
                              const float* d_x, int32_t batch, float* d_y, void* d_ws,
                              void* stream) {
  qg_status st = check_common(desc, batch, d_ws);
  if (st != QG_OK) return st;
  if (!d_params16 || !d_x || !d_y) return qg::fail(QG_ERR_ARG, "null buffer");
  qg_mlp_layout L;
  layout(desc, &L);
  const Ws w = carve(desc, batch, d_ws);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int B = batch;
  const void* in = d_x;
  int fan_in = desc->d_in;
  hipError_t e = hipSuccess;
  for (int i = 0; i < desc->depth && e == hipSuccess; ++i) {
    EpiArgs ep{};
    ep.kind = kBiasGeluBf16;
    ep.bias16 = d_params16 + L.b_off[i];
    ep.out16 = w.a16[i & 1];
    const int sl = fit_slices(slices_bf16(B, desc->width, fan_in), B, desc->width, w);
    e = product16(s, in, i == 0, fan_in, d_params16 + L.w_off[i], B, desc->width, fan_in, sl, false,
                  ep, w);
    in = w.a16[i & 1];
    fan_in = desc->width;
  }
  if (e == hipSuccess) {
    EpiArgs ep{};
    ep.kind = kBias;
    ep.bias16 = d_params16 + L.b_off[desc->depth];
    ep.out = d_y;
    // one launch where the output has tiles enough: no second kernel
    const bool whole = tiles_of(B, desc->d_out) >= 64 && fan_in <= 1024;
    const int sl = fit_slices(slices_bf16(B, desc->d_out, fan_in), B, desc->d_out, w);
    e = product16(s, in, false, fan_in, d_params16 + L.w_off[desc->depth], B, desc->d_out, fan_in,
                  sl, whole, ep, w);
  }
  if (e == hipSuccess) e = hipGetLastError();
  return e == hipSuccess ? QG_OK : dev_fail(e, "mlp bf16 forward");
}

}  // extern "C"
