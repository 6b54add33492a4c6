// FP32 "NT" GEMM on CDNA4 matrix cores: C = P * Q^T with P (M x K) and
// Q (N x K) both K-contiguous.  Both products of an AM iteration have this
// shape once A is held column-major (for A^T Y) and row-major (for A X):
//   V^T (r x p) = Y^T (r x n) * [A columns] (p x n)^T     K = n
//   U^T (r x n) = X^T (r x p) * [A rows]    (n x p)^T     K = p
//
// Tiling: a workgroup of WM x WN waves owns a BM x BN tile of C; each wave
// owns (BM/WM) x (BN/WN) built from 32 x 32 v_mfma_f32_32x32x2_f32 blocks.
// K advances 32 at a time through two LDS stages: while the waves multiply
// out of one stage, the next K slab is already in registers and is written
// to the other stage, so one barrier per slab suffices.
// Within an 8-wide K chunk, lane l feeds row (l % 32) at k offset
// 4 * (l / 32) .. +3 as one 16-byte LDS read; the i-th of the four MFMAs of
// the chunk takes element i.  The order in which k terms enter the sum does
// not change the product, so every LDS read is 16 bytes wide.
// LDS rows are 128 bytes with no padding; the 16-byte chunk c of row r is
// stored at chunk c ^ ((r ^ (r >> 3)) & 7), so that any 8 consecutive rows
// (and any 16 rows of alternating parity pairs) read at one chunk index
// fall in distinct banks for 32- and 64-bank LDS alike.
// Split-K: when splits > 1, slab range s of every tile writes its partial
// product to C + s * split_stride; the consumer sums the partials in order.
// BF16 operands: the same 128-byte LDS rows hold 64 bf16 of K; each 16-byte
// chunk (8 bf16 of one row) feeds one v_mfma_f32_32x32x16_bf16 instead of
// four FP32 MFMAs, and the products accumulate in FP32.
#include <cmath>
#include <cstdio>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace spca {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kBK = 32;              // floats per LDS row (128 bytes)
constexpr int kChunks = kBK / 4;     // 16-byte chunks per LDS row

// Element traits: how many K elements a 16-byte chunk holds.
template <typename T>
struct Elem;
template <>
struct Elem<float> {
  static constexpr int kPerChunk = 4;
};
template <>
struct Elem<uint16_t> {  // bf16 bit patterns
  static constexpr int kPerChunk = 8;
};

template <int BM, int BN, int WM, int WN>
struct GemmCfg {
  static constexpr int kThreads = WM * WN * kWave;
  static constexpr int kTM = BM / WM;  // rows per wave
  static constexpr int kTN = BN / WN;  // cols per wave
  static constexpr int kFM = kTM / 32;
  static constexpr int kFN = kTN / 32;
  static constexpr int kPVec = BM * kChunks / kThreads;  // float4 per thread
  static constexpr int kQVec = BN * kChunks / kThreads;
  static constexpr int kStage = (BM + BN) * kBK;  // floats per LDS stage
  static_assert(kTM % 32 == 0 && kTN % 32 == 0, "wave tile must be 32-aligned");
  static_assert((BM * kChunks) % kThreads == 0, "P slab load must divide");
  static_assert((BN * kChunks) % kThreads == 0, "Q slab load must divide");
};

__device__ __forceinline__ int swz(int row, int chunk) {
  return row * kBK + ((chunk ^ ((row ^ (row >> 3)) & 7)) << 2);
}

// 16 bytes of row `row` starting at element k (zero past kend or nrows).
template <typename T>
__device__ __forceinline__ floatx4 load_chunk(const T* __restrict__ base,
                                              int64_t ld, int row, int nrows,
                                              int k, int kend) {
  constexpr int E = Elem<T>::kPerChunk;
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  if (row < nrows) {
    const T* p = base + (int64_t)row * ld + k;
    if (k + E - 1 < kend) {
      v = *reinterpret_cast<const floatx4*>(p);
    } else {
      T tmp[E];
#pragma unroll
      for (int e = 0; e < E; ++e) tmp[e] = k + e < kend ? p[e] : T(0);
      v = *reinterpret_cast<const floatx4*>(tmp);
    }
  }
  return v;
}

// One BM x BN tile of C = P * Q^T over K range [kbeg, kend): rows m0.. of P
// and C, rows n0.. of Q (columns of C); lds holds 2 * kStage floats.
// DEPTH = slabs in flight between global memory and LDS: 1 (one register
// set), or 2 (two register sets, the slab loop taken two at a time).
template <typename T, int BM, int BN, int WM, int WN, int DEPTH = 1>
__device__ __forceinline__ void gemm_tile(const T* __restrict__ P, int64_t ldp,
                                          const T* __restrict__ Q, int64_t ldq,
                                          float* __restrict__ Cs, int64_t ldc, int M,
                                          int N, int m0, int n0, int kbeg, int kend,
                                          float* lds) {
  using Cfg = GemmCfg<BM, BN, WM, WN>;
  constexpr int E = Elem<T>::kPerChunk;
  constexpr int SK = kChunks * E;  // K elements per slab
  const int nslabs = kend > kbeg ? (kend - kbeg + SK - 1) / SK : 0;

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = tid / kWave;
  const int wm = wave % WM;
  const int wn = wave / WM;
  const int lrow = lane % 32;
  const int lhalf = lane / 32;

  const T* Pblk = P + (int64_t)m0 * ldp;
  const T* Qblk = Q + (int64_t)n0 * ldq;
  const int mrows = M - m0;
  const int nrows = N - n0;

  floatx16 acc[Cfg::kFM][Cfg::kFN];
#pragma unroll
  for (int i = 0; i < Cfg::kFM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::kFN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  static_assert(DEPTH == 1 || DEPTH == 2, "one or two slabs in flight");
  floatx4 pre_p[DEPTH][Cfg::kPVec];
  floatx4 pre_q[DEPTH][Cfg::kQVec];

  // Small wave tiles (at most two MFMA blocks) load interior slabs of full
  // tiles without per-row or per-K guards, and read the operands of the
  // next 8-wide K chunk from LDS while the current chunk's MFMAs run (two
  // register sets).  Larger wave tiles issue enough MFMAs per LDS read to
  // cover its latency, and measured slower with either change.
  constexpr bool kPrefetch = Cfg::kFM * Cfg::kFN <= 2;
  const bool full_rows = mrows >= BM && nrows >= BN;
  auto fetch = [&](auto set_tag, int k0) {
    constexpr int R = decltype(set_tag)::value;
    if (kPrefetch && full_rows && k0 + SK <= kend) {
#pragma unroll
      for (int v = 0; v < Cfg::kPVec; ++v) {
        const int f = tid + v * Cfg::kThreads;
        pre_p[R][v] = *reinterpret_cast<const floatx4*>(
            Pblk + (int64_t)(f / kChunks) * ldp + k0 + (f % kChunks) * E);
      }
#pragma unroll
      for (int v = 0; v < Cfg::kQVec; ++v) {
        const int f = tid + v * Cfg::kThreads;
        pre_q[R][v] = *reinterpret_cast<const floatx4*>(
            Qblk + (int64_t)(f / kChunks) * ldq + k0 + (f % kChunks) * E);
      }
      return;
    }
#pragma unroll
    for (int v = 0; v < Cfg::kPVec; ++v) {
      int f = tid + v * Cfg::kThreads;
      pre_p[R][v] = load_chunk<T>(Pblk, ldp, f / kChunks, mrows, k0 + (f % kChunks) * E, kend);
    }
#pragma unroll
    for (int v = 0; v < Cfg::kQVec; ++v) {
      int f = tid + v * Cfg::kThreads;
      pre_q[R][v] = load_chunk<T>(Qblk, ldq, f / kChunks, nrows, k0 + (f % kChunks) * E, kend);
    }
  };
  auto stash = [&](auto set_tag, float* st) {
    constexpr int R = decltype(set_tag)::value;
#pragma unroll
    for (int v = 0; v < Cfg::kPVec; ++v) {
      int f = tid + v * Cfg::kThreads;
      *reinterpret_cast<floatx4*>(&st[swz(f / kChunks, f % kChunks)]) = pre_p[R][v];
    }
    float* sq = st + BM * kBK;
#pragma unroll
    for (int v = 0; v < Cfg::kQVec; ++v) {
      int f = tid + v * Cfg::kThreads;
      *reinterpret_cast<floatx4*>(&sq[swz(f / kChunks, f % kChunks)]) = pre_q[R][v];
    }
  };

  // the MFMAs of slab ks, from LDS stage ks & 1
  auto compute = [&](int ks) {
    const float* sp = lds + (ks & 1) * Cfg::kStage;
    const float* sq = sp + BM * kBK;
    floatx4 a[2][Cfg::kFM];
    floatx4 bq[2][Cfg::kFN];
    auto read_ops = [&](int buf, int c8) {
      const int chunk = c8 + lhalf;  // k offset 4 * chunk within the slab
#pragma unroll
      for (int i = 0; i < Cfg::kFM; ++i)
        a[buf][i] = *reinterpret_cast<const floatx4*>(
            &sp[swz(wm * Cfg::kTM + i * 32 + lrow, chunk)]);
#pragma unroll
      for (int j = 0; j < Cfg::kFN; ++j)
        bq[buf][j] = *reinterpret_cast<const floatx4*>(
            &sq[swz(wn * Cfg::kTN + j * 32 + lrow, chunk)]);
    };
    if (kPrefetch) read_ops(0, 0);
#pragma unroll
    for (int c8 = 0; c8 < kChunks; c8 += 2) {
      const int cur = kPrefetch ? (c8 / 2) & 1 : 0;
      if (!kPrefetch) {
        read_ops(0, c8);
      } else if (c8 + 2 < kChunks) {
        read_ops(cur ^ 1, c8 + 2);
        // keep the scheduler from sinking those reads below the MFMAs
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (E == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < Cfg::kFM; ++i)
#pragma unroll
            for (int j = 0; j < Cfg::kFN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][i][e], bq[cur][j][e],
                                                               acc[i][j], 0, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < Cfg::kFM; ++i)
#pragma unroll
          for (int j = 0; j < Cfg::kFN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, a[cur][i]), __builtin_bit_cast(bf16x8, bq[cur][j]),
                acc[i][j], 0, 0, 0);
      }
    }
  };
  using S0 = std::integral_constant<int, 0>;
  if constexpr (DEPTH == 1) {
    if (nslabs > 0) {
      fetch(S0{}, kbeg);
      stash(S0{}, lds);
    }
    __syncthreads();
    for (int ks = 0; ks < nslabs; ++ks) {
      if (ks + 1 < nslabs) fetch(S0{}, kbeg + (ks + 1) * SK);
      compute(ks);
      if (ks + 1 < nslabs) stash(S0{}, lds + ((ks + 1) & 1) * Cfg::kStage);
      __syncthreads();
    }
  } else {
    // slab ks + 2 loads into the register set that slab ks left while
    // slab ks is multiplied and slab ks + 1 waits in the other set
    using S1 = std::integral_constant<int, 1>;
    if (nslabs > 0) {
      fetch(S0{}, kbeg);
      stash(S0{}, lds);
    }
    if (nslabs > 1) fetch(S1{}, kbeg + SK);
    __syncthreads();
    int ks = 0;
    for (; ks + 1 < nslabs; ks += 2) {
      if (ks + 2 < nslabs) fetch(S0{}, kbeg + (ks + 2) * SK);
      compute(ks);
      stash(S1{}, lds + Cfg::kStage);
      __syncthreads();
      if (ks + 3 < nslabs) fetch(S1{}, kbeg + (ks + 3) * SK);
      compute(ks + 1);
      if (ks + 2 < nslabs) stash(S0{}, lds);
      __syncthreads();
    }
    if (ks < nslabs) compute(ks);
  }

  // Accumulator layout of the 32x32 block: register e of lane l holds
  // row 8 * (e / 4) + 4 * (l / 32) + e % 4, column l % 32.
#pragma unroll
  for (int i = 0; i < Cfg::kFM; ++i) {
#pragma unroll
    for (int j = 0; j < Cfg::kFN; ++j) {
      const int col = n0 + wn * Cfg::kTN + j * 32 + lrow;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm * Cfg::kTM + i * 32 + 8 * (e / 4) + 4 * lhalf + (e % 4);
        if (row < M && col < N) Cs[(int64_t)row * ldc + col] = acc[i][j][e];
      }
    }
  }
}

// MARKS: only the tiles that hold a mark (a kernel of its own: one argument more
// cost the products of a solve 1%).
// DEPTH 2 holds two register sets of slabs; its one compiled shape
// (64 x 128) is held to 168 registers so that a CU keeps three workgroups.
template <typename T, int BM, int BN, int WM, int WN, int DEPTH = 1, bool MARKS = false>
__global__ __launch_bounds__(WM* WN* kWave, DEPTH == 2 ? 3 : 1) void gemm_nt_kernel(
    const T* __restrict__ P, int64_t ldp, const T* __restrict__ Q,
    int64_t ldq, float* __restrict__ C, int64_t ldc, int M, int N, int K,
    int tiles_m, int tiles_mn, int splits, int kslabs_per_split,
    int64_t split_stride, const int32_t* __restrict__ gate, int32_t gate_run,
    const int32_t* __restrict__ kdev) {
  using Cfg = GemmCfg<BM, BN, WM, WN>;
  constexpr int SK = kChunks * Elem<T>::kPerChunk;  // K elements per slab
  if (gate != nullptr && *gate != gate_run) return;
  if (kdev != nullptr) {
    K = *kdev;
    kslabs_per_split = (K + SK - 1) / SK;
  }

  __shared__ __attribute__((aligned(16))) float lds[2 * Cfg::kStage];

  // Blocks are dealt to the 8 XCDs round-robin (block b to XCD b mod 8).
  // Unsplit, renumber so that runs of consecutive tiles (the M tiles sharing
  // one Q tile) stay on one XCD and reuse its L2.  Split, keep the split
  // index fastest: with a power-of-two split count the blocks of one K range
  // share XCDs, so each XCD reads only its K ranges of P and Q (the whole P
  // on every XCD cost 12% at 256 x 5000 x 50000 with 8 splits).
  int b = blockIdx.x;
  if (splits == 1) {
    const int per_xcd = tiles_mn / 8;
    if (b < per_xcd * 8) b = (b % 8) * per_xcd + b / 8;
  }
  const int split = b % splits;
  const int t = b / splits;
  const int tm = t % tiles_m;
  const int tn = t / tiles_m;
  const int kbeg = split * kslabs_per_split * SK;
  int kend = kbeg + kslabs_per_split * SK;
  kend = kend < K ? kend : K;
  // (a wave stores only after the barriers of the K loop: all have looked)
  if (MARKS && !marked<BM, BN>(C, ldc, M, N, tm * BM, tn * BN)) return;
  gemm_tile<T, BM, BN, WM, WN, DEPTH>(P, ldp, Q, ldq, C + (int64_t)split * split_stride, ldc,
                               M, N, tm * BM, tn * BN, kbeg, kend, lds);
}

// Compiled tile shapes.  occ = workgroups a CU holds at once (LDS and
// registers); eff = relative MFMA efficiency of the shape measured on
// MI355X (larger per-wave tiles reuse each LDS read for more MFMAs); eff16
// the same for BF16 operands, where a tile's operand bytes per MFMA (global
// and LDS) limit it long before the matrix cores do, so the largest tiles
// win (measured on 256 x 50000 x 5000 and 256 x 5000 x 50000); with one
// workgroup per CU, 8 waves (two per SIMD) hide more of its load latency
// than 4.  A shape with eff (eff16) 0 is never planned for FP32 (BF16) by
// the model, only by the autotuner.
struct Shape {
  int bm, bn, occ;
  double eff, eff16;
};
constexpr Shape kShapes[] = {
    {128, 128, 2, 1.00, 0.73},  // 2x2 waves of 64x64
    {128, 160, 2, 1.00, 0.80},  // 4x1 waves of 32x160
    {128, 96, 2, 0.92, 0.73},   // 4x1 waves of 32x96
    {128, 64, 3, 0.85, 0.64},   // 2x2 waves of 64x32
    {64, 128, 3, 0.85, 0.65},   // 2x2 waves of 32x64
    {32, 128, 3, 0.70, 0.48},   // 1x4 waves of 32x32
    {64, 256, 2, 0.85, 0.57},   // 1x4 waves of 64x64
    {256, 128, 1, 0.90, 0.85},  // 2x2 waves of 128x64
    {256, 256, 1, 0.90, 1.25},  // 2x2 waves of 128x128
    {256, 256, 1, 0.0, 1.36},   // 2x4 waves of 128x64: BF16 only (2 waves per SIMD)
    {256, 256, 1, 0.0, 0.0},    // 4x2 waves of 64x128: tuning candidate only
    {64, 128, 3, 0.0, 0.0},     // 2x2 waves of 32x64, two slabs in flight: tuning candidate only
};
constexpr int kNumShapes = (int)(sizeof(kShapes) / sizeof(kShapes[0]));

template <typename T, int BM, int BN, int WM, int WN, int DEPTH = 1>
void launch(hipStream_t st, const T* P, int64_t ldp, const T* Q,
            int64_t ldq, float* C, int64_t ldc, int64_t M, int64_t N,
            int64_t K, int splits, int64_t split_stride, const int32_t* gate,
            int32_t gate_run, const int32_t* kdev, bool marks) {
  const int tiles_m = (int)ceil_div(M, BM);
  const int tiles_n = (int)ceil_div(N, BN);
  const int kslabs = (int)ceil_div(K, kChunks * Elem<T>::kPerChunk);
  const int per_split = (int)ceil_div(kslabs, splits);
  const int total = tiles_m * tiles_n * splits;
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(total), dim3(WM * WN * kWave), 0, st, P, ldp, Q, ldq, C, ldc,
                       (int)M, (int)N, (int)K, tiles_m, tiles_m * tiles_n, splits, per_split,
                       split_stride, gate, gate_run, kdev);
  };
  if constexpr (std::is_same_v<T, float>) {
    if (marks) {
      run(gemm_nt_kernel<T, BM, BN, WM, WN, DEPTH, true>);
      return;
    }
  }
  run(gemm_nt_kernel<T, BM, BN, WM, WN, DEPTH>);
}

template <typename T>
void dispatch(int shape, hipStream_t st, const T* P, int64_t ldp,
              const T* Q, int64_t ldq, float* C, int64_t ldc, int64_t M,
              int64_t N, int64_t K, int splits, int64_t split_stride,
              const int32_t* gate, int32_t gate_run, const int32_t* kdev, bool marks) {
  switch (shape) {
    case 0:
      launch<T, 128, 128, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 1:
      launch<T, 128, 160, 4, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 2:
      launch<T, 128, 96, 4, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 3:
      launch<T, 128, 64, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 4:
      launch<T, 64, 128, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 5:
      launch<T, 32, 128, 1, 4>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 6:
      launch<T, 64, 256, 1, 4>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 7:
      launch<T, 256, 128, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 8:
      launch<T, 256, 256, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 9:
      launch<T, 256, 256, 2, 4>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    case 10:
      launch<T, 256, 256, 4, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
    default:
      launch<T, 64, 128, 2, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, splits, split_stride, gate, gate_run, kdev, marks);
      break;
  }
}

}  // namespace

// Choice of tile shape and K split: a measured winner from the tuning table
// when there is one, else the deterministic model below.
// Model of one launch, in cycles of one CU:
//   a workgroup's MFMA work  w = BM * BN * (K slabs per split * 32)
//                               / (128 MACs per cycle * eff);
//   the workgroups fill rounds of 256 CUs x occ slots; a CU running k
//   workgroups at once takes w * max(k, 1.5) (one workgroup alone cannot
//   keep the matrix cores busy), so the partial last round costs
//   w * max(ceil(rest / 256), 1.5);
//   split partials cost their HBM traffic, 8 bytes per element per split at
//   about 1.7 KB per cycle for the whole chip.
// ---------------------------------------------------------------------------
// Tuning table: measured winners keyed by element width, max splits and the
// half-octave buckets of M, N and K (round(2 log2 x)).  Filled by the
// autotuner of the solve (or imported as text); consulted before the model.
// ---------------------------------------------------------------------------
namespace {
struct TuneKey {
  int eb, ms, bm, bn, bk;
  bool operator<(const TuneKey& o) const {
    if (eb != o.eb) return eb < o.eb;
    if (ms != o.ms) return ms < o.ms;
    if (bm != o.bm) return bm < o.bm;
    if (bn != o.bn) return bn < o.bn;
    return bk < o.bk;
  }
};
std::mutex g_tune_mu;
std::map<TuneKey, GemmPlan> g_tune;

int bucket(int64_t x) { return (int)std::lround(2.0 * std::log2((double)(x > 0 ? x : 1))); }
// a workgroup tile, or (FP32 only) a one-wave or a BF16-part tile
bool shape_known(int shape, int eb) {
  return (shape >= 0 && shape < kNumShapes) ||
         (eb == 4 && shape >= kStreamShape0 && shape < kStreamShape0 + gemm_num_stream_shapes()) ||
         (eb == 4 && shape >= kSplitShape0 && shape < kSplitShape0 + gemm_num_split_shapes());
}
TuneKey key_of(int64_t M, int64_t N, int64_t K, int ms, int eb) {
  return TuneKey{eb, ms, bucket(M), bucket(N), bucket(K)};
}
}  // namespace

bool tuned_plan(int64_t M, int64_t N, int64_t K, int max_splits, int elem_bytes,
                GemmPlan* out) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(key_of(M, N, K, max_splits, elem_bytes));
  if (it == g_tune.end()) return false;
  *out = it->second;
  return true;
}

void record_tuned_plan(int64_t M, int64_t N, int64_t K, int max_splits,
                       int elem_bytes, GemmPlan plan) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune[key_of(M, N, K, max_splits, elem_bytes)] = plan;
}

std::string tune_table_text() {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  std::ostringstream os;
  for (const auto& kv : g_tune)
    os << kv.first.eb << ' ' << kv.first.ms << ' ' << kv.first.bm << ' ' << kv.first.bn
       << ' ' << kv.first.bk << ' ' << kv.second.shape << ' ' << kv.second.splits << '\n';
  return os.str();
}

bool tune_table_load(const char* text, std::string* err) {
  std::map<TuneKey, GemmPlan> t;
  std::istringstream is(text);
  std::string line;
  int ln = 0;
  while (std::getline(is, line)) {
    ++ln;
    if (line.find_first_not_of(" \t\r") == std::string::npos) continue;
    std::istringstream ls(line);
    TuneKey k;
    GemmPlan g;
    if (!(ls >> k.eb >> k.ms >> k.bm >> k.bn >> k.bk >> g.shape >> g.splits) ||
        (k.eb != 2 && k.eb != 4) || !shape_known(g.shape, k.eb) || g.splits < 1 ||
        g.splits > k.ms) {
      *err = "bad tuning entry on line " + std::to_string(ln);
      return false;
    }
    t[k] = g;
  }
  std::lock_guard<std::mutex> lock(g_tune_mu);
  for (const auto& kv : t) g_tune[kv.first] = kv.second;
  return true;
}

void tune_table_clear() {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune.clear();
}

int max_feasible_splits(int64_t K, int max_splits, int elem_bytes) {
  const int64_t kslabs = ceil_div(K, 128 / elem_bytes);
  int s = 1;
  while (s * 2 <= max_splits && ceil_div(kslabs, (int64_t)s * 2) >= 8) s *= 2;
  return s;
}

GemmPlan plan_gemm_nt(int64_t M, int64_t N, int64_t K, int max_splits,
                      int elem_bytes) {
  {
    // a tuning-table entry covers a size bucket: its split count is capped
    // at what this K allows, which is what callers size split buffers for
    GemmPlan t;
    if (tuned_plan(M, N, K, max_splits, elem_bytes, &t)) {
      const int cap = max_feasible_splits(K, max_splits, elem_bytes);
      if (t.splits > cap) t.splits = cap;
      if (t.splits < 1) t.splits = 1;
      return t;
    }
  }
  return model_plan_gemm_nt(M, N, K, max_splits, elem_bytes);
}

namespace {
// modelled time of a plan of model_plan_gemm_nt: its cycles take 1.2 times as
// long as at 2.4 GHz, plus the launch
double f32_model_us(double cycles) { return cycles * 1.2 / 2400.0 + 3.0; }
}  // namespace

GemmPlan plan_f32(int64_t M, int64_t N, int64_t K, int max_splits, double* us_out) {
  GemmPlan t;
  if (us_out != nullptr) *us_out = 0.0;
  if (tuned_plan(M, N, K, max_splits, 4, &t) && t.shape < kSplitShape0)
    return plan_gemm_nt(M, N, K, max_splits, 4);
  double cycles = 0.0, stream_us = 0.0;
  GemmPlan g = model_plan_gemm_nt(M, N, K, max_splits, 4, &cycles);
  double us = f32_model_us(cycles);
  // One-wave tiles where few tiles and a long K loop leave the workgroup
  // tiles waiting for memory: 16 x 1000 x 8000 24 to 12 us, 12 x 162 x 24937
  // 57 to 21, 339 x 653 x 10114 76 to 61, 64 x 2000 x 20000 72 to 65.  From 128
  // rows on the workgroup tiles without padding do up to a tenth better than
  // their model, hence the margin there: 128 x 10000 x 1000 35 us on them and
  // 40 on one-wave tiles, 1024 x 1000 x 1250 34 and 36, 256 x 10000 x 1000
  // (in a solve) 56.5 and 62.
  const int v = model_stream(M, N, K, g.splits, &stream_us);
  if (stream_us < (M >= 128 ? 0.9 : 1.0) * us) {
    us = stream_us;
    g.shape = kStreamShape0 + v;
  }
  if (us_out != nullptr) *us_out = us;
  return g;
}

GemmPlan plan_product_f32(int64_t M, int64_t N, int64_t K, int64_t ldp, int64_t ldq) {
  const bool split = split_possible(K, ldp, ldq);
  GemmPlan t;
  if (tuned_plan(M, N, K, 1, 4, &t)) {
    // an entry covers a size bucket, in which K may be too small for it
    if (t.shape >= kSplitShape0 && !split) return model_plan_gemm_nt(M, N, K, 1, 4);
    return plan_gemm_nt(M, N, K, 1, 4);
  }
  // Both models in microseconds, and 3 us for a launch, 7 for the two of the large
  // tiles.  Over 140 sizes of 1 to 1024 rows, K from 192 to 50000, the choice is 2%
  // from the better one of both, the parts up to 20 times faster; the FP32 tiles
  // stay ahead where K is short (300 x 45359 x 240: 87 us on them, 100 on parts;
  // 62 x 24975 x 434: 27 and 34).
  double us = 0.0, parts_us = 0.0;
  const GemmPlan f32 = plan_f32(M, N, K, 1, &us);
  if (!split) return f32;
  const int parts = model_plan_split(M, N, K, &parts_us);
  return parts_us + (split_own_redo(parts) ? 3.0 : 7.0) < us ? GemmPlan{parts, 1} : f32;
}

GemmPlan model_plan_gemm_nt(int64_t M, int64_t N, int64_t K, int max_splits,
                            int elem_bytes, double* cycles_out) {
  GemmPlan best{0, 1};
  double best_cost = 1e300;
  const int64_t slab_k = 128 / elem_bytes;
  const int64_t kslabs = ceil_div(K, slab_k);
  // MACs per cycle per CU: FP32 MFMA 128; BF16 operands are limited by
  // operand traffic well below their MFMA rate, taken as 4x FP32 times the
  // shape's BF16 efficiency
  const double macs = elem_bytes == 4 ? 128.0 : 512.0;
  for (int s = 0; s < kNumShapes; ++s) {
    const Shape& sh = kShapes[s];
    if (sh.bm > 32 && M <= sh.bm / 2) continue;  // mostly padding rows
    const int64_t tiles = ceil_div(M, sh.bm) * ceil_div(N, sh.bn);
    for (int splits = 1; splits <= max_splits; splits *= 2) {
      const int64_t per = ceil_div(kslabs, splits);
      if (splits > 1 && per < 8) break;  // too little K per split
      const int64_t wgs = tiles * splits;
      const int64_t slots = 256LL * sh.occ;
      const double eff = elem_bytes == 4 ? sh.eff : sh.eff16;
      const double w = (double)sh.bm * sh.bn * (double)(per * slab_k) / (macs * eff);
      const int64_t full = wgs / slots;
      const int64_t rest = wgs % slots;
      double cost = (double)full * w * (sh.occ > 1.5 ? sh.occ : 1.5);
      if (rest > 0) {
        double k = (double)ceil_div(rest, 256);
        cost += w * (k > 1.5 ? k : 1.5);
      }
      if (splits > 1) cost += (double)splits * M * N * 8.0 / 1700.0;
      if (cost < best_cost * 0.999) {
        best_cost = cost;
        best = GemmPlan{s, splits};
      }
    }
  }
  if (cycles_out != nullptr) *cycles_out = best_cost;
  return best;
}

// Microseconds per slab of 64 K and round of workgroups, by shape, on a chip that
// is less than full: a workgroup waits for each slab (measured over the same
// products as the tiles of gemm_bf16.hip; long K costs up to half more, which
// leaves the other side ahead there all the more).
double gemm_bf16_us(int64_t M, int64_t N, int64_t K, int shape) {
  constexpr double kStep[] = {1.5, 1.7, 1.15, 1.2, 1.5, 0.78, 1.5, 2.0, 2.6, 2.6, 2.6, 1.3};
  static_assert(sizeof(kStep) / sizeof(kStep[0]) == kNumShapes, "one step per shape");
  const Shape& sh = kShapes[shape];
  const int64_t tiles = ceil_div(M, (int64_t)sh.bm) * ceil_div(N, (int64_t)sh.bn);
  double step = kStep[shape];
  if (sh.bm == 32) step += 0.3 * (tiles < 300 ? (double)tiles / 300.0 : 1.0);
  return 3.0 + (double)ceil_div(tiles, (int64_t)256 * sh.occ) *
                   (double)ceil_div(K, (int64_t)64) * step;
}

int gemm_num_shapes() { return kNumShapes; }
int gemm_shape_bm(int shape) {
  if (shape >= kSplitShape0) return split_shape_bm(shape);
  if (shape >= kStreamShape0) return stream_shape_bm(shape);
  return shape >= 0 && shape < kNumShapes ? kShapes[shape].bm : 0;
}

void gemm_nt_f32(hipStream_t st, const float* P, int64_t ldp, const float* Q,
                 int64_t ldq, float* C, int64_t ldc, int64_t M, int64_t N,
                 int64_t K, const int32_t* gate, int32_t gate_run,
                 GemmPlan plan, int64_t split_stride, const int32_t* kdev, bool marks) {
  if (M <= 0 || N <= 0) return;
  if (plan.shape >= kSplitShape0) {
    gemm_nt_split(st, P, ldp, Q, ldq, C, ldc, M, N, K, plan.shape);
    return;
  }
  if (plan.shape >= kStreamShape0) {
    gemm_nt_stream(st, P, ldp, Q, ldq, C, ldc, M, N, K, gate, gate_run, plan, split_stride,
                   marks);
    return;
  }
  if (kdev != nullptr) plan.splits = 1;
  dispatch<float>(plan.shape, st, P, ldp, Q, ldq, C, ldc, M, N, K, plan.splits,
                  split_stride, gate, gate_run, kdev, marks);
}

void gemm_nt_bf16(hipStream_t st, const uint16_t* P, int64_t ldp,
                  const uint16_t* Q, int64_t ldq, float* C, int64_t ldc,
                  int64_t M, int64_t N, int64_t K, const int32_t* gate,
                  int32_t gate_run, GemmPlan plan, int64_t split_stride) {
  if (M <= 0 || N <= 0) return;
  dispatch<uint16_t>(plan.shape, st, P, ldp, Q, ldq, C, ldc, M, N, K,
                     plan.splits, split_stride, gate, gate_run, nullptr, false);
}

}  // namespace spca
