// FP32 products C = P * Q^T on FP32 MFMAs with one wave per tile and no
// barrier: the tiles of few starts, whose cost is the latency of the K loop
// and not arithmetic, and of the grouped solves.
//
// A wave owns a 16 FM x 16 FN tile over the whole K range of its split.  It
// keeps D slabs of 32 K in flight from global memory to registers (8 lanes
// of 16 bytes a row, coalesced), passes each through an LDS slab of its own
// into fragment order, and multiplies with v_mfma_f32_16x16x4_f32.  Within
// 8 consecutive K the MFMAs take k = 0 4 1 5 and 2 6 3 7, so that a sum is
// formed term by term in the order of the 32x32x2 MFMAs of gemm_nt_kernel:
// the same bits as its tiles, whatever the tile.
//
// Bound: latency.  A 16 x 16 tile takes 0.38 us a slab, where its chain of eight
// dependent MFMAs takes 0.11: a slab is written to LDS and read back before its
// first MFMA, and half of the LDS cycles are bank conflicts (8 requests of 16 x 300
// x 1500: matrix cores busy 15% of the CUs' cycles, LDS 43%).  gemm_nt_kernel keeps
// one slab of a workgroup in flight and pays the memory latency, about 2 us, per
// slab: those requests took 47 us per launch there, 14 here.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace spca {
namespace {

typedef float fx4 __attribute__((ext_vector_type(4)));

constexpr int kSlabK = 32;
constexpr int kStreamWaves = 4;  // waves (tiles) per workgroup

template <int FM, int FN>
struct StreamTile {
  static constexpr int kRows = (FM + FN) * 16;     // of P, then of Q
  static constexpr int kLoads = kRows / 8;         // 16-byte loads per lane and slab
  static constexpr int kFloats = kRows * kSlabK;   // LDS floats per wave
};

// One tile: C rows m0.., columns n0.. over K range [kbeg, kend).
template <int FM, int FN, int D>
__device__ __forceinline__ void stream_tile(const float* __restrict__ P, int64_t ldp,
                                            const float* __restrict__ Q, int64_t ldq,
                                            float* __restrict__ Cs, int64_t ldc, int M, int N,
                                            int m0, int n0, int kbeg, int kend, float* slab) {
  using T = StreamTile<FM, FN>;
  const int lane = threadIdx.x % kWave;
  const int lr = lane % 16, lc = lane / 16;
  const int nslabs = kend > kbeg ? (kend - kbeg + kSlabK - 1) / kSlabK : 0;
  const int nfull = kend > kbeg ? (kend - kbeg) / kSlabK : 0;

  // this lane's loads: row 8 v + lane / 8, 16-byte chunk lane % 8
  const int r8 = lane / 8, c8 = lane % 8;
  const float* src[T::kLoads];
#pragma unroll
  for (int v = 0; v < T::kLoads; ++v) {
    const bool isp = v < 2 * FM;
    int row = (isp ? m0 : n0) + (isp ? v : v - 2 * FM) * 8 + r8;
    const int last = isp ? M - 1 : N - 1;
    row = row < last ? row : last;
    src[v] = (isp ? P + (int64_t)row * ldp : Q + (int64_t)row * ldq) + kbeg + 4 * c8;
  }
  fx4 ring[D][T::kLoads];
  auto load = [&](fx4 (&r)[T::kLoads], int s) {
#pragma unroll
    for (int v = 0; v < T::kLoads; ++v)
      r[v] = *reinterpret_cast<const fx4*>(src[v] + s * kSlabK);
  };

  // LDS slab: row r is 128 bytes, its 16-byte chunk c at position c ^ (r & 7)
  const int wr = (r8 * 8 + (c8 ^ r8)) * 4;
  auto put = [&](const fx4 (&r)[T::kLoads]) {
#pragma unroll
    for (int v = 0; v < T::kLoads; ++v) *reinterpret_cast<fx4*>(slab + wr + v * 256) = r[v];
  };
  // fragment of chunk pair c (8 K): lane group lc takes elements lc / 2 and
  // lc / 2 + 2 of 16-byte chunk 2 c + (lc & 1) (reading the whole chunk and
  // selecting put vector instructions between the MFMAs: 15% slower)
  int rd[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    rd[c] = lr * kSlabK + (((2 * c + (lc & 1)) ^ (lr & 7)) << 2) + (lc >> 1);
  struct Frag {
    float x[2][FM + FN];
  };
  auto read = [&](Frag& f, int c) {
#pragma unroll
    for (int b = 0; b < FM + FN; ++b) {
      f.x[0][b] = slab[b * 16 * kSlabK + rd[c]];
      f.x[1][b] = slab[b * 16 * kSlabK + rd[c] + 2];
    }
  };
  fx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
  auto mult = [&](const Frag& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.x[h][FM + j], f.x[h][i], acc[i][j],
                                                           0, 0, 0);
  };
  Frag fr[2];
  // the slab in LDS: four chunk pairs, each read one ahead of its MFMAs (a
  // second LDS slab, written ahead, measured the same)
  auto multiply_slab = [&]() {
    read(fr[0], 0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c + 1 < 4) read(fr[(c + 1) & 1], c + 1);
      mult(fr[c & 1]);
    }
  };
  if (nfull > 0) {
    // D slabs at a time without a branch, so that every wait is for the
    // oldest slab alone; past the last full slab the loads repeat it
    const int last = nfull - 1;
#pragma unroll
    for (int d = 0; d < D; ++d) load(ring[d], d < last ? d : last);
    int s = 0;
    for (; s + D <= nfull; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        put(ring[d]);
        load(ring[d], s + d + D < last ? s + d + D : last);
        multiply_slab();
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (s + d < nfull) {  // wave-uniform
        put(ring[d]);
        multiply_slab();
      }
  }
  if (nfull < nslabs) {  // the partial last slab: zeros from kend on
    const int k = kbeg + nfull * kSlabK + 4 * c8;
#pragma unroll
    for (int v = 0; v < T::kLoads; ++v) {
      const float* x = src[v] + nfull * kSlabK;
      fx4 t = {0.f, 0.f, 0.f, 0.f};
      if (k + 3 < kend) {
        t = *reinterpret_cast<const fx4*>(x);
      } else {
        if (k < kend) t.x = x[0];
        if (k + 1 < kend) t.y = x[1];
        if (k + 2 < kend) t.z = x[2];
      }
      ring[0][v] = t;
    }
    put(ring[0]);
    multiply_slab();
  }

  // C layout (operands swapped): lane holds row lr, columns 4 lc .. 4 lc + 3
  const bool vec = ldc % 4 == 0 && ((uintptr_t)Cs & 15) == 0;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0 + i * 16 + lr;
    if (row >= M) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + j * 16 + 4 * lc;
      float* c = Cs + (int64_t)row * ldc + col;
      if (vec && col + 3 < N) {
        *reinterpret_cast<fx4*>(c) = acc[i][j];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < N) c[e] = acc[i][j][e];
      }
    }
  }
}

// MARKS: only the tiles that hold a mark (common.hpp)
template <int FM, int FN, int D, int OCC, bool MARKS = false>
__global__ __launch_bounds__(kStreamWaves* kWave, OCC) void stream_kernel(
    const float* __restrict__ P, int64_t ldp, const float* __restrict__ Q, int64_t ldq,
    float* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m, int items, int splits,
    int kslabs_per_split, int64_t split_stride, const int32_t* __restrict__ gate,
    int32_t gate_run) {
  __shared__ __attribute__((aligned(16))) float lds[kStreamWaves * StreamTile<FM, FN>::kFloats];
  if (gate != nullptr && *gate != gate_run) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // blocks are dealt to the 8 XCDs in turn: runs of consecutive tiles (the M
  // tiles of one Q tile) stay on one of them
  int b = blockIdx.x;
  const int per_xcd = gridDim.x / 8;
  if (b < per_xcd * 8) b = (b % 8) * per_xcd + b / 8;
  const int item = b * kStreamWaves + wave;
  if (item >= items) return;
  const int per_split = items / splits;
  const int split = item / per_split, t = item % per_split;
  const int kbeg = split * kslabs_per_split * kSlabK;
  int kend = kbeg + kslabs_per_split * kSlabK;
  kend = kend < K ? kend : K;
  const int m0 = (t % tiles_m) * FM * 16, n0 = (t / tiles_m) * FN * 16;
  if (MARKS && !marked<FM * 16, FN * 16>(C, ldc, M, N, m0, n0)) return;
  stream_tile<FM, FN, D>(P, ldp, Q, ldq, C + (int64_t)split * split_stride, ldc, M, N, m0, n0,
                         kbeg, kend, lds + wave * StreamTile<FM, FN>::kFloats);
}

// Grouped products: the tiles of several independent products, each owned
// by the product whose item range holds it.
template <int FM, int FN, int D, int OCC>
__global__ __launch_bounds__(kStreamWaves* kWave, OCC) void stream_group_kernel(
    const GemmGroupDesc* __restrict__ d, int count, int items,
    const int32_t* __restrict__ running) {
  __shared__ __attribute__((aligned(16))) float lds[kStreamWaves * StreamTile<FM, FN>::kFloats];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int item = blockIdx.x * kStreamWaves + wave;
  if (item >= items) return;
  // the last product whose first item is at or below this one (ascending)
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (d[mid].tile0 <= item) lo = mid; else hi = mid - 1;
  }
  const GemmGroupDesc g = d[lo];
  if (running != nullptr && running[g.req] == 0) return;
  const int local = item - g.tile0;
  const int split = local % g.splits, t = local / g.splits;
  const int kbeg = split * g.kslabs_per_split * kSlabK;
  int kend = kbeg + g.kslabs_per_split * kSlabK;
  kend = kend < g.K ? kend : g.K;
  stream_tile<FM, FN, D>(g.P, g.ldp, g.Q, g.ldq, g.C + (int64_t)split * g.split_stride, g.ldc,
                         g.M, g.N, (t % g.tiles_m) * FM * 16, (t / g.tiles_m) * FN * 16, kbeg,
                         kend, lds + wave * StreamTile<FM, FN>::kFloats);
}

// Compiled tiles (FM, FN) and the time of a slab in microseconds, measured over
// 80 products of 1 to 1024 rows.  A workgroup puts one wave on each SIMD of a
// CU; with more workgroups than CUs the times add up.
struct StreamShape {
  int fm, fn;
  double slab_us;
};
constexpr StreamShape kStreamShapes[] = {{4, 2, 1.60}, {2, 4, 1.45}, {2, 2, 0.92},
                                         {4, 1, 1.00}, {1, 2, 0.66}, {1, 1, 0.38}};
constexpr int kNumStream = (int)(sizeof(kStreamShapes) / sizeof(kStreamShapes[0]));

template <int FM, int FN, int D, int OCC>
void launch_stream(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq,
                   float* C, int64_t ldc, int64_t M, int64_t N, int64_t K, int splits,
                   int64_t split_stride, const int32_t* gate, int32_t gate_run, bool marks) {
  const int tm = (int)ceil_div(M, 16 * FM), tn = (int)ceil_div(N, 16 * FN);
  const int per = (int)ceil_div(ceil_div(K, (int64_t)kSlabK), (int64_t)splits);
  const int items = tm * tn * splits;
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(items, kStreamWaves)),
                       dim3(kStreamWaves * kWave), 0, st, P, ldp, Q, ldq, C, ldc, (int)M, (int)N,
                       (int)K, tm, items, splits, per, split_stride, gate, gate_run);
  };
  if (marks)
    run(stream_kernel<FM, FN, D, OCC, true>);
  else
    run(stream_kernel<FM, FN, D, OCC>);
}

}  // namespace

int gemm_num_stream_shapes() { return kNumStream; }
int stream_shape_bm(int shape) {
  const int v = shape - kStreamShape0;
  return v >= 0 && v < kNumStream ? 16 * kStreamShapes[v].fm : 0;
}

// The tile with the least modelled time at a given K split (which the sums
// depend on): 5 us of launch and first loads, then the slabs of a round of
// 256 workgroups one after another.
int model_stream(int64_t M, int64_t N, int64_t K, int splits, double* us_out) {
  int best = 0;
  double best_us = 1e300;
  const int64_t per = ceil_div(ceil_div(K, (int64_t)kSlabK), (int64_t)splits);
  for (int v = 0; v < kNumStream; ++v) {
    const StreamShape& sh = kStreamShapes[v];
    if (sh.fm > 1 && M <= 8 * sh.fm) continue;  // mostly padding rows
    const int64_t items =
        ceil_div(M, (int64_t)16 * sh.fm) * ceil_div(N, (int64_t)16 * sh.fn) * splits;
    const double rounds = (double)ceil_div(items, (int64_t)256 * kStreamWaves);
    const double us = 5.0 + (double)per * sh.slab_us * rounds;
    if (us < best_us) {
      best_us = us;
      best = v;
    }
  }
  *us_out = best_us;
  return best;
}

void gemm_nt_stream(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq,
                    float* C, int64_t ldc, int64_t M, int64_t N, int64_t K, const int32_t* gate,
                    int32_t gate_run, GemmPlan plan, int64_t stride, bool marks) {
  if (M <= 0 || N <= 0) return;
  const int s = plan.splits;
  switch (plan.shape - kStreamShape0) {
    case 0: launch_stream<4, 2, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
    case 1: launch_stream<2, 4, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
    case 2: launch_stream<2, 2, 4, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
    case 3: launch_stream<4, 1, 3, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
    case 4: launch_stream<1, 2, 5, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
    default: launch_stream<1, 1, 8, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K, s, stride, gate, gate_run, marks); break;
  }
}

// Tile of a group's products: 16 x 16 while its tiles fit the chip's SIMDs
// about twice over (the K chain decides), else 32 x 32, which loads each
// operand half as often.
int gemm_group_tiles(GemmGroupDesc* d, int count, int* total_items) {
  auto fill = [&](int f) {
    int64_t t = 0;
    for (int q = 0; q < count; ++q) {
      d[q].tiles_m = (int32_t)ceil_div((int64_t)d[q].M, (int64_t)16 * f);
      const int64_t tiles_n = ceil_div((int64_t)d[q].N, (int64_t)16 * f);
      const int64_t kslabs = ceil_div((int64_t)d[q].K, (int64_t)kSlabK);
      if (d[q].splits < 1) d[q].splits = 1;
      d[q].kslabs_per_split = (int32_t)ceil_div(kslabs, (int64_t)d[q].splits);
      d[q].tile0 = (int32_t)t;
      t += d[q].tiles_m * tiles_n * d[q].splits;
    }
    return t;
  };
  int f = 1;
  int64_t t = fill(f);
  if (t > 2 * 256 * kStreamWaves) t = fill(f = 2);
  *total_items = (int)t;
  return f;
}

void gemm_nt_f32_group(hipStream_t st, const GemmGroupDesc* d_dev, int count, int tile, int items,
                       const int32_t* running) {
  if (count <= 0 || items <= 0) return;
  const dim3 grid((unsigned)ceil_div(items, kStreamWaves)), block(kStreamWaves * kWave);
  if (tile == 1)
    hipLaunchKernelGGL((stream_group_kernel<1, 1, 8, 2>), grid, block, 0, st, d_dev, count, items,
                       running);
  else
    hipLaunchKernelGGL((stream_group_kernel<2, 2, 4, 2>), grid, block, 0, st, d_dev, count, items,
                       running);
}

}  // namespace spca
