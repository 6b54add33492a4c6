// BF16 products C = P * Q^T (FP32 accumulation and output) with the operands
// loaded straight to LDS.
//
// Small tiles whose K is shared by the waves of a workgroup: wave w of a 16 FM x 16 FN tile takes the slabs
// w, w + waves, ... of 64 K (one 128-byte line a row), keeps D of them in
// flight from global memory to LDS buffers of its own, and multiplies with no
// barrier in the loop; the partial tiles are summed in wave order at the end.
// A workgroup so has up to 128 KB under way, which is what reading operands at
// the memory's rate takes, and a product of few tiles still has eight waves a
// CU.  Bound: the operands' way from L2, 64 bytes a cycle and CU.
// The tiles of gemm_nt_kernel, which share a slab in LDS, load it once per
// workgroup and stay ahead where many workgroups of large tiles fill the chip
// (1024 x 10000 x 1000: 37 us, 73 us here); with few tiles they
// wait 0.8 to 1.5 us for every slab: 22 x 3040 x 15296 348 us, 20 us here;
// 64 x 1000 x 10000 126 and 12.6; 1024 x 1000 x 10000 216 and 50;
// 485 x 4931 x 26761 661 and 346.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace spca {
namespace {

typedef float fx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int kSlabK = 64;  // K per slab

template <int FM, int FN, int W, int D>
constexpr size_t lds_bytes() {
  const size_t slabs = (size_t)W * D * (FM + FN) * 2048;
  const size_t parts = (size_t)(W / 2) * FM * FN * 1024;
  return slabs > parts ? slabs : parts;
}

// the 8 K from k on of a row, zero from kend on
__device__ __forceinline__ bf8 load_tail(const uint16_t* __restrict__ row, int k, int kend) {
  uint16_t t[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = k + e < kend ? row[k + e] : (uint16_t)0;
  bf8 v;
  __builtin_memcpy(&v, t, sizeof(v));
  return v;
}

template <int FM, int FN, int W, int D>
__global__ __launch_bounds__(W* kWave, (W + 3) / 4) void bf16_ks_kernel(
    const uint16_t* __restrict__ P, int64_t ldp, const uint16_t* __restrict__ Q, int64_t ldq,
    float* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m) {
  constexpr int RB = (FM + FN) * 16;  // rows of a slab: P's, then Q's
  constexpr int NL = RB / 8;          // loads of a slab
  static_assert((D - 1) * NL < 64, "vmcnt counts to 63");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lr = lane % 16, lc = lane / 16;
  // runs of consecutive tiles (the M tiles sharing one Q tile) on one XCD
  int b = blockIdx.x;
  const int per_xcd = (int)gridDim.x / 8;
  if (b < per_xcd * 8) b = (b % 8) * per_xcd + b / 8;
  const int m0 = (b % tiles_m) * 16 * FM, n0 = (b / tiles_m) * 16 * FN;
  const int nfull = K / kSlabK;
  const char* Pb = reinterpret_cast<const char*>(P + (int64_t)m0 * ldp);
  const char* Qb = reinterpret_cast<const char*>(Q + (int64_t)n0 * ldq);

  fx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
  bf8 p[FM][2], q[FN][2];
  auto multiply = [&] {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q[j][h], p[i][h], acc[i][j], 0, 0, 0);
  };

  // buffers of this wave: row r is 128 bytes, its 16-byte chunk c at position
  // c ^ (r & 7); 8 lanes load a row, rows past the end repeat the last one
  char* mine = lds + wave * (D * RB * 128);
  int64_t off[NL];
  {
    const int r8 = lane / 8, ch = (lane % 8) ^ r8;
#pragma unroll
    for (int v = 0; v < NL; ++v) {
      const bool isp = v < 2 * FM;
      int row = (isp ? v : v - 2 * FM) * 8 + r8;
      const int last = isp ? M - 1 - m0 : N - 1 - n0;
      row = row < last ? row : last;
      off[v] = (int64_t)row * (isp ? ldp : ldq) * 2 + 16 * ch;
    }
  }
  auto load_slab = [&](int ks, int buf) {
#pragma unroll
    for (int v = 0; v < NL; ++v)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)((v < 2 * FM ? Pb : Qb) +
                                                          (int64_t)ks * (2 * kSlabK) + off[v]),
          (__attribute__((address_space(3))) void*)(mine + buf * (RB * 128) + v * 1024), 16, 0, 0);
  };
  const int rd0 = lr * 128 + ((lc ^ (lr & 7)) * 16);
  const int rd1 = lr * 128 + (((4 + lc) ^ (lr & 7)) * 16);
  if (wave < nfull) {
    // slabs past the end repeat the last one, so that the count of loads in
    // flight is always the same
    const int last = nfull - 1 - (nfull - 1 - wave) % W;
    auto slab = [&](int t) { return wave + t * W < nfull ? wave + t * W : last; };
#pragma unroll
    for (int d = 0; d < D; ++d) load_slab(slab(d), d);
    const int steps = (nfull - wave + W - 1) / W;
    int buf = 0;
    for (int t = 0; t < steps; ++t) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * NL) : "memory");  // slab t is in LDS
      const char* sl = mine + buf * (RB * 128);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        p[i][0] = *reinterpret_cast<const bf8*>(sl + i * 2048 + rd0);
        p[i][1] = *reinterpret_cast<const bf8*>(sl + i * 2048 + rd1);
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        q[j][0] = *reinterpret_cast<const bf8*>(sl + (FM + j) * 2048 + rd0);
        q[j][1] = *reinterpret_cast<const bf8*>(sl + (FM + j) * 2048 + rd1);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // and now in registers
      load_slab(slab(t + D), buf);
      __builtin_amdgcn_sched_barrier(0);
      multiply();
      buf = buf + 1 < D ? buf + 1 : 0;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  if (nfull * kSlabK < K && wave == nfull % W) {  // the partial last slab
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = i * 16 + lr < M - m0 ? i * 16 + lr : M - 1 - m0;
      const uint16_t* s = P + (int64_t)(m0 + row) * ldp;
      p[i][0] = load_tail(s, nfull * kSlabK + 8 * lc, K);
      p[i][1] = load_tail(s, nfull * kSlabK + 32 + 8 * lc, K);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int row = j * 16 + lr < N - n0 ? j * 16 + lr : N - 1 - n0;
      const uint16_t* s = Q + (int64_t)(n0 + row) * ldq;
      q[j][0] = load_tail(s, nfull * kSlabK + 8 * lc, K);
      q[j][1] = load_tail(s, nfull * kSlabK + 32 + 8 * lc, K);
    }
    multiply();
  }

  // the waves' partial tiles: the upper half through LDS to the lower half,
  // which adds them, then every wave sums its share of the blocks
  constexpr int FB = FM * FN, H = W / 2;
  fx4* L = reinterpret_cast<fx4*>(lds);
  __syncthreads();  // the slabs are read
  if (wave >= H) {
#pragma unroll
    for (int x = 0; x < FB; ++x) L[((wave - H) * FB + x) * kWave + lane] = acc[x / FN][x % FN];
  }
  __syncthreads();
  if (wave < H) {
#pragma unroll
    for (int x = 0; x < FB; ++x) {
      fx4* s = &L[(wave * FB + x) * kWave + lane];
      *s = acc[x / FN][x % FN] + *s;
    }
  }
  __syncthreads();
  const bool vec = ldc % 4 == 0 && ((uintptr_t)C & 15) == 0;
  for (int x = wave; x < FB; x += W) {
    fx4 s = L[x * kWave + lane];
#pragma unroll
    for (int w = 1; w < H; ++w) s += L[(w * FB + x) * kWave + lane];
    // register e of lane (lr, lc): row lr of P, column 4 lc + e
    const int row = m0 + (x / FN) * 16 + lr, col = n0 + (x % FN) * 16 + 4 * lc;
    if (row >= M) continue;
    float* c = C + (int64_t)row * ldc + col;
    if (vec && col + 3 < N) {
      *reinterpret_cast<fx4*>(c) = s;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e < N) c[e] = s[e];
    }
  }
}

template <int FM, int FN, int W, int D>
void launch_ks(hipStream_t st, const uint16_t* P, int64_t ldp, const uint16_t* Q, int64_t ldq,
               float* C, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  constexpr size_t lds = lds_bytes<FM, FN, W, D>();
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  const int64_t tm = ceil_div(M, (int64_t)16 * FM), tn = ceil_div(N, (int64_t)16 * FN);
  hipLaunchKernelGGL((bf16_ks_kernel<FM, FN, W, D>), dim3((unsigned)(tm * tn)), dim3(W * kWave),
                     lds, st, P, ldp, Q, ldq, C, ldc, (int)M, (int)N, (int)K, (int)tm);
}

// ---------------------------------------------------------------------------
// Large tiles, 256 x 224 per workgroup of 8 waves (4 of 64 rows by 2 of 112
// columns): the products that fill most CUs with those and are bound by
// reading Q once, 256 x 50000 x 5000 in one round of 224 workgroups.  Q's
// slabs of 64 K go straight to LDS two stages ahead (three buffers), P's, which
// come from L2, one (two buffers): 148 KB.  The two waves of a SIMD work in
// turns, one multiplying from registers while the other reads its fragments,
// and the loads go out between the MFMAs.  Bound: the loads to LDS, 30 GB/s a
// CU; 159 us at that size (gemm_nt_kernel, slabs through registers one stage
// ahead: 200 us; 32 K a stage, half lines: 214; the loads in one burst: 171).
// ---------------------------------------------------------------------------
constexpr int kTM = 256, kTN = 224, kTW = 8;
constexpr int kStageP = kTM * 128, kStageQ = kTN * 128;  // bytes
constexpr int kQ0 = 2 * kStageP;                         // Q's stages in LDS
constexpr size_t kTileLds = kQ0 + 3 * kStageQ;

__global__ __launch_bounds__(kTW* kWave, 2) void bf16_tile_kernel(
    const uint16_t* __restrict__ P, int64_t ldp, const uint16_t* __restrict__ Q, int64_t ldq,
    float* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m) {
  constexpr int FM = 4, FN = 7;
  constexpr int NLP = kTM / 8 / kTW;              // a wave's loads of a stage
  constexpr int NLQ = (kTN / 8 + kTW - 1) / kTW;  // (some repeat the last)
  static_assert(NLP <= FN && NLQ <= FN, "loads between the MFMAs");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wm = wave % 4, wn = wave / 4;
  const int lr = lane % 16, lc = lane / 16;
  int b = blockIdx.x;
  const int per_xcd = (int)gridDim.x / 8;
  if (b < per_xcd * 8) b = (b % 8) * per_xcd + b / 8;
  const int m0 = (b % tiles_m) * kTM, n0 = (b / tiles_m) * kTN;
  const int nfull = K / kSlabK;

  fx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
  bf8 p[FM], q[FN];

  // a wave load: 8 rows of 128 bytes, row r's chunk c at position c ^ (r % 8);
  // rows past the end repeat the last
  const char* src_p[NLP];
  const char* src_q[NLQ];
  int dst_q[NLQ];
  {
    const int r8 = lane / 8, ch = (lane % 8) ^ r8;
#pragma unroll
    for (int v = 0; v < NLP; ++v) {
      const int row = m0 + (wave + v * kTW) * 8 + r8;
      src_p[v] = reinterpret_cast<const char*>(P + (int64_t)(row < M ? row : M - 1) * ldp) + 16 * ch;
    }
#pragma unroll
    for (int v = 0; v < NLQ; ++v) {
      int g = wave + v * kTW;
      g = g < kTN / 8 ? g : kTN / 8 - 1;
      const int row = n0 + g * 8 + r8;
      src_q[v] = reinterpret_cast<const char*>(Q + (int64_t)(row < N ? row : N - 1) * ldq) + 16 * ch;
      dst_q[v] = g * 1024;
    }
  }
  auto to_lds = [&](const char* src, int t, int at) {
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src + (int64_t)(t < nfull ? t : nfull - 1) *
                                                                  (2 * kSlabK)),
        (__attribute__((address_space(3))) void*)(lds + at), 16, 0, 0);
  };
  auto load_p = [&](int t, int v) {
    to_lds(src_p[v], t, (t & 1) * kStageP + (wave + v * kTW) * 1024);
  };
  auto load_q = [&](int t, int buf, int v) {
    to_lds(src_q[v], t, kQ0 + buf * kStageQ + dst_q[v]);
  };
  const int rd[2] = {lr * 128 + ((lc ^ (lr & 7)) * 16), lr * 128 + (((4 + lc) ^ (lr & 7)) * 16)};
  if (nfull > 0) {
#pragma unroll
    for (int v = 0; v < NLQ; ++v) load_q(0, 0, v);
#pragma unroll
    for (int v = 0; v < NLP; ++v) load_p(0, v);
#pragma unroll
    for (int v = 0; v < NLQ; ++v) load_q(1, 1, v);
  }
  auto read = [&](int t, int buf, int h) {
    const char* sp = lds + (t & 1) * kStageP + wm * 8192 + rd[h];
    const char* sq = lds + kQ0 + buf * kStageQ + wn * (FN * 2048) + rd[h];
#pragma unroll
    for (int i = 0; i < FM; ++i) p[i] = *reinterpret_cast<const bf8*>(sp + i * 2048);
#pragma unroll
    for (int j = 0; j < FN; ++j) q[j] = *reinterpret_cast<const bf8*>(sq + j * 2048);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the MFMAs of what was read, a load issued every four
  auto multiply = [&](auto load) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      load(j);
#pragma unroll
      for (int i = 0; i < FM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q[j], p[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto turn = [&] { asm volatile("s_barrier" ::: "memory"); };
  auto begin = [&] {  // behind the barrier stage t is in LDS, stage t - 1 read
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NLQ) : "memory");
  };
  auto none = [](int) {};
  int buf = 0, prev = 2;  // Q's stages of t and t - 1 (then t + 2)
  auto next = [&] {
    prev = buf;
    buf = buf < 2 ? buf + 1 : 0;
  };
  if (wn == 0) {
    for (int t = 0; t < nfull; ++t) {
      auto lp = [&](int v) { if (v < NLP) load_p(t + 1, v); };
      auto lq = [&](int v) { if (v < NLQ) load_q(t + 2, prev, v); };
      begin();
      read(t, buf, 0);
      turn();
      multiply(lp);
      turn();
      read(t, buf, 1);
      turn();
      multiply(lq);
      next();
    }
  } else if (nfull > 0) {
    begin();
#pragma unroll
    for (int v = 0; v < NLP; ++v) load_p(1, v);
    turn();
    read(0, buf, 0);
    turn();
    multiply([&](int v) { if (v < NLQ) load_q(2, prev, v); });
    turn();
    read(0, buf, 1);
    next();
    for (int t = 1; t < nfull; ++t) {
      auto lp = [&](int v) { if (v < NLP) load_p(t + 1, v); };
      auto lq = [&](int v) { if (v < NLQ) load_q(t + 2, prev, v); };
      begin();
      multiply(lp);
      turn();
      read(t, buf, 0);
      turn();
      multiply(lq);
      turn();
      read(t, buf, 1);
      next();
    }
    multiply(none);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (nfull * kSlabK < K) {  // the partial last slab, straight from memory
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = nfull * kSlabK + 32 * h + 8 * lc;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = m0 + wm * 64 + i * 16 + lr;
        p[i] = load_tail(P + (int64_t)(row < M ? row : M - 1) * ldp, k, K);
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int row = n0 + wn * 16 * FN + j * 16 + lr;
        q[j] = load_tail(Q + (int64_t)(row < N ? row : N - 1) * ldq, k, K);
      }
      multiply(none);
    }
  }
  const bool vec = ldc % 4 == 0 && ((uintptr_t)C & 15) == 0;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0 + wm * 64 + i * 16 + lr;
    if (row >= M) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * 16 * FN + j * 16 + 4 * lc;
      float* c = C + (int64_t)row * ldc + col;
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

void launch_tile(hipStream_t st, const uint16_t* P, int64_t ldp, const uint16_t* Q, int64_t ldq,
                 float* C, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  const int64_t tm = ceil_div(M, (int64_t)kTM), tn = ceil_div(N, (int64_t)kTN);
  hipLaunchKernelGGL(bf16_tile_kernel, dim3((unsigned)(tm * tn)), dim3(kTW * kWave), kTileLds, st,
                     P, ldp, Q, ldq, C, ldc, (int)M, (int)N, (int)K, (int)tm);
}

// Compiled tiles.  One workgroup per CU takes, in microseconds, `fixed` and
// `step` per slab of a wave, up to `step_full` with a workgroup on every CU
// (measured over 90 products of 16 to 1024 rows; good to a quarter).  The large
// tile's waves take every slab.
struct KsShape {
  int bm, bn, waves;
  double step, step_full, fixed;
};
constexpr KsShape kKsShapes[] = {
    {16, 16, 8, 0.40, 0.50, 0.7}, {16, 32, 8, 0.42, 1.05, 1.3}, {32, 32, 8, 0.55, 1.10, 1.5},
    {64, 64, 8, 2.10, 3.20, 2.0}, {128, 64, 4, 1.60, 2.80, 3.0}, {kTM, kTN, 1, 1.40, 2.00, 9.0},
};
constexpr int kNumKs = (int)(sizeof(kKsShapes) / sizeof(kKsShapes[0]));

// The quickest of those, and its time.
int plan_ks(int64_t M, int64_t N, int64_t K, double* us_out) {
  int best = 0;
  double best_us = 1e300;
  for (int v = 0; v < kNumKs; ++v) {
    const KsShape& s = kKsShapes[v];
    if (M <= s.bm / 2 && s.bm > 64) continue;  // mostly padding rows
    const int64_t wgs = ceil_div(M, (int64_t)s.bm) * ceil_div(N, (int64_t)s.bn);
    const double steps = (double)ceil_div(ceil_div(K, (int64_t)kSlabK), (int64_t)s.waves);
    const int64_t full = wgs / 256, rest = wgs % 256;
    double us = 3.0 + (double)full * (steps * s.step_full + s.fixed);
    if (rest > 0)
      us += steps * (s.step + (s.step_full - s.step) * (double)rest / 256.0) + s.fixed;
    if (us < best_us) {
      best_us = us;
      best = v;
    }
  }
  *us_out = best_us;
  return best;
}

}  // namespace

bool bf16_direct_possible(int shape, int64_t K) {
  return shape >= kBf16Shape0 && shape < kBf16Shape0 + kNumKs && K >= kSlabK;
}

int plan_bf16_direct(int64_t M, int64_t N, int64_t K, double other_us) {
  if (K < kSlabK) return -1;
  double us;
  const int v = plan_ks(M, N, K, &us);
  return us >= 0.9 * other_us ? -1 : kBf16Shape0 + v;
}

void gemm_nt_bf16_direct(hipStream_t st, const uint16_t* P, int64_t ldp, const uint16_t* Q,
                         int64_t ldq, float* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                         int shape) {
  if (M <= 0 || N <= 0) return;
  switch (shape - kBf16Shape0) {
    case 0: launch_ks<1, 1, 8, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 1: launch_ks<1, 2, 8, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 2: launch_ks<2, 2, 8, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 3: launch_ks<4, 4, 8, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 4: launch_ks<8, 4, 4, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    default: launch_tile(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
  }
}

}  // namespace spca
