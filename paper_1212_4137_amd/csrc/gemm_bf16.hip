// BF16 products C = P * Q^T (FP32 accumulation and output) whose K is shared
// by the waves of a workgroup: wave w of a 16 FM x 16 FN tile takes the slabs
// w, w + waves, ... of 64 K (one 128-byte line a row), keeps D of them in
// flight from global memory to LDS buffers of its own, and multiplies with no
// barrier in the loop; the partial tiles are summed in wave order at the end.
// A workgroup so has up to 128 KB under way, which is what reading operands at
// the memory's rate takes, and a product of few tiles still has eight waves a
// CU.  Bound: the operands' way from L2, 64 bytes a cycle and CU.
// The tiles of gemm_nt_kernel, which share a slab in LDS, load it once per
// workgroup and stay ahead where many workgroups of the largest tiles fill
// the chip (256 x 50000 x 5000: 200 us, 355 us here); with few tiles they
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

// Compiled tiles.  One workgroup per CU takes, in microseconds, `fixed` and
// `step` per slab of a wave, up to `step_full` with a workgroup on every CU
// (measured over 90 products of 16 to 1024 rows; good to a quarter).
struct KsShape {
  int bm, bn, waves;
  double step, step_full, fixed;
};
constexpr KsShape kKsShapes[] = {
    {16, 16, 8, 0.40, 0.50, 0.7}, {16, 32, 8, 0.42, 1.05, 1.3}, {32, 32, 8, 0.55, 1.10, 1.5},
    {64, 64, 8, 2.10, 3.20, 2.0}, {128, 64, 4, 1.60, 2.80, 3.0},
};

// The quickest of those, and its time.
int plan_ks(int64_t M, int64_t N, int64_t K, double* us_out) {
  int best = 0;
  double best_us = 1e300;
  for (int v = 0; v < (int)(sizeof(kKsShapes) / sizeof(kKsShapes[0])); ++v) {
    const KsShape& s = kKsShapes[v];
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

bool gemm_nt_bf16_ks(hipStream_t st, const uint16_t* P, int64_t ldp, const uint16_t* Q,
                     int64_t ldq, float* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                     double other_us) {
  if (M <= 0 || N <= 0 || K < kSlabK) return false;
  double us;
  const int v = plan_ks(M, N, K, &us);
  if (us >= 0.9 * other_us) return false;
  switch (v) {
    case 0: launch_ks<1, 1, 8, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 1: launch_ks<1, 2, 8, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 2: launch_ks<2, 2, 8, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 3: launch_ks<4, 4, 8, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    default: launch_ks<8, 4, 4, 1>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
  }
  return true;
}

}  // namespace spca
