// FP32 products on the BF16 matrix cores: C = P * Q^T with FP32 operands,
// each operand split on the fly into three BF16 parts whose sum is the FP32
// value exactly (8 significant bits each, round to nearest),
//   x = h + m + l,  h = bf16(x),  m = bf16(x - h),  l = bf16(x - h - m),
// and the products h h', h m', m h', m m', h l', l h' accumulated in FP32.
// The three left out (m l', l m', l l') are below 2^-24 of the product, the
// size of one FP32 rounding; a sum of K terms is rounded up to six times per 32
// K instead of once per term, so that of dense rows the error against FP64 is
// below that of the FP32 matrix instructions (normwise, unit Gaussian rows, K =
// 1000: 2.1e-7 and 1.6e-7 for the two kernels below, FP32 MFMA 5.7e-7).  The
// BF16 rate is 16 times the FP32 one (2.5 PFLOP/s against 157 TFLOP/s), so six
// products cost 3/8 of the FP32 ones.
//
// What the parts do not serve, the FP32 MFMAs compute, in the order and with the
// bits of the FP32 tiles: rows with many zeros (see kFull), and 16 x 16 blocks of
// C with a sum that overflows, holds an infinity or NaN, or lies so low that parts
// of an operand fall under the BF16 or FP32 range (see suspect).  The small tiles
// do so themselves; the large ones mark such blocks (common.hpp), and a second
// launch computes the FP32 tiles that hold a mark, which takes 3 to 5 us where it
// finds none.  1024 x 10000 x 1000: 113 us dense, 189 with 5 nonzeros in each row
// of P, 280 with a NaN in every sum, on the FP32 tiles 180; 64 x 2000 x 20000: 90,
// 150, 232 and 770.
//
// split_pp_kernel, large tiles (256 x 160 or 256 x 128 per workgroup of 8
// waves, 64 x 80 or 64 x 64 per wave): both operands staged through LDS as
// BF16 parts in MFMA fragment order, two stages of 32 K.  The two waves of a
// SIMD work in turns (an s_barrier per half step): while one issues its 120
// MFMAs from registers, converting its share of a later slab between them,
// the other writes converted parts to LDS and reads its next fragments.
// Bound: the matrix cores and the vector ALUs that feed them, at the clock that the
// chip's power allows (1024 x 10000 x 1000: busy 59% and 55% of the CUs' cycles at
// 2.06 GHz, 86% of the CUs holding a tile).  There 113 us with the second launch
// (FP32 MFMA 180 us); of that 7 us go to the separate small sums; without the turns
// (one barrier per slab) 112 us where the loop as of then took 100, with 32 x 32
// MFMAs 119-123.
//
// split_ks_kernel, small tiles (16 FM x 16 FN) of which the waves of a
// workgroup share K: wave w takes the slabs w, w + waves, ..., loads them
// into an LDS slab of its own (coalesced, global to LDS), converts them in
// fragment order and multiplies, with no barrier in the loop; the partial
// tiles are summed in wave order at the end.  Bound: the conversions (7 vector
// instructions per operand element; one of them finds thin rows, 2 to 12% of the
// time; vector ALUs busy 68% of the CUs' cycles, matrix cores 46%).  Used where
// large tiles leave CUs idle: 1024 x 1000 x 10000 135 us (FP32 MFMA 401 us), 64 x
// 2000 x 20000 90 us (770 us), 16 x 300 x 1500 11 us (55 us).
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"

namespace spca {
namespace {

typedef float fx4 __attribute__((ext_vector_type(4)));
typedef float fx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef uint32_t ux2 __attribute__((ext_vector_type(2)));
typedef uint32_t ux4 __attribute__((ext_vector_type(4)));
typedef uint16_t us2 __attribute__((ext_vector_type(2)));

constexpr int kSlab = 32;  // K per slab: one 16x16x32 MFMA deep
static_assert(kSplitMinK >= kSlab, "split_pp_kernel may load the first slab of any row");

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const fx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2));
}
__device__ __forceinline__ float low_of(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ float high_of(uint32_t h) { return __uint_as_float(h & 0xffff0000u); }

// The BF16 parts of four consecutive FP32 values; amax gathers the largest
// magnitude.
constexpr int NP = 3;  // parts of a value
__device__ __forceinline__ void split4(fx4 x, ux2 (&w)[NP], float& amax) {
  amax = fmaxf(fmaxf(amax, fabsf(x.x)), fabsf(x.y));
  amax = fmaxf(fmaxf(amax, fabsf(x.z)), fabsf(x.w));
  uint32_t a = pack_bf16(x.x, x.y), b = pack_bf16(x.z, x.w);
  w[0] = ux2{a, b};
  const float r0 = x.x - low_of(a), r1 = x.y - high_of(a);
  const float r2 = x.z - low_of(b), r3 = x.w - high_of(b);
  a = pack_bf16(r0, r1);
  b = pack_bf16(r2, r3);
  w[1] = ux2{a, b};
  w[2] = ux2{pack_bf16(r0 - low_of(a), r1 - high_of(a)),
             pack_bf16(r2 - low_of(b), r3 - high_of(b))};
}

// Marks a register value as changed, so that what is derived from it is computed
// again and not held.
__device__ __forceinline__ void reload(int& x) { asm volatile("" : "+v"(x)); }

// Four consecutive values of a row from K position k (zero from kend on).
__device__ __forceinline__ fx4 load_tail(const float* s, int k, int kend) {
  fx4 r = {0.f, 0.f, 0.f, 0.f};
  if (k + 3 < kend) {
    r = *reinterpret_cast<const fx4*>(s);
  } else {
    if (k < kend) r.x = s[0];
    if (k + 1 < kend) r.y = s[1];
    if (k + 2 < kend) r.z = s[2];
  }
  return r;
}

// the part products of one block column, smallest terms first: all but h h'
// into small[i], h h' into acc[i] (the two may be the same)
template <int FM>
__device__ __forceinline__ void mfma_parts(const bf8 (&q)[3], const bf8 (&p)[FM][NP],
                                           fx4 (&small)[FM], fx4 (&acc)[FM]) {
  auto mm = [&](int a, int b, fx4 (&c)[FM]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
      c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q[b], p[i][a], c[i], 0, 0, 0);
  };
  mm(0, 2, small);
  mm(2, 0, small);
  mm(1, 1, small);
  mm(0, 1, small);
  mm(1, 0, small);
  mm(0, 0, acc);
}

// Which rows the parts serve.  A sum over n nonzero terms is rounded n times by
// the FP32 instructions and up to six times per slab of 32 K by the parts, so
// these are more exact where a slab holds more terms than that and less exact
// where most terms are zero (P with 5 nonzeros a row, K = 1000 and 10000:
// 5.5e-8 against 4.4e-8).  A row is fit if at least 5/8 of its quads (4
// consecutive K; in the small tiles, of its octets) hold values of 2^-40 and more
// alone: two such rows share a quarter of all quads, 8 terms a slab.  A row of
// zeros is fit as well, its sums are exact.  Rows are looked at while they are
// converted.
constexpr float kFull = 0x1p-40f;
constexpr int kZeroRow = -(1 << 30);

// the lanes whose quad is not full, from the first parts of its values
__device__ __forceinline__ uint64_t thin_quad(ux2 h) {
  const ux2 m = h & 0x7fff7fffu;
  const us2 least = __builtin_elementwise_min(__builtin_bit_cast(us2, m.x),
                                              __builtin_bit_cast(us2, m.y));
  const us2 full = {0x2b80, 0x2b80};  // 2^-40 in BF16
  return __ballot(__builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(full, least)) != 0u);
}

// What a workgroup knows of its ROWS rows, P's first (in LDS).
template <int ROWS>
struct Fitness {
  int thin[ROWS];       // thin quads; negative for a row of zeros
  int unfit, nonzero;   // unfit_start: by the counts, by the rows looked through
  int n, list[64];      // those
  __device__ __forceinline__ void clear() {
    for (int i = threadIdx.x; i < ROWS; i += blockDim.x) thin[i] = 0;
    if (threadIdx.x == 0) unfit = nonzero = n = 0;
  }
};

// behind an s_barrier that waits for LDS alone: loads stay in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// From the first slabs, `seen` counts a row in thin[] and `pad` in each that lie
// past K: whether the tile is to go to the FP32 instructions at once, because a row
// has most of its quads thin, beyond what a fit row would show by chance (P with 5
// nonzeros a row, 1024 x 10000 x 1000: 189 us; 278 when that shows at the end).
// Rows that have shown nothing are looked through in memory: rows of zeros are fit
// (up to 64 of them), rows with a nonzero are not.
// All threads call it, behind a barrier, and get the same answer.
template <int ROWS>
__device__ __forceinline__ bool unfit_start(Fitness<ROWS>& f, int rows_p, int seen, int pad,
                                            const char* Pb, int64_t ldp, int last_p,
                                            const char* Qb, int64_t ldq, int last_q, int K) {
  constexpr int kMost = sizeof(f.list) / sizeof(f.list[0]);
  for (int row = threadIdx.x; row < ROWS; row += blockDim.x) {
    const int t = f.thin[row] - pad;
    if (t >= seen) {
      const int at = atomicAdd(&f.n, 1);
      if (at < kMost)
        f.list[at] = row;
      else
        f.unfit = 1;
    } else if (t > 5 * seen / 8 + 2) {
      f.unfit = 1;
    }
  }
  lds_barrier();
  const int n = f.n;
  if (f.unfit) return true;  // (not written any more)
  if (n == 0) return false;
  for (int c = 0; c < n; ++c) {
    const bool isp = f.list[c] < rows_p;
    const int i = isp ? f.list[c] : f.list[c] - rows_p, last = isp ? last_p : last_q;
    const float* x = reinterpret_cast<const float*>(isp ? Pb : Qb) +
                     (int64_t)(i < last ? i : last) * (isp ? ldp : ldq);
    bool any = false;
#pragma unroll 4
    for (int k = 4 * threadIdx.x; k < K; k += 4 * blockDim.x) {
      const fx4 v = load_tail(x + k, k, K);
      any |= v.x != 0.f || v.y != 0.f || v.z != 0.f || v.w != 0.f;
    }
    if (any) __hip_atomic_store(&f.nonzero, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    // (seen early or late: the answer is the same)
    if (__hip_atomic_load(&f.nonzero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
  }
  lds_barrier();
  if (f.nonzero) return true;
  if ((int)threadIdx.x < n) f.thin[f.list[threadIdx.x]] = kZeroRow;
  lds_barrier();
  return false;
}

// Whether a sum of fit rows may have lost accuracy to the range of the parts.
// With K <= 2^31 terms, B the largest magnitude of the operands in the tile:
// parts under 2^-133 lose at most 2^-134 B per term and products under
// 2^-126 at most their own size, so sums of at least 2^-80 (1 + B) keep
// FP32 accuracy for K up to 2^20.  A sum of exactly zero lost no more than that
// either, and its terms, an eighth of them 2^-80 or more, are rounded to 2^-104
// and more by the FP32 instructions: for B up to 2^28.  Overflow, infinities and
// NaN show as a sum that is not finite.
__device__ __forceinline__ bool suspect(float s, bool zero_row, float big) {
  const float a = fabsf(s);
  if (!(a <= 3.4028234e38f)) return true;
  if (a == 0.f) return !zero_row && big > 0x1p28f;
  return a < 0x1p-80f * (1.f + big);
}

// Four consecutive columns of C (16-byte aligned)
__device__ __forceinline__ void store_cols(float* c, int col, int N, fx4 v) {
  if (col + 3 < N) {
    *reinterpret_cast<fx4*>(c) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (col + e < N) c[e] = v[e];
  }
}

__device__ __forceinline__ void mark_block(float* C, int64_t ldc, int M, int N, int row,
                                           int col) {
  if (row < M && col < N) C[(int64_t)row * ldc + col] = __uint_as_float(kMark);
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, kWave));
  return x;
}

// Block -> tile as in gemm_nt_kernel: runs of consecutive tiles stay on one XCD
// (blocks are dealt to the 8 XCDs in turn).
__device__ __forceinline__ int tile_of(int b, int tiles) {
  const int per_xcd = tiles / 8;
  return b < per_xcd * 8 ? (b % 8) * per_xcd + b / 8 : b;
}

// ---------------------------------------------------------------------------
// Large tiles
// ---------------------------------------------------------------------------

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(WM* WN* kWave, 2) void split_pp_kernel(
    const float* __restrict__ P, int64_t ldp, const float* __restrict__ Q, int64_t ldq,
    float* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m, int tiles_mn) {
  constexpr int NT = WM * WN * kWave;
  constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
  constexpr int RPV = NT / 8;  // rows per load round (8 lanes of 16 bytes a row)
  constexpr int VP = BM / RPV, VQ = (BN + RPV - 1) / RPV, VN = VP + VQ;
  constexpr int kPBytes = BM / 16 * NP * 1024;
  constexpr int kStage = kPBytes + BN / 16 * 3 * 1024;
  static_assert(BM % RPV == 0 && TM % 16 == 0 && TN % 16 == 0, "tile split");
  __shared__ __attribute__((aligned(16))) char lds[2 * kStage];
  __shared__ __attribute__((aligned(16))) Fitness<BM + BN> fit;

  const int tile = tile_of(blockIdx.x, tiles_mn);
  const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
  // slabs: a partial one (K not a multiple of 32) goes first, where the
  // loop's loads need no guard for it
  const int nfull = K / kSlab;
  const int part = K % kSlab != 0 ? 1 : 0;
  const int nslabs = nfull + part;

  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave % WM, wn = wave / WM;
  const int frow = tid / 8, c4 = tid % 8;

  // byte offsets of this lane's loads from the tile's first rows
  const char* Pb = reinterpret_cast<const char*>(P + (int64_t)m0 * ldp);
  const char* Qb = reinterpret_cast<const char*>(Q + (int64_t)n0 * ldq);
  uint32_t po[VP], qo[VQ];
#pragma unroll
  for (int v = 0; v < VP; ++v) {
    int row = frow + v * RPV;
    row = m0 + row < M ? row : M - 1 - m0;
    po[v] = (uint32_t)row * (uint32_t)ldp * 4u + 16u * c4;
  }
#pragma unroll
  for (int v = 0; v < VQ; ++v) {
    int row = frow + v * RPV;
    row = n0 + row < N ? row : N - 1 - n0;
    qo[v] = (uint32_t)row * (uint32_t)ldq * 4u + 16u * c4;
  }
  struct Regs {
    fx4 p[VP], q[VQ];
  };
  auto kbyte = [&](int sl) {  // byte offset of a full slab within a row
    return (sl - part) * 4 * kSlab;
  };
  auto fetch = [&](Regs& r, int sl) {
    if (sl < part) {
      const int k = nfull * kSlab + 4 * c4;
#pragma unroll
      for (int v = 0; v < VP; ++v)
        r.p[v] = load_tail(reinterpret_cast<const float*>(Pb + nfull * 4 * kSlab + po[v]), k, K);
#pragma unroll
      for (int v = 0; v < VQ; ++v)
        r.q[v] = load_tail(reinterpret_cast<const float*>(Qb + nfull * 4 * kSlab + qo[v]), k, K);
    } else {
      const int kb = kbyte(sl);
#pragma unroll
      for (int v = 0; v < VP; ++v) r.p[v] = *reinterpret_cast<const fx4*>(Pb + kb + po[v]);
#pragma unroll
      for (int v = 0; v < VQ; ++v) r.q[v] = *reinterpret_cast<const fx4*>(Qb + kb + qo[v]);
    }
  };
  Regs rg;

  // LDS: blocks of 16 rows x 32 K per part (1 KB), the 16-byte chunk c of
  // row r at slot 16 c + (r ^ 2 c), so that the 8-byte writes of two rows
  // and the fragment reads (lane l: row l % 16, chunk l / 16) are both free
  // of bank conflicts
  float big = 0.f;
  ux2 kp[VP][NP], kq[VQ][3];
  auto convert = [&](const Regs& r, int v) {
    if (v < VP)
      split4(r.p[v], kp[v], big);
    else
      split4(r.q[v - VP], kq[v - VP], big);
  };
  // of the slab in kp and kq (thin quads are few)
  auto count_thin = [&] {
    uint64_t thins[VN], any = 0;
#pragma unroll
    for (int v = 0; v < VN; ++v) {
      thins[v] = thin_quad(v < VP ? kp[v][0] : kq[v - VP][0]);
      any |= thins[v];
    }
    if (any == 0) return;
    int first = threadIdx.x;
    reload(first);  // nothing of this is held through the loop
    first /= 8;
#pragma unroll
    for (int v = 0; v < VN; ++v) {
      const int row = first + (v < VP ? v : v - VP) * RPV;
      if (__builtin_amdgcn_inverse_ballot_w64(thins[v]) && (v < VP || row < BN))
        atomicAdd(&fit.thin[v < VP ? row : BM + row], 1);
    }
  };
  const int wc = c4 / 2;
  const int woff = (wc * 16 + ((frow & 15) ^ (2 * wc))) * 16 + (c4 & 1) * 8;
  auto write_parts = [&](char* st) {
#pragma unroll
    for (int v = 0; v < VP; ++v) {
      char* b = st + ((frow + v * RPV) / 16) * NP * 1024 + woff;
#pragma unroll
      for (int q = 0; q < NP; ++q) *reinterpret_cast<ux2*>(b + q * 1024) = kp[v][q];
    }
#pragma unroll
    for (int v = 0; v < VQ; ++v) {
      if (BN % RPV == 0 || v + 1 < VQ || frow + v * RPV < BN) {
        char* b = st + kPBytes + ((frow + v * RPV) / 16) * 3072 + woff;
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<ux2*>(b + q * 1024) = kq[v][q];
      }
    }
  };
  const int slot = ((lane / 16) * 16 + ((lane % 16) ^ (2 * (lane / 16)))) * 16;
  bf8 pf[FM][NP], qf[FN][3];
  auto read_frags = [&](const char* st) {
    const char* sp = st + wm * FM * NP * 1024 + slot;
    const char* sq = st + kPBytes + wn * FN * 3072 + slot;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int q = 0; q < NP; ++q)
        pf[i][q] = *reinterpret_cast<const bf8*>(sp + (i * NP + q) * 1024);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        qf[j][q] = *reinterpret_cast<const bf8*>(sq + (j * 3 + q) * 1024);
  };
  // end of a half step: this wave's LDS accesses are done, then all meet
  auto turn = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  fx4 acc[FN][FM];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int i = 0; i < FM; ++i) acc[j][i] = fx4{0.f, 0.f, 0.f, 0.f};

  fit.clear();
  __syncthreads();
  const int pad = part ? 8 - K % kSlab / 4 : 0;  // quads of the partial slab that are not full
  {
    // slab 0 in stage 0, slab 1 converted in registers, slab 2 in flight;
    // past the last slab the loads repeat it (the copies are never read)
    const int last = nslabs - 1;
    {
      Regs r0, r1;
      fetch(r0, 0);
      fetch(r1, last < 1 ? last : 1);
      fetch(rg, last < 2 ? last : 2);
#pragma unroll
      for (int v = 0; v < VN; ++v) convert(r0, v);
      write_parts(lds);
      count_thin();
#pragma unroll
      for (int v = 0; v < VN; ++v) convert(r1, v);
      count_thin();
    }
    const bool second = wave >= WM * WN / 2;  // the other wave of each SIMD
    __syncthreads();
    if (unfit_start(fit, BM, 16 - pad, pad, Pb, ldp, M - 1 - m0, Qb, ldq, N - 1 - n0, K)) {
      for (int b = tid; b < BM / 16 * (BN / 16); b += NT)
        mark_block(C, ldc, M, N, m0 + b % (BM / 16) * 16, n0 + b / (BM / 16) * 16);
      return;
    }
    // Order of LDS accesses, half step by half step (first | second waves):
    // slab s is written to stage s & 1 in half steps 2s - 2 | 2s - 1 and
    // read in 2s | 2s + 1; it replaces slab s - 2, read in 2s - 4 | 2s - 3.
    if (second) turn();
    for (int ks = 0; ks < nslabs; ++ks) {
      write_parts(lds + ((ks + 1) & 1) * kStage);
      if (ks > 0 && ks < last) count_thin();  // (slabs 0 and 1 are counted)
      read_frags(lds + (ks & 1) * kStage);
      turn();
      // (with a single, partial slab: the rows' first 32 entries, which K >=
      // kSplitMinK makes sure of; never used)
      const int kn = ks + 3 < last ? ks + 3 : last;
      const int kb = kn < part ? 0 : kbyte(kn);
      const char* Pn = Pb + kb;
      const char* Qn = Qb + kb;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        // the small products from zero, then added to the sum that takes
        // h h': two roundings at its size per slab instead of six
        fx4 small[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) small[i] = fx4{0.f, 0.f, 0.f, 0.f};
        mfma_parts<FM>(qf[j], pf, small, acc[j]);
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[j][i] += small[i];
#pragma unroll
        for (int v = 0; v < VN; ++v) {
          if (v * FN / VN != j) continue;
          convert(rg, v);
          if (v < VP)
            rg.p[v] = *reinterpret_cast<const fx4*>(Pn + po[v]);
          else
            rg.q[v - VP] = *reinterpret_cast<const fx4*>(Qn + qo[v - VP]);
        }
        // two vector instructions in the shadow of every MFMA
#pragma unroll
        for (int g = 0; g < FM * 6; ++g) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 2, 0);
        }
      }
      turn();
    }
    if (!second) turn();
  }
  // the operands' largest magnitudes over the whole tile
  float* red = reinterpret_cast<float*>(lds);
  big = wave_max(big);
  if (lane == 0) red[wave] = big;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WM * WN; ++w) big = fmaxf(big, red[w]);

  float* Cs = C;
  const bool vec = ldc % 4 == 0 && ((uintptr_t)Cs & 15) == 0;
  const int lr = lane % 16, lc = lane / 16;
  // Rows of C that are not 16-byte aligned go through LDS, 16 rows of the
  // wave's tile at a time, so that the 4-byte stores of a wave still cover
  // whole rows (387 x 22611 x 334: 74 to 71 us)
  constexpr int kRow = TN + 4;
  float* strip = reinterpret_cast<float*>(lds) + 64 + wave * 16 * kRow;
  static_assert((64 + WM * WN * 16 * kRow) * 4 <= 2 * kStage, "row strips fit in the stages");
  auto store_blocks = [&](int i, auto block) {  // the FN blocks of row block i
    const int r0 = m0 + wm * TM + i * 16, c0 = n0 + wn * TN;
    if (vec) {
      if (r0 + lr < M) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int col = c0 + j * 16 + 4 * lc;
          store_cols(Cs + (int64_t)(r0 + lr) * ldc + col, col, N, block(j));
        }
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < FN; ++j)
      *reinterpret_cast<fx4*>(strip + lr * kRow + j * 16 + 4 * lc) = block(j);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int e = lane; e < 16 * TN; e += kWave) {
      const int r = e / TN, c = e % TN;
      if (r0 + r < M && c0 + c < N) Cs[(int64_t)(r0 + r) * ldc + c0 + c] = strip[r * kRow + c];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  };
  // a row of blocks with a sum that the parts cannot serve is marked instead
  const int limit = K / 4 * 3 / 8 + pad;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int tp = fit.thin[wm * TM + i * 16 + lr];
    bool bad = tp > limit;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int* tq = &fit.thin[BM + wn * TN + j * 16 + 4 * lc];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        bad |= tq[e] > limit || suspect(acc[j][i][e], tp < 0 || tq[e] < 0, big);
    }
    if (!__any(bad)) {  // wave-uniform
      store_blocks(i, [&](int j) { return acc[j][i]; });
    } else if (lane < FN) {
      mark_block(Cs, ldc, M, N, m0 + wm * TM + i * 16, n0 + wn * TN + lane * 16);
    }
  }
}

// ---------------------------------------------------------------------------
// Small tiles, K shared by the waves
// ---------------------------------------------------------------------------

// Tiles of at most 8 blocks compute what the parts cannot serve themselves, a
// block a wave, and need no second launch (61 x 3001 x 777: 11.4 us, with one 14.7).
template <int FM, int FN>
constexpr bool kOwnRedo = FM * FN <= 8;
constexpr int kRing = 4;  // slabs in flight to LDS there

// LDS bytes of a workgroup: the slabs of its waves, at the end the partial tiles
// of half of them, and the rings of f32_block
template <int FM, int FN>
constexpr size_t ks_lds_bytes(int waves) {
  const size_t slabs = (size_t)waves * (FM + FN) * 2048;
  const size_t parts = (size_t)((waves + 1) / 2) * FM * FN * 1024;
  const size_t rings =
      kOwnRedo<FM, FN> ? (size_t)(FM * FN < waves ? FM * FN : waves) * kRing * 4096 : 0;
  const size_t most = slabs > parts ? slabs : parts;
  return most > rings ? most : rings;
}

// One 16 x 16 block (C layout of the 16x16 MFMAs; rows m0.. of P, n0.. of Q) on
// FP32 MFMAs in the order of gemm_nt_kernel (8 K at a time: 0 4, 1 5, 2 6, 3 7):
// its bits.  One wave; kRing slabs go straight to its ring of LDS.  Bound: the
// chain of MFMAs, and the slabs' way from memory.
__device__ __forceinline__ fx4 f32_block(const float* __restrict__ P, int64_t ldp,
                                         const float* __restrict__ Q, int64_t ldq, int M, int N,
                                         int m0, int n0, int K, char* ring) {
  const int lane = threadIdx.x % kWave, lr = lane % 16, lc = lane / 16;
  const int nfull = K / kSlab;
  // a slab: P's 16 rows, then Q's, of 128 bytes; row r's chunk c at position c ^ (r & 7)
  const float* src[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r8 = lane / 8, row = (v < 2 ? m0 : n0) + v % 2 * 8 + r8;
    const int last = v < 2 ? M - 1 : N - 1;
    src[v] = (v < 2 ? P + (int64_t)(row < last ? row : last) * ldp
                    : Q + (int64_t)(row < last ? row : last) * ldq) + 4 * ((lane % 8) ^ r8);
  }
  auto load = [&](int s, int buf) {
    const int at = s < nfull ? s : nfull - 1;  // past the end the last one again
#pragma unroll
    for (int v = 0; v < 4; ++v)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(src[v] + (int64_t)at * kSlab),
          (__attribute__((address_space(3))) void*)(ring + buf * 4096 + v * 1024), 16, 0, 0);
  };
  fx4 c = {0.f, 0.f, 0.f, 0.f};
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads below are the only ones counted
#pragma unroll
  for (int d = 0; d < kRing; ++d) load(d, d);
  for (int s = 0, buf = 0; s < nfull; ++s, buf = buf + 1 < kRing ? buf + 1 : 0) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kRing - 1) * 4) : "memory");
    const float* x = reinterpret_cast<const float*>(ring + buf * 4096);
    float p[4][2], q[4][2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int at = lr * kSlab + (((2 * e + (lc & 1)) ^ (lr & 7)) << 2) + (lc >> 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        p[e][h] = x[at + 2 * h];
        q[e][h] = x[16 * kSlab + at + 2 * h];
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // in registers
    load(s + kRing, buf);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(q[e][h], p[e][h], c, 0, 0, 0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (nfull * kSlab < K) {  // the partial last slab
    const float* pr = P + (int64_t)(m0 + lr < M ? m0 + lr : M - 1) * ldp;
    const float* qr = Q + (int64_t)(n0 + lr < N ? n0 + lr : N - 1) * ldq;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = nfull * kSlab + 4 * (2 * e + (lc & 1)) + (lc >> 1) + 2 * h;
        const float a = k < K ? qr[k] : 0.f, b = k < K ? pr[k] : 0.f;
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
      }
  }
  return c;
}

template <int FM, int FN>
__device__ __forceinline__ void ks_tile(const float* __restrict__ P, int64_t ldp,
                                        const float* __restrict__ Q, int64_t ldq,
                                        float* __restrict__ Cs, int64_t ldc, int M, int N, int m0,
                                        int n0, int K, char* lds, float* red,
                                        Fitness<(FM + FN) * 16>& fit) {
  constexpr int RB = (FM + FN) * 16;  // rows of a slab: P's, then Q's
  constexpr int FB = FM * FN;
  const int nslabs = (K + kSlab - 1) / kSlab, nfull = K / kSlab;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nw = blockDim.x / kWave;
  const int lr = lane % 16, lc = lane / 16;
  const char* Pb = reinterpret_cast<const char*>(P + (int64_t)m0 * ldp);
  const char* Qb = reinterpret_cast<const char*>(Q + (int64_t)n0 * ldq);

  float big = 0.f;
  // a fragment: lane (row lr, lc) holds k = 4 lc .. +3 and 16 + 4 lc .. +3
  auto split_frag = [&](const fx4 (&x)[2], bf8 (&out)[NP]) {
    ux2 a[NP], b[NP];
    split4(x[0], a, big);
    split4(x[1], b, big);
#pragma unroll
    for (int q = 0; q < NP; ++q)
      out[q] = __builtin_bit_cast(bf8, ux4{a[q].x, a[q].y, b[q].x, b[q].y});
  };
  fx4 acc[FN][FM];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int i = 0; i < FM; ++i) acc[j][i] = fx4{0.f, 0.f, 0.f, 0.f};
  bf8 pf[FM][NP];
  fx4 rp[FM][2], rq[FN][2];
  // thin octets (two quads) of this lane's part of every row, two rows a register
  uint32_t thin[(FM + FN + 1) / 2];
#pragma unroll
  for (int f = 0; f < (FM + FN + 1) / 2; ++f) thin[f] = 0;
  auto find_thin = [&](const fx4 (&x)[2], int f) {
    float least = fminf(fminf(fabsf(x[0].x), fabsf(x[0].y)), fabsf(x[0].z));
    least = fminf(fminf(least, fabsf(x[0].w)), fabsf(x[1].x));
    least = fminf(fminf(least, fabsf(x[1].y)), fabsf(x[1].z));
    least = fminf(least, fabsf(x[1].w));
    thin[f / 2] += least >= kFull ? 0u : f % 2 == 0 ? 1u : 0x10000u;
  };
  auto count_thin = [&] {
#pragma unroll
    for (int f = 0; f < FM + FN; ++f) {
      const int n = f % 2 == 0 ? thin[f / 2] & 0xffffu : thin[f / 2] >> 16;
      if (n != 0) atomicAdd(&fit.thin[f * 16 + lr], n);
    }
#pragma unroll
    for (int f = 0; f < (FM + FN + 1) / 2; ++f) thin[f] = 0;
  };
  // after every wave's first slab (a wave without one counts none)
  auto unfit_tile = [&] {
    count_thin();
    lds_barrier();
    return unfit_start(fit, FM * 16, 4 * (nw < nfull ? nw : nfull), 0, Pb, ldp, M - 1 - m0, Qb,
                       ldq, N - 1 - n0, K);
  };
  auto redo_block = [&](int b) {
    const int rm = m0 + b / FN * 16, cn = n0 + b % FN * 16;
    const fx4 s = f32_block(P, ldp, Q, ldq, M, N, rm, cn, K, lds + wave * (kRing * 4096));
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (rm + lr < M && cn + 4 * lc + e < N)
        Cs[(int64_t)(rm + lr) * ldc + cn + 4 * lc + e] = s[e];
  };
  // an unfit tile
  auto leave_tile = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load to LDS outlives its use
    if constexpr (kOwnRedo<FM, FN>) {
      lds_barrier();  // the slabs make room
      for (int b = wave; b < FB; b += nw) redo_block(b);
      return;
    }
    for (int b = threadIdx.x; b < FB; b += blockDim.x)
      mark_block(Cs, ldc, M, N, m0 + b / FN * 16, n0 + b % FN * 16);
  };

  // this wave's slab in LDS: row r is 128 bytes, its 16-byte chunk c at
  // position c ^ (r & 7); 8 lanes load a row
  char* slab = lds + wave * RB * 128;
  uint32_t off[RB / 8];
  {
    const int r8 = lane / 8, ch = (lane % 8) ^ r8;
#pragma unroll
    for (int v = 0; v < RB / 8; ++v) {
      const bool isp = v < 2 * FM;
      int row = (isp ? v : v - 2 * FM) * 8 + r8;
      const int last = isp ? M - 1 - m0 : N - 1 - n0;
      row = row < last ? row : last;
      off[v] = (uint32_t)row * (uint32_t)(isp ? ldp : ldq) * 4u + 16u * ch;
    }
  }
  auto load_slab = [&](int ks) {
    const char* Pn = Pb + ks * 4 * kSlab;
    const char* Qn = Qb + ks * 4 * kSlab;
#pragma unroll
    for (int v = 0; v < RB / 8; ++v)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)((v < 2 * FM ? Pn : Qn) + off[v]),
          (__attribute__((address_space(3))) void*)(slab + v * 1024), 16, 0, 0);
  };
  const int rd0 = lr * 128 + ((lc ^ (lr & 7)) * 16);
  const int rd1 = lr * 128 + (((4 + lc) ^ (lr & 7)) * 16);
  int ks = wave;
  if (ks < nfull) load_slab(ks);
  fit.clear();
  lds_barrier();
  auto do_slab = [&] {
    const int kn = ks + nw < nfull ? ks + nw : ks;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the slab is in LDS
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      rp[i][0] = *reinterpret_cast<const fx4*>(slab + i * 2048 + rd0);
      rp[i][1] = *reinterpret_cast<const fx4*>(slab + i * 2048 + rd1);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      rq[j][0] = *reinterpret_cast<const fx4*>(slab + (FM + j) * 2048 + rd0);
      rq[j][1] = *reinterpret_cast<const fx4*>(slab + (FM + j) * 2048 + rd1);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // and now in registers
    load_slab(kn);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      find_thin(rp[i], i);
      split_frag(rp[i], pf[i]);
    }
    bf8 q[2][3];
    find_thin(rq[0], FM);
    split_frag(rq[0], q[0]);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      mfma_parts<FM>(q[j & 1], pf, acc[j], acc[j]);
      if (j + 1 < FN) {
        find_thin(rq[j + 1], FM + j + 1);
        split_frag(rq[j + 1], q[(j + 1) & 1]);
      }
      if constexpr (FM * FN >= 16) {
#pragma unroll
        for (int g = 0; g < FM * 6; ++g) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
        }
      }
    }
  };
  if (ks < nfull) do_slab();
  if (unfit_tile()) return leave_tile();
  for (ks += nw; ks < nfull; ks += nw) do_slab();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (nfull < nslabs && wave == nfull % nw) {  // the partial last slab
    const int k0 = nfull * kSlab;
    auto load_frag = [&](fx4 (&r)[2], const char* base, uint32_t ld, int row) {
      const float* s = reinterpret_cast<const float*>(base + nfull * 4 * kSlab +
                                                      (uint64_t)row * ld * 4u) + 4 * lc;
      r[0] = load_tail(s, k0 + 4 * lc, K);
      r[1] = load_tail(s + 16, k0 + 16 + 4 * lc, K);
    };
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = i * 16 + lr < M - m0 ? i * 16 + lr : M - 1 - m0;
      load_frag(rp[i], Pb, (uint32_t)ldp, row);
      split_frag(rp[i], pf[i]);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int row = j * 16 + lr < N - n0 ? j * 16 + lr : N - 1 - n0;
      bf8 q[3];
      load_frag(rq[j], Qb, (uint32_t)ldq, row);
      split_frag(rq[j], q);
      mfma_parts<FM>(q, pf, acc[j], acc[j]);
    }
  }
  big = wave_max(big);
  if (lane == 0) red[wave] = big;
  count_thin();

  // the waves' partial tiles: the upper half through LDS to the lower half,
  // which adds them, then every wave sums its share of the blocks
  fx4* L = reinterpret_cast<fx4*>(lds);
  const int half = (nw + 1) / 2;
  __syncthreads();  // the slabs are read; red is written
  for (int w = 0; w < nw; ++w) big = fmaxf(big, red[w]);
  const int limit = 4 * nfull * 3 / 8;  // thin octets of a fit row, in the full slabs
  if (wave >= half) {
#pragma unroll
    for (int b = 0; b < FB; ++b) L[((wave - half) * FB + b) * kWave + lane] = acc[b % FN][b / FN];
  }
  __syncthreads();
  if (wave < half) {
#pragma unroll
    for (int b = 0; b < FB; ++b) {
      fx4 s = acc[b % FN][b / FN];
      if (wave + half < nw) s += L[(wave * FB + b) * kWave + lane];
      L[(wave * FB + b) * kWave + lane] = s;
    }
  }
  __syncthreads();
  const bool vec = ldc % 4 == 0 && ((uintptr_t)Cs & 15) == 0;
  // C rows that are not 16-byte aligned: the sums go back to LDS and out in
  // whole rows of the tile with 4-byte stores
  uint32_t redo = 0;  // blocks of this wave that the parts cannot serve
  for (int b = wave; b < FB; b += nw) {
    fx4 s = L[b * kWave + lane];
    for (int w = 1; w < half; ++w) s += L[(w * FB + b) * kWave + lane];
    const int tp = fit.thin[b / FN * 16 + lr];
    const int* tq = &fit.thin[(FM + b % FN) * 16 + 4 * lc];
    bool bad = tp > limit;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      bad |= tq[e] > limit || suspect(s[e], tp < 0 || tq[e] < 0, big);
    const int rm = m0 + (b / FN) * 16, cn = n0 + (b % FN) * 16;
    const int row = rm + lr, col = cn + 4 * lc;
    bad = __any(bad);  // wave-uniform
    const float m = __uint_as_float(kMark);
    redo |= (uint32_t)bad << b;
    if (!vec)
      L[b * kWave + lane] = bad ? fx4{m, m, m, m} : s;
    else if (bad && lane == 0)
      mark_block(Cs, ldc, M, N, rm, cn);
    else if (!bad && row < M)
      store_cols(Cs + (int64_t)row * ldc + col, col, N, s);
  }
  if (!vec) {
    __syncthreads();
    const float* T = reinterpret_cast<const float*>(lds);
    for (int e = threadIdx.x; e < FB * 256; e += blockDim.x) {
      const int r = e / (16 * FN), c = e % (16 * FN);
      const int b = (r / 16) * FN + c / 16, l = r % 16 + 16 * ((c % 16) / 4);
      if (m0 + r < M && n0 + c < N)
        Cs[(int64_t)(m0 + r) * ldc + n0 + c] = T[(b * kWave + l) * 4 + c % 4];
    }
  }
  if constexpr (kOwnRedo<FM, FN>) {
    __syncthreads();  // what lies in LDS is read, what was stored is stored
    for (int b = wave; b < FB; b += nw)
      if (redo >> b & 1) redo_block(b);
  }
}

constexpr int kKsWaves = 8;

template <int FM, int FN, int OCC>
__global__ __launch_bounds__(kKsWaves* kWave, OCC) void split_ks_kernel(
    const float* __restrict__ P, int64_t ldp, const float* __restrict__ Q, int64_t ldq,
    float* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m, int tiles_mn) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ float red[kKsWaves];
  __shared__ __attribute__((aligned(16))) Fitness<(FM + FN) * 16> fit;
  const int tile = tile_of(blockIdx.x, tiles_mn);
  ks_tile<FM, FN>(P, ldp, Q, ldq, C, ldc, M, N, (tile % tiles_m) * FM * 16,
                  (tile / tiles_m) * FN * 16, K, lds, red, fit);
}

// Compiled tiles.  Times of one workgroup step in microseconds, as measured
// with few workgroups and with all CUs busy (the clock falls as the matrix
// cores fill): a large tile takes `step` per slab, a small one `step` per
// round of its waves over their slabs; `fixed` per workgroup is the first
// loads, the sums over the waves and the store.
struct SplitShape {
  int bm, bn, waves;  // waves > 0: K shared by that many waves
  bool own_redo;      // no second launch
  double step, step_full, fixed;
};
constexpr SplitShape kSplitShapes[] = {
    {256, 160, 0, false, 2.13, 2.87, 12.0},
    {256, 128, 0, false, 1.75, 2.35, 12.0},
    {64, 80, 8, kOwnRedo<4, 5>, 3.30, 4.10, 4.0},
    {64, 64, 8, kOwnRedo<4, 4>, 2.70, 3.40, 3.5},
    {64, 32, 8, kOwnRedo<4, 2>, 1.85, 2.30, 2.5},
    {32, 32, 8, kOwnRedo<2, 2>, 1.20, 1.50, 2.2},
    {64, 16, 8, kOwnRedo<4, 1>, 1.43, 1.80, 2.2},
    {16, 16, 8, kOwnRedo<1, 1>, 0.60, 0.75, 2.0},
};
constexpr int kNumSplit = (int)(sizeof(kSplitShapes) / sizeof(kSplitShapes[0]));

template <int BM, int BN, int WM, int WN>
void launch_pp(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq, float* C,
               int64_t ldc, int64_t M, int64_t N, int64_t K) {
  const int tm = (int)ceil_div(M, BM), tn = (int)ceil_div(N, BN);
  hipLaunchKernelGGL((split_pp_kernel<BM, BN, WM, WN>), dim3((unsigned)(tm * tn)),
                     dim3(WM * WN * kWave), 0, st, P, ldp, Q, ldq, C, ldc, (int)M, (int)N, (int)K,
                     tm, tm * tn);
}

template <int FM, int FN, int OCC>
void launch_ks(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq, float* C,
               int64_t ldc, int64_t M, int64_t N, int64_t K) {
  const int tm = (int)ceil_div(M, 16 * FM), tn = (int)ceil_div(N, 16 * FN);
  const int slabs = (int)ceil_div(K, (int64_t)kSlab);
  // few slabs and workgroups for every CU anyway: fewer waves, two slabs
  // each, and more workgroups at once (24 x 26299 x 219: 13.0 to 10.9 us)
  int waves = kKsWaves;
  if (slabs < 2 * waves && (int64_t)tm * tn >= 512) waves = slabs < 4 ? 2 : (slabs + 1) / 2;
  hipLaunchKernelGGL((split_ks_kernel<FM, FN, OCC>), dim3((unsigned)(tm * tn)),
                     dim3(waves * kWave), (ks_lds_bytes<FM, FN>(waves)), st, P, ldp, Q, ldq, C,
                     ldc, (int)M, (int)N, (int)K, tm, tm * tn);
}

void launch_parts(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq,
                  float* C, int64_t ldc, int64_t M, int64_t N, int64_t K, int shape) {
  switch (shape - kSplitShape0) {
    case 0: launch_pp<256, 160, 4, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 1: launch_pp<256, 128, 4, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 2: launch_ks<4, 5, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 3: launch_ks<4, 4, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 4: launch_ks<4, 2, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 5: launch_ks<2, 2, 4>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    case 6: launch_ks<4, 1, 2>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
    default: launch_ks<1, 1, 4>(st, P, ldp, Q, ldq, C, ldc, M, N, K); break;
  }
}

}  // namespace

int gemm_num_split_shapes() { return kNumSplit; }
bool split_own_redo(int shape) { return kSplitShapes[shape - kSplitShape0].own_redo; }
int split_shape_bm(int shape) {
  const int v = shape - kSplitShape0;
  return v >= 0 && v < kNumSplit ? kSplitShapes[v].bm : 0;
}

// Products with K below kSplitMinK stay on the FP32 tiles, which are as fast or
// faster there (66 x 43429 x 210: 27 us, 49 on parts; 191 x 1555 x 282: 12 and 12),
// and both kernels count on several slabs.  The tiles' byte offsets are 32 bits
// wide, which bounds the leading dimensions.
bool split_possible(int64_t K, int64_t ldp, int64_t ldq) {
  return K >= kSplitMinK && ldp <= (1 << 21) && ldq <= (1 << 21);
}

int model_plan_split(int64_t M, int64_t N, int64_t K, double* us_out) {
  int best = kSplitShape0;
  double best_us = 1e300;
  const int64_t slabs = ceil_div(K, (int64_t)kSlab);
  for (int v = 0; v < kNumSplit; ++v) {
    const SplitShape& sh = kSplitShapes[v];
    if (sh.bm > 16 && M <= sh.bm / 2) continue;  // mostly padding rows
    const int64_t wgs = ceil_div(M, (int64_t)sh.bm) * ceil_div(N, (int64_t)sh.bn);
    const double steps = (double)(sh.waves > 0 ? ceil_div(slabs, (int64_t)sh.waves) : slabs);
    // rounds of 256 workgroups, the last one partly filled (and faster)
    const int64_t full = wgs / 256, rest = wgs % 256;
    double us = (double)full * (steps * sh.step_full + sh.fixed);
    if (rest > 0)
      us += steps * (sh.step + (sh.step_full - sh.step) * (double)rest / 256.0) + sh.fixed;
    if (us < best_us * 0.999) {
      best_us = us;
      best = kSplitShape0 + v;
    }
  }
  *us_out = best_us;
  return best;
}

void gemm_nt_split(hipStream_t st, const float* P, int64_t ldp, const float* Q, int64_t ldq,
                   float* C, int64_t ldc, int64_t M, int64_t N, int64_t K, int shape) {
  if (M <= 0 || N <= 0) return;
  launch_parts(st, P, ldp, Q, ldq, C, ldc, M, N, K, shape);
  if (split_own_redo(shape)) return;
  // the tiles that it marked
  gemm_nt_f32(st, P, ldp, Q, ldq, C, ldc, M, N, K, nullptr, 0, plan_f32(M, N, K, 1), 0, nullptr,
              true);
}

}  // namespace spca
