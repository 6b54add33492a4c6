// x-update for long rows (p beyond what one workgroup keeps in registers):
// each row of V is cut into chunks of kWCH elements and every chunk gets its
// own workgroup, so a launch has (chunks x starts) workgroups instead of one
// per start.  Row-level decisions are taken by small per-row kernels between
// the chunk passes; every sum is reduced in a fixed order, so results do not
// depend on timing.  Operators (Table 3, rows S3-S6):
//   T_s   exact top-s by |v| with ties to the lowest index.  Large s: a radix select
//         over the 31-bit keys of |v| in three digit passes (11, 10, 10
//         bits); each pass histograms the keys that share the prefix fixed
//         so far (LDS histogram per chunk, integer atomics into one global
//         histogram per row) and a per-row kernel picks the digit holding
//         the s-th largest key.  When the s-th key is shared by more
//         elements than are still needed, a counting pass gives each chunk
//         the number of such ties before it.
//   U_g   keep v_i with v_i^2 > g;  V_g  soft threshold at g.
// Then: per-chunk FP64 partial sums (count, ||w||^2, sum (w^2 - g)), a
// per-row kernel that adds them in chunk order, applies the stop test and
// turns the counts into list offsets, and an emit pass that writes
// x = w / ||w|| (and the index list and column marks).
// T_s and V_{lambda_s} of the usual small s go in two launches instead, from
// candidates: see wide_cand_kernel.  Other V_{lambda_s} take one workgroup a
// row: see wide_lambda_kernel.
#include "../../include/spca.h"
#include "common.hpp"
#include "kernels.hpp"
#include "select.hpp"

namespace spca {
namespace {

static_assert(kRT == 256, "chunks of 256 threads");
constexpr int kWT = kRT;              // threads per chunk workgroup
constexpr int kWN = 16;               // elements per thread
constexpr int kWCH = kWT * kWN;       // chunk length
constexpr int kWBins = 2048;          // largest digit (11 bits)
constexpr int kNWv = kWT / kWave;

struct alignas(64) WRow {
  uint32_t prefix;   // key bits fixed so far (the full key after pass 3)
  int32_t need;      // elements still to take at or below the prefix
  int32_t eq_total;  // elements whose key equals the final key
  int32_t straddle;  // 1 when only part of those are taken
  int32_t live;      // row processed in this x-update
  int32_t listed;    // the index list is written
  int32_t zero;      // w = 0
  int32_t marking;   // kept columns get colmark = epoch
  int32_t epoch;
  double inv;        // 1 / ||w||
  double lam;        // gamma of the row under the warm-up
};

struct Wide {
  uint32_t* ghist;  // r x kWBins
  WRow* rows;       // r
  int32_t* eqcnt;   // r x nch
  int32_t* cnt;     // r x nch: kept count, then list offset
  double* part;     // r x nch x 2
  int nch;
  int len;          // entries of a chunk, the last one's aside
  float* xrec;      // without scratch (no lists, every row live): the chunk records
  int64_t ldx;      // at the start of each chunk's part of X
  int32_t warm_K;   // sparsity-targeted warm-up (0: off)
  int32_t warm_target;
  double* gam;      // r: parameter of each start under the warm-up
};

// The scratch of r rows of p entries at base; *bytes: its size.
Wide carve_wide(void* base, int64_t r, int64_t p, size_t* bytes = nullptr) {
  Wide w;
  w.nch = (int)ceil_div(p, kWCH);
  w.len = (int)round_up(ceil_div(p, w.nch), 4);
  w.xrec = nullptr;
  w.ldx = 0;
  uintptr_t c = (uintptr_t)base;
  auto take = [&](size_t n) {
    const uintptr_t q = c;
    c += (n + 255) / 256 * 256;
    return (void*)q;
  };
  w.ghist = (uint32_t*)take(sizeof(uint32_t) * kWBins * r);
  w.rows = (WRow*)take(sizeof(WRow) * r);
  w.eqcnt = (int32_t*)take(sizeof(int32_t) * r * w.nch);
  w.cnt = (int32_t*)take(sizeof(int32_t) * r * w.nch);
  w.part = (double*)take(sizeof(double) * 2 * r * w.nch);
  if (bytes != nullptr) *bytes = (size_t)(c - (uintptr_t)base);
  w.warm_K = 0;
  w.warm_target = 0;
  w.gam = nullptr;
  return w;
}

__device__ __forceinline__ bool row_live(const StartState& s, int64_t j) {
  return s.status == nullptr || s.status[j] == kRunning;
}

// Element 4 (q kRT + tid) + e of [0, n) is v[4 q + e]; zeros beyond.
template <int NPT>
__device__ __forceinline__ void load_striped(const float* __restrict__ src, int n,
                                             float (&v)[NPT]) {
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    const int i = 4 * ((q / 4) * kRT + (int)threadIdx.x);
    if (i + 3 < n) {
      const floatx4 t = *reinterpret_cast<const floatx4*>(src + i);
      v[q] = t.x;
      v[q + 1] = t.y;
      v[q + 2] = t.z;
      v[q + 3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q + e] = i + e < n ? src[i + e] : 0.f;
    }
  }
}

// the place in its chunk of register k after load_striped
__device__ __forceinline__ int at(int k) { return 4 * ((k / 4) * kRT + (int)threadIdx.x) + k % 4; }

// digit pass PASS: bits [shift, shift + bits) of the key, among keys whose
// higher bits equal the prefix
template <int PASS>
struct Digit {
  static constexpr int kShift = PASS == 0 ? 20 : PASS == 1 ? 10 : 0;
  static constexpr int kBits = PASS == 0 ? 11 : 10;
  static constexpr int kBins = 1 << kBits;
};

template <int PASS>
__global__ __launch_bounds__(kWT) void wide_hist_kernel(
    const float* __restrict__ V, int64_t ldv, int p, StartState s, Wide w) {
  using D = Digit<PASS>;
  __shared__ uint32_t lh[D::kBins];
  const int64_t j = blockIdx.x / w.nch;
  const int chunk = blockIdx.x % w.nch;
  if (!row_live(s, j)) return;
  const int tid = threadIdx.x;
  for (int b = tid; b < D::kBins; b += kWT) lh[b] = 0u;
  const uint32_t prefix = PASS == 0 ? 0u : w.rows[j].prefix;
  __syncthreads();
  const int base = chunk * w.len;
  const int n = p - base < w.len ? p - base : w.len;
  float v[kWN];
  load_striped<kWN>(V + j * ldv + base, n, v);
#pragma unroll
  for (int k = 0; k < kWN; ++k) {
    const uint32_t key = key_of(v[k]);
    const bool in = at(k) < n &&
                    (PASS == 0 || (key >> (D::kShift + D::kBits)) == prefix);
    if (in) atomicAdd(&lh[(key >> D::kShift) & (D::kBins - 1)], 1u);
  }
  __syncthreads();
  uint32_t* gh = w.ghist + j * kWBins;
  for (int b = tid; b < D::kBins; b += kWT)
    if (lh[b] != 0u) atomicAdd(&gh[b], lh[b]);
}

// per row: the digit holding the need-th largest key; clears the histogram
template <int PASS>
__global__ __launch_bounds__(kWT) void wide_decide_kernel(StartState s, Wide w,
                                                          int32_t s_need) {
  using D = Digit<PASS>;
  constexpr int kPer = D::kBins / kWT;
  __shared__ int scan[kNWv + 1];
  const int64_t j = blockIdx.x;
  if (!row_live(s, j)) return;
  const int tid = threadIdx.x;
  WRow* R = w.rows + j;
  const int need = PASS == 0 ? s_need : R->need;
  const uint32_t prefix = PASS == 0 ? 0u : R->prefix;
  uint32_t* gh = w.ghist + j * kWBins;
  // thread 0 owns the highest bins
  const int hi = D::kBins - kPer * tid;
  int c[kPer];
  int sum = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    c[e] = (int)gh[hi - 1 - e];
    sum += c[e];
  }
  int total;
  int run = block_exclusive_scan(sum, scan, &total);
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (run < need && need <= run + c[e]) {
      const uint32_t key = (prefix << D::kBits) | (uint32_t)(hi - 1 - e);
      R->prefix = key;
      R->need = need - run;
      if (PASS == 2) {
        R->eq_total = c[e];
        R->straddle = key != 0u && c[e] > need - run;
      }
    }
    run += c[e];
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) gh[hi - 1 - e] = 0u;
}

__global__ __launch_bounds__(kWT) void wide_eqcount_kernel(
    const float* __restrict__ V, int64_t ldv, int p, StartState s, Wide w) {
  __shared__ int red[kNWv + 1];
  const int64_t j = blockIdx.x / w.nch;
  const int chunk = blockIdx.x % w.nch;
  if (!row_live(s, j) || !w.rows[j].straddle) return;
  const uint32_t t = w.rows[j].prefix;
  const int base = chunk * w.len;
  const int n = p - base < w.len ? p - base : w.len;
  float v[kWN];
  load_striped<kWN>(V + j * ldv + base, n, v);
  int eq = 0;
#pragma unroll
  for (int k = 0; k < kWN; ++k) eq += at(k) < n && key_of(v[k]) == t;
  eq = block_sum(eq, red);
  if (threadIdx.x == 0) w.eqcnt[j * w.nch + chunk] = eq;
}

// Membership and value of each element of the thread's slice.  For T_s the
// rank of an element among the ties at the final key decides (lowest
// indices first).
template <int KIND>
struct Keep {
  uint32_t t = 0;
  int straddle = 0, need = 0;
  int rank[kWN / 4] = {};
  double lam = 0.0;

  __device__ void setup(const Wide& w, int64_t j, double param,
                        const float (&v)[kWN], int n, uint64_t* pscan, int* red) {
    if (KIND == kTopS) {
      const WRow& R = w.rows[j];
      t = R.prefix;
      straddle = R.straddle;
      need = R.need;
      if (straddle) {
        int before = 0;
        for (int c = threadIdx.x; c < (int)(blockIdx.x % w.nch); c += kWT)
          before += w.eqcnt[j * w.nch + c];
        before = block_sum(before, red);
        int eq[kWN / 4] = {};
#pragma unroll
        for (int k = 0; k < kWN; ++k) eq[k / 4] += at(k) < n && key_of(v[k]) == t;
        rank_rows<kWN / 4>(eq, rank, pscan);
#pragma unroll
        for (int q = 0; q < kWN / 4; ++q) rank[q] += before;
      }
    } else if (w.warm_K > 0) {
      lam = w.rows[j].lam;  // per row: gamma under the warm-up
    } else {
      lam = param;
    }
  }

  // register k, in order
  __device__ bool operator()(int k, float vv, bool valid, double* wv) {
    if (!valid) return false;
    if (KIND == kTopS) {
      const uint32_t key = key_of(vv);
      *wv = (double)vv;
      if (key == 0u || key < t) return false;
      if (key > t || !straddle) return true;
      return rank[k / 4]++ < need;
    } else if (KIND == kHardGamma) {
      *wv = (double)vv;
      return (double)vv * (double)vv > lam;
    } else {  // soft threshold
      const double a = fabs((double)vv);
      *wv = vv > 0.f ? a - lam : lam - a;
      return a > lam;
    }
  }
};

template <int KIND>
__global__ __launch_bounds__(kWT) void wide_partial_kernel(
    const float* __restrict__ V, int64_t ldv, int p, double param, StartState s,
    Wide w) {
  __shared__ uint64_t pscan[3 * kRW];
  __shared__ int red[kNWv + 1];
  __shared__ double dred[2 * (kNWv + 1)];
  const int64_t j = blockIdx.x / w.nch;
  const int chunk = blockIdx.x % w.nch;
  if (!row_live(s, j)) return;
  const int base = chunk * w.len;
  const int n = p - base < w.len ? p - base : w.len;
  float v[kWN];
  load_striped<kWN>(V + j * ldv + base, n, v);
  Keep<KIND> keep;
  keep.setup(w, j, param, v, n, pscan, red);
  int cnt = 0;
  double acc[2] = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kWN; ++k) {
    double wv;
    if (keep(k, v[k], at(k) < n, &wv)) {
      ++cnt;
      acc[0] += wv * wv;
      if (KIND == kHardGamma) acc[1] += wv * wv - keep.lam;
    }
  }
  block_sum_n<double, 2>(acc, dred);
  cnt = block_sum(cnt, red);
  if (threadIdx.x == 0 && w.xrec != nullptr) {
    const Words<double> a0(acc[0]), a1(acc[1]);
    float* rec = w.xrec + j * w.ldx + base;
    rec[0] = __int_as_float(a0.w[0]);
    rec[1] = __int_as_float(a0.w[1]);
    rec[2] = __int_as_float(a1.w[0]);
    rec[3] = __int_as_float(a1.w[1]);
    rec[4] = __int_as_float(cnt);
  } else if (threadIdx.x == 0) {
    const int64_t c = j * w.nch + chunk;
    w.cnt[c] = cnt;
    w.part[2 * c] = acc[0];
    w.part[2 * c + 1] = acc[1];
  }
}

// phi, counters and the stop test of a row (one thread; the same state
// machine as the one-workgroup kernels)
__device__ __forceinline__ void finish_row(const StartState& s, int64_t j, double phi, int total,
                                           bool zero, double tol, int maxit, int warm_K) {
  if (s.status == nullptr) {
    s.phi[j] = phi;
    s.nnz[j] = zero ? 0 : total;
    return;
  }
  const int it = s.iters[j] + 1;
  const double prev = s.phi[j];
  s.iters[j] = it;
  s.phi_prev[j] = prev;
  s.phi[j] = phi;
  s.nnz[j] = zero ? 0 : total;
  if (zero)
    s.status[j] = SPCA_ZERO;
  else if (it >= 2 && tol >= 0.0 && (warm_K == 0 || it >= warm_K + 1) &&
           phi <= (1.0 + tol) * prev)
    s.status[j] = SPCA_CONVERGED;
  else if (it >= maxit)
    s.status[j] = SPCA_MAXIT;
}

__device__ __forceinline__ double words_of(float a, float b) {
  Words<double> w(0.0);
  w.w[0] = __float_as_int(a);
  w.w[1] = __float_as_int(b);
  return w.value();
}

// One wave per row: chunk sums (lane l adds chunks l, l + 64, ..., then the
// butterfly), phi, the stop test and list offsets.  64 x 200000: 16 us with
// one thread a row, a chain of loads over its 49 chunks; 3 us so.
template <int KIND>
__global__ __launch_bounds__(kWave) void wide_row_kernel(
    StartState s, double tol, int maxit, int list_cap, int have_list, const Plan* plan,
    int have_marks, Wide w) {
  const int64_t j = blockIdx.x;
  const int lane = threadIdx.x;
  const bool in_x = w.xrec != nullptr;
  float* rec = in_x ? w.xrec + j * w.ldx : nullptr;
  WRow* R = in_x ? nullptr : w.rows + j;
  const bool live = row_live(s, j);
  if (!in_x && lane == 0) R->live = live;
  if (!live) return;
  double a0 = 0.0, a1 = 0.0;
  int total = 0;
  for (int c0 = 0; c0 < w.nch; c0 += kWave) {
    const int c = c0 + lane;
    const int64_t q = j * w.nch + c;
    int k = 0;
    if (c < w.nch && in_x) {
      const float* rc = rec + (int64_t)c * w.len;
      a0 += words_of(rc[0], rc[1]);
      a1 += words_of(rc[2], rc[3]);
      k = __float_as_int(rc[4]);
    } else if (c < w.nch) {
      a0 += w.part[2 * q];
      a1 += w.part[2 * q + 1];
      k = w.cnt[q];
    }
    const int incl = wave_scan(k);
    if (c < w.nch && !in_x) w.cnt[q] = total + incl - k;
    total += __shfl(incl, kWave - 1, kWave);
  }
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
  const double nrm = sqrt(a0);
  const double phi = KIND == kHardGamma ? a1 : nrm;
  const bool zero = !(nrm > 0.0);
  if (in_x) {  // every chunk's emit block finds 1 / nrm (-1: w = 0) in its own part
    const Words<double> inv(zero ? -1.0 : 1.0 / nrm);
    for (int c = lane; c < w.nch; c += kWave) {
      rec[(int64_t)c * w.len] = __int_as_float(inv.w[0]);
      rec[(int64_t)c * w.len + 1] = __int_as_float(inv.w[1]);
    }
    if (lane == 0) finish_row(s, j, phi, total, zero, tol, maxit, 0);
    return;
  }
  if (lane != 0) return;
  R->zero = zero;
  R->inv = zero ? 0.0 : 1.0 / nrm;
  R->listed = have_list && !zero && total <= list_cap;
  R->marking = have_marks && !zero && plan != nullptr && plan->mark != 0;
  R->epoch = R->marking ? plan->epoch : 0;
  if (KIND != kTopS && w.warm_K > 0 && s.status != nullptr && s.iters[j] + 1 <= w.warm_K)
    w.gam[j] = R->lam;
  finish_row(s, j, phi, total, zero, tol, maxit, w.warm_K);
}

template <int KIND>
__global__ __launch_bounds__(kWT) void wide_emit_kernel(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int32_t* __restrict__ colmark,
    Wide w) {
  __shared__ uint64_t pscan[3 * kRW];
  __shared__ int red[kNWv + 1];
  const int64_t j = blockIdx.x / w.nch;
  const int chunk = blockIdx.x % w.nch;
  WRow R;
  const int base = chunk * w.len;
  const int n = p - base < w.len ? p - base : w.len;
  if (w.xrec != nullptr) {
    const float* rec = w.xrec + j * w.ldx + base;
    R.inv = words_of(rec[0], rec[1]);
    R.zero = R.inv < 0.0;
    R.live = 1;
    R.listed = R.marking = 0;
    __syncthreads();  // the record lies in what this block writes
  } else {
    R = w.rows[j];
  }
  if (!R.live) return;
  float v[kWN];
  load_striped<kWN>(V + j * ldv + base, n, v);
  Keep<KIND> keep;
  keep.setup(w, j, param, v, n, pscan, red);
  float xo[kWN];
  bool kp[kWN];
  int cnt[kWN / 4] = {};
#pragma unroll
  for (int k = 0; k < kWN; ++k) {
    double wv = 0.0;
    kp[k] = keep(k, v[k], at(k) < n, &wv) && !R.zero;
    xo[k] = kp[k] ? (float)(wv * R.inv) : 0.f;
    cnt[k / 4] += kp[k];
  }
  if (R.listed) {
    int off[kWN / 4];
    rank_rows<kWN / 4>(cnt, off, pscan);
    const int first = w.cnt[j * w.nch + chunk];
    int32_t* li = list_idx + j * ldl;
    float* lv = list_val + j * ldl;
#pragma unroll
    for (int k = 0; k < kWN; ++k) {
      if (kp[k]) {
        li[first + off[k / 4]] = base + at(k);
        lv[first + off[k / 4]] = xo[k];
        ++off[k / 4];
      }
    }
  }
  if (R.marking) {
#pragma unroll
    for (int k = 0; k < kWN; ++k)
      if (kp[k]) colmark[base + at(k)] = R.epoch;
  }
  float* x = X + j * ldx + base;
#pragma unroll
  for (int q = 0; q < kWN; q += 4) {
    const int i = at(q);
    if (i + 3 < n) {
      floatx4 t = {xo[q], xo[q + 1], xo[q + 2], xo[q + 3]};
      *reinterpret_cast<floatx4*>(x + i) = t;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + e < n) x[i + e] = xo[q + e];
    }
  }
}

// ---------------------------------------------------------------------------
// T_s and lambda_s from candidates, without scratch.  Every chunk finds a
// threshold that at least `need` (and fewer than cap) of its entries reach,
// by the counting search over registers, and writes its part of X: cap places
// with that threshold (0: no other entry is nonzero) and the values of those
// entries in index order, cap / 2 words with their 16-bit indices in the chunk,
// zeros after that.  (Indices alone, and a gather from V, read most of V's
// lines again: 45 us in place of 23 at 64 x 200000.)
// One workgroup per row then loads its nch * cap <= 12288 candidates into
// registers, decides as for a short row, clears the places and writes the
// kept entries.
//   T_s       need = s: the s largest of a row are among its chunks' s largest.
//   lambda_s  the candidates from the largest of the chunks' thresholds on are
//             complete; the root lies among them unless the large entries
//             crowd in few chunks: such a row is flagged (nnz = -1) and left
//             to wide_lambda_kernel.
// V is read once and X written once (64 x 200000, s = 200: T_s 118 us in
// three histogram passes, their decisions, a counting, a summing and an
// emitting pass, 45 us so; lambda_s 3100 us, 41 us so).
// ---------------------------------------------------------------------------
constexpr int kCandCapW = 1024;  // places of a chunk
constexpr int kCandChunks = 192;
constexpr int kMergeSlots = 48 * kRT;  // places of a row

struct CandPlan {
  int nch = 0;   // chunks of a row
  int len = 0;   // entries of a chunk (a multiple of 4)
  int cap = 0;   // places of a chunk (a multiple of 8); 0: not this way
  int need = 0;  // entries a chunk names at least, if it has as many
  uint32_t cap_inv = 0;  // ceil(2^32 / cap)
};

bool overlap(const float* V, int64_t ldv, const float* X, int64_t ldx, int64_t r, int64_t p) {
  const uintptr_t v0 = (uintptr_t)V, v1 = (uintptr_t)(V + (r - 1) * ldv + p);
  const uintptr_t x0 = (uintptr_t)X, x1 = (uintptr_t)(X + (r - 1) * ldx + p);
  return x0 < v1 && v0 < x1;
}

// U_g and V_g of a call without state, lists and marks keep their chunk sums in
// X itself, five words a chunk: the allocation, and its release, took 20 to 50
// us of 70 to 98 (64 x 200000; 500 x 20003).
bool records_in_x(XKind kind, const StartState& s, bool lists, const float* V, int64_t ldv,
                  const float* X, int64_t ldx, int64_t r, int64_t p) {
  return (kind == kHardGamma || kind == kSoftGamma) && s.status == nullptr && !lists &&
         ceil_div(p, kWCH) <= kCandChunks && !overlap(V, ldv, X, ldx, r, p);
}

// T_s: s places and some slack (the search ends early in a wide window).
// lambda_s: 16 s candidates over the row, three times what a row of noise and
// s larger entries keeps.  A chunk is never shorter than its places and their
// indices: more than 12288 / 4 - 4 * 192 entries.  X must not overlap V, which
// rows that are left to wide_lambda_kernel read again.
CandPlan plan_cand(XKind kind, double par, const float* V, int64_t ldv, const float* X,
                   int64_t ldx, int64_t r, int64_t p, int warm_K) {
  CandPlan c;
  const int64_t nch = ceil_div(p, kWCH);
  if (nch > kCandChunks || warm_K > 0) return c;
  if (overlap(V, ldv, X, ldx, r, p)) return c;
  int64_t need;
  if (kind == kTopS) {
    need = par < (double)kCandCapW ? (int64_t)par : kCandCapW;
  } else if (kind == kLambdaS) {
    const double n = 16.0 * par / (double)nch;
    need = n < 32.0 ? 32 : n < (double)kCandCapW ? (int64_t)n : kCandCapW;
  } else {
    return c;
  }
  int64_t cap = kMergeSlots / nch / 8 * 8;
  cap = cap < kCandCapW ? cap : kCandCapW;
  cap = cap < need + need / 4 + 32 ? cap : round_up(need + need / 4 + 32, 8);
  if (need > cap - 1) return c;
  c.nch = (int)nch;
  c.len = (int)round_up(ceil_div(p, nch), 4);
  c.cap = (int)cap;
  c.need = (int)need;
  c.cap_inv = (uint32_t)(((uint64_t(1) << 32) + cap - 1) / cap);
  return c;
}

__global__ __launch_bounds__(kRT, 4) void wide_cand_kernel(const float* __restrict__ V,
                                                           int64_t ldv, int p,
                                                           float* __restrict__ X, int64_t ldx,
                                                           StartState s, CandPlan cp, int ties) {
  constexpr int R = kWN / 4;
  __shared__ RSmem sm;
  __shared__ __align__(16) uint32_t place[kCandCapW + kCandCapW / 2];
  const int64_t j = blockIdx.x / cp.nch;
  const int base = (int)(blockIdx.x % cp.nch) * cp.len;
  if (!row_live(s, j)) return;
  const int tid = threadIdx.x;
  const int n = p - base < cp.len ? p - base : cp.len;
  const int words = cp.cap + cp.cap / 2;
  for (int i = tid; i < words; i += kRT) place[i] = 0u;
  uint16_t* index = reinterpret_cast<uint16_t*>(place + cp.cap);
  float v[kWN];
  load_striped<kWN>(V + j * ldv + base, n, v);
  Bracket b;
  const bool fit = narrow<kWN>(v, n, (uint32_t)cp.need, (uint32_t)cp.cap - 1u, sm, b);
  // entries of a key from t0 on, and the first `ties_left` at the key below it
  uint32_t t0 = b.lo > 1u ? b.lo : 1u;
  uint32_t head = b.lo;
  int ties_left = 0;
  if (b.nan) {
    t0 = 0x7f800001u;  // the row is to be found NaN
  } else if (!fit && b.lo > 0u) {
    t0 = head = b.hi;  // more than cap - 1 entries share the key below
    ties_left = ties ? cp.need - (int)b.nhi : 0;
  }
  int cnt[R], off[R], eq[R], eq_off[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    cnt[q] = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) cnt[q] += key_of(v[4 * q + e]) >= t0;
  }
  if (ties_left > 0) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      eq[q] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) eq[q] += key_of(v[4 * q + e]) == t0 - 1u;
    }
    rank_rows<R>(eq, eq_off, sm.pscan);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int left = ties_left - eq_off[q];
      cnt[q] += left <= 0 ? 0 : eq[q] < left ? eq[q] : left;
    }
  }
  rank_rows<R>(cnt, off, sm.pscan);
#pragma unroll
  for (int q = 0; q < R; ++q) {
    int o = off[q] + 1;
    int left = ties_left > 0 ? ties_left - eq_off[q] : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = key_of(v[4 * q + e]);
      const bool tie = ties_left > 0 && key == t0 - 1u && left-- > 0;
      if (key >= t0 || tie) {
        if (o < cp.cap) {
          place[o] = __float_as_uint(v[4 * q + e]);
          index[o] = (uint16_t)(4 * (q * kRT + tid) + e);
        }
        ++o;
      }
    }
  }
  if (tid == 0) place[0] = head;
  __syncthreads();
  float* x = X + j * ldx + base;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int i = 4 * (q * kRT + tid);
    floatx4 t = {0.f, 0.f, 0.f, 0.f};
    if (i < words) {
      t.x = __uint_as_float(place[i]);
      t.y = __uint_as_float(place[i + 1]);
      t.z = __uint_as_float(place[i + 2]);
      t.w = __uint_as_float(place[i + 3]);
    }
    if (i + 3 < n) {
      *reinterpret_cast<floatx4*>(x + i) = t;
    } else {
      if (i < n) x[i] = t.x;
      if (i + 1 < n) x[i + 1] = t.y;
      if (i + 2 < n) x[i + 2] = t.z;
    }
  }
}

// Thread t holds places [t NPT, (t + 1) NPT) of the row, so that thread order
// is index order.  A few counting passes over them leave at most 1024 (T_s) or
// 2048 entries, PER a thread, and all else goes over those.
template <int KIND, int NPT>
__global__ __launch_bounds__(kRT, 2) void wide_merge_kernel(
    int p, double param, float* __restrict__ X, int64_t ldx,
    int32_t* __restrict__ list_idx, float* __restrict__ list_val, int64_t ldl, int list_cap,
    StartState s, double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan,
    CandPlan cp) {
  constexpr int kPer = KIND == kTopS ? 4 : 8;
  constexpr int kFew = kPer * kRT;
  __shared__ uint32_t ured[2 * kRW];
  __shared__ int scan[kRW];
  __shared__ double dred[3 * kRW];
  __shared__ float cval[kFew];
  __shared__ int cplace[kFew];
  __shared__ int cut_at;
  const int64_t j = blockIdx.x;
  if (!row_live(s, j)) return;
  const int tid = threadIdx.x;
  const int slots = cp.nch * cp.cap;
  float* x = X + j * ldx;
  // the chunk of place i: i / cap, exact for i < 2^14 and cap < 2^11
  auto chunk_of = [&](int i) { return (int)__umulhi((uint32_t)i, cp.cap_inv); };
  // the row index of place i
  auto index_of = [&](int i) {
    const int ch = chunk_of(i), t = i - ch * cp.cap;
    const uint32_t w = __float_as_uint(x[ch * cp.len + cp.cap + t / 2]);
    return ch * cp.len + (int)(t % 2 != 0 ? w >> 16 : w & 0xffffu);
  };
  float v[NPT];
  uint32_t head = 0u, mk = 0u;
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    const int i = tid * NPT + q;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[q + e] = 0.f;
    if (i < slots) {
      const int ch = chunk_of(i), place = i - ch * cp.cap;
      const floatx4 t = *reinterpret_cast<const floatx4*>(x + ch * cp.len + place);
      v[q] = t.x;
      v[q + 1] = t.y;
      v[q + 2] = t.z;
      v[q + 3] = t.w;
      if (place == 0) {
        const uint32_t h = __float_as_uint(v[q]);
        head = h > head ? h : head;
        v[q] = 0.f;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const uint32_t key = key_of(v[k]);
    mk = key > mk ? key : mk;
  }
  head = block_max(head, ured);
  mk = block_max(mk, ured);
  const bool nan = mk > 0x7f800000u;
  if (KIND == kLambdaS && nan) {
    if (tid == 0) s.nnz[j] = -1;
    return;
  }
  Bracket b{0u, mk + 1u, (uint32_t)slots, 0u, 0u, mk, nan, false};
  uint32_t need, t;
  if (KIND == kTopS) {
    // the chunks' thresholds are what cp.need of cp.len entries reach
    need = (uint32_t)cp.need;
    t = key_of(__uint_as_float(head) * tail_quantile((float)p / (1.4f * (float)need + 16.f)) /
               tail_quantile((float)cp.len / (float)cp.need));
  } else {
    const double want = 8.0 * param < 0.75 * kFew ? 8.0 * param : 0.75 * kFew;
    need = (uint32_t)want;
    b.lo = head > 1u ? head : 1u;
    b.nlo = count_from(v, b.lo, 0u, ured);
    b.parity = 1u;
    t = 0u;
  }
  const bool fit = narrow_from<NPT>(v, need, (uint32_t)kFew, t, ured, b);
  if (KIND == kLambdaS && !fit) {
    if (tid == 0) s.nnz[j] = -1;
    return;
  }
  // the entries from key t0 on; T_s: with those below it that complete `need`
  // where more share their key than fit (in index order)
  const uint32_t t0 = fit || b.lo == 0u ? (b.lo > 1u ? b.lo : 1u) : b.hi;
  int ties_left = KIND == kTopS && !fit && b.lo > 0u ? (int)need - (int)b.nhi : 0;
  if (ties_left > 0) {
    int eq = 0, all;
#pragma unroll
    for (int k = 0; k < NPT; ++k) eq += key_of(v[k]) == t0 - 1u;
    ties_left -= block_exclusive_scan(eq, scan, &all);
  }
  int mine = 0, left = ties_left;
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const uint32_t key = key_of(v[k]);
    mine += key >= t0 || (key == t0 - 1u && left-- > 0);
  }
  int n;
  int o = block_exclusive_scan(mine, scan, &n);
  left = ties_left;
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      reload(v[q + e]);  // compare again rather than hold the masks
      const uint32_t key = key_of(v[q + e]);
      if (key >= t0 || (key == t0 - 1u && left-- > 0)) {
        if (o < kFew) {
          cval[o] = v[q + e];
          cplace[o] = tid * NPT + q + e;
        }
        ++o;
      }
    }
  }
  __syncthreads();
  n = n < kFew ? n : kFew;
  float c[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) c[e] = kPer * tid + e < n ? cval[kPer * tid + e] : 0.f;

  uint32_t thr_key = 0u;
  int cut = kFew;  // T_s: of the entries at thr_key, those up to here
  double lam = 0.0;
  if (KIND == kTopS) {
    settle<kPer>(c, need, ured, b);
    thr_key = b.lo;
    const int tied = (int)need - (int)b.nhi;
    if (thr_key != 0u && b.nlo > need) {
      int eq = 0, all;
#pragma unroll
      for (int e = 0; e < kPer; ++e) eq += key_of(c[e]) == thr_key;
      int seen = block_exclusive_scan(eq, scan, &all);
#pragma unroll
      for (int e = 0; e < kPer; ++e)
        if (key_of(c[e]) == thr_key && ++seen == tied) cut_at = kPer * tid + e;
      __syncthreads();
      cut = cut_at;
    }
  } else {
    // as lambda_root, from these entries alone
    const double rs = sqrt(param);
    double set3[3];
    bool done = false;
    float f = __uint_as_float(b.lo);
    sums_from<kPer>(c, f, set3, dred);
    bool ok = true;
    if (b.lo > 1u || head > 0u) {
      lam = (double)f;
      ok = rho_above(set3, lam, rs);
    } else {
      done = !(set3[1] > rs * sqrt(set3[2]));  // all of the row: inactive
    }
    for (int round = 0; ok && !done && round < kLamRoundsFull; ++round) {
      const double kk = set3[0];
      ok = kk > param;
      if (!ok) break;
      double l = lambda_of(set3, param);
      const bool held = !(l > lam);
      if (held) l = lam;
      sums_from<kPer>(c, float_above(l), set3, dred);
      lam = l;
      ok = !held || set3[0] != kk;  // (else rounding)
      done = ok && (set3[0] == kk || set3[0] == 0.0);
      if (set3[0] == 0.0) lam = fmin(l, (double)__uint_as_float(mk));
    }
    if (!done) {
      if (tid == 0) s.nnz[j] = -1;
      return;
    }
  }
  const float lamf = float_above(lam);
  auto kept = [&](int e) {
    if (KIND == kLambdaS) return fabsf(c[e]) >= lamf;
    const uint32_t key = key_of(c[e]);
    return key > thr_key || (key == thr_key && key != 0u && kPer * tid + e <= cut);
  };
  double acc[1] = {0.0};
  int cnt = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (!kept(e)) continue;
    const double w = KIND == kTopS ? (double)c[e] : fabs((double)c[e]) - lam;
    acc[0] += w * w;
    ++cnt;
  }
  block_sum_n<double, 1>(acc, dred);
  int total;
  o = block_exclusive_scan(cnt, scan, &total);
  // the kept entries' indices are read: clear the places
  int at[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) at[e] = kept(e) ? index_of(cplace[kPer * tid + e]) : 0;
  __syncthreads();
  const int words = cp.cap + cp.cap / 2;
  for (int ch = tid / kWave; ch < cp.nch; ch += kRW)
    for (int i = 4 * (tid % kWave); i < words; i += 4 * kWave)
      *reinterpret_cast<floatx4*>(x + ch * cp.len + i) = floatx4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  const double nrm = nan ? __longlong_as_double(0x7ff8000000000000ll) : sqrt(acc[0]);
  const bool zero = !(nrm > 0.0);
  const double inv = zero ? 0.0 : 1.0 / nrm;
  const bool listed = list_idx != nullptr && !zero && total <= list_cap;
  const bool marking = colmark != nullptr && !zero && plan != nullptr && plan->mark != 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (zero || !kept(e)) continue;
    const int idx = at[e];
    const double a = fabs((double)c[e]);
    const double w = KIND == kTopS ? (double)c[e] : c[e] > 0.f ? a - lam : lam - a;
    const float val = (float)(w * inv);
    x[idx] = val;
    if (listed) {
      list_idx[j * ldl + o] = idx;
      list_val[j * ldl + o] = val;
      ++o;
    }
    if (marking) colmark[idx] = plan->epoch;
  }
  if (tid == 0)
    finish_row(s, j, KIND == kLambdaS ? lam * sqrt(param) + nrm : nrm, total, zero, tol, maxit, 0);
}

// ---------------------------------------------------------------------------
// lambda_s, one workgroup per row from memory: every row, or those flagged by
// wide_merge_kernel (only = 1).  The rounds of lambda_root from all nonzero
// entries, a pass over the row each; what they do not settle takes an FP64
// search over float intervals.
// ---------------------------------------------------------------------------
constexpr int kLT = 1024;
constexpr int kLW = kLT / kWave;

__global__ __launch_bounds__(kLT) void wide_lambda_kernel(
    const float* V, int64_t ldv, int p, double s_par, float* X, int64_t ldx,
    int32_t* __restrict__ list_idx, float* __restrict__ list_val, int64_t ldl, int list_cap,
    StartState s, double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan, Warm wm,
    int only) {
  __shared__ double dred[2 * kNCd * kLW];
  __shared__ uint32_t ured[kLW];
  __shared__ int scan[kLW];
  const int64_t j = blockIdx.x;
  if (!row_live(s, j) || (only && s.nnz[j] >= 0)) return;
  const int tid = threadIdx.x;
  const float* vg = V + j * ldv;
  const double rs = sqrt(s_par);
  const bool warm = wm.K > 0 && s.status != nullptr;
  const bool frozen = warm && s.iters[j] + 1 > wm.K;  // after the warm-up
  double lam = 0.0;
  // f(entry) over the row in a fixed order per thread
  auto each = [&](auto f) {
    const int n4 = p / 4;
#pragma unroll 4
    for (int i = tid; i < n4; i += kLT) {
      const floatx4 t = *reinterpret_cast<const floatx4*>(vg + 4 * (int64_t)i);
      f(t.x);
      f(t.y);
      f(t.z);
      f(t.w);
    }
    if (tid < p - 4 * n4) f(vg[4 * n4 + tid]);
  };
  auto sums = [&](float from, double (&b)[3]) {
    b[0] = b[1] = b[2] = 0.0;
    each([&](float vv) {
      const bool in = fabsf(vv) >= from;
      const double a = (double)(in ? fabsf(vv) : 0.f);
      b[0] += in ? 1.0 : 0.0;
      b[1] += a;
      b[2] += a * a;
    });
    block_sum_n<double, 3>(b, dred);
  };
  if (frozen) {
    lam = wm.gam[j];
  } else {
    double set3[3] = {0.0, 0.0, 0.0};
    uint32_t mk = 0u;
    each([&](float vv) {  // all nonzero entries
      const uint32_t key = key_of(vv);
      mk = key > mk ? key : mk;
      const bool in = fabsf(vv) > 0.f;
      const double a = (double)(in ? fabsf(vv) : 0.f);
      set3[0] += in ? 1.0 : 0.0;
      set3[1] += a;
      set3[2] += a * a;
    });
    mk = block_max(mk, ured);
    block_sum_n<double, 3>(set3, dred);
    // inactive (or NaN): lambda = 0
    bool done = mk > 0x7f800000u || !(set3[1] > rs * sqrt(set3[2]));
    for (int round = 0; !done && round < kLamRoundsFull; ++round) {
      const double kk = set3[0];
      if (!(kk > s_par)) break;
      const double l = lambda_of(set3, s_par);
      if (!(l > lam)) break;
      sums(float_above(l), set3);
      lam = l;
      done = set3[0] == kk || set3[0] == 0.0;
      if (set3[0] == 0.0) lam = fmin(l, (double)__uint_as_float(mk));
    }
    if (!done) {
      // the largest key t with ||(|v| - t)_+||_1 >= sqrt(s) ||(|v| - t)_+||_2,
      // then the closed form on the interval, where the active set is fixed
      uint32_t lo = 0u, hi = mk;
      while (hi - lo > 1u) {
        uint32_t t[kNCd];
        spread<kNCd>(lo, hi, t);
        double acc[2 * kNCd], tf[kNCd];
#pragma unroll
        for (int c = 0; c < kNCd; ++c) {
          acc[2 * c] = acc[2 * c + 1] = 0.0;
          tf[c] = (double)__uint_as_float(t[c]);
        }
        for (int i = tid; i < p; i += kLT) {
          const double a = fabs((double)vg[i]);
#pragma unroll
          for (int c = 0; c < kNCd; ++c) {
            double d = a - tf[c];
            d = d > 0.0 ? d : 0.0;
            acc[2 * c] += d;
            acc[2 * c + 1] += d * d;
          }
        }
        block_sum_n<double, 2 * kNCd>(acc, dred);
        lambda_step<kNCd>(t, acc, rs, lo, hi);
      }
      const double tl = (double)__uint_as_float(lo), th = (double)__uint_as_float(hi);
      sums(__uint_as_float(lo + 1u), set3);
      lam = set3[0] > s_par ? lambda_of(set3, s_par) : tl;
      lam = lam < tl ? tl : lam;
      lam = lam > th ? th : lam;
    }
  }
  const float lamf = float_above(lam);
  double acc[2] = {0.0, 0.0};
  each([&](float vv) {
    if (fabsf(vv) >= lamf) {
      const double w = fabs((double)vv) - lam;
      acc[0] += w * w;
      acc[1] += 1.0;
    }
  });
  block_sum_n<double, 2>(acc, dred);
  const int total = (int)acc[1];
  const double nrm = sqrt(acc[0]);
  const bool zero = !(nrm > 0.0);
  const double inv = zero ? 0.0 : 1.0 / nrm;
  const bool listed = list_idx != nullptr && !zero && total <= list_cap;
  const bool marking = colmark != nullptr && !zero && plan != nullptr && plan->mark != 0;
  float* x = X + j * ldx;
  int done = 0;
  for (int i0 = 0; i0 < p; i0 += kLT) {
    const int i = i0 + tid;
    const float vv = i < p ? vg[i] : 0.f;
    const bool kp = i < p && !zero && fabsf(vv) >= lamf;
    const double a = fabs((double)vv);
    const float xo = kp ? (float)((vv > 0.f ? a - lam : lam - a) * inv) : 0.f;
    if (i < p) x[i] = xo;
    if (kp && marking) colmark[i] = plan->epoch;
    if (listed) {
      int in_tile;
      const int o = done + block_exclusive_scan((int)kp, scan, &in_tile);
      if (kp) {
        list_idx[j * ldl + o] = i;
        list_val[j * ldl + o] = xo;
      }
      done += in_tile;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (warm && !frozen) wm.gam[j] = lam;
    finish_row(s, j, lam * rs + nrm, total, zero, tol, maxit, wm.K);
  }
}

template <int KIND>
void launch_merge(hipStream_t st, double param, int64_t r, int64_t p, float* X,
                  int64_t ldx, int32_t* li, float* lv, int64_t ldl, int list_cap,
                  StartState s, double tol, int maxit, int32_t* colmark, const Plan* plan,
                  const CandPlan& cp) {
  const int per = (int)ceil_div(cp.nch * cp.cap, kRT);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)r), dim3(kRT), 0, st, (int)p, param, X, ldx, li,
                       lv, ldl, list_cap, s, tol, maxit, colmark, plan, cp);
  };
  if (per <= 4)
    run(wide_merge_kernel<KIND, 4>);
  else if (per <= 8)
    run(wide_merge_kernel<KIND, 8>);
  else if (per <= 16)
    run(wide_merge_kernel<KIND, 16>);
  else if (per <= 24)
    run(wide_merge_kernel<KIND, 24>);
  else if (per <= 32)
    run(wide_merge_kernel<KIND, 32>);
  else
    run(wide_merge_kernel<KIND, 48>);
}

void launch_wide_cand(hipStream_t st, XKind kind, const CandPlan& cp, double param,
                      const float* V, int64_t ldv, int64_t r, int64_t p, float* X, int64_t ldx,
                      int32_t* li, float* lv, int64_t ldl, int list_cap, StartState s, double tol,
                      int maxit, int32_t* colmark, const Plan* plan, Warm wm) {
  const bool top = kind == kTopS;
  if (cp.cap > 0)
    hipLaunchKernelGGL(wide_cand_kernel, dim3((unsigned)(cp.nch * r)), dim3(kRT), 0, st, V, ldv,
                       (int)p, X, ldx, s, cp, top ? 1 : 0);
  if (top) {
    launch_merge<kTopS>(st, param, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit,
                        colmark, plan, cp);
    return;
  }
  if (cp.cap > 0)
    launch_merge<kLambdaS>(st, param, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit,
                           colmark, plan, cp);
  hipLaunchKernelGGL(wide_lambda_kernel, dim3((unsigned)r), dim3(kLT), 0, st, V, ldv, (int)p,
                     param, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm,
                     cp.cap > 0 ? 1 : 0);
}

// warm-up of the penalties: gamma of the row from the (target + 1)-th largest
// key found by the digit passes, or the frozen value
template <int KIND>
__global__ __launch_bounds__(64) void gam_row_kernel(int64_t r, int p, StartState s,
                                                     Wide w) {
  const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (j >= r || !row_live(s, j)) return;
  WRow* R = w.rows + j;
  const bool warming = s.status == nullptr || s.iters[j] + 1 <= w.warm_K;
  if (!warming) {
    R->lam = w.gam[j];
  } else if ((int64_t)w.warm_target >= (int64_t)p) {
    R->lam = 0.0;
  } else {
    const double t = (double)__uint_as_float(R->prefix);
    R->lam = KIND == kHardGamma ? t * t : t;
  }
}

template <int KIND>
void launch_wide_kind(hipStream_t st, double param, const float* V,
                      int64_t ldv, int64_t r, int64_t p, float* X, int64_t ldx,
                      int32_t* li, float* lv, int64_t ldl, int list_cap,
                      StartState s, double tol, int maxit, int32_t* colmark,
                      const Plan* plan, const Wide& w) {
  const dim3 g2((unsigned)(w.nch * r));  // chunk fastest
  const int ip = (int)p;
  const bool warm_gamma = (KIND == kHardGamma || KIND == kSoftGamma) && w.warm_K > 0;
  if (KIND == kTopS || warm_gamma) {
    const int64_t want = warm_gamma ? (int64_t)w.warm_target + 1 : (int64_t)param;
    const int32_t need = (int32_t)(want < p ? want : p);
    const dim3 g1((unsigned)r);
    hipLaunchKernelGGL(wide_hist_kernel<0>, g2, dim3(kWT), 0, st, V, ldv, ip, s, w);
    hipLaunchKernelGGL(wide_decide_kernel<0>, g1, dim3(kWT), 0, st, s, w, need);
    hipLaunchKernelGGL(wide_hist_kernel<1>, g2, dim3(kWT), 0, st, V, ldv, ip, s, w);
    hipLaunchKernelGGL(wide_decide_kernel<1>, g1, dim3(kWT), 0, st, s, w, need);
    hipLaunchKernelGGL(wide_hist_kernel<2>, g2, dim3(kWT), 0, st, V, ldv, ip, s, w);
    hipLaunchKernelGGL(wide_decide_kernel<2>, g1, dim3(kWT), 0, st, s, w, need);
  }
  if (KIND == kTopS)
    hipLaunchKernelGGL(wide_eqcount_kernel, g2, dim3(kWT), 0, st, V, ldv, ip, s, w);
  if (warm_gamma)
    hipLaunchKernelGGL(gam_row_kernel<KIND>, dim3((unsigned)ceil_div(r, 64)), dim3(64), 0,
                       st, r, ip, s, w);
  hipLaunchKernelGGL(wide_partial_kernel<KIND>, g2, dim3(kWT), 0, st, V, ldv, ip,
                     param, s, w);
  hipLaunchKernelGGL(wide_row_kernel<KIND>, dim3((unsigned)r), dim3(kWave), 0, st, s, tol,
                     maxit, list_cap, li != nullptr ? 1 : 0, plan,
                     colmark != nullptr ? 1 : 0, w);
  hipLaunchKernelGGL(wide_emit_kernel<KIND>, g2, dim3(kWT), 0, st, V, ldv, ip, param,
                     X, ldx, li, lv, ldl, colmark, w);
}

}  // namespace

bool x_update_wide_scratch(int fid, double s_or_gamma, const float* V, int64_t ldv, int64_t r,
                           int64_t p, const float* X, int64_t ldx) {
  if (x_update_wide_bytes(fid, r, p) == 0) return false;
  const XKind kind = xkind_of(fid);
  return kind != kLambdaS && plan_cand(kind, s_or_gamma, V, ldv, X, ldx, r, p, 0).cap == 0 &&
         !records_in_x(kind, StartState{}, false, V, ldv, X, ldx, r, p);
}

size_t x_update_wide_bytes(int fid, int64_t r, int64_t p) {
  (void)fid;
  if (p <= kWideMinP || r < 1) return 0;
  size_t bytes = 0;
  (void)carve_wide(nullptr, r, p, &bytes);
  return bytes;
}

hipError_t x_update_wide_reset(hipStream_t st, void* scratch, int64_t r) {
  return hipMemsetAsync(scratch, 0, sizeof(uint32_t) * kWBins * r, st);
}

int64_t x_update_wide_clear_words(int64_t r) { return (int64_t)kWBins * r; }

bool x_update_wide(hipStream_t st, int fid, double s_or_gamma, const float* V,
                   int64_t ldv, int64_t r, int64_t p, float* X, int64_t ldx,
                   int32_t* list_idx, float* list_val, int64_t ldl, int list_cap,
                   StartState s, double tol, int32_t maxit, int32_t* colmark,
                   const Plan* plan, void* scratch, Warm wm) {
  if (x_update_wide_bytes(fid, r, p) == 0) return false;
  const XKind kind = xkind_of(fid);
  const CandPlan cp = plan_cand(kind, s_or_gamma, V, ldv, X, ldx, r, p, wm.K);
  if (kind == kLambdaS || cp.cap > 0) {
    launch_wide_cand(st, kind, cp, s_or_gamma, V, ldv, r, p, X, ldx, list_idx, list_val, ldl,
                     list_cap, s, tol, maxit, colmark, plan, wm);
    return true;
  }
  Wide w = carve_wide(scratch, r, p);
  if (scratch == nullptr) {
    if (!records_in_x(kind, s, list_idx != nullptr || colmark != nullptr, V, ldv, X, ldx, r, p))
      return false;
    w.xrec = X;
    w.ldx = ldx;
  }
  w.warm_K = wm.K;
  w.warm_target = wm.target;
  w.gam = wm.gam;
  switch (kind) {
    case kTopS:
      launch_wide_kind<kTopS>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx, list_val,
                              ldl, list_cap, s, tol, maxit, colmark, plan, w);
      return true;
    case kHardGamma:
      launch_wide_kind<kHardGamma>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                                   list_val, ldl, list_cap, s, tol, maxit, colmark, plan, w);
      return true;
    case kSoftGamma:
      launch_wide_kind<kSoftGamma>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                                   list_val, ldl, list_cap, s, tol, maxit, colmark, plan, w);
      return true;
    default:
      return false;
  }
}

}  // namespace spca
