// Selection in a block of 256 threads that holds a row, or a part of one, in
// registers: the threshold of the s largest magnitudes and lambda_s, by
// counting passes and closed-form rounds (the device side that the x-updates
// of short and long rows share).
#pragma once

#include "common.hpp"

namespace spca {
namespace {

constexpr int kNCd = 7;    // thresholds per FP64 search step

__device__ __forceinline__ uint32_t key_of(float v) {
  return __float_as_uint(v) & 0x7fffffffu;
}

// NC thresholds that split (lo, hi) evenly; hi stands for none.
template <int NC>
__device__ __forceinline__ void spread(uint32_t lo, uint32_t hi, uint32_t (&t)[NC]) {
  const uint32_t span = hi - lo;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    uint32_t d = span > NC + 1
                     ? (uint32_t)(((uint64_t)span * (uint64_t)(c + 1)) / (NC + 1))
                     : (uint32_t)(c + 1);
    t[c] = d < span ? lo + d : hi;
  }
}

// A step of the search for lambda_s among keys: the sums of (|v| - t)_+ and of
// its square at the thresholds t of spread() halve [lo, hi) around the largest
// key with ||.||_1 >= rs ||.||_2.  The first threshold that fails bounds it
// from above and those before it from below, so that the bracket shrinks with
// every step even where rounding makes the comparison fall either way (s equal
// entries: the two sides agree at every t).
template <int NC>
__device__ __forceinline__ void lambda_step(const uint32_t (&t)[NC], const double (&acc)[2 * NC],
                                            double rs, uint32_t& lo, uint32_t& hi) {
  bool open = true;  // no threshold has failed yet
  uint32_t nlo = lo, nhi = hi;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const bool in = open && t[c] < hi;
    const bool above = acc[2 * c + 1] > 0.0 && acc[2 * c] >= rs * sqrt(acc[2 * c + 1]);
    nlo = in && above ? t[c] : nlo;
    nhi = in && !above ? t[c] : nhi;
    open = in && above;
  }
  lo = nlo;
  hi = nhi;
}

// Four floats of a row, loaded and stored with one 16-byte instruction: global
// memory asks for 4-byte alignment only, so rows of any leading dimension
// and offset take it (900 x 12285: T_s 31 us, lambda_s 50, U_g 19; one
// 1024-thread workgroup a row from LDS took 290, 712 and 28).
typedef float floatx4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRT = 256;  // threads per start
constexpr int kRW = kRT / kWave;
constexpr int kSelPer = 4;
constexpr int kSelCap = kSelPer * kRT;  // entries that a selection goes on with alone
constexpr int kLamRoundsFull = 40;  // closed-form rounds of lambda_s from the whole row

struct RSmem {
  double dred[2 * kNCd * (kRW + 1)];
  uint32_t ured[2 * kRW];
  int scan[kRW + 1];
  float cand[kSelCap];
  int cut;
  uint64_t pscan[3 * (kRW + 1)];  // packed per-row counts (rank_rows)
};

// Index-order ranks over the striped row layout of the one-workgroup
// x-update: thread t holds elements 4 (q kRT + t) + e, e < 4, for rows q <
// R.  Given per-thread counts c[q] <= 4 of the elements that satisfy a
// predicate, returns in base[q] the number of such elements at a lower
// index than this thread's row-q group (earlier rows of the whole block,
// then lower threads of the same row), and the block total.  Four 16-bit
// fields per 64-bit word hold row counts up to 4 kRT without carries.
template <int R>
__device__ __forceinline__ int rank_rows(const int (&c)[R], int (&base)[R], uint64_t* scratch) {
  constexpr int W = (R + 3) / 4;
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  uint64_t in[W], inc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) in[w] = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) in[q / 4] |= (uint64_t)c[q] << (16 * (q % 4));
#pragma unroll
  for (int w = 0; w < W; ++w) inc[w] = wave_scan(in[w]);
  if (lane == kWave - 1) {
#pragma unroll
    for (int w = 0; w < W; ++w) scratch[wave * W + w] = inc[w];
  }
  __syncthreads();
  uint64_t before[W], tot[W];
#pragma unroll
  for (int w = 0; w < W; ++w) before[w] = tot[w] = 0;
#pragma unroll
  for (int u = 0; u < kRW; ++u) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint64_t x = scratch[u * W + w];
      if (u < wave) before[w] += x;
      tot[w] += x;
    }
  }
  __syncthreads();
  int run = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int sh = 16 * (q % 4);
    const int mine = (int)(((before[q / 4] + inc[q / 4] - in[q / 4]) >> sh) & 0xffffu);
    base[q] = run + mine;
    run += (int)((tot[q / 4] >> sh) & 0xffffu);
  }
  return run;
}

// Marks a register value as changed, so that the compiler recomputes what
// it derives from it (keys, bins) instead of holding copies across passes.
__device__ __forceinline__ void reload(float& x) { asm volatile("" : "+v"(x)); }

// Number of the block's entries with |v| at or above the float of key t; one
// compare an entry and one barrier a call (parity: consecutive calls alternate
// it, so that a wave may write its count while another still reads the last).
template <int N>
__device__ __forceinline__ uint32_t count_from(float (&v)[N], uint32_t t, uint32_t parity,
                                               uint32_t* scratch) {
  const float f = __uint_as_float(t);
  uint32_t n = 0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    reload(v[k]);
    n += (uint32_t)__popcll(__ballot(fabsf(v[k]) >= f));
  }
  uint32_t* c = scratch + kRW * parity;
  if (threadIdx.x % kWave == 0) c[threadIdx.x / kWave] = n;
  __syncthreads();
  n = 0;
#pragma unroll
  for (int w = 0; w < kRW; ++w) n += c[w];
  return n;
}

// Compacts the entries with |v| >= f, at most kSelCap, into LDS in thread
// order and deals them out again, kSelPer a thread (zeros beyond them).
template <int NPT>
__device__ __forceinline__ void compact(float (&v)[NPT], float f, RSmem& sm,
                                        float (&c)[kSelPer]) {
  int mine = 0;
#pragma unroll
  for (int k = 0; k < NPT; ++k) mine += fabsf(v[k]) >= f;
  int n;
  int off = block_exclusive_scan(mine, sm.scan, &n);
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    reload(v[k]);  // compare again rather than hold the masks
    if (fabsf(v[k]) >= f) sm.cand[off++] = fabsf(v[k]);
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kSelPer; ++e) {
    const int i = threadIdx.x + e * kRT;
    c[e] = i < n ? sm.cand[i] : 0.f;
  }
}

// The magnitude that about one in `ratio` entries of standard normal noise
// exceeds (asymptotic tail quantile): where searches start.  Any value is a
// valid start.
__device__ __forceinline__ float tail_quantile(float ratio) {
  const float q = logf(fmaxf(ratio, 1.05f));
  return q > 1.f ? sqrtf(2.f * q - logf(3.f * q)) : 0.95f * q;
}

// Search for the need-th largest key of a row (1 <= need <= p): the bracket
// #{key >= lo} >= need > #{key >= hi} with those counts.
struct Bracket {
  uint32_t lo, hi, nlo, nhi, parity;
  uint32_t mk;  // the largest key
  bool nan;     // the row holds NaN
  bool slack;   // lambda_s: certainly 0 (see narrow)
};

// Halves the bracket in key space (a float's bits are monotone and about
// logarithmic in it) by counting passes over the registers, from the start t,
// until at most cap entries lie from lo on; false if that needs lo = 0 or
// ties forbid it.  Counting takes one compare an entry, where a histogram of
// the key's bits takes an LDS atomic, most of them on the few bins that hold
// most of a row.  ured: 2 kRW words of LDS.
template <int NPT>
__device__ __forceinline__ bool narrow_from(float (&v)[NPT], uint32_t need, uint32_t cap,
                                            uint32_t t, uint32_t* ured, Bracket& b) {
  uint32_t step = 1u << 21;  // a quarter of a binade: brackets a start that is nearly right
  bool first = true, down = false;
  while (b.hi - b.lo > 1u && b.nlo > cap) {
    if (!(t > b.lo && t < b.hi)) t = b.lo + (b.hi - b.lo) / 2u;
    const uint32_t n = count_from(v, t, b.parity, ured);
    b.parity ^= 1u;
    const bool in = n >= need;
    if (in) {
      b.lo = t;
      b.nlo = n;
    } else {
      b.hi = t;
      b.nhi = n;
    }
    // steps in one direction double; the first turn brackets the threshold
    if (!first && down == in) step = 0u;
    first = false;
    down = !in;
    t = step == 0u ? 0u : (in ? t + step : (t > step ? t - step : 0u));
    step *= 2u;
  }
  return b.lo > 0u && b.nlo <= cap;
}

// The same from the whole row of p entries, from a start by tail_quantile; false
// for a row with NaN too: the whole-row passes give its norm as NaN.
// LAMBDA: with rs = sqrt(s), a row whose FP32 sums place ||v||_1 below rs
// ||v||_2 by a thousandth, far beyond their rounding (a few 1e-6; the sum of
// squares within its range), has an inactive constraint: b.slack, no search
// (1024 x 10000, 1% nonzero, s = 1000: 57 us with the search, 23 without).
template <int NPT, bool LAMBDA = false>
__device__ __forceinline__ bool narrow(float (&v)[NPT], int p, uint32_t need, uint32_t cap,
                                       RSmem& sm, Bracket& b, float rs = 0.f) {
  constexpr int NS = LAMBDA ? 2 : 1;
  float sum[NS] = {};
  uint32_t mk = 0;
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const uint32_t key = key_of(v[k]);
    mk = key > mk ? key : mk;
    sum[0] += v[k] * v[k];
    if (LAMBDA) sum[NS - 1] += fabsf(v[k]);
  }
  block_sum_n<float, NS>(sum, reinterpret_cast<float*>(sm.dred));
  const float sq = sum[0];
  mk = block_max(mk, sm.ured);
  b = Bracket{0u, mk + 1u, (uint32_t)p, 0u, 0u, mk, sq != sq, false};
  if (LAMBDA && sq > 1e-30f && sq < 1e30f && sum[NS - 1] < 0.999f * rs * sqrtf(sq)) {
    b.slack = true;
    return false;
  }
  const float want = fminf(1.4f * (float)need + 16.f, 0.5f * (float)(need + cap));
  const uint32_t t = key_of(sqrtf(sq / (float)p) * tail_quantile((float)p / want));
  return narrow_from<NPT>(v, need, cap, t, sm.ured, b) && !b.nan;
}

// Halves the bracket over v down to one key: the need-th largest.
template <int N>
__device__ __forceinline__ void settle(float (&v)[N], uint32_t need, uint32_t* ured,
                                       Bracket& b) {
  while (b.hi - b.lo > 1u) {
    const uint32_t t = b.lo + (b.hi - b.lo) / 2u;
    const uint32_t n = count_from(v, t, b.parity, ured);
    b.parity ^= 1u;
    if (n >= need) {
      b.lo = t;
      b.nlo = n;
    } else {
      b.hi = t;
      b.nhi = n;
    }
  }
}

// The need-th largest key of the row is b.lo, with b.nlo keys from it on and
// b.nhi above it; true if all of those are in c.
template <int NPT>
__device__ __forceinline__ bool select_key(float (&v)[NPT], int p, uint32_t need, RSmem& sm,
                                           float (&c)[kSelPer], Bracket& b) {
  const bool few = narrow<NPT>(v, p, need, kSelCap, sm, b);
  if (few) {
    compact(v, __uint_as_float(b.lo), sm, c);
    settle<kSelPer>(c, need, sm.ured, b);
  } else {
    settle<NPT>(v, need, sm.ured, b);
  }
  return few;
}

// The smallest float above l >= 0: |v| >= float_above(l) is |v| > l.
__device__ __forceinline__ float float_above(double l) {
  const float f = (float)l;
  if (!((double)f <= l)) return f;
  return f == 0.f ? __uint_as_float(1u) : __uint_as_float(__float_as_uint(f) + 1u);
}

// Count, sum and sum of squares of the entries with |v| >= f.
template <int N>
__device__ __forceinline__ void sums_from(float (&v)[N], float f, double (&b)[3],
                                          double* scratch) {
  int n = 0;
  b[1] = b[2] = 0.0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // few conversions live at once
    reload(v[k]);
    const bool in = fabsf(v[k]) >= f;
    n += in;
    const double a = (double)(in ? fabsf(v[k]) : 0.f);
    b[1] += a;
    b[2] += a * a;
  }
  b[0] = (double)n;
  block_sum_n<double, 3>(b, scratch);
}

// From the count, sum and sum of squares over {|v| >= t}: is rho(t) > sqrt(s)
// beyond rounding?  Then the row's root lies above t.
__device__ __forceinline__ bool rho_above(const double (&set3)[3], double t, double rs) {
  const double l1 = set3[1] - set3[0] * t;
  const double l2 = set3[2] - 2.0 * t * set3[1] + set3[0] * t * t;
  return l2 > 1e-12 * set3[2] && l1 > (1.0 + 1e-9) * rs * sqrt(l2);
}

// The root on a set of more than s entries with these sums.
__device__ __forceinline__ double lambda_of(const double (&set3)[3], double s_par) {
  double disc = set3[0] * set3[2] - set3[1] * set3[1];
  disc = disc > 0.0 ? disc : 0.0;
  return (set3[1] - sqrt(s_par * disc / (set3[0] - s_par))) / set3[0];
}

// lambda_s of the row (0 where the constraint is inactive); false if the
// rounds do not settle it.
//
// The root on a set S of entries, l = (S1 - sqrt(s (k S2 - S1^2) / (k - s))) /
// k with k = |S|, S1 = sum |v|, S2 = sum v^2 over S, lies at or below the
// row's while S holds every entry above that one (entries below l only lower
// the sum and raise the norm).  So each round takes S to {|v| > l}, and l
// rises to the row's root, reached when S no longer changes.  S begins as
// {|v| >= t} if rho(t) > sqrt(s) there, which places the root above t, else
// as all nonzero entries.  t has the 8 s largest entries or more above it (a
// row of noise and s larger entries keeps about 5 s) and at most kSelCap, and
// the rounds run over those alone (c, if few); S from the whole row does so
// once it has come down to that.  Entries equal to the bound itself (ties at t)
// can place l below it: the bound then stays, and S loses them.  Where more
// than s entries equal the largest, no root lies below that: l ends there, S is
// empty and w = 0, as from the search.
template <int NPT>
__device__ __forceinline__ bool lambda_root(float (&v)[NPT], int p, double s_par, RSmem& sm,
                                            float (&c)[kSelPer], bool& few, Bracket& b,
                                            double& lam) {
  const double rs = sqrt(s_par);
  double set3[3] = {0.0, 0.0, 0.0};
  const double want = 8.0 * s_par < 800.0 ? 8.0 * s_par : 800.0;
  float f = 0.f;
  few = narrow<NPT, true>(v, p, want < (double)p ? (uint32_t)want : (uint32_t)p, kSelCap, sm, b,
                          (float)rs);
  if (b.slack) {
    lam = 0.0;
    return true;
  }
  if (few) {
    f = __uint_as_float(b.lo);
    lam = (double)f;
    compact(v, f, sm, c);
    sums_from<kSelPer>(c, f, set3, sm.dred);
    few = rho_above(set3, lam, rs);
  }
  if (!few) {
    lam = 0.0;
    f = __uint_as_float(1u);
    sums_from<NPT>(v, f, set3, sm.dred);
    if (b.nan || !(set3[1] > rs * sqrt(set3[2]))) return true;  // inactive, or NaN
  }
#pragma unroll 1
  for (int round = 0; round < kLamRoundsFull; ++round) {
    const double kk = set3[0];
    if (!(kk > s_par)) break;
    double l = lambda_of(set3, s_par);
    const bool held = !(l > lam);
    if (held) l = lam;
    if (!few && kk <= (double)kSelCap) {
      compact(v, f, sm, c);
      few = true;
    }
    f = float_above(l);
    if (few)
      sums_from<kSelPer>(c, f, set3, sm.dred);
    else
      sums_from<NPT>(v, f, set3, sm.dred);
    lam = l;
    if (set3[0] == 0.0) {
      const double top = (double)__uint_as_float(b.mk);
      lam = l < top ? l : top;
      return true;
    }
    if (set3[0] == kk) {  // nested sets of equal size: unchanged
      if (held) break;    // rounding: left to the caller's search
      return true;
    }
  }
  few = false;
  return false;
}

}  // namespace
}  // namespace spca
