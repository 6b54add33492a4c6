// x-update of Algorithm 2 (Table 3, rows S3-S6), one workgroup per start:
//   L0 constraint  x = T_s(v) / ||T_s(v)||             phi = ||T_s(v)||
//   L1 constraint  x = V_l(v) / ||V_l(v)||, l = lambda_s(v)
//                                                      phi = l sqrt(s) + ||V_l(v)||
//   L0 penalty     x = U_g(v) / ||U_g(v)||             phi = sum_kept (v_i^2 - g)
//   L1 penalty     x = V_g(v) / ||V_g(v)||             phi = ||V_g(v)||
// followed by the ratio stop test of Section 2.2.
//
// Selection without a sort.  The bit pattern of a non-negative float is
// monotone in its value, so thresholds are searched over the 31-bit keys of
// |v_i| by counting passes over register-resident rows.
//   T_s       largest key t with #{key >= t} >= s; ties at that key go to the
//             lowest indices (a block-wide prefix count finds the cut index).
//   lambda_s  the derivative of l sqrt(s) + ||V_l(v)|| is sqrt(s) - rho(l)
//             with rho = ||V_l||_1 / ||V_l||_2 non-increasing, so lambda = 0
//             when rho(0) <= sqrt(s), and otherwise the root on the k
//             largest entries, where it keeps exactly those, is
//             l = (S1_k - sqrt(s (k S2_k - S1_k^2) / (k - s))) / k.
//             Rounds of that formula rise to the root from below; rows they
//             do not settle (rounding; k <= s) take a search over keys with
//             FP64 sums of (|v| - t)_+ and its square for the float interval
//             holding the root, on which the active set is fixed.
// Comparisons that decide membership use FP64 on the FP32 inputs (squares
// and differences of floats are exact or correctly rounded there).
#include "../../include/spca.h"
#include "common.hpp"
#include "kernels.hpp"
#include "select.hpp"

namespace spca {
namespace {

// Exclusive prefix sums of two doubles per thread in thread order (kRT).
__device__ __forceinline__ void rscan2(double (&v)[2], double* scratch) {
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  double inc[2] = {v[0], v[1]};
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double o = __shfl_up(inc[c], off, kWave);
      if (lane >= off) inc[c] += o;
    }
  }
  if (lane == kWave - 1) {
    scratch[2 * wave] = inc[0];
    scratch[2 * wave + 1] = inc[1];
  }
  __syncthreads();
  double b0 = 0.0, b1 = 0.0;
  for (int w = 0; w < wave; ++w) {
    b0 += scratch[2 * w];
    b1 += scratch[2 * w + 1];
  }
  v[0] = b0 + inc[0] - v[0];
  v[1] = b1 + inc[1] - v[1];
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Register-resident rows, p <= 256 * NPT: a 256-thread block per start, so
// that every pass is register arithmetic and all starts of a batch are
// resident on the chip at once (1024 x 10000: 4 blocks a CU).  Reading V and
// writing X, 82 MB there, takes 17 us of the 27 us of T_s and 32 us of
// lambda_s; the rest is the passes and their barriers, which all blocks go
// through in step.  Norm, count and rounds therefore run over the at most
// 1024 entries that the search left, where there are such (over the whole
// row: 40 and 50 us; with three LDS histograms a selection and a sort of
// lambda_s candidates: 53 and 232 us).
// ---------------------------------------------------------------------------
// WARM: the sparsity-targeted warm-up (Section 4.1) of the parameter.
template <int KIND, int NPT, bool WARM>
__device__ __forceinline__ void full_update(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* __restrict__ X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int list_cap, const StartState& s,
    double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan,
    const Warm& wm, RSmem& sm) {
  static_assert(NPT % 4 == 0, "NPT must be a multiple of 4");
  const int64_t j = blockIdx.x;
  const bool full = s.status != nullptr;
  const int tid = threadIdx.x;
  // Striped rows: element 4 (q kRT + tid) + e is v[4 q + e], so that each
  // 16-byte load and store instruction covers 1 KB of contiguous memory.
  constexpr int R = NPT / 4;
  auto gidx = [&](int k) { return 4 * ((k / 4) * kRT + tid) + k % 4; };
  const float* vg = V + j * ldv;
  float v[NPT];
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    const int i = gidx(q);
    if (i + 3 < p) {
      const floatx4 t = *reinterpret_cast<const floatx4*>(vg + i);
      v[q] = t.x;
      v[q + 1] = t.y;
      v[q + 2] = t.z;
      v[q + 3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q + e] = i + e < p ? vg[i + e] : 0.f;
    }
  }

  uint32_t thr_key = 0;
  int cut = -1;
  int tied = 0;       // T_s: entries kept at the threshold itself
  double lam = 0.0;
  float c[kSelPer];   // the magnitudes of all entries from the threshold on, if few
  bool few = false;
  Bracket br;
  const int itc = full ? s.iters[j] + 1 : 1;  // this x-update's number
  const bool warming = WARM && itc <= wm.K;
  if (KIND == kTopS) {
    const uint32_t s_int = (uint32_t)((int64_t)param < (int64_t)p ? (int64_t)param : (int64_t)p);
    few = select_key<NPT>(v, p, s_int, sm, c, br);
    thr_key = br.lo;
    cut = p;
    tied = thr_key == 0u ? 0 : (int)((br.nlo < s_int ? br.nlo : s_int) - br.nhi);
    if (thr_key != 0u && br.nlo > s_int) {
      // ties at thr_key: keep the first (s - #{key > thr_key}) in index
      // order; rare, so from memory, a run of the row a thread
      const int need = (int)(s_int - br.nhi);
      const int run = (p + kRT - 1) / kRT;
      const int i0 = run * tid, i1 = i0 + run < p ? i0 + run : p;
      int eq = 0, total_eq;
#pragma unroll 1
      for (int i = i0; i < i1; ++i) eq += key_of(vg[i]) == thr_key;
      int seen = block_exclusive_scan(eq, sm.scan, &total_eq);
      if (tid == 0) sm.cut = -1;
      __syncthreads();
      if (seen < need && need <= seen + eq) {
#pragma unroll 1
        for (int i = i0; i < i1; ++i)
          if (key_of(vg[i]) == thr_key && ++seen == need) sm.cut = i;
      }
      __syncthreads();
      cut = sm.cut;
    }
  } else if (KIND == kLambdaS && WARM && !warming) {
    lam = wm.gam[j];  // frozen after the warm-up
  } else if (KIND == kLambdaS) {
    const double s_par = param;
    const double rs = sqrt(s_par);
    const bool done = lambda_root<NPT>(v, p, s_par, sm, c, few, br, lam);
    const uint32_t mk = br.mk;
    if (!done) {
      // fallback: FP64 search of the float interval holding the root; reads
      // the row from memory so that the fast path keeps its registers
      uint32_t lo = 0, hi = mk;
      while (hi - lo > 1) {
        uint32_t t[kNCd];
        spread<kNCd>(lo, hi, t);
        double acc[2 * kNCd];
#pragma unroll
        for (int c = 0; c < 2 * kNCd; ++c) acc[c] = 0.0;
        double tf[kNCd];
#pragma unroll
        for (int c = 0; c < kNCd; ++c) tf[c] = (double)__uint_as_float(t[c]);
#pragma unroll 1
        for (int i = tid; i < p; i += kRT) {
          const double a = fabs((double)vg[i]);
#pragma unroll
          for (int c = 0; c < kNCd; ++c) {
            double d = a - tf[c];
            d = d > 0.0 ? d : 0.0;
            acc[2 * c] += d;
            acc[2 * c + 1] += d * d;
          }
        }
        block_sum_n<double, 2 * kNCd>(acc, sm.dred);
        lambda_step<kNCd>(t, acc, rs, lo, hi);
      }
      const double tl = (double)__uint_as_float(lo);
      const double th = (double)__uint_as_float(hi);
      double ks[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
      for (int i = tid; i < p; i += kRT) {
        const double a = fabs((double)vg[i]);
        if (a > tl) {
          ks[0] += 1.0;
          ks[1] += a;
          ks[2] += a * a;
        }
      }
      block_sum_n<double, 3>(ks, sm.dred);
      const double k = ks[0], S1 = ks[1], S2 = ks[2];
      double l = tl;
      if (k > s_par) {
        double disc = k * S2 - S1 * S1;
        disc = disc > 0.0 ? disc : 0.0;
        l = (S1 - sqrt(s_par * disc / (k - s_par))) / k;
      }
      l = l < tl ? tl : l;
      l = l > th ? th : l;
      lam = l;
    }
  } else if (WARM && warming) {
    // gamma for target nonzeros: the (target + 1)-th largest |v_i| (or its
    // square for U_gamma), which the strict threshold then excludes
    if ((int64_t)wm.target >= (int64_t)p) {
      lam = 0.0;
    } else {
      (void)select_key<NPT>(v, p, (uint32_t)wm.target + 1u, sm, c, br);
      const double t = (double)__uint_as_float(br.lo);
      lam = KIND == kHardGamma ? t * t : t;
    }
  } else if (WARM) {
    lam = wm.gam[j];
  } else {
    lam = param;
  }

  const float lamf = float_above(lam);
  auto kept = [&](int i, float vv, double* w) -> bool {
    if (KIND == kTopS) {
      uint32_t k = key_of(vv);
      *w = (double)vv;
      return k != 0 && (k > thr_key || (k == thr_key && i <= cut));
    } else if (KIND == kHardGamma) {
      *w = (double)vv;
      return (double)vv * (double)vv > lam;
    } else {
      double a = fabs((double)vv);
      *w = vv > 0.f ? a - lam : lam - a;
      return fabsf(vv) >= lamf;
    }
  };

  // the kept entries' number and squares, from the candidates where there are
  // such, and their offsets in the list if one is written
  double acc[3] = {0.0, 0.0, 0.0};
  auto add = [&](float vv) {
    bool in;
    double w;
    if (KIND == kTopS) {
      in = key_of(vv) > thr_key;
      w = (double)vv;
    } else {
      in = kept(0, vv, &w);
    }
    if (in) {
      acc[0] += w * w;
      if (KIND == kHardGamma) acc[1] += w * w - lam;
      acc[2] += 1.0;
    }
  };
  if (few) {
#pragma unroll
    for (int e = 0; e < kSelPer; ++e) add(c[e]);
  } else {
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      if (k % 8 == 0) __builtin_amdgcn_sched_barrier(0);
      reload(v[k]);
      add(v[k]);
    }
  }
  block_sum_n<double, 3>(acc, sm.dred);
  if (KIND == kTopS && tied > 0) {
    const double w = (double)__uint_as_float(thr_key);
    acc[0] += (double)tied * (w * w);
    acc[2] += (double)tied;
  }
  const int total = (int)acc[2];
  int cnt[R], off[R];
  if (list_idx != nullptr) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      cnt[q] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 4 * q + e;
        double w;
        reload(v[k]);
        cnt[q] += kept(gidx(k), v[k], &w);
      }
    }
    rank_rows<R>(cnt, off, sm.pscan);
  }
  const double nrm = sqrt(acc[0]);
  double phi;
  if (KIND == kHardGamma)
    phi = acc[1];
  else if (KIND == kLambdaS)
    phi = lam * sqrt(param) + nrm;
  else
    phi = nrm;
  const bool zero = !(nrm > 0.0);
  const double inv = zero ? 0.0 : 1.0 / nrm;

  // the list is written only when it can serve the list-based product
  const bool listed = list_idx != nullptr && !zero && total <= list_cap;
  const bool marking = colmark != nullptr && !zero && plan->mark != 0;
  const int32_t epoch = marking ? plan->epoch : 0;
  int32_t* li = listed ? list_idx + j * ldl : nullptr;
  float* lv = listed ? list_val + j * ldl : nullptr;
  float* x = X + j * ldx;
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    float xo[4];
    int o = li != nullptr ? off[q / 4] : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double w;
      const int gi = gidx(q + e);
      reload(v[q + e]);  // recompute w here rather than hold it since the count pass
      const bool kp = kept(gi, v[q + e], &w) && !zero;
      xo[e] = kp ? (float)(w * inv) : 0.f;
      if (kp && li != nullptr) {
        li[o] = gi;
        lv[o] = xo[e];
        ++o;
      }
      if (kp && marking) colmark[gi] = epoch;
    }
    const int i = gidx(q);
    if (i + 3 < p) {
      floatx4 t = {xo[0], xo[1], xo[2], xo[3]};
      *reinterpret_cast<floatx4*>(x + i) = t;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + e < p) x[i + e] = xo[e];
    }
  }

  if (tid == 0) {
    if (WARM && warming && KIND != kTopS) wm.gam[j] = lam;
    // the selection threshold, a first guess for the next x-update
    if (full && s.thr != nullptr) {
      if (KIND == kTopS) s.thr[j] = zero ? 0.f : __uint_as_float(thr_key);
      if (KIND == kLambdaS) s.thr[j] = zero ? 0.f : (float)lam;
    }
    if (!full) {
      s.phi[j] = phi;
      s.nnz[j] = zero ? 0 : total;
    } else {
      const int it = s.iters[j] + 1;
      const double prev = s.phi[j];
      s.iters[j] = it;
      s.phi_prev[j] = prev;
      s.phi[j] = phi;
      s.nnz[j] = zero ? 0 : total;
      if (zero)
        s.status[j] = SPCA_ZERO;
      else if (it >= 2 && tol >= 0.0 && (!WARM || it >= wm.K + 1) &&
               phi <= (1.0 + tol) * prev)
        s.status[j] = SPCA_CONVERGED;
      else if (it >= maxit)
        s.status[j] = SPCA_MAXIT;
    }
  }
}

// The request of a grouped solve's start (its settings replace the launch's);
// false when it takes another operator.
__device__ __forceinline__ bool start_settings(const StartState& s, int64_t j, int kind,
                                               double& param, double& tol, int& maxit) {
  if (s.cfg == nullptr) return true;
  if (s.cfg[j].kind != kind) return false;
  param = s.cfg[j].param;
  tol = s.cfg[j].tol;
  maxit = s.cfg[j].maxit;
  return true;
}

template <int KIND, int NPT, bool WARM>
__global__ __launch_bounds__(kRT, WARM ? 2 : 4) void x_update_reg_kernel(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* __restrict__ X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int list_cap, StartState s,
    double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan,
    Warm wm) {
  __shared__ RSmem sm;
  const int64_t j = blockIdx.x;
  if (s.status != nullptr && s.status[j] != kRunning) return;
  if (!start_settings(s, j, KIND, param, tol, maxit)) return;
  // after the candidate kernel: only the rows it could not settle
  if (s.redo != nullptr && s.redo[j] == 0) return;
  full_update<KIND, NPT, WARM>(V, ldv, p, param, X, ldx, list_idx, list_val, ldl, list_cap, s,
                               tol, maxit, colmark, plan, wm, sm);
}

// ---------------------------------------------------------------------------
// Candidate x-update for T_s and V_{lambda_s} (register-resident rows,
// inside a solve).  Near convergence the selection threshold moves little
// between x-updates, so the entries with |v_i| at least 90% of the last
// threshold (the s-th largest |v_i|, or lambda) are few, and they contain
// every entry the operator keeps:
//   T_s       when at least s of them exist, the s largest |v_i| (ties to
//             the lower index) are the s first candidates in (|v| desc,
//             index asc) order;
//   lambda_s  when rho(t) = ||(|v| - t)_+||_1 / ||(|v| - t)_+||_2 >= sqrt(s)
//             at the guess t, the root lies above t (rho is non-increasing),
//             and the segment scan over the sorted candidates finds it.
// The candidates (at most kCandCap) are sorted in registers (a bitonic
// network: shuffles within a wave, LDS across waves, register swaps within
// a thread), and the norm, phi, list (sorted again, by index) and column
// marks all come from them; one more pass over the registers writes x.  A
// row whose guess does not hold (the first x-update, or a threshold that
// moved by more than 10%) is flagged in s.redo and left to
// x_update_reg_kernel, launched right after.  Reductions run in a fixed
// order, so results are deterministic.
// lambda_s first tries the last x-update's kept set S = {|v_i| > lambda'}:
// restricted to S, the root condition sum (|v| - l) = sqrt(s) ||(|v| - l)||_2
// is a quadratic in l whose smaller root is (S1 - sqrt(s (k S2 - S1^2) /
// (k - s))) / k (k = |S|, S1 = sum |v|, S2 = sum v^2 over S); when exactly
// the entries of S lie above that l, it is the root of the whole row, and
// the row is finished from registers without candidates or sorts.
// ---------------------------------------------------------------------------
constexpr int kCandCap = 1024;
constexpr int kCandPer = kCandCap / kRT;  // sorted positions per thread
constexpr float kGuessLow = 0.9f;
constexpr float kGuessRetry = 0.7f;  // the next guesses: this factor lower
constexpr int kLamRounds = 6;        // closed-form rounds of lambda_s before the candidates
constexpr uint32_t kIdxMask = 0x3fffu;    // row indices below 16384

struct CSmem {
  // candidate sort keys, (|v| bits) << 32 | (kIdxMask - index) << 1 | sign:
  // descending order is |v| descending, then index ascending
  uint64_t k64[kCandCap];
  int scan[kRW + 1];
  double dscan[2 * (kRW + 1)];
  double red[2];
  int kbest;
  double seg[4];
};

// Ascending bitonic sort of kRT E keys: x[e] is element tid + kRT e.
// Partners fewer than 64 apart are in the same wave (shuffles), 64 and 128
// apart in another wave (through buf, kRT E keys of LDS), kRT and more
// apart in the same thread.
template <int E>
__device__ __forceinline__ void block_sort_asc(uint64_t (&x)[E], uint64_t* buf) {
  const int tid = threadIdx.x;
  constexpr int N = kRT * E;
#pragma unroll
  for (int size = 2; size <= N; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride >= kRT) {
        const int d = stride / kRT;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int e2 = e ^ d;
          if (e2 > e) {
            const bool asc = ((tid + kRT * e) & size) == 0;
            const uint64_t a = x[e], b = x[e2];
            const bool sw = asc ? a > b : a < b;
            x[e] = sw ? b : a;
            x[e2] = sw ? a : b;
          }
        }
      } else {
        if (stride >= kWave) {
#pragma unroll
          for (int e = 0; e < E; ++e) buf[tid + kRT * e] = x[e];
          __syncthreads();
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int i = tid + kRT * e;
          const uint64_t b = stride >= kWave ? buf[i ^ stride] : lane_xor_by(x[e], stride);
          const bool lower = (i & stride) == 0;
          const bool asc = (i & size) == 0;
          const uint64_t mn = x[e] < b ? x[e] : b;
          const uint64_t mx = x[e] < b ? b : x[e];
          x[e] = lower == asc ? mn : mx;
        }
        if (stride >= kWave) __syncthreads();
      }
    }
  }
}

// Sorts arr[0, n) ascending in place (n <= kCandCap), padding with pad.
// Entries may have been written by any thread before the call.
template <int E>
__device__ __forceinline__ void sort_in_lds(uint64_t* arr, int n, uint64_t pad) {
  __syncthreads();
  uint64_t x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = threadIdx.x + kRT * e;
    x[e] = i < n ? arr[i] : pad;
  }
  __syncthreads();
  block_sort_asc<E>(x, arr);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = threadIdx.x + kRT * e;
    if (i < n) arr[i] = x[e];
  }
  __syncthreads();
}

// The same for n <= 64: the first wave sorts with shuffles alone.
__device__ __forceinline__ void sort_wave_lds(uint64_t* arr, int n, uint64_t pad) {
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    uint64_t x = lane < n ? arr[lane] : pad;
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1) {
#pragma unroll
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        const uint64_t b = lane_xor_by(x, stride);
        const bool lower = (lane & stride) == 0;
        const bool asc = (lane & size) == 0;
        const uint64_t mn = x < b ? x : b;
        const uint64_t mx = x < b ? b : x;
        x = lower == asc ? mn : mx;
      }
    }
    if (lane < n) arr[lane] = x;
  }
  __syncthreads();
}

__device__ __forceinline__ void sort_lds(uint64_t* arr, int n, uint64_t pad) {
  if (n <= kWave)
    sort_wave_lds(arr, n, pad);
  else if (n <= kRT)
    sort_in_lds<1>(arr, n, pad);
  else if (n <= 2 * kRT)
    sort_in_lds<2>(arr, n, pad);
  else
    sort_in_lds<4>(arr, n, pad);
}

// Sum over positions [0, m) of f(q), FP64, in a fixed order: lane l of the
// first wave adds positions l, l + 64, ..., then an xor butterfly.  The
// result is returned to every thread of the block.
template <typename F>
__device__ __forceinline__ double fixed_sum(int m, F f, double* slot) {
  if (threadIdx.x < kWave) {
    double a = 0.0;
    for (int q = threadIdx.x; q < m; q += kWave) a += f(q);
    a = wave_sum(a);
    if (threadIdx.x == 0) *slot = a;
  }
  __syncthreads();
  const double r = *slot;
  __syncthreads();
  return r;
}

// False (nothing written) for a row it cannot settle.
template <int KIND, int NPT>
__device__ __forceinline__ bool cand_update(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* __restrict__ X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int list_cap, const StartState& s,
    double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan, CSmem& sm) {
  static_assert(KIND == kTopS || KIND == kLambdaS, "T_s and lambda_s only");
  static_assert(kRT * NPT <= (int)kIdxMask + 1, "row indices must fit the sort key");
  const int64_t j = blockIdx.x;
  const int tid = threadIdx.x;
  const uint32_t t0 = key_of(s.thr[j] * kGuessLow);
  if (t0 == 0u) {  // no guess yet
    return false;
  }
  auto gidx = [&](int k) { return 4 * ((k / 4) * kRT + tid) + k % 4; };
  const float* vg = V + j * ldv;
  float v[NPT];
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    const int i = gidx(q);
    if (i + 3 < p) {
      const floatx4 w4 = *reinterpret_cast<const floatx4*>(vg + i);
      v[q] = w4.x;
      v[q + 1] = w4.y;
      v[q + 2] = w4.z;
      v[q + 3] = w4.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q + e] = i + e < p ? vg[i + e] : 0.f;
    }
  }
  if constexpr (KIND == kLambdaS) {
    // closed-form root on the last kept set (every branch below depends on
    // block totals only, so all threads take it together)
    constexpr int R = NPT / 4;
    // S_0 = {|v| > lambda'}; each round takes the root l of S_t's quadratic
    // and S_{t+1} = {|v| > l}, until S_{t+1} = S_t (l is then the root of the
    // row) or kLamRounds rounds; a row that does not settle takes the
    // candidate path below
    const double lprev = (double)s.thr[j];
    double set3[3] = {0.0, 0.0, 0.0};  // |S|, sum |v| and sum v^2 over S
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      reload(v[k]);  // each pass derives its doubles afresh (no copies held across passes)
      const double a = fabs((double)v[k]);
      if (a > lprev) {
        set3[0] += 1.0;
        set3[1] += a;
        set3[2] += a * a;
      }
    }
    block_sum_n<double, 3>(set3, reinterpret_cast<double*>(sm.k64));
    double lam = -1.0;
    int cnt[R], off[R];
    double acc[2] = {0.0, 0.0};
    bool settled = false;
#pragma unroll 1
    for (int round = 0; round < kLamRounds; ++round) {
      const double kk = set3[0];
      if (!(kk > param)) break;
      double disc = kk * set3[2] - set3[1] * set3[1];
      disc = disc > 0.0 ? disc : 0.0;
      lam = (set3[1] - sqrt(param * disc / (kk - param))) / kk;
      if (!(lam > 0.0)) break;
      // the set above lam: its size and sums (the next round's), and the
      // squared distances to lam (the norm, if the set is unchanged)
      double b4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < R; ++q) {
        cnt[q] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          reload(v[4 * q + e]);
          const double a = fabs((double)v[4 * q + e]);
          if (a > lam) {
            ++cnt[q];
            b4[0] += 1.0;
            b4[1] += a;
            b4[2] += a * a;
            b4[3] += (a - lam) * (a - lam);
          }
        }
      }
      block_sum_n<double, 4>(b4, reinterpret_cast<double*>(sm.k64));
      if (b4[0] == kk) {  // nested sets of equal size: unchanged
        acc[0] = b4[3];
        acc[1] = b4[0];
        settled = true;
        break;
      }
      set3[0] = b4[0];
      set3[1] = b4[1];
      set3[2] = b4[2];
    }
    if (settled) {  // {|v| > lam} is the set lam came from: lam is the root
      const int total = rank_rows<R>(cnt, off, sm.k64);
      const double nrm = sqrt(acc[0]);
      const double phi = lam * sqrt(param) + nrm;
      const bool zero = !(nrm > 0.0);
      const double inv = zero ? 0.0 : 1.0 / nrm;
      const bool listed = list_idx != nullptr && !zero && total <= list_cap;
      const bool marking = colmark != nullptr && !zero && plan->mark != 0;
      const int32_t epoch = marking ? plan->epoch : 0;
      int32_t* li = listed ? list_idx + j * ldl : nullptr;
      float* lv = listed ? list_val + j * ldl : nullptr;
      float* x = X + j * ldx;
#pragma unroll
      for (int q = 0; q < NPT; q += 4) {
        float xo[4];
        int o = off[q / 4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          reload(v[q + e]);
          const float vv = v[q + e];
          const double a = fabs((double)vv);
          const bool kp = a > lam && !zero;
          const double w = vv > 0.f ? a - lam : lam - a;
          xo[e] = kp ? (float)(w * inv) : 0.f;
          const int gi = gidx(q + e);
          if (kp && li != nullptr) {
            li[o] = gi;
            lv[o] = xo[e];
            ++o;
          }
          if (kp && marking) colmark[gi] = epoch;
        }
        const int i = gidx(q);
        if (i + 3 < p) {
          floatx4 w4 = {xo[0], xo[1], xo[2], xo[3]};
          *reinterpret_cast<floatx4*>(x + i) = w4;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (i + e < p) x[i + e] = xo[e];
        }
      }
      if (tid == 0) {
        s.thr[j] = zero ? 0.f : (float)lam;
        const int it = s.iters[j] + 1;
        const double prev = s.phi[j];
        s.iters[j] = it;
        s.phi_prev[j] = prev;
        s.phi[j] = phi;
        s.nnz[j] = zero ? 0 : total;
        if (zero)
          s.status[j] = SPCA_ZERO;
        else if (it >= 2 && tol >= 0.0 && phi <= (1.0 + tol) * prev)
          s.status[j] = SPCA_CONVERGED;
        else if (it >= maxit)
          s.status[j] = SPCA_MAXIT;
      }
      return true;
    }
  }
  // the candidate at sorted position q
  auto cval = [&](int q) -> float {  // signed value
    const uint64_t k = ~sm.k64[q];
    const uint32_t bits = (uint32_t)(k >> 32) | ((uint32_t)k << 31);
    return __uint_as_float(bits);
  };
  auto cidx = [&](int q) -> int {
    return (int)(kIdxMask - (((uint32_t)~sm.k64[q] >> 1) & kIdxMask));
  };
  const uint32_t s_int =
      (uint32_t)((int64_t)param < (int64_t)p ? (int64_t)param : (int64_t)p);

  // the guess t: accepted when it brackets the threshold (at least s keys
  // at or above it for T_s; for lambda_s more than s keys and
  // rho(t) >= sqrt(s), i.e. the root at or above t) with at most kCandCap
  // candidates; otherwise lowered twice by a factor 0.7 (too many
  // candidates leave the row to the full kernel at once)
  const double rs = sqrt(param);
  uint32_t t = t0;
  bool ok = false;
  int mine = 0;
#pragma unroll 1
  for (int attempt = 0; attempt < 3; ++attempt) {
    if (attempt > 0) t = key_of(__uint_as_float(t) * kGuessRetry);
    if (t == 0u) break;
    // (the rho test only picks the guess, so FP32 sums do: a guess
    // accepted by rounding finds no root segment below and is left to the
    // full kernel)
    mine = 0;
    float a[2] = {0.f, 0.f};
    const float tf = __uint_as_float(t);
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const bool in = key_of(v[k]) >= t;
      mine += in;
      if (KIND == kLambdaS) {
        const float d = in ? fabsf(v[k]) - tf : 0.f;
        a[0] += d;
        a[1] += d * d;
      }
    }
    const int n_in = block_sum(mine, sm.scan);
    if (KIND == kLambdaS) block_sum_n<float, 2>(a, reinterpret_cast<float*>(sm.dscan));
    if (n_in > kCandCap) break;
    if (KIND == kTopS ? n_in >= (int)s_int
                      : (double)n_in > param && a[1] > 0.f &&
                            (double)a[0] >= rs * sqrt((double)a[1])) {
      ok = true;
      break;
    }
  }
  if (!ok) {
    return false;
  }
  int nc;
  int off = block_exclusive_scan(mine, sm.scan, &nc);
  // sort keys, complemented so that an ascending sort gives (|v| desc,
  // index asc); the pads (all ones) go last
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const uint32_t key = key_of(v[k]);
    if (key >= t) {
      const uint32_t lo = ((kIdxMask - (uint32_t)gidx(k)) << 1) | (__float_as_uint(v[k]) >> 31);
      sm.k64[off++] = ~(((uint64_t)key << 32) | lo);
    }
  }
  sort_lds(sm.k64, nc, ~0ull);

  uint32_t thr_key = 0;
  int64_t cut = -1;
  double lam = 0.0;
  int nkept;
  if (KIND == kTopS) {
    thr_key = key_of(cval(s_int - 1));
    cut = cidx(s_int - 1);
    nkept = (int)s_int;
  } else {
    const double s_par = param;
    const double tf = (double)__uint_as_float(t);
    // prefix sums of c and c^2 over the sorted candidates; thread t owns
    // positions kCandPer t onward; the segment holding the root
    double cv[kCandPer], pre[2] = {0.0, 0.0};
#pragma unroll
    for (int e = 0; e < kCandPer; ++e) {
      const int q = kCandPer * tid + e;
      cv[e] = q < nc ? fabs((double)cval(q)) : 0.0;
      pre[0] += cv[e];
      pre[1] += cv[e] * cv[e];
    }
    rscan2(pre, sm.dscan);
    if (tid == 0) sm.kbest = INT32_MAX;
    __syncthreads();
    double S1 = pre[0], S2 = pre[1];
    int myk = INT32_MAX;
    double seg[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < kCandPer; ++e) {
      const int q = kCandPer * tid + e;
      S1 += cv[e];
      S2 += cv[e] * cv[e];
      const int k = q + 1;
      if (q >= nc || (double)k <= s_par || myk != INT32_MAX) continue;
      const double lo = k < nc ? fabs((double)cval(k)) : tf;
      const double l1 = S1 - (double)k * lo;
      const double l2 = S2 - 2.0 * lo * S1 + (double)k * lo * lo;
      if (l2 > 0.0 && l1 >= rs * sqrt(l2)) {
        myk = k;
        seg[0] = S1;
        seg[1] = S2;
        seg[2] = lo;
        seg[3] = cv[e];
      }
    }
    if (myk != INT32_MAX) atomicMin(&sm.kbest, myk);
    __syncthreads();
    const int kb = sm.kbest;
    if (myk == kb && kb != INT32_MAX) {
      sm.seg[0] = seg[0];
      sm.seg[1] = seg[1];
      sm.seg[2] = seg[2];
      sm.seg[3] = seg[3];
    }
    __syncthreads();
    if (kb == INT32_MAX) {  // rounding at the lower end: leave it to the full kernel
      return false;
    }
    const double k = (double)kb, S1b = sm.seg[0], S2b = sm.seg[1];
    double disc = k * S2b - S1b * S1b;
    disc = disc > 0.0 ? disc : 0.0;
    double l = (S1b - sqrt(s_par * disc / (k - s_par))) / k;
    l = l < sm.seg[2] ? sm.seg[2] : l;
    l = l > sm.seg[3] ? sm.seg[3] : l;
    lam = l;
    // kept: |v| > lambda, a prefix of the sorted candidates
    int cnt = 0;
    for (int q = tid; q < nc; q += kRT) cnt += fabs((double)cval(q)) > lam;
    nkept = block_sum(cnt, sm.scan);
  }
  // w of the kept candidate at sorted position q
  auto wsorted = [&](int q) -> double {
    const float x = cval(q);
    if (KIND == kTopS) return (double)x;
    const double a = fabs((double)x);
    return x > 0.f ? a - lam : lam - a;
  };
  const double nrm2 = fixed_sum(nkept, [&](int q) {
    const double w = wsorted(q);
    return w * w;
  }, &sm.red[0]);
  const double nrm = sqrt(nrm2);
  const double phi = KIND == kLambdaS ? lam * sqrt(param) + nrm : nrm;
  const bool zero = !(nrm > 0.0);
  const double inv = zero ? 0.0 : 1.0 / nrm;
  // list (index order) and column marks, from the kept candidates: their
  // (index, x value) pairs sorted by index
  const bool listed = list_idx != nullptr && !zero && nkept <= list_cap;
  const bool marking = colmark != nullptr && !zero && plan->mark != 0;
  const int32_t epoch = marking ? plan->epoch : 0;
  if (listed || marking) {
    uint64_t pr[kCandPer];
#pragma unroll
    for (int e = 0; e < kCandPer; ++e) {
      const int q = tid + kRT * e;
      pr[e] = q < nkept ? ((uint64_t)(uint32_t)cidx(q) << 32) |
                              __float_as_uint((float)(wsorted(q) * inv))
                        : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kCandPer; ++e) {
      const int q = tid + kRT * e;
      if (q < nkept) sm.k64[q] = pr[e];
    }
    sort_lds(sm.k64, nkept, ~0ull);
    for (int q = tid; q < nkept; q += kRT) {
      const uint64_t k = sm.k64[q];
      const int iq = (int)(k >> 32);
      if (listed) {
        list_idx[j * ldl + q] = iq;
        list_val[j * ldl + q] = __uint_as_float((uint32_t)k);
      }
      if (marking) colmark[iq] = epoch;
    }
  }
  // x, from the registers
  float* x = X + j * ldx;
#pragma unroll
  for (int q = 0; q < NPT; q += 4) {
    float xo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float vv = v[q + e];
      const uint32_t kk = key_of(vv);
      bool kp;
      double w;
      if (KIND == kTopS) {
        w = (double)vv;
        kp = kk != 0u && (kk > thr_key || (kk == thr_key && (int64_t)gidx(q + e) <= cut));
      } else {
        const double a = fabs((double)vv);
        w = vv > 0.f ? a - lam : lam - a;
        kp = a > lam;
      }
      xo[e] = (kp && !zero) ? (float)(w * inv) : 0.f;
    }
    const int i = gidx(q);
    if (i + 3 < p) {
      floatx4 w4 = {xo[0], xo[1], xo[2], xo[3]};
      *reinterpret_cast<floatx4*>(x + i) = w4;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + e < p) x[i + e] = xo[e];
    }
  }
  if (tid == 0) {
    s.thr[j] = zero ? 0.f : (KIND == kTopS ? __uint_as_float(thr_key) : (float)lam);
    const int it = s.iters[j] + 1;
    const double prev = s.phi[j];
    s.iters[j] = it;
    s.phi_prev[j] = prev;
    s.phi[j] = phi;
    s.nnz[j] = zero ? 0 : nkept;
    if (zero)
      s.status[j] = SPCA_ZERO;
    else if (it >= 2 && tol >= 0.0 && phi <= (1.0 + tol) * prev)
      s.status[j] = SPCA_CONVERGED;
    else if (it >= maxit)
      s.status[j] = SPCA_MAXIT;
  }
  return true;
}

template <int KIND, int NPT>
__global__ __launch_bounds__(kRT, 4) void x_update_cand_kernel(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* __restrict__ X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int list_cap, StartState s,
    double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan) {
  __shared__ CSmem sm;
  const int64_t j = blockIdx.x;
  if (s.status[j] != kRunning) return;
  if (!start_settings(s, j, KIND, param, tol, maxit)) return;
  const bool done = cand_update<KIND, NPT>(V, ldv, p, param, X, ldx, list_idx, list_val, ldl,
                                           list_cap, s, tol, maxit, colmark, plan, sm);
  if (threadIdx.x == 0) s.redo[j] = !done;
}

// Both in one launch, for rows short enough that the registers of the two fit
// together without spills: the launch after the candidates, mostly empty, costs
// 2 to 5 us of an iteration of 40 to 60 (100 x 500 with one start; 8 requests
// of 16 starts).
constexpr int kBothMax = 24;  // floats a thread

template <int KIND, int NPT>
__global__ __launch_bounds__(kRT, 4) void x_update_both_kernel(
    const float* __restrict__ V, int64_t ldv, int p, double param,
    float* __restrict__ X, int64_t ldx, int32_t* __restrict__ list_idx,
    float* __restrict__ list_val, int64_t ldl, int list_cap, StartState s,
    double tol, int maxit, int32_t* __restrict__ colmark, const Plan* plan) {
  __shared__ union {
    CSmem cand;
    RSmem full;
  } sm;
  const int64_t j = blockIdx.x;
  if (s.status[j] != kRunning) return;
  if (!start_settings(s, j, KIND, param, tol, maxit)) return;
  if (cand_update<KIND, NPT>(V, ldv, p, param, X, ldx, list_idx, list_val, ldl, list_cap, s, tol,
                             maxit, colmark, plan, sm.cand))
    return;
  __syncthreads();  // the shared memory changes hands
  full_update<KIND, NPT, false>(V, ldv, p, param, X, ldx, list_idx, list_val, ldl, list_cap, s,
                                tol, maxit, colmark, plan, Warm{}, sm.full);
}

template <int KIND, int NPT>
void launch_reg(hipStream_t st, double param, const float* V, int64_t ldv,
                int64_t r, int64_t p, float* X, int64_t ldx, int32_t* li,
                float* lv, int64_t ldl, int list_cap, StartState s, double tol,
                int maxit, int32_t* colmark, const Plan* plan, Warm wm) {
  // inside a solve, T_s and lambda_s first try the candidate kernel; the
  // full kernel then takes only the rows it flagged
  constexpr bool kCand = KIND == kTopS || KIND == kLambdaS;
  const bool cand = kCand && wm.K == 0 && s.status != nullptr && s.thr != nullptr &&
                    s.redo != nullptr;
  if (!cand) s.redo = nullptr;
  if constexpr (kCand && NPT <= kBothMax) {
    if (cand) {
      hipLaunchKernelGGL((x_update_both_kernel<KIND, NPT>), dim3((unsigned)r), dim3(kRT), 0, st, V,
                         ldv, (int)p, param, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark,
                         plan);
      return;
    }
  } else if constexpr (kCand) {
    if (cand)
      hipLaunchKernelGGL((x_update_cand_kernel<KIND, NPT>), dim3((unsigned)r), dim3(kRT),
                         0, st, V, ldv, (int)p, param, X, ldx, li, lv, ldl, list_cap, s,
                         tol, maxit, colmark, plan);
  }
  if (KIND != kTopS && wm.K > 0)
    hipLaunchKernelGGL((x_update_reg_kernel<KIND, NPT, true>), dim3((unsigned)r),
                       dim3(kRT), 0, st, V, ldv, (int)p, param, X, ldx, li, lv,
                       ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else
    hipLaunchKernelGGL((x_update_reg_kernel<KIND, NPT, false>), dim3((unsigned)r),
                       dim3(kRT), 0, st, V, ldv, (int)p, param, X, ldx, li, lv,
                       ldl, list_cap, s, tol, maxit, colmark, plan, wm);
}

template <int KIND>
void launch_kind(hipStream_t st, double param, const float* V, int64_t ldv,
                 int64_t r, int64_t p, float* X, int64_t ldx, int32_t* li,
                 float* lv, int64_t ldl, int list_cap, StartState s, double tol,
                 int maxit, int32_t* colmark, const Plan* plan, Warm wm) {
  const int64_t per = ceil_div(p, kRT);
  if (per <= 8)
    launch_reg<KIND, 8>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else if (per <= 16)
    launch_reg<KIND, 16>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else if (per <= 24)
    launch_reg<KIND, 24>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else if (per <= 32)
    launch_reg<KIND, 32>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else if (per <= 40)
    launch_reg<KIND, 40>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
  else
    launch_reg<KIND, 48>(st, param, V, ldv, r, p, X, ldx, li, lv, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
}

}  // namespace

void x_update(hipStream_t st, int fid, double s_or_gamma, const float* V,
              int64_t ldv, int64_t r, int64_t p, float* X, int64_t ldx,
              int32_t* list_idx, float* list_val, int64_t ldl, int list_cap,
              StartState s, double tol, int32_t maxit, int32_t* colmark,
              const Plan* plan, void* wide, Warm wm) {
  if (p > kWideMinP) {
    (void)x_update_wide(st, fid, s_or_gamma, V, ldv, r, p, X, ldx, list_idx, list_val,
                        ldl, list_cap, s, tol, maxit, colmark, plan, wide, wm);
    return;
  }
  switch (xkind_of(fid)) {
    case kTopS:
      launch_kind<kTopS>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                         list_val, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
      break;
    case kLambdaS:
      launch_kind<kLambdaS>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                            list_val, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
      break;
    case kHardGamma:
      launch_kind<kHardGamma>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                              list_val, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
      break;
    case kSoftGamma:
      launch_kind<kSoftGamma>(st, s_or_gamma, V, ldv, r, p, X, ldx, list_idx,
                              list_val, ldl, list_cap, s, tol, maxit, colmark, plan, wm);
      break;
  }
}

}  // namespace spca
