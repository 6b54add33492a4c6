// Internal helpers of libspca: error reporting, launch checks and
// deterministic block reductions for gfx950 (wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

namespace spca {

constexpr int kWave = 64;

// Thread-local last-error message (exported through spca_last_error).
void set_error(const std::string& msg);
const char* last_error();

struct Status {
  int code;
};

#define SPCA_HIP_TRY(expr)                                                   \
  do {                                                                       \
    hipError_t _e = (expr);                                                  \
    if (_e != hipSuccess) {                                                  \
      ::spca::set_error(std::string(#expr) + ": " + hipGetErrorString(_e));  \
      return SPCA_EHIP;                                                      \
    }                                                                        \
  } while (0)

#define SPCA_LAUNCH_CHECK(what)                                              \
  do {                                                                       \
    hipError_t _e = hipGetLastError();                                       \
    if (_e != hipSuccess) {                                                  \
      ::spca::set_error(std::string("launch of ") + (what) + ": " +          \
                        hipGetErrorString(_e));                              \
      return SPCA_EHIP;                                                      \
    }                                                                        \
  } while (0)

#define SPCA_REQUIRE(cond, msg)                                              \
  do {                                                                       \
    if (!(cond)) {                                                           \
      ::spca::set_error(msg);                                                \
      return SPCA_EINVAL;                                                    \
    }                                                                        \
  } while (0)

__host__ __device__ inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
__host__ __device__ inline int64_t ceil_div(int64_t x, int64_t m) { return (x + m - 1) / m; }

// ---------------------------------------------------------------------------
// Exchanges between the lanes of a wave by DPP and row swaps, in registers: a
// shuffle through LDS (ds_bpermute) takes 60 to 100 cycles until its value is
// there, and the six steps of a reduction or a scan wait for one another.
// All 64 lanes must be active.
// ---------------------------------------------------------------------------
template <typename T>
struct Words {  // a 4- or 8-byte value as 32-bit words
  static constexpr int N = sizeof(T) / 4;
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "4- or 8-byte values");
  int w[N];
  __device__ __forceinline__ explicit Words(T v) { __builtin_memcpy(w, &v, sizeof(T)); }
  __device__ __forceinline__ T value() const {
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
  }
};

// DPP move; lanes without a source, or outside the rows of ROWS, get 0.
template <int CTRL, int ROWS = 0xf, typename T>
__device__ __forceinline__ T dpp(T v) {
  Words<T> a(v);
#pragma unroll
  for (int i = 0; i < Words<T>::N; ++i)
    a.w[i] = __builtin_amdgcn_update_dpp(0, a.w[i], CTRL, ROWS, 0xf, false);
  return a.value();
}

// For M = 16 or 32: *lo is the value of lane & ~M, *hi that of lane | M.
template <int M, typename T>
__device__ __forceinline__ void lane_pair(T v, T* lo, T* hi) {
  static_assert(M == 16 || M == 32, "rows or halves");
  Words<T> a(v), b(v);
#pragma unroll
  for (int i = 0; i < Words<T>::N; ++i) {
    const auto r = M == 16 ? __builtin_amdgcn_permlane16_swap(a.w[i], b.w[i], false, false)
                           : __builtin_amdgcn_permlane32_swap(a.w[i], b.w[i], false, false);
    a.w[i] = (int)r[0];
    b.w[i] = (int)r[1];
  }
  *lo = a.value();
  *hi = b.value();
}

constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppXor3 = 0x1b;  // within 4 lanes
constexpr int kDppXor7 = 0x141;                                   // half row mirror
constexpr int kDppRor = 0x120;                                    // rotate a row of 16
constexpr int kDppShr = 0x110;                                    // shift a row up
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;

// The value of lane ^ M.
template <int M, typename T>
__device__ __forceinline__ T lane_xor(T v) {
  if constexpr (M == 1) {
    return dpp<kDppXor1>(v);
  } else if constexpr (M == 2) {
    return dpp<kDppXor2>(v);
  } else if constexpr (M == 4) {
    return dpp<kDppXor7>(dpp<kDppXor3>(v));
  } else if constexpr (M == 8) {
    return dpp<kDppRor + 8>(v);
  } else {
    T lo, hi;
    lane_pair<M>(v, &lo, &hi);
    return (threadIdx.x & M) != 0 ? lo : hi;
  }
}

// The same for a power of two m that is a constant once the caller's loop is
// unrolled.
template <typename T>
__device__ __forceinline__ T lane_xor_by(T v, int m) {
  switch (m) {
    case 1: return lane_xor<1>(v);
    case 2: return lane_xor<2>(v);
    case 4: return lane_xor<4>(v);
    case 8: return lane_xor<8>(v);
    case 16: return lane_xor<16>(v);
    default: return lane_xor<32>(v);
  }
}

// op over the wave by the butterfly lane ^ 32, 16, 8, 4, 2, 1 (op commutes;
// from the third step on all rows of 16 agree, so a rotation serves as xor).
template <typename T, typename Op>
__device__ __forceinline__ T wave_all(T v, Op op) {
  T lo, hi;
  lane_pair<32>(v, &lo, &hi);
  v = op(lo, hi);
  lane_pair<16>(v, &lo, &hi);
  v = op(lo, hi);
  v = op(v, dpp<kDppRor + 8>(v));
  v = op(v, dpp<kDppRor + 4>(v));
  v = op(v, dpp<kDppXor2>(v));
  return op(v, dpp<kDppXor1>(v));
}

// Inclusive prefix sum over the wave's lanes (integers).
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {
  v += dpp<kDppShr + 1>(v);
  v += dpp<kDppShr + 2>(v);
  v += dpp<kDppShr + 4>(v);
  v += dpp<kDppShr + 8>(v);
  v += dpp<kDppBcast15, 0xa>(v);  // rows 1 and 3: the sum of the row below
  v += dpp<kDppBcast31, 0xc>(v);  // rows 2 and 3: the sum of the lower half
  return v;
}

// ---------------------------------------------------------------------------
// Deterministic reductions.  A wave reduces with a fixed xor butterfly; waves
// are then summed in wave order.  The result does not depend on timing, only
// on the block size.
// ---------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  return wave_all(v, [](T a, T b) { return a + b; });
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  return wave_all(v, [](T a, T b) { return b > a ? b : a; });
}

// Sums NV values per thread over the block; every thread receives the
// totals.  scratch must hold NV * (blockDim/64) elements of T.
template <typename T, int NV>
__device__ __forceinline__ void block_sum_n(T (&v)[NV], T* scratch) {
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int nwaves = blockDim.x / kWave;
#pragma unroll
  for (int c = 0; c < NV; ++c) v[c] = wave_sum(v[c]);
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < NV; ++c) scratch[wave * NV + c] = v[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NV; ++c) v[c] = 0;
#pragma unroll 4
  for (int w = 0; w < nwaves; ++w) {
#pragma unroll
    for (int c = 0; c < NV; ++c) v[c] += scratch[w * NV + c];
  }
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ T block_sum(T v, T* scratch) {
  T a[1] = {v};
  block_sum_n<T, 1>(a, scratch);
  return a[0];
}

// Block max; scratch holds blockDim/64 elements.
template <typename T>
__device__ __forceinline__ T block_max(T v, T* scratch) {
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int nwaves = blockDim.x / kWave;
  v = wave_max(v);
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  v = scratch[0];
#pragma unroll 4
  for (int w = 1; w < nwaves; ++w) v = scratch[w] > v ? scratch[w] : v;
  __syncthreads();
  return v;
}

// Exclusive prefix sum of one integer per thread in thread order; returns the
// thread's offset and writes the block total to *total.  scratch holds
// blockDim/64 values.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* scratch, T* total) {
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int nwaves = blockDim.x / kWave;
  const T incl = wave_scan(v);
  if (lane == kWave - 1) scratch[wave] = incl;
  __syncthreads();
  T before = 0, sum = 0;
#pragma unroll 4
  for (int w = 0; w < nwaves; ++w) {
    const T t = scratch[w];
    before += w < wave ? t : (T)0;
    sum += t;
  }
  __syncthreads();
  *total = sum;
  return before + incl - v;
}

// FP32 -> BF16 bit pattern, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}

// Marks in C: a product on BF16 parts leaves one at the first element of every 16
// x 16 block that it cannot serve, and a second launch on FP32 tiles, each of
// which looks for marks in its own part of C, computes the tiles that hold one.
// The mark is a quiet NaN with a payload that no sum of the first launch stores.
constexpr uint32_t kMark = 0x7fc5a9a5u;
constexpr int kMarkBlock = 16;

// Whether rows [m0, m0 + BM) by columns [n0, n0 + BN) of C hold a mark
// (wave-uniform, the same in every wave that asks).
template <int BM, int BN>
__device__ __forceinline__ bool marked(const float* C, int64_t ldc, int M, int N, int m0, int n0) {
  constexpr int NM = BM / kMarkBlock, NB = NM * (BN / kMarkBlock);
  bool hit = false;
  for (int b = threadIdx.x % kWave; b < NB; b += kWave) {
    const int row = m0 + (b % NM) * kMarkBlock, col = n0 + (b / NM) * kMarkBlock;
    if (row < M && col < N) hit |= __float_as_uint(C[(int64_t)row * ldc + col]) == kMark;
  }
  return __any(hit);
}

// Per-start state machine shared by the iteration kernels.
constexpr int32_t kRunning = -1;

}  // namespace spca
