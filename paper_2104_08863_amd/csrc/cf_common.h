// Shared device/host helpers for the chanflow HIP kernels: a plain complex
// type and the handful of operations the transforms and solves need.
//
// Everything here is usable from host code as well, so the per-thread math of
// the kernels can be exercised on the CPU.
#pragma once

#include <cstddef>
#include <cstdint>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define CF_HD __host__ __device__ __forceinline__
#else
#define CF_HD inline
#endif

namespace cf {

template <typename T>
struct alignas(2 * sizeof(T)) cx {
  T re, im;
};

template <typename T> CF_HD cx<T> mk(T r, T i) { cx<T> z; z.re = r; z.im = i; return z; }
template <typename T> CF_HD cx<T> operator+(cx<T> a, cx<T> b) { return mk(a.re + b.re, a.im + b.im); }
template <typename T> CF_HD cx<T> operator-(cx<T> a, cx<T> b) { return mk(a.re - b.re, a.im - b.im); }
template <typename T> CF_HD cx<T> operator*(cx<T> a, T s) { return mk(a.re * s, a.im * s); }
template <typename T> CF_HD cx<T> cmul(cx<T> a, cx<T> b) {
  return mk(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
// a * conj(b)
template <typename T> CF_HD cx<T> cmulc(cx<T> a, cx<T> b) {
  return mk(a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im);
}
template <typename T> CF_HD cx<T> conj(cx<T> a) { return mk(a.re, -a.im); }
// multiply by -i (forward sign) or +i (inverse sign)
template <bool INV, typename T> CF_HD cx<T> mul_mi(cx<T> a) {
  return INV ? mk(-a.im, a.re) : mk(a.im, -a.re);
}

// Reciprocal: on the device the hardware estimate refined by Newton steps
// (error about one ulp, no IEEE division sequence); on the host 1/x.
CF_HD double rcp(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
#else
  return 1.0 / x;
#endif
}
CF_HD float rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  float r = __builtin_amdgcn_rcpf(x);
  float e = __builtin_fmaf(-x, r, 1.0f);
  return __builtin_fmaf(r, e, r);
#else
  return 1.0f / x;
#endif
}

template <typename T> CF_HD T cf_max(T a, T b) { return a > b ? a : b; }
template <typename T> CF_HD T cf_min(T a, T b) { return a < b ? a : b; }

// A load and a store of a value that a kernel touches once: non-temporal when
// NT (streamed past the caches; the launches choose it for fields larger than
// the XCDs' L2s together), plain otherwise.
#if defined(__HIPCC__)
template <bool NT, typename T>
__device__ __forceinline__ T ld_once(const T* a) {
  if constexpr (NT) return __builtin_nontemporal_load(a);
  else return *a;
}
template <bool NT, typename T>
__device__ __forceinline__ void st_once(T v, T* a) {
  if constexpr (NT) __builtin_nontemporal_store(v, a);
  else *a = v;
}
template <bool NT, typename T>
__device__ __forceinline__ cx<T> ld_once(const cx<T>* a) {
  if constexpr (NT) {
    const T* p = reinterpret_cast<const T*>(a);
    return mk(__builtin_nontemporal_load(p), __builtin_nontemporal_load(p + 1));
  } else {
    return *a;
  }
}
template <bool NT, typename T>
__device__ __forceinline__ void st_once(cx<T> v, cx<T>* a) {
  if constexpr (NT) {
    T* p = reinterpret_cast<T*>(a);
    __builtin_nontemporal_store(v.re, p);
    __builtin_nontemporal_store(v.im, p + 1);
  } else {
    *a = v;
  }
}

// Orders the LDS accesses of a line's threads (TPL consecutive threads, a power
// of two).  A line that lies within one wave needs no barrier: a wave's LDS
// accesses execute in order, and only the compiler has to keep them so.  (Block
// barriers held all waves of a block to the slowest at every exchange.)
template <int TPL>
__device__ __forceinline__ void line_sync() {
  if constexpr (TPL <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}
#endif
// Data size from which the stencils and corrections take non-temporal loads and
// stores for the arrays they touch once: the 8 XCDs' L2s together (32 MiB).
// Smaller arrays stay cached for the next kernel (streamed, the 64^3 time loop
// was 2-4 % slower).
constexpr long kStreamBytes = 32L << 20;
// The spectrum sizes from which the z transforms and the one-pass wall-normal
// solve stream.  What they store without it is partly still in the 256 MB cache
// behind the L2s when the next kernel of the solve reads it: FP64 Poisson solve,
// both cached against both streamed, 64 MiB 148 -> 131 us, 109 MiB 232 -> 212, 128
// MiB 263 -> 246.  Beyond that two cached neighbours push each other out (193 MiB,
// the solve cached and the z transforms streamed 949 us, both cached 1031, both
// streamed 998).
constexpr long kStreamZ = 160L << 20;
// The wall-normal solve beside streamed z transforms, whole Poisson solve in us,
// its arrays cached / streamed:
//   FP64  257 MiB 473 / 490, 514 MiB 953 / 964, 770 MiB 1484 / 1492, 1.0 GiB 1943 /
//         1947, 1.25 GiB 2603 / 2624, 1.5 GiB 3058 / 3080, 2 GiB 4016 / 4025 (within
//         a step 11000 / 10984), 3 GiB 6369 / 6334, 4 GiB 8108 / 8078, 8 GiB 17031 /
//         16927
//   FP32  256 MiB 1308 / 1363, 513 MiB 2674 / 2703, 770 MiB 4058 / 4070, 1.0 GiB
//         5515 / 5507, 1.25 GiB 7096 / 7035, 1.5 GiB 8377 / 8272, 4 GiB 23105 / 22897
// The kernel alone gains earlier (FP64 1.0 GiB, in a step: 399 / 387 us) what the
// kernels next to it lose (the step: 5471 / 5467).
template <typename T>
constexpr long kStreamSolve = (sizeof(T) == 8 ? 2048L : 1024L) << 20;

// Compute units of the chip (8 XCDs of 32).
constexpr int kCus = 256;

// Work order for the 8 XCDs, each with its own L2.  The hardware deals
// blocks round-robin (block b to XCD b mod 8); for a grid made of groups of n
// consecutive work items (n a multiple of 8), block b is given the item that
// puts XCD x on the contiguous run [x n/8, (x+1) n/8) of every group, so items
// beside each other, which read each other's edge cells, do so from one L2.
// With n the whole grid each XCD gets one run.  A permutation of the grid
// either way (identity when n is not a multiple of 8).
CF_HD int xcd_slab_block(int b, int n) {
  if (n & 7) return b;
  const int x = b & 7, s = b >> 3, per = n >> 3;
  return (s / per) * n + x * per + s % per;
}

// Modes of the partitioned solve.  kWhole: every partition of a line in one
// block.  The two slab modes split the same computation at the point where a
// partition needs data from the others (the paper's exchange across
// processes): kSlabLocal runs the local solves of the partitions [pa, pb) and
// writes their interface rows; kSlabFinish reads every partition's interface
// rows, solves the reduced system, redoes the local solves of [pa, pb) and
// writes their corrected rows.
enum YMode { kWhole = 0, kSlabLocal = 1, kSlabFinish = 2 };

}  // namespace cf
