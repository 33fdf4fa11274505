// Launch of the wall-normal line solves.
#include "cf_internal.h"
#include "cf_ysolve_kernels.h"

namespace cf {

// Rows per partition compiled for both precisions, and the longer partitions
// compiled for FP32 only (in FP64 their rows no longer fit the registers).
#define CF_FOR_EACH_M(X) X(1) X(2) X(3) X(4) X(6) X(8) X(12) X(16)
#define CF_FOR_EACH_M_FP32(X) X(24) X(32)

bool ysolve_m_compiled(int m, bool fp64) {
  switch (m) {
#define CF_CASE(M) case M:
    CF_FOR_EACH_M(CF_CASE)
    return true;
    CF_FOR_EACH_M_FP32(CF_CASE)
    return !fp64;
#undef CF_CASE
    default:
      return false;
  }
}

// Default lines per block, from timings of every admissible partitioning of
// 512 x ny x 256 with 24 <= ny <= 768.  A row access of a block should be whole
// 128-byte lines, 8 FP64 or 16 FP32 values.
//   FP64: at most 256 threads (two blocks per CU at 192 VGPRs; 288 threads of 18
//     partitions are 20-30 % slower than 216), and of those the most lines in
//     multiples of 8 (9 x 16 rows: 59 us at 24 lines, 65 at 28, 69 at 16), or 12
//     lines where 16 do not fit (19 x 16 rows: 143 us at 12 lines, 165 at 8; at
//     13 lines, which 256 threads would take, 255).
//   FP32: 16 lines (25 x 12 rows: 104 us, 204 at 10; 13 x 24 rows: 167 us at 19),
//     32 where at most 8 partitions leave the block small, 8 above 32 partitions
//     (at most 512 threads), and 32 for 13 to 16 partitions of 24 rows, whose
//     instance is held to 128 VGPRs so that two blocks of 512 threads share a CU.
//     us at 16 / 32 lines on 512 x 24P x 256, 1024 x 24P x 512 and 1024 x 24P x
//     1024: P = 11 64 / 70, 243 / 250, 476 / 478; 12 73 / 77, 268 / 263, 527 / 505;
//     13 79 / 76, 285 / 273, 560 / 529; 14 84 / 84, 308 / 291, 561 / 537; 15 89 / 87,
//     327 / 297, 606 / 543; 16 95 / 91, 356 / 317, 648 / 577.  Other rows are slower
//     at 32 lines from P = 9 on (512 x 16P x 256: P = 9 33 / 41, 16 52 / 57; of 32
//     rows: 83 / 110, 123 / 151).
// At least one wave.
int ysolve_default_lb(int P, int M, bool fp64) {
  int lb;
  if (fp64) {
    lb = 256 / P;
    lb = lb >= 16 ? lb & ~7 : (lb >= 12 ? 12 : 8);
    if (lb > 48) lb = 48;
  } else {
    lb = P <= 8 || (M == 24 && P >= 13 && P <= 16) ? 32 : P <= 32 ? 16 : 8;
  }
  if (lb * P < 64) lb = (64 + P - 1) / P;
  return lb;
}

template <typename T, int M, int MODE, bool DROP>
static hipError_t ysolve_go(long blocks, const int* blist, const YArgs& ya, int threads, const cx<T>* fin,
                            cx<T>* pout, const T* a, const T* c, const T* kx2, const T* kz2, hipStream_t s,
                            const SpecialLines& sp = SpecialLines{}) {
  blocks += special_blocks(sp.n);
  if (blocks <= 0) return hipSuccess;
  const int nyp = ya.P * M;  // rows of the partitions (padded past ny)
  size_t lds = MODE == kSlabLocal ? sizeof(T) * 2 * (size_t)nyp : ysolve_lds_bytes<T>(nyp, ya.P, ya.LB, DROP);
  if (sp.n > 0 && lds < special_lds_bytes(ya.ny)) lds = special_lds_bytes(ya.ny);
  if constexpr (MODE == kWhole) {
    // the slab passes read their right-hand side twice: only the one-pass
    // solve streams it
    if ((long)ya.nlines * ya.ny * (long)sizeof(cx<T>) >= kStreamSolve<T>) {
      hipLaunchKernelGGL((k_ysolve<T, M, MODE, DROP, true>), dim3(blocks), dim3(threads), lds, s, fin, pout, a, c,
                         kx2, kz2, blist, ya, sp);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_ysolve<T, M, MODE, DROP, false>), dim3(blocks), dim3(threads), lds, s, fin, pout, a, c, kx2,
                     kz2, blist, ya, sp);
  return hipGetLastError();
}

template <typename T, int M>
static hipError_t ysolve_m(const YLaunch& y, const YArgs& ya, int threads, const cx<T>* fin, cx<T>* pout, const T* a,
                           const T* c, const T* kx2, const T* kz2, hipStream_t s) {
  const long all = (y.nlines + ya.LB - 1) / ya.LB;
  if (y.mode == kSlabLocal) return ysolve_go<T, M, kSlabLocal, false>(all, nullptr, ya, threads, fin, pout, a, c,
                                                                      kx2, kz2, s);
  // blocks whose lines all allow the drop take the dropped reduced system, the
  // others the exact one (two launches over the plan's block lists; without
  // lists every block is exact)
  const long ne = y.blocks_exact ? y.n_exact : all;
  hipError_t e;
  if (y.mode == kSlabFinish) {
    e = ysolve_go<T, M, kSlabFinish, false>(ne, y.blocks_exact, ya, threads, fin, pout, a, c, kx2, kz2, s);
    if (e == hipSuccess && y.blocks_drop)
      e = ysolve_go<T, M, kSlabFinish, true>(y.n_drop, y.blocks_drop, ya, threads, fin, pout, a, c, kx2, kz2, s);
  } else {
    // the special lines go with the first launch: the exact blocks, or the
    // dropped ones when every block drops
    const bool with_exact = ne > 0 || !y.blocks_drop;
    const SpecialLines none{};
    e = ysolve_go<T, M, kWhole, false>(ne, y.blocks_exact, ya, threads, fin, pout, a, c, kx2, kz2, s,
                                       with_exact ? y.special : none);
    if (e == hipSuccess && y.blocks_drop)
      e = ysolve_go<T, M, kWhole, true>(y.n_drop, y.blocks_drop, ya, threads, fin, pout, a, c, kx2, kz2, s,
                                        with_exact ? none : y.special);
  }
  return e;
}

template <typename T>
hipError_t launch_ysolve(YLaunch y, const cx<T>* fin, cx<T>* pout, const T* a, const T* c,
                         const T* kx2, const T* kz2, hipStream_t s) {
  YArgs ya;
  ya.ny = y.ny;
  ya.nz = y.nz;
  ya.nkx = y.nkx;
  ya.P = y.P;
  ya.LB = y.LB > 0 ? y.LB : ysolve_default_lb(y.P, y.M, std::is_same<T, double>::value);
  ya.nlines = y.nlines;
  ya.skip_kx = y.skip_kx;
  ya.skip_kz = y.skip_kz;
  ya.pa = y.mode == kWhole ? 0 : y.pa;
  ya.pb = y.mode == kWhole ? y.P : y.pb;
  ya.iface = y.iface;
  ya.G = y.G > 0 ? y.G : y.P;
  if (y.mode != kWhole && (ya.pa < 0 || ya.pb > y.P || ya.pa >= ya.pb || y.iface == nullptr))
    return hipErrorInvalidValue;
  if (y.P % ya.G != 0) return hipErrorInvalidValue;
  // A local-mode block holds the threads of its slab's partitions only and no
  // interface data, so it takes more lines (about 256 threads) and only the
  // coefficient rows in LDS.
  if (y.mode == kSlabLocal) {
    const int np = ya.pb - ya.pa;
    while (2 * ya.LB * np <= 256) ya.LB *= 2;
  }
  const int threads = ya.LB * (y.mode == kSlabLocal ? ya.pb - ya.pa : y.P);
  // A special line needs a whole wave; beside smaller blocks the lines get a
  // launch of their own (the order does not matter: the other blocks discard
  // what they read of these lines).
  if (threads < 64 && y.special.n > 0) {
    const hipError_t e = launch_special_lines<T>(fin, pout, y.special, y.ny, y.nz, s);
    if (e != hipSuccess) return e;
    y.special = SpecialLines{};
  }
  switch (y.M) {
#define CF_CASE(M) \
  case M:          \
    return ysolve_m<T, M>(y, ya, threads, fin, pout, a, c, kx2, kz2, s);
    CF_FOR_EACH_M(CF_CASE)
#undef CF_CASE
    default:
      break;
  }
  if constexpr (std::is_same<T, float>::value) {
    switch (y.M) {
#define CF_CASE(M) \
  case M:          \
    return ysolve_m<T, M>(y, ya, threads, fin, pout, a, c, kx2, kz2, s);
      CF_FOR_EACH_M_FP32(CF_CASE)
#undef CF_CASE
      default:
        break;
    }
  }
  return hipErrorInvalidValue;
}

// Dynamic LDS needed by a y-solve launch over P partitions of nyp / P rows
// (checked by the plan against the device limit).
size_t ysolve_lds_needed(int nyp, int P, int LB, bool fp64) {
  return fp64 ? ysolve_lds_bytes<double>(nyp, P, LB, true) : ysolve_lds_bytes<float>(nyp, P, LB, true);
}

template <typename T>
hipError_t launch_special_lines(const cx<T>* fin, cx<T>* pout, const SpecialLines& sp, int ny, int nz, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_special_lines<T>), dim3(sp.n), dim3(256), special_lds_bytes(ny), s, fin, pout, sp, ny, nz);
  return hipGetLastError();
}

#define CF_INST(T)                                                                                  \
  template hipError_t launch_ysolve<T>(YLaunch, const cx<T>*, cx<T>*, const T*, const T*,   \
                                       const T*, const T*, hipStream_t);                           \
  template hipError_t launch_special_lines<T>(const cx<T>*, cx<T>*, const SpecialLines&, int, int, hipStream_t);
CF_INST(double)
CF_INST(float)
#undef CF_INST

}  // namespace cf
