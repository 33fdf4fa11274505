// Launch of the adjoint (transpose) kernels of the projection step.
#include "cf_adjoint_kernels.h"
#include "cf_internal.h"

namespace cf {

// Tile of the transposed stencil (six LDS fields x two planes), chunks of at
// most 32 planes.  Both launches of an adjoint step on 1024x256x512 in FP64: 64 x
// 4 columns 5.32 ms, 128 x 4 5.52, 32 x 8 5.45 (three planes in LDS and branches
// for the walls, as before: 5.78), 64 x 8, 32 x 16 and 16 x 16 5.8-6.0; capped at
// 128 VGPRs for a fourth block per CU they spill and take 6.5-6.8.  FP32 on
// 1024x384x1024: 128 x 4 columns 8.03 ms, 64 x 8 8.37 (8.99 before), 256 x 4 8.18,
// 256 x 2 11.7.
template <typename T>
struct AdjTile {
  static constexpr int TX = 64, TZ = 4, BPC = 3;
};
template <>
struct AdjTile<float> {
  static constexpr int TX = 128, TZ = 4, BPC = 2;
};

template <typename T>
hipError_t launch_rhs_adjoint(const T* u, const T* v, const T* w, const T* au, const T* av, const T* aw,
                              const T* bu, const T* bv, const T* bw, T c1, T c2, const AdjGeo<T>& g, T nu, T s,
                              int add, T* gu, T* gv, T* gw, hipStream_t st) {
  constexpr int ADJ_TX = AdjTile<T>::TX, ADJ_TZ = AdjTile<T>::TZ;
  AdjPtrs P{u, v, w, au, av, aw, bu, bv, bw, gu, gv, gw};
  const long cols = (long)((g.g.nx + ADJ_TX - 1) / ADJ_TX) * ((g.g.nz + ADJ_TZ - 1) / ADJ_TZ);
  const int cy = chunk_planes(cols, g.g.ny, AdjTile<T>::BPC * kCus, kMaxChunk, 2);
  const long blocks = cols * ((g.g.ny + cy - 1) / cy);
  const dim3 grid(blocks), block(ADJ_TX * ADJ_TZ);
  const bool nt = (long)g.g.nx * g.g.ny * g.g.nz * (long)sizeof(T) >= kStreamBytes;
#define CF_ADJ_GO(HASB, ADD)                                                                                     \
  if (nt)                                                                                                        \
    hipLaunchKernelGGL((k_rhs_adjoint<T, ADJ_TX, ADJ_TZ, HASB, ADD, true>), grid, block, 0, st, P, c1, c2, g, nu, \
                       s, cy);                                                                                \
  else                                                                                                           \
    hipLaunchKernelGGL((k_rhs_adjoint<T, ADJ_TX, ADJ_TZ, HASB, ADD, false>), grid, block, 0, st, P, c1, c2, g, nu, \
                       s, cy)
  if (bu != nullptr && add) {
    CF_ADJ_GO(true, true);
  } else if (bu != nullptr) {
    CF_ADJ_GO(true, false);
  } else if (add) {
    CF_ADJ_GO(false, true);
  } else {
    CF_ADJ_GO(false, false);
  }
#undef CF_ADJ_GO
  return hipGetLastError();
}

template <typename T>
hipError_t launch_correct_w(const T* gu, const T* gv, const T* gw, T* ou, T* ov, T* ow, const double* phi,
                            const AdjGeo<T>& g, hipStream_t st) {
  const long n = (long)g.g.nx * g.g.ny * g.g.nz;
  const int th = correction_threads(g.g.nx);
  const dim3 blocks((g.g.nx / 2 * g.g.nz + th - 1) / th, g.g.ny);
  if (n * (long)sizeof(T) >= kStreamBytes)
    hipLaunchKernelGGL((k_correct_w<T, true>), blocks, dim3(th), 0, st, gu, gv, gw, ou, ov, ow, phi, g);
  else
    hipLaunchKernelGGL((k_correct_w<T, false>), blocks, dim3(th), 0, st, gu, gv, gw, ou, ov, ow, phi, g);
  return hipGetLastError();
}

#define CF_INST(T)                                                                                         \
  template hipError_t launch_rhs_adjoint<T>(const T*, const T*, const T*, const T*, const T*, const T*,    \
                                            const T*, const T*, const T*, T, T, const AdjGeo<T>&, T, T, int, \
                                            T*, T*, T*, hipStream_t);                                      \
  template hipError_t launch_correct_w<T>(const T*, const T*, const T*, T*, T*, T*, const double*,         \
                                          const AdjGeo<T>&, hipStream_t);
CF_INST(double)
CF_INST(float)
#undef CF_INST

}  // namespace cf
