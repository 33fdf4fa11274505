// Both stages of the RK2 (Heun) momentum update in one marching pass.
//
// ub = u + dt R(u) and u2 = (u + ub)/2 + dt/2 R(ub) are computed plane by
// plane: while a block marches up its y-chunk, stage 1 runs one plane ahead
// of stage 2 on the tile grown by one cell in x and z (the cells stage 2's
// stencil reads), and ub lives only in LDS.  The pass reads u, v, w once and
// writes u2 once, instead of the two passes of the split stages (read u, write
// ub; read ub and u, write u2).  The stencil arithmetic is the same function as
// in the split stages.
//
// Both stages use the edge products carried up from the plane below and the
// plane-below values of the thread's own column from registers, so the input
// ring keeps two planes (j, j+1).  Stage 2 runs two planes behind stage 1 (the
// ub ring keeps three planes), so within one barrier interval the two stages
// are independent and their LDS reads and arithmetic interleave: neither has a
// branch (the row factors hold the walls, see YRow).  A chunk starts four
// iterations early with nothing in the carries: each iteration makes the next
// one's valid, and the first results stored are those of its first plane.
#pragma once

#include "cf_step_kernels.h"

namespace cf {

// Two-plane LDS ring (planes j and j+1, row stride SXX) with the thread's own
// column at plane j-1 held in registers.  Off-column values of plane j-1 are
// never requested: the stencil is always called with its lower-face products
// carried.
template <typename T, int SXX>
struct Ring2Acc {
  const T* su;
  const T* sv;
  const T* sw;
  int s0, sp;  // slot offsets of planes j and j+1
  int base;    // this point within a slot
  T um, vm, wm;
  __device__ __forceinline__ int off(int dj, int dk, int di) const { return (dj > 0 ? sp : s0) + base + dk * SXX + di; }
  __device__ __forceinline__ T u(int dj, int dk, int di) const { return dj < 0 ? um : su[off(dj, dk, di)]; }
  __device__ __forceinline__ T v(int dj, int dk, int di) const { return dj < 0 ? vm : sv[off(dj, dk, di)]; }
  __device__ __forceinline__ T w(int dj, int dk, int di) const { return dj < 0 ? wm : sw[off(dj, dk, di)]; }
};

// Per-column marching state of one stencil point: the values of the plane
// below and the edge products at the lower face of the current plane.
template <typename T>
struct ColState {
  T um, vm, wm;
  FaceFlux<T> c;
};

// Stage 1 at plane j for one point of the grown tile: reads u at planes j and
// j+1 from the ring (slot offsets s0, sp; point offset ubase), writes ub of
// plane j into the ub ring at boff (zero outside 0 <= j < ny, v zero on the
// top wall) and advances the column state.
template <typename T, int UX>
__device__ __forceinline__ void rk_stage1_point(const T* su, const T* sv, const T* sw, T* bu, T* bv, T* bw, int s0,
                                                int sp, int ubase, int boff, ColState<T>& st, const Geo<T>& g,
                                                const YRow<T>& Y, int j, T dt, T nu, T fx) {
  const Ring2Acc<T, UX> A{su, sv, sw, s0, sp, ubase, st.um, st.vm, st.wm};
  const T uc = A.u(0, 0, 0), vc = A.v(0, 0, 0), wc = A.w(0, 0, 0);
  FaceFlux<T> up;
  const RhsOut<T> r = momentum_rhs<T>(A, g, Y, nu, fx, st.c, up);
  const bool in = j >= 0 && j < g.ny;
  const T ou = uc + dt * r.ru, ov = vc + dt * r.rv, ow = wc + dt * r.rw;
  st.c = up;
  st.um = uc;
  st.vm = vc;
  st.wm = wc;
  bu[boff] = in ? ou : T(0);
  bv[boff] = in && j != g.ny - 1 ? ov : T(0);
  bw[boff] = in ? ow : T(0);
}

// Most planes of one y-chunk.
constexpr int kRkfMaxChunk = 128;

template <int TX, int TZ>
struct RkFusedTile {
  static constexpr int TH = TX * TZ;
  static constexpr int EX = TX + 2, EZ = TZ + 2, EPL = EX * EZ;  // grown tile (stage 1)
  static constexpr int UX = TX + 4, UZ = TZ + 4, UPL = UX * UZ;  // input tile
  static constexpr int NRING = 2 * EX + 2 * TZ;                  // grown-tile cells outside the block's own
  static constexpr int PER = (UPL + TH - 1) / TH;                // input values per thread per plane
};

// At least four waves per SIMD in FP64 (128 VGPRs, five spilled) and six in FP32
// (three blocks per CU).  The row factors in scalar registers, the walls without
// branches and the folded averages took the FP64 pass from 357 to 281 VALU and 57
// to 39 LDS instructions per wave and plane and from 2.18 to 1.88 ms on
// 1024x256x512 (6.44 GB, 3.4 TB/s), and FP32 from 3.78 to 3.07 ms on
// 1024x384x1024.  VALU issue takes 0.61 of the cycles and LDS 0.48, at a 2.0 GHz
// clock; the three waves with outer cells finish last.  Outer cells first, or
// with a raised priority, are 2-4 % slower.
// The tile index is remapped (xcd_slab_block over the whole grid) so that each
// XCD walks one contiguous run of tiles and neighbouring tiles share the halo
// lines in one L2 (runs within each y-chunk instead: within 1.5 %, either way).
// NT: the outputs, written once, are streamed (non-temporal) for large fields
// (the FP64 pass on 1024x256x512: about 2 % faster).
// cy: planes of a block's chunk, at most kRkfMaxChunk (see chunk_planes).
template <typename T, int TX, int TZ, bool NT>
__global__ void __launch_bounds__(TX * TZ, sizeof(T) == 8 ? 4 : 6)
k_rk2_fused(const T* __restrict__ u, const T* __restrict__ v, const T* __restrict__ w, T* uo, T* vo, T* wo,
            Geo<T> g, T dt, T nu, T fx, int cy) {
  using Tl = RkFusedTile<TX, TZ>;
  constexpr int TH = Tl::TH, EX = Tl::EX, EPL = Tl::EPL, UX = Tl::UX, UPL = Tl::UPL, PER = Tl::PER;
  static_assert(Tl::NRING <= TH, "the grown tile's outer cells must fit one pass of the block");
  __shared__ T su[2 * UPL], sv[2 * UPL], sw[2 * UPL];
  __shared__ T bu[3 * EPL], bv[3 * EPL], bw[3 * EPL];
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int ntx = (nx + TX - 1) / TX, ntz = (nz + TZ - 1) / TZ;
  int b = xcd_slab_block(blockIdx.x, gridDim.x);
  const int bx = b % ntx;
  b /= ntx;
  const int bz = b % ntz;
  const int by = b / ntz;
  const int i0 = bx * TX, k0 = bz * TZ;
  const int j0 = by * cy, j1 = (j0 + cy < ny) ? j0 + cy : ny;
  const int t = threadIdx.x;
  const int tx = t % TX, tz = t / TX;
  const int i = i0 + tx, k = k0 + tz;
  const bool mine = (i < nx) && (k < nz);
  const long plane = (long)nx * nz;
  // input tile: two-cell halo, periodic wrap
  int toff[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = t + q * TH;
    const int zz = idx / UX, xx = idx % UX;
    int gi = (i0 + xx - 2) % nx;
    if (gi < 0) gi += nx;
    int gk = (k0 + zz - 2) % nz;
    if (gk < 0) gk += nz;
    toff[q] = (idx < UPL) ? gk * nx + gi : -1;
  }
  T ru[PER], rv[PER], rw[PER];
#define CF_RKF_FETCH(jj)                                         \
  _Pragma("unroll") for (int q = 0; q < PER; ++q) {             \
    ru[q] = rv[q] = rw[q] = T(0);                               \
    if (toff[q] >= 0 && (jj) >= 0 && (jj) < ny) {               \
      const long o = (long)(jj) * plane + toff[q];              \
      ru[q] = u[o];                                             \
      rw[q] = w[o];                                             \
      if ((jj) < ny - 1) rv[q] = v[o];                          \
    }                                                           \
  }
#define CF_RKF_STORE(jj)                                         \
  _Pragma("unroll") for (int q = 0; q < PER; ++q) {             \
    if (toff[q] >= 0) {                                         \
      const int idx = ((jj) & 1) * UPL + t + q * TH;            \
      su[idx] = ru[q];                                          \
      sv[idx] = rv[q];                                          \
      sw[idx] = rw[q];                                          \
    }                                                           \
  }
  // point A: the block's own cell (tx, tz); point B (t < NRING): one cell of
  // the grown tile's outer ring
  const int ubA = (tz + 2) * UX + tx + 2, eA = (tz + 1) * EX + tx + 1;
  const bool hasB = t < Tl::NRING;
  int exB, ezB;
  if (t < EX) {
    exB = t, ezB = 0;
  } else if (t < 2 * EX) {
    exB = t - EX, ezB = Tl::EZ - 1;
  } else if (t < 2 * EX + TZ) {
    exB = 0, ezB = 1 + t - 2 * EX;
  } else {
    exB = EX - 1, ezB = 1 + (t - 2 * EX - TZ) % TZ;
  }
  const int ubB = (ezB + 1) * UX + exB + 1, eB = ezB * EX + exB;
#define CF_US(jj) (((jj) & 1) * UPL)
#define CF_BS(jj) ((((jj) + 6) % 3) * EPL)

  ColState<T> sA{}, sB{}, s2{};
  CF_RKF_FETCH(j0 - 2)
  CF_RKF_STORE(j0 - 2)
  CF_RKF_FETCH(j0 - 1)
  const T hh = T(0.5), hd = T(0.5) * dt;
  // iteration s: stage 1 at plane s+1 and stage 2 at plane s-1, independent of
  // each other within the barrier interval (three ub planes in LDS).  Valid from
  // s = j0-3 on: the carries of stage 1; from j0-2: ub of plane j0-1; from j0:
  // the carries of stage 2; from j0+1: the results
  T p0u = T(0), p0v = T(0), p0w = T(0);
  for (int s = j0 - 3; s <= j1; ++s) {
    CF_RKF_STORE(s + 2)
    __syncthreads();
    CF_RKF_FETCH(s + 3)
    const YRow<T> Y1 = load_row(g.rows, s + 1), Y2 = load_row(g.rows, s - 1);
    const T c0u = sA.um, c0v = sA.vm, c0w = sA.wm;  // u, v, w of this cell at plane s
    rk_stage1_point<T, UX>(su, sv, sw, bu, bv, bw, CF_US(s + 1), CF_US(s + 2), ubA, CF_BS(s + 1) + eA, sA, g, Y1,
                           s + 1, dt, nu, fx);
    {
      const int q = s - 1;
      const Ring2Acc<T, EX> B{bu, bv, bw, CF_BS(q), CF_BS(q + 1), eA, s2.um, s2.vm, s2.wm};
      const T uc = B.u(0, 0, 0), vc = B.v(0, 0, 0), wc = B.w(0, 0, 0);
      FaceFlux<T> up;
      const RhsOut<T> r = momentum_rhs<T>(B, g, Y2, nu, fx, s2.c, up);
      s2.c = up;
      s2.um = uc;
      s2.vm = vc;
      s2.wm = wc;
      if (mine && s > j0) {
        const long id = (long)q * plane + (long)k * nx + i;
        st_once<NT>(hh * (p0u + uc) + hd * r.ru, &uo[id]);
        st_once<NT>((q == ny - 1) ? T(0) : hh * (p0v + vc) + hd * r.rv, &vo[id]);
        st_once<NT>(hh * (p0w + wc) + hd * r.rw, &wo[id]);
      }
    }
    if (hasB && s < j1)
      rk_stage1_point<T, UX>(su, sv, sw, bu, bv, bw, CF_US(s + 1), CF_US(s + 2), ubB, CF_BS(s + 1) + eB, sB, g, Y1,
                             s + 1, dt, nu, fx);
    p0u = c0u;
    p0v = c0v;
    p0w = c0w;
    __syncthreads();
  }
#undef CF_RKF_FETCH
#undef CF_RKF_STORE
#undef CF_US
#undef CF_BS
}

}  // namespace cf
