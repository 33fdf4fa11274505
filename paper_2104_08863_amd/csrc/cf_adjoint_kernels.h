// Transposes for the adjoint of the projection step (Euclidean gradients).
//
// Momentum RHS.  R(u) = -N(u) + nu lap(u) + fx e_x with the flux-form
// N(u) = [Dx(uc^2) + Dy(Exy) + Dz(Exz), Dx(Exy) + Dyc(vc^2) + Dz(Eyz),
//         Dx(Exz) + Dy(Eyz) + Dz(wc^2)] built from
//   uc = (u_i + u_{i-1})/2,  vc = (v_j + v_{j-1})/2,  wc = (w_k + w_{k-1})/2,
//   Exy = Iy(u) Ax(v),  Exz = Az(u) Ax(w),  Eyz = Iy(w) Az(v),
//   Iy(q)_j = q_j wl_j + q_{j+1} wu_j (face j+1),  Ax(q)_i = (q_i + q_{i+1})/2,
//   Az(q)_k = (q_k + q_{k+1})/2.
// Its Jacobian transpose applied to an adjoint field lam is gathered at every
// velocity point: each edge product E contributes mu * dE/du, where mu is the
// transpose of the two differences that consume E (for Exy: Dy^T lam_u +
// Dx^T lam_v), and each centre square c^2 contributes 2 c (D^T lam).  The
// Laplacian is self-adjoint in the face-volume inner product, so its transpose
// is the same flux stencil applied to lam / W with the outer 1/W dropped
// (W = dy_j for u, w and dyc_j for v).  v on the top wall is not a variable.
//
// Projection.  P = I - G L^+ D is self-adjoint in the face-volume inner
// product, so P^T g = g - W G L^+ D (g / W): the forward solve applied to
// g / W (k_divergence-style source with row weights, SrcDivW) and a weighted
// correction (k_correct_w).
#pragma once

#include "cf_common.h"
#include "cf_step_kernels.h"

namespace cf {

template <typename T>
struct AdjGeo {
  Geo<T> g;
  const T* dy;    // dy_j
  T rdxh, rdzh;   // rdx / 2, rdz / 2
  const T* rows;  // AdjRow rows of planes -kRowPad .. ny + kRowPad - 1; points at plane 0
};

// The wall-normal factors of the transposed stencil at plane j, zero outside
// [0, ny) except what plane -1 needs to give the bottom wall's carries (rdyp,
// fc and rcp).  The weights carry the 1/2 of the velocity averages and are zero
// on the walls; fc holds 2/dy on the wall faces (see YRow): no case for the
// walls is left in the stencil.
template <typename T>
struct AdjRow {
  T rdy, rdyp;    // 1/dy_j, 1/dy_{j+1}
  T wl, wu, wum;  // half the weights at face j+1, and of the upper cell at face j
  T fc;           // 1/dyc at the upper face, 2/dy on a wall
  T rc, rcp;      // 1/dyc at faces j+1 and j+2, 0 on the walls
};

// The row by a scalar load (see load_row).
template <typename T>
__device__ __forceinline__ AdjRow<T> load_adj_row(const T* rows, int j) {
  using CP = const __attribute__((address_space(4))) T*;
  const CP p = (CP)(uintptr_t)(rows + (long)j * 8);
  return AdjRow<T>{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]};
}

// J_R(u)^T lam at point (i, j, k) from an accessor with relative offsets in
// planes j and j+1: A.U(dj, dk, di) etc. for the state and A.LU(...) for lam; A
// returns 0 outside [0, ny) and for v / lam_v on the top wall.  gv is
// meaningless on the top wall's plane.
template <typename T>
struct AdjOut {
  T gu, gv, gw;
};

// Lower-face terms of plane j that equal upper-face terms of plane j-1: twice
// the x-y and y-z edge factors mu A(v) at face j, twice the centre term vc xi_y
// at centre j, and the viscous fluxes of lam_u / W, lam_w / W and lam_v / W
// through the cell's lower side.
template <typename T>
struct AdjCarry {
  T exy, eyz, cy, fu, fw, fv;
};

template <typename T, class Acc>
__device__ __forceinline__ AdjOut<T> rhs_adjoint_point(const Acc& A, const AdjGeo<T>& G, const AdjRow<T>& Y, T nu,
                                                       AdjCarry<T>& c) {
  const Geo<T>& g = G.g;
  const T rdx = g.rdx, rdz = g.rdz;
  AdjOut<T> o;
  const T U0 = A.U(0, 0, 0), V0 = A.V(0, 0, 0), W0 = A.W(0, 0, 0);
  const T lu0 = A.LU(0, 0, 0), lv0 = A.LV(0, 0, 0), lw0 = A.LW(0, 0, 0);
  const T luip = A.LU(0, 0, 1), luim = A.LU(0, 0, -1), lukp = A.LU(0, 1, 0), lukm = A.LU(0, -1, 0);
  const T lwip = A.LW(0, 0, 1), lwim = A.LW(0, 0, -1), lwkp = A.LW(0, 1, 0), lwkm = A.LW(0, -1, 0);
  const T lvip = A.LV(0, 0, 1), lvim = A.LV(0, 0, -1), lvkp = A.LV(0, 1, 0), lvkm = A.LV(0, -1, 0);
  const T lu1 = A.LU(1, 0, 0), lw1 = A.LW(1, 0, 0), lv1 = A.LV(1, 0, 0);
  const T Uim = A.U(0, 0, -1), Wkm = A.W(0, -1, 0);
  // the transposed differences mu that consume the edge products, each used by
  // the two velocities of its product
  const T qu0 = lu0 * Y.rdy, qu1 = lu1 * Y.rdyp, qw0 = lw0 * Y.rdy, qw1 = lw1 * Y.rdyp;
  const T muxy = (qu0 - qu1) + (lv0 - lvip) * rdx;
  const T muyz = (qw0 - qw1) + (lv0 - lvkp) * rdz;
  const T muxz = (lu0 - lukp) * rdz + (lw0 - lwip) * rdx;
  const T exy = muxy * (V0 + A.V(0, 0, 1)), eyz = muyz * (V0 + A.V(0, 1, 0));
  {
    // u point (i+1/2, j, k)
    const T mk1 = (lukm - lu0) * rdz + (lwkm - A.LW(0, -1, 1)) * rdx;
    const T s = (U0 + Uim) * (luim - lu0) + (A.U(0, 0, 1) + U0) * (lu0 - luip);
    const T t = muxz * (W0 + A.W(0, 0, 1)) + mk1 * (Wkm + A.W(0, -1, 1));
    const T acc = s * G.rdxh + t * T(0.25) + exy * Y.wl + c.exy * Y.wum;
    const T fu = (qu1 - qu0) * Y.fc;
    const T lap = (luip - T(2) * lu0 + luim) * g.rdx2 + (lukp - T(2) * lu0 + lukm) * g.rdz2 + (fu - c.fu);
    o.gu = nu * lap - acc;
    c.fu = fu;
  }
  {
    // w point (i, j, k+1/2)
    const T m1 = (luim - A.LU(0, 1, -1)) * rdz + (lwim - lw0) * rdx;
    const T s = (W0 + Wkm) * (lwkm - lw0) + (A.W(0, 1, 0) + W0) * (lw0 - lwkp);
    const T t = muxz * (U0 + A.U(0, 1, 0)) + m1 * (Uim + A.U(0, 1, -1));
    const T acc = s * G.rdzh + t * T(0.25) + eyz * Y.wl + c.eyz * Y.wum;
    const T fw = (qw1 - qw0) * Y.fc;
    const T lap = (lwip - T(2) * lw0 + lwim) * g.rdx2 + (lwkp - T(2) * lw0 + lwkm) * g.rdz2 + (fw - c.fw);
    o.gw = nu * lap - acc;
    c.fw = fw;
  }
  {
    // v point (i, face j+1, k)
    const T q0 = lv0 * Y.rc, q1 = lv1 * Y.rcp;
    const T cy = (A.V(1, 0, 0) + V0) * (q0 - q1);
    const T m1 = luim * Y.rdy - A.LU(1, 0, -1) * Y.rdyp + (lvim - lv0) * rdx;
    const T m2 = lwkm * Y.rdy - A.LW(1, -1, 0) * Y.rdyp + (lvkm - lv0) * rdz;
    const T s = muxy * (U0 * Y.wl + A.U(1, 0, 0) * Y.wu) + m1 * (Uim * Y.wl + A.U(1, 0, -1) * Y.wu);
    const T t = muyz * (W0 * Y.wl + A.W(1, 0, 0) * Y.wu) + m2 * (Wkm * Y.wl + A.W(1, -1, 0) * Y.wu);
    const T acc = (c.cy + cy) * T(0.5) + s + t;
    const T fv = (q1 - q0) * Y.rdyp;
    const T lap = (lvip - T(2) * lv0 + lvim) * g.rdx2 + (lvkp - T(2) * lv0 + lvkm) * g.rdz2 + (fv - c.fv);
    o.gv = nu * lap - acc;
    c.cy = cy;
    c.fv = fv;
  }
  c.exy = exy;
  c.eyz = eyz;
  return o;
}

// LDS accessor: six fields (u, v, w, lam_u, lam_v, lam_w), two plane slots each.
template <typename T, int TX, int TZ>
struct AdjLdsAcc {
  const T* s;  // 6 fields x 2 slots x PLANE
  int s0, sp;  // slot offsets (in elements) of planes j and j+1 within a field
  int base;
  static constexpr int SX = TX + 2, PLANE = (TX + 2) * (TZ + 2);
  __device__ __forceinline__ int off(int f, int dj, int dk, int di) const {
    return f * 2 * PLANE + (dj > 0 ? sp : s0) + base + dk * SX + di;
  }
  __device__ __forceinline__ T U(int dj, int dk, int di) const { return s[off(0, dj, dk, di)]; }
  __device__ __forceinline__ T V(int dj, int dk, int di) const { return s[off(1, dj, dk, di)]; }
  __device__ __forceinline__ T W(int dj, int dk, int di) const { return s[off(2, dj, dk, di)]; }
  __device__ __forceinline__ T LU(int dj, int dk, int di) const { return s[off(3, dj, dk, di)]; }
  __device__ __forceinline__ T LV(int dj, int dk, int di) const { return s[off(4, dj, dk, di)]; }
  __device__ __forceinline__ T LW(int dj, int dk, int di) const { return s[off(5, dj, dk, di)]; }
};

struct AdjPtrs {
  const void *u, *v, *w, *au, *av, *aw, *bu, *bv, *bw;
  void *gu, *gv, *gw;
};

// out = s * J_R(state)^T lam (+ A + B when ADD), lam = c1 A (+ c2 B when HASB).
// 2.5D tiling as in k_rk_stage: a TX x TZ column tile marches over cy planes
// keeping planes j and j+1 of the six fields in LDS (what a plane needs of the
// one below it is carried in registers, see AdjCarry), the raw values of plane
// j+2 fetched into registers while plane j is computed.  lam is formed only when a
// plane moves from registers to LDS, and every global load is unconditional
// (clamped address, masked on the move), so the compiler's waits never cover
// a load still in flight for a later plane.  Each thread fetches its own cell
// first (a wave reads aligned x runs), so the A + B term of the ADD output is
// taken from that fetch (two planes kept in registers) instead of a second
// load.  Each XCD takes a contiguous run of every y-chunk's tiles
// (xcd_slab_block; one run over the whole grid is as fast in FP32 and 12 %
// slower in FP64).  Bound by its reads: the tiles' halos come to about 1.5 times
// the fields (FP32 on 2048x768x2048 1.6 and 1.9), mostly from beyond the L2; VALU and
// LDS are each busy 0.4 of the time in FP64.
// NT: outputs, written once, stored non-temporally for large fields (the
// two launches of an FP32 adjoint step on 2048x768x2048 in 64 x 8 tiles: 72-74 ->
// 71.5 ms; 64.5 in the present ones).
template <typename T, int TX, int TZ, bool HASB, bool ADD, bool NT>
__global__ void __launch_bounds__(TX * TZ)
k_rhs_adjoint(AdjPtrs P, T c1, T c2, AdjGeo<T> G, T nu, T s, int cy) {
  constexpr int SX = TX + 2, SZ = TZ + 2, PLANE = SX * SZ, TH = TX * TZ;
  constexpr int NHALO = PLANE - TH;                // 2 SX + 2 TZ ring cells
  constexpr int PER = 1 + (NHALO + TH - 1) / TH;  // own cell first, then ring cells
  constexpr int NF = HASB ? 9 : 6;  // raw fields fetched per tile value
  __shared__ T sm[6 * 2 * PLANE];
  const T* src[9] = {static_cast<const T*>(P.u),  static_cast<const T*>(P.v),  static_cast<const T*>(P.w),
                     static_cast<const T*>(P.au), static_cast<const T*>(P.av), static_cast<const T*>(P.aw),
                     static_cast<const T*>(P.bu), static_cast<const T*>(P.bv), static_cast<const T*>(P.bw)};
  const Geo<T>& g = G.g;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int ntx = (nx + TX - 1) / TX, ntz = (nz + TZ - 1) / TZ;
  int b = xcd_slab_block(blockIdx.x, ntx * ntz);
  const int bx = b % ntx;
  b /= ntx;
  const int bz = b % ntz;
  const int by = b / ntz;
  const int i0 = bx * TX, k0 = bz * TZ;
  const int j0 = by * cy, j1 = (j0 + cy < ny) ? j0 + cy : ny;
  const int tx = threadIdx.x % TX, tz = threadIdx.x / TX;
  const int i = i0 + tx, k = k0 + tz;
  const bool mine = (i < nx) && (k < nz);
  const long plane = (long)nx * nz;
  // tile cells of this thread: q = 0 its own cell (tz+1, tx+1), q >= 1 the
  // ring cells (top row, bottom row, left column, right column)
  unsigned toff[PER];
  int cidx[PER];
  bool tin[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    int zz, xx;
    if (q == 0) {
      zz = tz + 1;
      xx = tx + 1;
      tin[q] = true;
    } else {
      const int h = threadIdx.x + (q - 1) * TH;
      tin[q] = h < NHALO;
      if (h < SX) {
        zz = 0, xx = h;
      } else if (h < 2 * SX) {
        zz = SZ - 1, xx = h - SX;
      } else if (h < 2 * SX + TZ) {
        zz = 1 + h - 2 * SX, xx = 0;
      } else {
        zz = 1 + (h - 2 * SX - TZ) % TZ, xx = SX - 1;
      }
    }
    int gi = (i0 + xx - 1) % nx;
    if (gi < 0) gi += nx;
    int gk = (k0 + zz - 1) % nz;
    if (gk < 0) gk += nz;
    toff[q] = tin[q] ? unsigned(gk * nx + gi) : 0u;
    cidx[q] = zz * SX + xx;
  }
  T r[NF][PER];
#define CF_ADJ_FETCH(jj)                                                        \
  {                                                                            \
    const long b_ = (long)min(max((jj), 0), ny - 1) * plane;                   \
    _Pragma("unroll") for (int f = 0; f < NF; ++f) {                           \
      const T* p_ = src[f] + b_;                                               \
      _Pragma("unroll") for (int q = 0; q < PER; ++q) r[f][q] = p_[toff[q]];   \
    }                                                                          \
  }
#define CF_ADJ_STORE(jj)                                                        \
  {                                                                            \
    const int sl_ = (jj) & 1;                                                  \
    const bool pin_ = (jj) >= 0 && (jj) < ny, vin_ = (jj) >= 0 && (jj) < ny - 1; \
    _Pragma("unroll") for (int q = 0; q < PER; ++q) {                          \
      if (tin[q]) {                                                            \
        const int idx = sl_ * PLANE + cidx[q];                                 \
        _Pragma("unroll") for (int f = 0; f < 3; ++f) {                        \
          const bool in_ = (f == 1) ? vin_ : pin_;                             \
          const T lam_ = HASB ? c1 * r[3 + f][q] + c2 * r[(6 + f) % NF][q] : c1 * r[3 + f][q]; \
          sm[f * 2 * PLANE + idx] = in_ ? r[f][q] : T(0);                      \
          sm[(3 + f) * 2 * PLANE + idx] = in_ ? lam_ : T(0);                   \
        }                                                                      \
      }                                                                        \
    }                                                                          \
    if (ADD) {                                                                 \
      _Pragma("unroll") for (int f = 0; f < 3; ++f) {                          \
        ps0[f] = ps1[f];                                                       \
        ps1[f] = HASB ? r[3 + f][0] + r[(6 + f) % NF][0] : r[3 + f][0];        \
      }                                                                        \
    }                                                                          \
  }
  const long pid = (long)k * nx + i;
  // A (+ B) at the own cell of planes j and j+1, kept from the move of the
  // planes into LDS for the ADD output
  T ps0[3] = {T(0), T(0), T(0)}, ps1[3] = {T(0), T(0), T(0)};
  CF_ADJ_FETCH(j0 - 1)
  CF_ADJ_STORE(j0 - 1)
  CF_ADJ_FETCH(j0)
  AdjLdsAcc<T, TX, TZ> A{sm, 0, 0, (tz + 1) * SX + tx + 1};
  T* gu = static_cast<T*>(P.gu);
  T* gv = static_cast<T*>(P.gv);
  T* gw = static_cast<T*>(P.gw);
  AdjCarry<T> carry{};
  // plane j0 - 1 only gives the carries of the chunk's first plane
  for (int j = j0 - 1; j < j1; ++j) {
    CF_ADJ_STORE(j + 1)
    __syncthreads();
    CF_ADJ_FETCH(j + 2)
    const AdjRow<T> Y = load_adj_row(G.rows, j);
    A.s0 = (j & 1) * PLANE;
    A.sp = ((j + 1) & 1) * PLANE;
    const AdjOut<T> o = rhs_adjoint_point<T>(A, G, Y, nu, carry);
    T ou = s * o.gu, ov = s * o.gv, ow = s * o.gw;
    if (ADD) {
      ou += ps0[0];
      ov += ps0[1];
      ow += ps0[2];
    }
    if (mine && j >= j0) {
      const long id = (long)j * plane + pid;
      st_once<NT>(ou, &gu[id]);
      st_once<NT>((j == ny - 1) ? T(0) : ov, &gv[id]);
      st_once<NT>(ow, &gw[id]);
    }
    __syncthreads();
  }
#undef CF_ADJ_FETCH
#undef CF_ADJ_STORE
}

// g* = g - W G phi (weighted correction of the projection transpose);
// W = dy_j for u and w, dyc_j for v (so the v part is g - (phi_{j+1} - phi_j)).
// Pairs and planes as in k_correct.
template <typename T, bool NT>
__global__ void __launch_bounds__(256)
k_correct_w(const T* __restrict__ gu, const T* __restrict__ gv, const T* __restrict__ gw, T* ou, T* ov, T* ow,
            const double* __restrict__ phi, AdjGeo<T> G) {
  const Geo<T>& g = G.g;
  const unsigned nh = g.nx / 2, m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nh * g.nz) return;
  const int j = blockIdx.y, k = int(m / nh), i = int(m - k * nh), kp = (k + 1 == g.nz) ? 0 : k + 1;
  const long row = (long)j * g.nz + k, id = row * nh + i;
  const cx<double>* p2 = reinterpret_cast<const cx<double>*>(phi);
  const cx<double> p0 = p2[id], pk = p2[((long)j * g.nz + kp) * nh + i];
  const double pn = phi[row * g.nx + (2 * i + 2 == g.nx ? 0 : 2 * i + 2)];
  const T dyj = G.dy[j];
  auto in = [&](const T* a) { return ld_once<NT>(reinterpret_cast<const cx<T>*>(a) + id); };
  auto out = [&](T* a, T r0, T r1) { st_once<NT>(mk(r0, r1), reinterpret_cast<cx<T>*>(a) + id); };
  // g and g* are touched once (streamed when NT, as in the forward correction)
  const cx<T> a = in(gu), c = in(gw);
  out(ou, a.re - dyj * (T(p0.im - p0.re) * g.rdx), a.im - dyj * (T(pn - p0.im) * g.rdx));
  out(ow, c.re - dyj * (T(pk.re - p0.re) * g.rdz), c.im - dyj * (T(pk.im - p0.im) * g.rdz));
  cx<T> b = mk(T(0), T(0));
  if (j != g.ny - 1) {
    const cx<double> pj = p2[id + (long)g.nz * nh];
    b = in(gv);
    b = mk(b.re - T(pj.re - p0.re), b.im - T(pj.im - p0.im));
  }
  out(ov, b.re, b.im);
}

}  // namespace cf
