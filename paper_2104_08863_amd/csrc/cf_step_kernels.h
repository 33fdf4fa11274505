// Momentum right-hand side, RK2 stages and pressure-gradient correction of the
// projection step (Section 2, Eq. (3)-(6) and Eq. (4)).
//
//   R(u) = -N(u) + nu lap(u) + fx e_x,  N(u) = div(u u) in flux form on the
//   staggered grid (linear interpolation; y-interpolation to a face weighted by
//   the two cell heights), lap with the no-slip ghost mirrored about the wall
//   (wall distance half a cell), v = 0 on both walls.
//   stage 1: ub = u + dt R(u)
//   stage 2: us = (u + ub)/2 + dt/2 R(ub)   (= u + dt/2 [R(u) + R(ub)])
//   correction: u1 = us - dt G p
//
// The RK stages march in y over LDS-resident planes (2.5D tiling, see
// k_rk_stage); the correction is pointwise.  Fields are (ny, nz, nx), x
// fastest; v[ny-1] is the top wall (read as 0, written as 0).
#pragma once

#include "cf_common.h"
#include "cf_rules.h"

namespace cf {

template <typename T>
struct Geo {
  const T* rdyc;  // 1/dyc_{j+1/2}, ny-1
  T rdx, rdz, rdx2, rdz2;
  T rdxq, rdzq;   // rdx / 4, rdz / 4
  int nx, ny, nz;
  const T* rows;  // YRow rows of planes -kRowPad .. ny + kRowPad - 1; points at plane 0
};

// The wall-normal factors of the momentum stencil at plane j (all zero outside
// [0, ny)): the interpolation weights carry the 1/2 of the velocity averages
// they multiply and are zero on the walls, and the wall faces hold 2/dy (the
// no-slip ghost mirrored about the wall, reached as a neighbour value of 0), so
// the stencil has no case for the walls.
template <typename T>
struct YRow {
  T rdy, rdyp;   // 1/dy_j, 1/dy_{j+1}
  T wl, wu;      // half the weights of planes j and j+1 at face j+1
  T fcm, fc;     // 1/dyc at the lower and the upper face
  T rdycq;       // 1/(4 dyc) at the upper face, 0 on the wall
  T pad;
};
constexpr int kRowPad = 4;

// Row j through the constant address space: j is the same for the whole block,
// so the row comes by one scalar load into scalar registers.  (Read from LDS it
// cost seven of the 25 LDS reads of a stencil and as many vector registers; a
// vector load would wait in order behind the next plane's prefetch.)
template <typename T>
__device__ __forceinline__ YRow<T> load_row(const T* rows, int j) {
  using CP = const __attribute__((address_space(4))) T*;
  const CP p = (CP)(uintptr_t)(rows + (long)j * 8);
  return YRow<T>{p[0], p[1], p[2], p[3], p[4], p[5], p[6], T(0)};
}

template <typename T>
struct RhsOut {
  T ru, rv, rw;
};

template <typename T>
struct FaceFlux {
  T exy, eyz;  // x-y and y-z edge products at the upper face of the cell
};

// R at point (i, j, k) from an accessor A with A.u(dj, dk, di) etc. returning
// the neighbour values (dj, dk, di in {-1, 0, 1}); A returns 0 for v on the top
// wall and for planes outside [0, ny).  below: the edge products at the lower
// face (the upper-face products of plane j-1); above receives those of face
// j+1.  The averages' factors 1/2 are folded into the difference factors (exact
// scalings by powers of two).  On the top wall's plane rv is meaningless.
template <typename T, class Acc>
__device__ __forceinline__ RhsOut<T> momentum_rhs(const Acc& A, const Geo<T>& g, const YRow<T>& Y, T nu, T fx,
                                                  FaceFlux<T> below, FaceFlux<T>& above) {
  const T u0 = A.u(0, 0, 0), uip = A.u(0, 0, 1), uim = A.u(0, 0, -1);
  const T ukp = A.u(0, 1, 0), ukm = A.u(0, -1, 0), ukpm = A.u(0, 1, -1);
  const T w0 = A.w(0, 0, 0), wip = A.w(0, 0, 1), wim = A.w(0, 0, -1);
  const T wkp = A.w(0, 1, 0), wkm = A.w(0, -1, 0), wkmp = A.w(0, -1, 1);
  const T v0 = A.v(0, 0, 0), vip = A.v(0, 0, 1), vim = A.v(0, 0, -1);
  const T vkp = A.v(0, 1, 0), vkm = A.v(0, -1, 0);
  const T uj1 = A.u(1, 0, 0), uj1m = A.u(1, 0, -1), wj1 = A.w(1, 0, 0), wj1m = A.w(1, -1, 0);
  const T vj1 = A.v(1, 0, 0);
  const T ujm = A.u(-1, 0, 0), wjm = A.w(-1, 0, 0), vjm = A.v(-1, 0, 0);
  // x-y and y-z edge products at face j+1 (u, w interpolated in y, v in x or z)
  const T exy_i = (u0 * Y.wl + uj1 * Y.wu) * (v0 + vip);
  const T exy_im = (uim * Y.wl + uj1m * Y.wu) * (vim + v0);
  const T eyz_k = (w0 * Y.wl + wj1 * Y.wu) * (v0 + vkp);
  const T eyz_km = (wkm * Y.wl + wj1m * Y.wu) * (vkm + v0);
  above.exy = exy_i;
  above.eyz = eyz_k;
  // four times the x-z edge products at (i+1/2, k+1/2) and the neighbours
  const T exz = (u0 + ukp) * (w0 + wip);
  const T exz_km = (ukm + u0) * (wkm + wkmp);
  const T exz_im = (uim + ukpm) * (wim + w0);
  RhsOut<T> o;
  {
    const T cp = uip + u0, cm = u0 + uim;
    const T n = (cp * cp - cm * cm) * g.rdxq + (exz - exz_km) * g.rdzq + (exy_i - below.exy) * Y.rdy;
    const T l = (uip - T(2) * u0 + uim) * g.rdx2 + (ukp - T(2) * u0 + ukm) * g.rdz2 +
                ((uj1 - u0) * Y.fc - (u0 - ujm) * Y.fcm) * Y.rdy;
    o.ru = (nu * l + fx) - n;
  }
  {
    const T cp = wkp + w0, cm = w0 + wkm;
    const T n = (cp * cp - cm * cm) * g.rdzq + (exz - exz_im) * g.rdxq + (eyz_k - below.eyz) * Y.rdy;
    const T l = (wip - T(2) * w0 + wim) * g.rdx2 + (wkp - T(2) * w0 + wkm) * g.rdz2 +
                ((wj1 - w0) * Y.fc - (w0 - wjm) * Y.fcm) * Y.rdy;
    o.rw = nu * l - n;
  }
  {
    const T cp = vj1 + v0, cm = v0 + vjm;
    const T n = (cp * cp - cm * cm) * Y.rdycq + (exy_i - exy_im) * g.rdx + (eyz_k - eyz_km) * g.rdz;
    const T l = (vip - T(2) * v0 + vim) * g.rdx2 + (vkp - T(2) * v0 + vkm) * g.rdz2 +
                ((vj1 - v0) * Y.rdyp - (v0 - vjm) * Y.rdy) * Y.fc;
    o.rv = nu * l - n;
  }
  return o;
}

// 2.5D tiling: a block owns TX x TZ columns (x, z) and marches over a chunk of
// cy planes in y, keeping three consecutive planes of u, v, w (with a one-cell
// halo in x and z, periodic wrap) in LDS; every field value is read from
// global memory once per plane step plus the halo.
template <int TX, int TZ>
struct RkTile {
  static constexpr int SX = TX + 2, SZ = TZ + 2, PLANE = SX * SZ, THREADS = TX * TZ;
};
template <typename T, int TX, int TZ>
struct LdsAcc {
  const T* su;  // three plane slots of u, each PLANE values
  const T* sv;
  const T* sw;
  int sm, s0, sp;  // slot offsets of planes j-1, j, j+1
  int base;        // (tz+1)*SX + tx+1
  static constexpr int SX = TX + 2;
  __device__ __forceinline__ int off(int dj, int dk, int di) const {
    return (dj < 0 ? sm : (dj > 0 ? sp : s0)) + base + dk * SX + di;
  }
  __device__ __forceinline__ T u(int dj, int dk, int di) const { return su[off(dj, dk, di)]; }
  __device__ __forceinline__ T v(int dj, int dk, int di) const { return sv[off(dj, dk, di)]; }
  __device__ __forceinline__ T w(int dj, int dk, int di) const { return sw[off(dj, dk, di)]; }
};

// STAGE 1: out = f + dt R(f).  STAGE 2: out = (f0 + f)/2 + dt/2 R(f).
// Plane j+2 is fetched into registers while plane j is computed from LDS.
// Each XCD takes a contiguous run of every y-chunk's tiles (xcd_slab_block):
// the FP32 stage on 2048x768x2048 runs in 17.2 ms instead of 22.0.
// NT: outputs, written once, stored non-temporally for large fields (FP64
// stage 1 on 1024x256x512: 1.37-1.43 -> 1.30 ms).
template <typename T, int STAGE, int TX, int TZ, bool NT>
__global__ void __launch_bounds__(TX * TZ, sizeof(T) == 8 ? 4 : 6)
k_rk_stage(const T* __restrict__ u, const T* __restrict__ v, const T* __restrict__ w,
           const T* u0, const T* v0, const T* w0, T* uo, T* vo, T* wo, Geo<T> g, T dt, T nu, T fx, int cy) {
  using Tl = RkTile<TX, TZ>;
  constexpr int PER = (Tl::PLANE + Tl::THREADS - 1) / Tl::THREADS;  // tile values per thread
  __shared__ T su[3 * Tl::PLANE], sv[3 * Tl::PLANE], sw[3 * Tl::PLANE];
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
  // in-plane offsets of this thread's tile values (periodic wrap); -1 = none
  int toff[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = threadIdx.x + q * Tl::THREADS;
    const int zz = idx / Tl::SX, xx = idx % Tl::SX;
    int gi = (i0 + xx - 1) % nx;
    if (gi < 0) gi += nx;
    int gk = (k0 + zz - 1) % nz;
    if (gk < 0) gk += nz;
    toff[q] = (idx < Tl::PLANE) ? gk * nx + gi : -1;
  }
  T ru[PER], rv[PER], rw[PER];
#define CF_RK_FETCH(jj)                                          \
  _Pragma("unroll") for (int q = 0; q < PER; ++q) {             \
    ru[q] = rv[q] = rw[q] = T(0);                               \
    if (toff[q] >= 0 && (jj) >= 0 && (jj) < ny) {               \
      const long o = (long)(jj) * plane + toff[q];              \
      ru[q] = u[o];                                             \
      rw[q] = w[o];                                             \
      if ((jj) < ny - 1) rv[q] = v[o];                          \
    }                                                           \
  }
#define CF_RK_STORE(s)                                           \
  _Pragma("unroll") for (int q = 0; q < PER; ++q) {             \
    if (toff[q] >= 0) {                                         \
      const int idx = threadIdx.x + q * Tl::THREADS;            \
      su[(s) * Tl::PLANE + idx] = ru[q];                        \
      sv[(s) * Tl::PLANE + idx] = rv[q];                        \
      sw[(s) * Tl::PLANE + idx] = rw[q];                        \
    }                                                           \
  }
  const long pid = (long)k * nx + i;  // this thread's in-plane offset
  CF_RK_FETCH(j0 - 1)
  CF_RK_STORE((j0 + 2) % 3)
  CF_RK_FETCH(j0)
  CF_RK_STORE(j0 % 3)
  CF_RK_FETCH(j0 + 1)
  T a0 = T(0), b0 = T(0), c0 = T(0);
  if (STAGE == 2 && mine) {
    a0 = u0[(long)j0 * plane + pid];
    b0 = (j0 < ny - 1) ? v0[(long)j0 * plane + pid] : T(0);
    c0 = w0[(long)j0 * plane + pid];
  }
  LdsAcc<T, TX, TZ> A{su, sv, sw, 0, 0, 0, (tz + 1) * Tl::SX + tx + 1};
  FaceFlux<T> carry{T(0), T(0)};
  // plane j0 - 1 only gives the edge products at the chunk's lowest face (its
  // plane below is not in LDS and what it makes of it is not used)
  for (int j = j0 - 1; j < j1; ++j) {
    if (j >= j0) {
      CF_RK_STORE((j + 1) % 3)
    }
    __syncthreads();
    if (j >= j0) {
      CF_RK_FETCH(j + 2)
    }
    const YRow<T> Y = load_row(g.rows, j);
    T a1 = T(0), b1 = T(0), c1 = T(0);
    if (STAGE == 2 && mine && j >= j0 && j + 1 < j1) {
      a1 = u0[(long)(j + 1) * plane + pid];
      b1 = (j + 1 < ny - 1) ? v0[(long)(j + 1) * plane + pid] : T(0);
      c1 = w0[(long)(j + 1) * plane + pid];
    }
    A.sm = ((j + 2) % 3) * Tl::PLANE;
    A.s0 = ((j + 3) % 3) * Tl::PLANE;
    A.sp = ((j + 1) % 3) * Tl::PLANE;
    FaceFlux<T> up;
    const RhsOut<T> r = momentum_rhs<T>(A, g, Y, nu, fx, carry, up);
    carry = up;
    if (mine && j >= j0) {
      const long id = (long)j * plane + pid;
      const bool top = (j == ny - 1);
      const T uc = A.u(0, 0, 0), vc = A.v(0, 0, 0), wc = A.w(0, 0, 0);
      if (STAGE == 1) {
        st_once<NT>(uc + dt * r.ru, &uo[id]);
        st_once<NT>(top ? T(0) : vc + dt * r.rv, &vo[id]);
        st_once<NT>(wc + dt * r.rw, &wo[id]);
      } else {
        const T hh = T(0.5), hd = T(0.5) * dt;
        st_once<NT>(hh * (a0 + uc) + hd * r.ru, &uo[id]);
        st_once<NT>(top ? T(0) : hh * (b0 + vc) + hd * r.rv, &vo[id]);
        st_once<NT>(hh * (c0 + wc) + hd * r.rw, &wo[id]);
      }
    }
    if (j >= j0) {
      a0 = a1;
      b0 = b1;
      c0 = c1;
    }
    __syncthreads();
  }
#undef CF_RK_FETCH
#undef CF_RK_STORE
}

// u1 = us - dt G p at the points 2i and 2i + 1 of row (j, k) (in place; the
// top-wall v plane is 0); returns the corrected values.  Two neighbours in x take
// one load and store per array (rows have an even length and the arrays are
// 16-byte aligned).  Each velocity value is read and written once,
// non-temporally when NT (the FP64 correction on 1024x256x512 runs 5 % faster
// than with plain loads and stores); p, whose values neighbouring points share,
// is read through the caches.
template <bool NT, typename T>
__device__ __forceinline__ void correct_pair(T* u, T* v, T* w, const double* __restrict__ p, const Geo<T>& g, T dt,
                                             int i, int k, int j, cx<T>& cu, cx<T>& cv, cx<T>& cw) {
  const int nh = g.nx / 2, kp = (k + 1 == g.nz) ? 0 : k + 1;
  const long row = (long)j * g.nz + k, id = row * nh + i;
  const cx<double>* p2 = reinterpret_cast<const cx<double>*>(p);
  const cx<double> p0 = p2[id], pk = p2[((long)j * g.nz + kp) * nh + i];
  const double pn = p[row * g.nx + (2 * i + 2 == g.nx ? 0 : 2 * i + 2)];
  cx<T>*u2 = reinterpret_cast<cx<T>*>(u) + id, *v2 = reinterpret_cast<cx<T>*>(v) + id,
       *w2 = reinterpret_cast<cx<T>*>(w) + id;
  cu = ld_once<NT>(u2);
  cw = ld_once<NT>(w2);
  cu = mk(cu.re - dt * (T(p0.im - p0.re) * g.rdx), cu.im - dt * (T(pn - p0.im) * g.rdx));
  cw = mk(cw.re - dt * (T(pk.re - p0.re) * g.rdz), cw.im - dt * (T(pk.im - p0.im) * g.rdz));
  st_once<NT>(cu, u2);
  st_once<NT>(cw, w2);
  cv = mk(T(0), T(0));
  if (j != g.ny - 1) {
    const cx<double> pj = p2[id + (long)g.nz * nh];
    cv = ld_once<NT>(v2);
    cv = mk(cv.re - dt * (T(pj.re - p0.re) * g.rdyc[j]), cv.im - dt * (T(pj.im - p0.im) * g.rdyc[j]));
  }
  st_once<NT>(cv, v2);
}

// u1 = us - dt G p, one thread per pair.  Memory-bound: six velocity passes and
// one of p.  A grid row of blocks holds one plane, so that a thread's indices
// take one 32-bit division.  Against one point per thread of the whole grid:
// FP64 1024x256x512 1.274 -> 1.271 ms (5.9 TB/s), 256x128x256 81 -> 74 us, FP32
// 512x192x512 338 -> 306 us (5.3 TB/s); of the scalar form with the plane's grid
// the last took 333.  Blocks of correction_threads.
template <typename T, bool NT>
__global__ void __launch_bounds__(256)
k_correct(T* u, T* v, T* w, const double* __restrict__ p, Geo<T> g, T dt) {
  const unsigned nh = g.nx / 2, m = blockIdx.x * blockDim.x + threadIdx.x;  // pair of plane j
  if (m >= nh * g.nz) return;
  const int k = int(m / nh);
  cx<T> cu, cv, cw;
  correct_pair<NT, T>(u, v, w, p, g, dt, int(m - k * nh), k, blockIdx.y, cu, cv, cw);
}

// Block reduction of six FP64 per-thread sums in a fixed order (wave shuffles,
// then the waves in order); thread f < 6 returns sum f.
template <int TH>
__device__ __forceinline__ double block_sum6(const double (&sm)[6], double (&red)[6][TH / 64]) {
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    double x = sm[f];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_down(x, d, 64);
    if ((threadIdx.x & 63) == 0) red[f][threadIdx.x >> 6] = x;
  }
  __syncthreads();
  double x = 0.0;
  if (threadIdx.x < 6)
    for (int k = 0; k < TH / 64; ++k) x += red[threadIdx.x][k];
  return x;
}

// The correction of k_correct (same per-point arithmetic) fused with the
// plane statistics of the corrected fields: block b corrects chunk b % nch of
// plane b / nch and writes the six FP64 sums of that chunk (u, v, w and their
// squares; fixed order: strided per-thread sums, then block_sum6) to
// part[b * 6 + f].  k_stats_gather adds the chunks of each plane in order.
template <typename T, int TH, bool NT>
__global__ void __launch_bounds__(TH)
k_correct_stats(T* __restrict__ u, T* __restrict__ v, T* __restrict__ w, const double* __restrict__ p, Geo<T> g,
                T dt, double* __restrict__ part, int nch) {
  __shared__ double red[6][TH / 64];
  const int nh = g.nx / 2, n2 = nh * g.nz;  // pairs of a plane
  const int j = blockIdx.x / nch, c = blockIdx.x % nch;
  const int len = (n2 + nch - 1) / nch;
  const int e0 = c * len, e1 = (e0 + len < n2) ? e0 + len : n2;
  double sm[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int e = e0 + threadIdx.x; e < e1; e += TH) {
    const int k = e / nh;
    cx<T> cu, cv, cw;
    correct_pair<NT, T>(u, v, w, p, g, dt, e - k * nh, k, j, cu, cv, cw);
    const double q[6] = {double(cu.re), double(cv.re), double(cw.re), double(cu.im), double(cv.im), double(cw.im)};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      sm[f % 3] += q[f];
      sm[f % 3 + 3] += q[f] * q[f];
    }
  }
  const double x = block_sum6<TH>(sm, red);
  if (threadIdx.x < 6) part[(long)blockIdx.x * 6 + threadIdx.x] = x;
}

// Plane statistics of a velocity field: for every y-plane j the means over the
// x-z plane of u, v, w and of their squares, summed in FP64.  One block per
// plane and a fixed reduction order (strided per-thread sums, wave shuffles,
// then the waves in order), so the result is bitwise repeatable.  st[j*6 + c]
// receives (or, with accumulate, gains) the means.
template <typename T, int TH>
__global__ void __launch_bounds__(TH)
k_plane_stats(const T* __restrict__ u, const T* __restrict__ v, const T* __restrict__ w, double* __restrict__ st,
              int nxz, double scale, int accumulate) {
  __shared__ double red[6][TH / 64];
  const long o = (long)blockIdx.x * nxz;
  double sm[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int e = threadIdx.x; e < nxz; e += TH) {
    const double a = double(u[o + e]), b = double(v[o + e]), c = double(w[o + e]);
    sm[0] += a;
    sm[1] += b;
    sm[2] += c;
    sm[3] += a * a;
    sm[4] += b * b;
    sm[5] += c * c;
  }
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    double x = sm[f];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_down(x, d, 64);
    if ((threadIdx.x & 63) == 0) red[f][threadIdx.x >> 6] = x;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    double x = 0.0;
    for (int k = 0; k < TH / 64; ++k) x += red[threadIdx.x][k];
    x *= scale;
    double* d = st + (long)blockIdx.x * 6 + threadIdx.x;
    *d = accumulate ? *d + x : x;
  }
}

}  // namespace cf
