// Level passes of the small and middle levels on whole tiles (arXiv
// 2602.01888, Section 3): the same down and up passes as the band-marching
// ones (fused.hip), for levels whose passes are bound by latency.
//
// A marching block runs a chain of eleven barrier phases for every two rows
// of its band and halo, and waits for each step's loads: 12 .. 22 us for
// levels of 65^2 .. 513^2 nodes, whatever the width.  Here a workgroup loads
// a whole tile with its halo at once, each thread one 2 x 2 quad (quad.h),
// and runs the colour phases over the tile: 4 nu barriers and one memory
// latency in all, every lane relaxing one node in each phase.  The price is
// the halo (4 nu + 2 columns, 2 nu + 2 rows), recomputed and read again by
// the neighbouring tiles, so large levels, bound by their bytes, stay with
// the marching passes.
//
// Halo.  Quads start at even nodes, and a region edge is not relaxed unless
// it is the grid's.  A sweep then leaves wrong values in the outer four
// columns and two rows on the low side, and one column and one row fewer on
// the high side; the residual and its restriction take one more each.
#include <type_traits>

#include "quad.h"
#include "tomg_internal.h"

namespace tomg {
namespace {

template <int NU, bool RES>
struct Halo {  // nodes around the owned tile (even, so that quads stay whole)
  static constexpr int W = 4 * NU + (RES ? 2 : 0), E = 4 * NU;
  static constexpr int S = 2 * NU + (RES ? 2 : 0), N = 2 * NU;
};

// CK, the grid transfer: 0 both axes halved, 1 x halved alone, 2 y halved alone.
template <typename T, bool EPS, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, int QX,
          int QY, int CK>
__device__ __forceinline__ void tile_body(const PassArgs<T> &a, const int bx, const int by,
                                          const double stop) {
  using H = Halo<NU, RESTRICT || NORM>;
  constexpr int PITCH = QX + 2, PS = PITCH * (QY + 2);
  __shared__ T S[4 * PS];
  __shared__ double red[QX * QY / 64];
  const int t = threadIdx.x, u = t % QX, w = t / QX;
  const int nx = a.nx, ny = a.ny;
  const int i0 = bx * a.W - H::W + 2 * u, j0 = by * a.CH - H::S + 2 * w;
  // columns are loaded in pairs from ib; a pair that would start at the last
  // column starts one before it
  const int ib = min(max(i0, 0), nx - 2);
  const bool last = i0 > ib;
  const size_t n = (size_t)nx * ny;
  auto row = [&](int j) { return (size_t)min(max(j, 0), ny - 1) * nx; };
  T *c = S + (w + 1) * PITCH + u + 1;

  std::conditional_t<EPS, QuadEps<T>, QuadSt<T>> q;
  bool in[4];  // node inside the grid
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const size_t at = row(j0 + b) + ib;
    const auto f = load_pair(a.b + at);
    q.f[2 * b] = last ? f[1] : f[0];
    q.f[2 * b + 1] = f[1];
    if constexpr (!ZERO) {
      const auto x = load_pair(a.xin + at);
      q.x[2 * b] = last ? x[1] : x[0];
      q.x[2 * b + 1] = x[1];
    }
    const uint8_t d0 = a.dir[last ? at + 1 : at], d1 = a.dir[at + 1];
    const bool rowin = j0 + b >= 0 && j0 + b < ny;
    in[2 * b] = rowin && i0 >= 0 && i0 < nx;
    in[2 * b + 1] = rowin && i0 + 1 >= 0 && i0 + 1 < nx;
    // provisional: 1 where the node may change
    q.ik[2 * b] = in[2 * b] && !d0 ? T(1) : T(0);
    q.ik[2 * b + 1] = in[2 * b + 1] && !d1 ? T(1) : T(0);
  }
  T dg[4];
  if constexpr (EPS) {
    // columns i0 - 1 .. i0 + 2, rows j0 - 1 .. j0 + 2 (clamped: only nodes
    // inside the grid's ring use them)
    const int iw = min(max(i0 - 1, 0), nx - 1), ie = min(max(i0 + 2, 0), nx - 1);
    T xx[2][4], xy[4][4], yy[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t at = row(j0 - 1 + r);
      const auto pxy = load_pair(a.exy + at + ib), pyy = load_pair(a.eyy + at + ib);
      xy[r][1] = last ? pxy[1] : pxy[0];
      xy[r][2] = pxy[1];
      yy[r][0] = last ? pyy[1] : pyy[0];
      yy[r][1] = pyy[1];
      if (r == 1 || r == 2) {
        const auto pxx = load_pair(a.exx + at + ib);
        xx[r - 1][1] = last ? pxx[1] : pxx[0];
        xx[r - 1][2] = pxx[1];
        xx[r - 1][0] = a.exx[at + iw];
        xx[r - 1][3] = a.exx[at + ie];
        xy[r][0] = a.exy[at + iw];
        xy[r][3] = a.exy[at + ie];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int x = k & 1, y = k >> 1;
      const T ax = xx[y][x + 1] * a.cx, ay = yy[y + 1][x] * a.cy;
      T gx, gy;
      eps_coefs(xx[y][x + 2] - xx[y][x], yy[y + 2][x] - yy[y][x], xy[y + 1][x + 2] - xy[y + 1][x],
                xy[y + 2][x + 1] - xy[y][x + 1], a.qx, a.qy, a.qxy, gx, gy);
      q.k1[k] = plain_add(ax, gx);
      q.k3[k] = plain_add(ax, -gx);
      q.k4[k] = plain_add(ay, gy);
      q.k5[k] = plain_add(ay, -gy);
      q.k6[k] = xy[y + 1][x + 1] * a.hxy;
      dg[k] = q.dg[k] = eps_diag(ax, ay);
    }
  } else {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const size_t at = row(j0 + b) + ib;
#pragma unroll
      for (int z = 0; z < 9; ++z) {
        const auto p = load_pair(a.st + z * n + at);
        q.a[2 * b][z] = last ? p[1] : p[0];
        q.a[2 * b + 1][z] = p[1];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dg[k] = q.a[k][4];
  }
  if constexpr (PROLONG && CK != 0) {
    T e[4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {  // along the halved axis: at the coarse node, half way
      T c0, c1;
      int k0, k1;
      if constexpr (CK == 1) {  // row j0 + b
        const T *r0 = a.xc + (size_t)min(max(j0 + b, 0), a.nyc - 1) * a.nxc;
        const int I = min(max(i0 >> 1, 0), a.nxc - 1);
        c0 = r0[I];
        c1 = r0[min(I + 1, a.nxc - 1)];
        k0 = 2 * b, k1 = 2 * b + 1;
      } else {  // column i0 + b
        const T *r0 = a.xc + min(max(i0 + b, 0), a.nxc - 1);
        const int J = min(max(j0 >> 1, 0), a.nyc - 1);
        c0 = r0[(size_t)J * a.nxc];
        c1 = r0[(size_t)min(J + 1, a.nyc - 1) * a.nxc];
        k0 = b, k1 = b + 2;
      }
      e[k0] = c0;
      e[k1] = T(0.5) * (c0 + c1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (q.ik[k] != T(0)) q.x[k] += e[k];
  } else if constexpr (PROLONG) {
    const int I = min(max(i0 >> 1, 0), a.nxc - 1), J = min(max(j0 >> 1, 0), a.nyc - 1);
    const int I1 = min(I + 1, a.nxc - 1), J1 = min(J + 1, a.nyc - 1);
    const T *r0 = a.xc + (size_t)J * a.nxc, *r1 = a.xc + (size_t)J1 * a.nxc;
    const T c00 = r0[I], c01 = r0[I1], c10 = r1[I], c11 = r1[I1];
    const T e01 = T(0.5) * (c00 + c01), e11 = T(0.5) * (c10 + c11);
    const T e[4] = {c00, e01, T(0.5) * (c00 + c10), T(0.5) * (e01 + e11)};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (q.ik[k] != T(0)) q.x[k] += e[k];
  }
  if (stop != 0.0) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (ZERO || !in[k]) q.x[k] = T(0);
    c[k * PS] = q.x[k];
    // the region's edge has no neighbours here and keeps its value (it is
    // outside the grid, or wrong and never reaches the owned tile)
    const bool edge = ((k & 1) ? u == QX - 1 : u == 0) || ((k >> 1) ? w == QY - 1 : w == 0);
    q.ik[k] = q.ik[k] != T(0) && !edge ? T(1) / dg[k] : T(0);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NU; ++s)
#pragma unroll
    for (int col = 0; col < 4; ++col) {
      quad_relax<T>(q, c, col, PS, PITCH);
      __syncthreads();
    }
  const bool own = u >= H::W / 2 && 2 * u < H::W + a.W && w >= H::S / 2 && 2 * w < H::S + a.CH;
  T res[4];
  double acc = 0.0;
  if constexpr (RESTRICT || NORM) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      res[k] = quad_resid<T>(q, c, k, PS, PITCH);
      if (own && in[k]) acc += (double)(res[k] * res[k]);
    }
  }
  if (own) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (in[k]) a.xout[(size_t)(j0 + (k >> 1)) * nx + i0 + (k & 1)] = q.x[k];
  }
  if constexpr (RESTRICT) {
    __syncthreads();  // the residuals take the iterate's place in LDS
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k * PS] = res[k];
    __syncthreads();
    if constexpr (CK != 0) {  // (1/4) [1 2 1] along the halved axis, two coarse nodes
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int k = CK == 1 ? 2 * b : b;
        if (own && in[k]) {
          const int I = CK == 1 ? i0 >> 1 : i0 + b, J = CK == 1 ? j0 + b : j0 >> 1;
          const bool ring = I == 0 || J == 0 || I == a.nxc - 1 || J == a.nyc - 1;
          const bool fixed = ring && (!a.dirc || a.dirc[(size_t)J * a.nxc + I]);
          const T lo = quad_nb(res, c, k, CK == 1 ? -1 : 0, CK == 1 ? 0 : -1, PS, PITCH);
          const T hi = quad_nb(res, c, k, CK == 1 ? 1 : 0, CK == 1 ? 0 : 1, PS, PITCH);
          a.bc[(size_t)J * a.nxc + I] = fixed ? T(0) : (lo + T(2) * res[k] + hi) * T(0.25);
        }
      }
    } else if (own && in[0]) {
      const int I = i0 >> 1, J = j0 >> 1;
      const bool ring = I == 0 || J == 0 || I == a.nxc - 1 || J == a.nyc - 1;
      // a coarse ring node is Dirichlet unless its edge is Neumann
      const bool fixed = ring && (!a.dirc || a.dirc[(size_t)J * a.nxc + I]);
      const T v = quad_full_weight(res, c, 0, PS, PITCH);
      a.bc[(size_t)J * a.nxc + I] = fixed ? T(0) : v;
    }
  }
  if constexpr (NORM) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((t & 63) == 0) red[t >> 6] = acc;
    __syncthreads();
    if (t == 0) {
      for (int k = 1; k < QX * QY / 64; ++k) acc += red[k];
      a.partials[(size_t)by * a.nbx + bx] = acc;
    }
  }
}

template <typename T, bool EPS, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, int QX,
          int QY, int CK>
__global__ __launch_bounds__(QX *QY) void k_tile(PassArgs<T> a) {
  // tested in the body once the tile's loads are under way: a launch is one
  // memory latency long, and the test first would be another
  const double stop = a.skip ? *a.skip : 0.0;
  tile_body<T, EPS, NU, ZERO, PROLONG, RESTRICT, NORM, QX, QY, CK>(a, blockIdx.x % a.nbx,
                                                                  blockIdx.x / a.nbx, stop);
}

template <typename T, bool EPS, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, int QX,
          int QY, int CK>
__global__ __launch_bounds__(QX *QY) void k_tile_b(BatchTab tab) {
  int bx, by;
  const PassArgs<T> a = batch_args<T>(tab, bx, by);
  tile_body<T, EPS, NU, ZERO, PROLONG, RESTRICT, NORM, QX, QY, CK>(a, bx, by, 0.0);
}

template <typename T, bool EPS, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, int QX,
          int QY, int CK>
void launch_shape(const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (tab)
    hipLaunchKernelGGL((k_tile_b<T, EPS, NU, ZERO, PROLONG, RESTRICT, NORM, QX, QY, CK>), nb,
                       QX * QY, 0, s, *tab);
  else
    hipLaunchKernelGGL((k_tile<T, EPS, NU, ZERO, PROLONG, RESTRICT, NORM, QX, QY, CK>),
                       a.nbx * a.nby, QX * QY, 0, s, a);
}
template <typename T, bool EPS, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, int CK>
void launch_nu(int nu, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  const bool large = a.form == kFormTileLarge;
  if (nu == 1 && large)
    launch_shape<T, EPS, 1, ZERO, PROLONG, RESTRICT, NORM, 32, 16, CK>(a, s, tab, nb);
  else if (nu == 1)
    launch_shape<T, EPS, 1, ZERO, PROLONG, RESTRICT, NORM, 16, 16, CK>(a, s, tab, nb);
  else if (large)
    launch_shape<T, EPS, 2, ZERO, PROLONG, RESTRICT, NORM, 32, 16, CK>(a, s, tab, nb);
  else
    launch_shape<T, EPS, 2, ZERO, PROLONG, RESTRICT, NORM, 16, 16, CK>(a, s, tab, nb);
}
// Three and four sweeps: FP64 levels below the first in a batch (pick_tile).
template <typename T, bool EPS, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
constexpr bool many_sweeps() {
  return std::is_same<T, double>::value && !EPS && !NORM && (ZERO || PROLONG);
}
template <typename T, bool EPS, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
void launch_ck(int nu, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if constexpr (many_sweeps<T, EPS, ZERO, PROLONG, RESTRICT, NORM>()) {
    if (nu == 3)
      return launch_shape<T, EPS, 3, ZERO, PROLONG, RESTRICT, NORM, 32, 16, 0>(a, s, tab, nb);
    if (nu == 4)
      return launch_shape<T, EPS, 4, ZERO, PROLONG, RESTRICT, NORM, 32, 16, 0>(a, s, tab, nb);
  }
  if (a.ck == 0)
    launch_nu<T, EPS, ZERO, PROLONG, RESTRICT, NORM, 0>(nu, a, s, tab, nb);
  else if (a.ck == 1)
    launch_nu<T, EPS, ZERO, PROLONG, RESTRICT, NORM, 1>(nu, a, s, tab, nb);
  else
    launch_nu<T, EPS, ZERO, PROLONG, RESTRICT, NORM, 2>(nu, a, s, tab, nb);
}

}  // namespace

// Gives the pass the tile form: up to two sweeps (of three or four the halo is
// wider than the tile), alone on levels up to 1.2 M nodes, where the bands in
// LDS, then the other form of these levels, took over: 65^2 13.1, 14.1 -> 5.8,
// 5.3 us a pass (down, up; FP64), 129^2 12.9, 12.4 -> 6.2, 5.8, 257^2 14.7, 16.4
// -> 7.9, 6.2, 513^2 21.7, 22.0 -> 15.7, 12.6, 1025^2 39.1, 38.7 -> 36.4, 36.4.
// Against the marching form, us a pass, marching / tiles, V(2,2):
//               FP64, tensor            FP64, stored            FP32, tensor
//               down       up           down       up           down       up
//   257^2       10.6/6.6   9.7/6.3      13.0/6.9   11.5/6.6     8.9/6.1    8.4/5.6
//   513^2       12.8/9.9   11.6/11.7    16.0/14.4  14.3/14.9    12.2/8.3   10.2/6.3
//   769^2       15.1/14.6  14.7/14.8    23.4/21.3  21.3/21.4    15.0/10.7  13.5/10.7
//   1025^2      20.4/22.1  20.0/21.0    31.1/36.5  27.5/35.4    16.8/15.6  15.0/14.2
//   1217x1025   23.0/25.1  22.3/24.8    33.6/42.8  30.7/43.4    17.3/17.2  15.7/15.9
//   1537^2      31.5/43.0  31.2/42.8    51.6/79.3  46.5/81.0    23.2/27.9  22.8/23.8
//   2049^2      50.8/71.7  51.3/72.9    97.0/139   93.9/139     29.7/46.1  27.3/42.4
// (coarse levels, stored, from zero: 1025^2 FP64 29.4/34.4, 27.6/34.7, FP32
// 19.7/21.5, 20.8/21.3; 769^2 21.2/20.2, 21.4/20.0 and 14.8/13.1, 14.1/14.1).
// So 1.2 M is where FP32 passes from the tensor change over; FP64 passes do at
// 0.6 M nodes, and those of a million lose 5 .. 30 % here.  Small grids take
// the 32 x 32 tiles, for more blocks; from 257^2 up there are enough of the
// larger ones, which recompute less halo (a 513^2 cycle 71.5 us with them, 77.7
// without).
// In a batch that fills the device the marching passes, which recompute less
// halo, are the faster from 257^2 up and even below.  256 problems of sides 65
// .. 1025, mixed precision and FP64, tiles on no level 19.5 and 25.4 ms, up to
// 65^2 19.55 and 25.8, 129^2 19.7 and 25.9, 257^2 20.2 and 26.6, 513^2 21.8 and
// 28.8; a burst of 24 requests 12.1, 12.1, 12.3, 12.6 and 12.7 ms.  (Before its
// arguments lay in scalar registers and the stored passes marched, a batch was
// fastest with tiles up to 129^2.)
// Three and four sweeps, FP64, in a batch: levels below the first up to 65^2.
// An FP32 batch has them in the tail, whose FP64 form starts at 33^2, and a
// band of 65^2 is a long chain on few blocks: 16 problems of 257^2, V(3,3), 2070
// us on bands, 1715 on tiles; 200 of 129^2 5300 and 4320.
// One axis halved (semi-annulus of 1537 x 769, stored, FP32; bands -> tiles):
// level 1, 769 x 769, 23, 22 -> 14, 14 us; level 0, whose bands ran chained
// in 66 us with the next cycle's downward pass, 23 + 27.
constexpr long kTileNodes = 1200000;      // largest level on tiles
constexpr long kSmallTileNodes = 20000;   // largest level on 32 x 32 tiles
constexpr long kTileNodesBatch = 20000;   // largest level on tiles in a batch
constexpr long kManySweepNodes = 65 * 65;  // largest level on tiles with three or four sweeps
template <typename T>
bool pick_tile(PassArgs<T> &a, int l, int nu, bool res, bool batch) {
  const long n = (long)a.nx * a.ny;
  if (nu > 2) {
    if (!std::is_same<T, double>::value || !batch || l == 0 || a.ck != 0 || n > kManySweepNodes)
      return false;
    a.form = kFormTileLarge;
  } else {
    if (n > (batch ? kTileNodesBatch : kTileNodes)) return false;
    a.form = n > kSmallTileNodes ? kFormTileLarge : kFormTileSmall;
  }
  const int hx = 8 * nu + (res ? 2 : 0), hy = 4 * nu + (res ? 2 : 0);
  a.W = (a.form == kFormTileLarge ? 64 : 32) - hx;
  a.CH = 32 - hy;
  a.nbx = (a.nx + a.W - 1) / a.W;
  a.nby = (a.ny + a.CH - 1) / a.CH;
  a.xcd_order = 0;
  return true;
}
template bool pick_tile<double>(PassArgs<double> &, int, int, bool, bool);
template bool pick_tile<float>(PassArgs<float> &, int, int, bool, bool);

template <typename T>
void tile_down(int nu, bool eps, bool zero, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (eps) {
    if (zero) launch_ck<T, true, true, false, true, false>(nu, a, s, tab, nb);
    else launch_ck<T, true, false, false, true, false>(nu, a, s, tab, nb);
  } else {
    if (zero) launch_ck<T, false, true, false, true, false>(nu, a, s, tab, nb);
    else launch_ck<T, false, false, false, true, false>(nu, a, s, tab, nb);
  }
}
template <typename T>
void tile_up(int nu, bool eps, bool norm, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (eps) {
    if (norm) launch_ck<T, true, false, true, false, true>(nu, a, s, tab, nb);
    else launch_ck<T, true, false, true, false, false>(nu, a, s, tab, nb);
  } else {
    if (norm) launch_ck<T, false, false, true, false, true>(nu, a, s, tab, nb);
    else launch_ck<T, false, false, true, false, false>(nu, a, s, tab, nb);
  }
}
template void tile_down<double>(int, bool, bool, const PassArgs<double> &, hipStream_t, const BatchTab *, int);
template void tile_down<float>(int, bool, bool, const PassArgs<float> &, hipStream_t, const BatchTab *, int);
template void tile_up<double>(int, bool, bool, const PassArgs<double> &, hipStream_t, const BatchTab *, int);
template void tile_up<float>(int, bool, bool, const PassArgs<float> &, hipStream_t, const BatchTab *, int);

}  // namespace tomg
