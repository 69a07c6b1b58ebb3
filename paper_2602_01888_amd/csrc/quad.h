// A 2 x 2 quad of grid nodes held by one thread: the four nodes of a quad
// have the four colours of the four-colour Gauss-Seidel sweep, so in every
// colour phase each thread relaxes exactly one node of its own and no lane
// idles.  The quad's stencils, right-hand side and iterate stay in registers;
// the iterate is mirrored in LDS, one plane per quad position, so that a
// phase reads the five neighbours outside the quad with unit stride across
// lanes.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "tomg_internal.h"

namespace tomg {

// ---- arithmetic of one node ---------------------------------------------
// Every kernel that relaxes nodes (level passes, tiles, tail) forms a node's
// value from these functions alone.  Each multiply-add is written out and
// contraction is off: left to the compiler, which product of a sum becomes
// the fused one depends on where its operands live, and a problem solved
// alone and in a batch, by different kernels, must agree bit for bit.

// f minus the off-centre part of a stored 9-point stencil.
template <typename T>
__device__ __forceinline__ T defect9(T f, const T *a, T sw, T s, T se, T w, T e, T nw, T n,
                                     T ne) {
#pragma clang fp contract(off)
  T o = a[1] * s;
  o = __builtin_elementwise_fma(a[0], sw, o);
  o = __builtin_elementwise_fma(a[2], se, o);
  o = __builtin_elementwise_fma(a[3], w, o);
  o = __builtin_elementwise_fma(a[5], e, o);
  o = __builtin_elementwise_fma(a[6], nw, o);
  o = __builtin_elementwise_fma(a[7], n, o);
  o = __builtin_elementwise_fma(a[8], ne, o);
  return f - o;
}
// The same for eq. 18: k1, k3, k4, k5 the E, W, N, S neighbours, k6 the
// diagonal difference.
template <typename T>
__device__ __forceinline__ T defect18(T f, T k1, T k3, T k4, T k5, T k6, T sw, T s, T se, T w,
                                      T e, T nw, T n, T ne) {
#pragma clang fp contract(off)
  T o = k3 * w;
  o = __builtin_elementwise_fma(k1, e, o);
  o = __builtin_elementwise_fma(k4, n, o);
  o = __builtin_elementwise_fma(k5, s, o);
  o = __builtin_elementwise_fma(k6, (ne - nw) - (se - sw), o);
  return f - o;
}
template <typename T>
__device__ __forceinline__ T relaxed(T defect, T ik) { return defect * ik; }
template <typename T>
__device__ __forceinline__ T residual_of(T defect, T dg, T x) {
  return __builtin_elementwise_fma(-dg, x, defect);
}
// Coefficients of eq. 18 at a node from the tensor there and the differences
// of its components across the node (dxx = eps_xx E - W, dyy = eps_yy N - S,
// xyx and xyy those of eps_xy); k1 = ax + gx, k3 = ax - gx, k4 = ay + gy,
// k5 = ay - gy, diagonal -2 (ax + ay).
template <typename T>
__device__ __forceinline__ void eps_coefs(T dxx, T dyy, T xyx, T xyy, T qx, T qy, T qxy, T &gx,
                                          T &gy) {
#pragma clang fp contract(off)
  gx = __builtin_elementwise_fma(xyy, qxy, dxx * qx);
  gy = __builtin_elementwise_fma(dyy, qy, xyx * qxy);
}
template <typename T>
__device__ __forceinline__ T plain_add(T a, T b) {
#pragma clang fp contract(off)
  return a + b;
}
template <typename T>
__device__ __forceinline__ T eps_diag(T ax, T ay) { return T(-2) * plain_add(ax, ay); }

// ---- quads -----------------------------------------------------------------

// Position k = a + 2 b of a node in its quad (a along x, b along y).
template <typename T>
struct Quad {
  T f[4], ik[4], x[4];  // ik: 1 / diagonal, 0 where the node is not relaxed
};
// Stored 9-point stencil (plane order of the level), and eq. 18's
// coefficients with the diagonal.
template <typename T>
struct QuadSt : Quad<T> {
  T a[4][9];
};
template <typename T>
struct QuadEps : Quad<T> {
  T k1[4], k3[4], k4[4], k5[4], k6[4], dg[4];
};

// Neighbour (di, dj) of position k: from the thread's own quad, or from the
// LDS plane of the neighbour's position.  c points at the thread's entry of
// plane 0; ps and pitch are the plane size and its row pitch.
template <typename T>
__device__ __forceinline__ T quad_nb(const T (&x)[4], const T *c, int k, int di, int dj, int ps,
                                     int pitch) {
  const int a = (k & 1) + di, b = (k >> 1) + dj;
  const int pos = (a & 1) + 2 * (b & 1);
  if (a >= 0 && a < 2 && b >= 0 && b < 2) return x[pos];
  const int du = a < 0 ? -1 : (a > 1 ? 1 : 0), dv = b < 0 ? -1 : (b > 1 ? 1 : 0);
  return c[pos * ps + dv * pitch + du];
}

// f minus the off-centre part of the operator at position k.
template <typename T, typename Q>
__device__ __forceinline__ T quad_defect(const Q &q, const T *c, int k, int ps, int pitch) {
  const T sw = quad_nb(q.x, c, k, -1, -1, ps, pitch), s = quad_nb(q.x, c, k, 0, -1, ps, pitch);
  const T se = quad_nb(q.x, c, k, 1, -1, ps, pitch), w = quad_nb(q.x, c, k, -1, 0, ps, pitch);
  const T e = quad_nb(q.x, c, k, 1, 0, ps, pitch), nw = quad_nb(q.x, c, k, -1, 1, ps, pitch);
  const T n = quad_nb(q.x, c, k, 0, 1, ps, pitch), ne = quad_nb(q.x, c, k, 1, 1, ps, pitch);
  if constexpr (std::is_same<Q, QuadSt<T>>::value)
    return defect9(q.f[k], q.a[k], sw, s, se, w, e, nw, n, ne);
  else
    return defect18(q.f[k], q.k1[k], q.k3[k], q.k4[k], q.k5[k], q.k6[k], sw, s, se, w, e, nw, n,
                    ne);
}
template <typename T>
__device__ __forceinline__ T quad_diag(const QuadSt<T> &q, int k) { return q.a[k][4]; }
template <typename T>
__device__ __forceinline__ T quad_diag(const QuadEps<T> &q, int k) { return q.dg[k]; }

// One colour phase: the node at position k, in registers and in LDS.
template <typename T, typename Q>
__device__ __forceinline__ void quad_relax(Q &q, T *c, int k, int ps, int pitch) {
  if (q.ik[k] != T(0)) {
    q.x[k] = relaxed(quad_defect<T>(q, c, k, ps, pitch), q.ik[k]);
    c[k * ps] = q.x[k];
  }
}

// Residual at position k, 0 where the node is not relaxed.
template <typename T, typename Q>
__device__ __forceinline__ T quad_resid(const Q &q, const T *c, int k, int ps, int pitch) {
  if (q.ik[k] == T(0)) return T(0);
  return residual_of(quad_defect<T>(q, c, k, ps, pitch), quad_diag(q, k), q.x[k]);
}

// Full weighting of the residuals around position kc of the thread's quad
// (res: its own; cr: its entry of the residual planes).
template <typename T>
__device__ __forceinline__ T quad_full_weight(const T (&res)[4], const T *cr, int kc, int ps,
                                              int pitch) {
  T col[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const T lo = quad_nb(res, cr, kc, d - 1, -1, ps, pitch);
    const T mid = quad_nb(res, cr, kc, d - 1, 0, ps, pitch);
    const T hi = quad_nb(res, cr, kc, d - 1, 1, ps, pitch);
    col[d] = lo + T(2) * mid + hi;
  }
  return (col[0] + T(2) * col[1] + col[2]) * T(0.0625);
}

// ---- tiles and bands of a launch -------------------------------------------

// Odd bands march down: then two neighbouring bands reach their common
// boundary at the same time -- at the start of the pass for one pair, at its
// end for the other -- and the halo rows both read are served by the cache
// instead of being fetched from memory twice.  FP64 passes only: the FP32
// passes move half the bytes and gain nothing from it.
template <typename T>
__device__ __forceinline__ bool mirrored(int by, int ny) {
  return std::is_same<T, double>::value && (by & 1) && (ny & 1);
}

// Tile of a block of a one-dimensional launch.  Workgroups go to the eight
// XCDs in turn (XCD = linear id mod 8); each XCD is given one contiguous run
// of tiles in strip-fastest order, so the neighbouring strips of a band --
// which read each other's halo columns at about the same time -- share that
// XCD's L2 instead of fetching the halo twice from memory.
__device__ __forceinline__ void xcd_tile(int id, int nbx, int nby, int &bx, int &by) {
  const int n = nbx * nby, per = n >> 3, rem = n & 7;
  const int xcd = id & 7, q = id >> 3;
  const int tile = xcd * per + min(xcd, rem) + q;
  bx = tile % nbx;
  by = tile / nbx;
}

// Entry of a batched launch holding block b (entries sorted by start).
__device__ __forceinline__ const BatchEntry &batch_locate(const BatchTab &tab, int b) {
  int lo = 0, hi = tab.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab.e[mid].start <= b) lo = mid; else hi = mid - 1;
  }
  return tab.e[lo];
}
// A value that is the same in every lane, in scalar registers.
template <typename S>
__device__ __forceinline__ S scalar(const S &s) {
  static_assert(sizeof(S) % 4 == 0, "whole words");
  struct W {
    int w[sizeof(S) / 4];
  };
  W x = __builtin_bit_cast(W, s);
#pragma unroll
  for (unsigned k = 0; k < sizeof(S) / 4; ++k) x.w[k] = __builtin_amdgcn_readfirstlane(x.w[k]);
  return __builtin_bit_cast(S, x);
}
// The pass arguments of a batched launch's block and its place among its
// problem's blocks, with the level-0 iterate of this solve.  In scalar
// registers, as a kernel's own arguments are: the compiler takes what it
// loads through the table for different in every lane, and the row addresses
// and bounds of the marching passes then cost vector registers and
// arithmetic (256 problems of sides 65 .. 1025, FP64 32.4 -> 27.6 ms, mixed
// precision 23.3 -> 21.1; a burst of 24 requests 13.9 -> 12.8 ms).
template <typename T>
__device__ __forceinline__ PassArgs<T> batch_args(const BatchTab &tab, int &bx, int &by) {
  const BatchEntry &e = batch_locate(tab, blockIdx.x);
  PassArgs<T> a = *static_cast<const PassArgs<T> *>(e.args);
  if (e.role == 1) a.xin = static_cast<const T *>(e.phi);
  if (e.role == 2) a.xout = static_cast<T *>(e.phi);
  const int local = __builtin_amdgcn_readfirstlane((int)blockIdx.x - e.start);
  const int nbx = __builtin_amdgcn_readfirstlane(a.nbx);
  bx = local % nbx;
  by = local / nbx;
  return scalar(a);
}

// Two neighbouring elements of a row in one load (rows have no alignment
// beyond that of an element).
template <typename T>
struct PairOf;
template <>
struct PairOf<double> {
  typedef double type __attribute__((ext_vector_type(2), aligned(8)));
};
template <>
struct PairOf<float> {
  typedef float type __attribute__((ext_vector_type(2), aligned(4)));
};
template <typename T>
__device__ __forceinline__ typename PairOf<T>::type load_pair(const T *p) {
  return *reinterpret_cast<const typename PairOf<T>::type *>(p);
}

}  // namespace tomg
