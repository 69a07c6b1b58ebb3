// Passes of the large levels (arXiv 2602.01888, Section 3), with the operator
// formed from the tensor (level 0, eq. 18) or stored: one wave marches up a
// band of rows, two columns per lane.
//
// A lane owns an even and the next odd column, so a step of two rows is one
// node of each colour per lane (quad.h's order without the quad's LDS): no
// lane idles in a colour phase.  The rows in flight -- node values and
// coefficients -- stay in registers, in rings indexed by compile-time slots,
// and a neighbour's value in the next lane comes by a one-lane wave shift
// (DPP), so a block is one wave without a barrier, and LDS holds only what a
// lane keeps for itself.  The passes that kept node values in LDS, one column
// per thread, spent a step's time in eleven barrier phases with half the lanes
// idle.  A pass of 4097^2, those -> this form: FP64 264 -> 200 us upward with
// its norm, 235 -> 195 us downward (856 MB, 4.3 and 4.4 TB/s); FP32 129 -> 115
// and 128 -> 108 us (436 MB, 3.8 and 4.0 TB/s); a batch of 256 problems of sides
// 65 .. 1025, FP64 39.1 -> 34.1 ms, mixed precision 26.7 -> 23.9 ms.  What is
// left is the walk itself: without its arithmetic it takes 180 us in FP64 and
// 107 us in FP32.
// With the stencil stored (nine planes: 2049^2 FP64 is 437 MB a pass) the same:
// the upward pass with its norm 115 -> 96 us, the downward pass 102 -> 97 us
// (4.5 TB/s), 256 problems of mixed precision 21.1 -> 20.3 ms.  Its six rows of
// coefficients take 360 .. 446 of a lane's 512 registers at FP64; the diagonal
// neighbours kept in LDS instead cost a step its LDS reads (107 us).
//
// Row order, colours and arithmetic are those of the other passes (fused.hip):
// at step m sweep s relaxes colours 0 and 1 of row 2m - 2s, then colours 2
// and 3 of row 2m - 2s - 1; the residual follows on rows 2m - 2 nu and the
// next.  A sweep leaves wrong values in four columns and two rows at the low
// edges of the block's region, and in one column and row fewer at the high
// edges (quads start at even nodes): 4 nu + 2 and 4 nu halo columns, 2 nu + 2
// and 2 nu halo rows.
#include <type_traits>

#include "quad.h"
#include "tomg_internal.h"

namespace tomg {
namespace {

// The value of the lane below (above) in the wave; 0 at the wave's end.
__device__ __forceinline__ int lane_below(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ int lane_above(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
template <bool ABOVE, typename T>
__device__ __forceinline__ T shift(T v) {
  if constexpr (sizeof(T) == 4) {
    const int x = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(T, ABOVE ? lane_above(x) : lane_below(x));
  } else {
    struct P {
      int lo, hi;
    };
    P p = __builtin_bit_cast(P, v);
    p.lo = ABOVE ? lane_above(p.lo) : lane_below(p.lo);
    p.hi = ABOVE ? lane_above(p.hi) : lane_below(p.hi);
    return __builtin_bit_cast(T, p);
  }
}
template <typename T>
__device__ __forceinline__ T below(T v) {
  return shift<false>(v);
}
template <typename T>
__device__ __forceinline__ T above(T v) {
  return shift<true>(v);
}

// The scheduler moves nothing across: it would otherwise overlap the phases
// and hold more values than the registers.
__device__ __forceinline__ void phase() { __builtin_amdgcn_sched_barrier(0); }

// One row as loaded: the lane's two columns.
template <typename T, bool ST>
struct Row;
template <typename T>
struct Row<T, false> {
  T x[2], f[2], xx[2], xy[2], yy[2];
  bool d[2];
};
template <typename T>
struct Row<T, true> {
  T x[2], f[2], a[9][2];
  bool d[2];
};
// One row's coefficients in registers.
template <typename T, bool ST>
struct Coef;
template <typename T>
struct Coef<T, false> {
  T k1[2], k3[2], k4[2], k5[2], k6[2], ik[2];
  bool on[2];  // the node is relaxed
};
template <typename T>
struct Coef<T, true> {
  T a[8][2], ik[2];  // S, W, E, N, SW, SE, NW, NE
  bool on[2];
};
// What a lane keeps in LDS for itself (no other lane reads it, so nothing is
// synchronised): values of the rows in flight that are read only now and
// then and would not fit the registers beside the rings.
template <typename T, int NS, bool ST>
struct Own {
  typedef T V2 __attribute__((ext_vector_type(2)));
  V2 f[NS][64], dg[NS][64];         // right-hand side and diagonal
  V2 xx[64], xy[2][64], yy[2][64];  // tensor of rows 2m-2 (xy, yy) and 2m-1
};
template <typename T, int NS>
struct Own<T, NS, true> {
  typedef T V2 __attribute__((ext_vector_type(2)));
  V2 f[NS][64], dg[NS][64];
};

template <typename T, bool ST, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, bool MIR>
__device__ __forceinline__ void march_body(const PassArgs<T> &a, const int bx, const int by) {
  constexpr int HL = 4 * NU + 2;
  // rows 2m+1 .. 2m-2nu are in flight in step m, and the value of the row below
  constexpr int NS = 2 * NU + 2, PER = NS / 2;  // ring slots; steps until they repeat
  typedef typename PairOf<T>::type Pair;
  __shared__ Own<T, NS, ST> own;
  typedef typename Own<T, NS, ST>::V2 V2;
  const int nx = a.nx, ny = a.ny;
  const int lane = threadIdx.x;
  const int x0 = bx * a.W;
  const int i0 = x0 - HL + 2 * lane;
  // Pairs are loaded from ib: never past the row.  Only the strip at the
  // grid's high edge has a lane whose pair starts one column early (last).
  const unsigned ib = (unsigned)min(max(i0, 0), nx - 2);
  const bool last = i0 == nx - 1, edge = x0 - HL + 127 >= nx - 1;
  const bool in0 = i0 >= 0 && i0 < nx, in1 = i0 + 1 >= 0 && i0 + 1 < nx;
  const bool out = lane >= HL / 2 && 2 * lane < HL + a.W && in0;
  const unsigned Ib = (unsigned)min(max(i0 >> 1, 0), a.nxc - 2);
  const size_t n = (size_t)nx * ny;
  (void)n;
  // MIR: the block marches down its band in flipped row coordinates (row r
  // is grid row ny-1-r; ny is odd, so parities and colours stay) and sums in
  // the order of the upward march
  const int ya = by * a.CH, yb = min(ny, ya + a.CH);
  const int y0 = MIR ? ny - yb : ya, y1 = MIR ? ny - ya : yb;
  const int ys = max(0, (y0 - (2 * NU + 1)) & ~1);
  const int ye = min(ny - 1, ((y1 - 1) | 1) + 2 * NU);
  // rows relaxed: those with both neighbours loaded, and the grid's edges
  // (Dirichlet, or free rows whose outer coefficients are zero)
  const int rlo = ys == 0 ? 0 : ys + 1, rn = (ye == ny - 1 ? ye : ye - 1) - rlo;
  const int m0 = ys >> 1;

  auto row_on = [&](int r) { return (unsigned)(r - rlo) <= (unsigned)rn; };

  // Nodes outside the grid hold whatever their clamped loads gave: none is
  // relaxed, and only nodes of the grid's edge have such neighbours, which
  // are not relaxed either (Dirichlet) or have zero coefficients there.
  auto load_row = [&](int r, Row<T, ST> &w) {
    const int rc = min(r, ny - 1);
    const size_t at = (size_t)(MIR ? ny - 1 - rc : rc) * nx;
    auto get = [&](const T *p, T(&v)[2]) {
      const Pair q = load_pair(p + at + ib);
      v[0] = q[0];
      v[1] = q[1];
    };
    if constexpr (!ZERO) get(a.xin, w.x);
    get(a.b, w.f);
    if constexpr (ST) {
#pragma unroll
      for (int z = 0; z < 9; ++z) get(a.st + z * n, w.a[z]);
    } else {
      get(a.exx, w.xx);
      get(a.exy, w.xy);
      get(a.eyy, w.yy);
    }
    const uint8_t *d = a.dir + at + ib;
    w.d[0] = d[0] != 0;
    w.d[1] = d[1] != 0;
  };
  auto fix_last = [&](Row<T, ST> &w) {
    if (!edge) return;
    if constexpr (!ZERO) w.x[0] = last ? w.x[1] : w.x[0];
    w.f[0] = last ? w.f[1] : w.f[0];
    if constexpr (ST) {
#pragma unroll
      for (int z = 0; z < 9; ++z) w.a[z][0] = last ? w.a[z][1] : w.a[z][0];
    } else {
      w.xx[0] = last ? w.xx[1] : w.xx[0];
      w.xy[0] = last ? w.xy[1] : w.xy[0];
      w.yy[0] = last ? w.yy[1] : w.yy[0];
    }
    w.d[0] = last ? w.d[1] : w.d[0];
  };
  auto load_coarse = [&](int J, T (&v)[2]) {  // coarse row J (flipped with the rows)
    const int j = min(J, a.nyc - 1);
    const Pair q = load_pair(a.xc + (size_t)(MIR ? a.nyc - 1 - j : j) * a.nxc + Ib);
    // (column nx-1 is Dirichlet without a stored stencil: its pair is not used)
    v[0] = ST && last ? q[1] : q[0];
    v[1] = q[1];
  };
  // value of a loaded row, with the correction of the coarse rows under row
  // r & ~1 (lo) and above it (hi)
  auto commit = [&](int q, const Row<T, ST> &w, const T (&lo)[2], const T (&hi)[2], T (&v)[2]) {
    v[0] = ZERO ? T(0) : w.x[0];
    v[1] = ZERO ? T(0) : w.x[1];
    if constexpr (PROLONG) {
      T e0 = lo[0], e1 = T(0.5) * (lo[0] + lo[1]);
      if (q) {
        e0 = T(0.5) * (e0 + hi[0]);
        e1 = T(0.5) * (e1 + T(0.5) * (hi[0] + hi[1]));
      }
      v[0] = w.d[0] ? v[0] : v[0] + e0;
      v[1] = w.d[1] ? v[1] : v[1] + e1;
    }
  };

  T V[NS][2], vb[2] = {T(0), T(0)};  // vb: row 2m-2nu-1
  Coef<T, ST> C[NS];
  auto slot = [](int rel) { return ((rel % NS) + NS) % NS; };
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      V[s][k] = T(0);
      if constexpr (ST) {
#pragma unroll
        for (int z = 0; z < 8; ++z) C[s].a[z][k] = T(0);
      } else {
        C[s].k1[k] = C[s].k3[k] = C[s].k4[k] = C[s].k5[k] = C[s].k6[k] = T(0);
      }
      C[s].ik[k] = T(0);
      C[s].on[k] = false;
    }
    own.f[s][lane] = own.dg[s][lane] = V2{T(0), T(0)};
  }
  if constexpr (!ST)
    own.xx[lane] = own.xy[0][lane] = own.xy[1][lane] = own.yy[0][lane] = own.yy[1][lane] =
        V2{T(0), T(0)};
  // a loaded row r into its ring slot s: right-hand side and, when stored, the stencil
  auto enter = [&](int r, int s, const Row<T, ST> &w) {
    own.f[s][lane] = V2{w.f[0], w.f[1]};
    if constexpr (ST) {
      constexpr int kOrder[8] = {1, 3, 5, 7, 0, 2, 6, 8};
      const bool ok = row_on(r);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int z = 0; z < 8; ++z) C[s].a[z][k] = w.a[kOrder[z]][k];
        C[s].ik[k] = T(1) / w.a[4][k];
        C[s].on[k] = ok && !w.d[k] && (k ? in1 : in0);
      }
      own.dg[s][lane] = V2{w.a[4][0], w.a[4][1]};
    }
  };
  bool pd0 = true, pd1 = true;  // Dirichlet flags of row 2m-1
  T rprev[2] = {T(0), T(0)};
  double acc = 0.0;
  Row<T, ST> cur[2], nxt[2];
  T c0[2] = {T(0), T(0)}, c1[2] = {T(0), T(0)}, c2[2] = {T(0), T(0)};  // coarse rows m .. m+2
  load_row(2 * m0, cur[0]);
  load_row(2 * m0 + 1, cur[1]);
  if constexpr (PROLONG) {
    load_coarse(m0, c0);
    load_coarse(m0 + 1, c1);
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    fix_last(cur[q]);
    commit(q, cur[q], c0, c1, V[slot(q)]);
    enter(2 * m0 + q, slot(q), cur[q]);
  }

  for (int sb = 0;; sb += PER) {
#pragma unroll
    for (int ph = 0; ph < PER; ++ph) {
      const int m = m0 + sb + ph;
      const int R0 = 2 * (m - NU);  // first row of the residual pair
      if (R0 > y1 - 1) goto done;
      {
        const int rel0 = 2 * ph;  // ring position of row 2m
        if constexpr (!ST) {  // coefficients of rows 2m-1 (v = 0) and 2m (v = 1)
          const V2 pxx = own.xx[lane], pxy = own.xy[1][lane], pyy = own.yy[1][lane];
          const V2 qxy = own.xy[0][lane], qyy = own.yy[0][lane];
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            Coef<T, ST> &c = C[slot(rel0 - 1 + v)];
            const bool rowok = row_on(2 * m - 1 + v);
            const T xx[2] = {v ? cur[0].xx[0] : pxx[0], v ? cur[0].xx[1] : pxx[1]};
            const T xy[2] = {v ? cur[0].xy[0] : pxy[0], v ? cur[0].xy[1] : pxy[1]};
            const T yy[2] = {v ? cur[0].yy[0] : pyy[0], v ? cur[0].yy[1] : pyy[1]};
            const T dxx[2] = {xx[1] - below(xx[1]), above(xx[0]) - xx[0]};
            const T dxy[2] = {xy[1] - below(xy[1]), above(xy[0]) - xy[0]};
            V2 dg;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const T lyy = v ? pyy[k] : qyy[k], lxy = v ? pxy[k] : qxy[k];
              const T hyy = v ? cur[1].yy[k] : cur[0].yy[k], hxy = v ? cur[1].xy[k] : cur[0].xy[k];
              const T ax = xx[k] * a.cx, ay = yy[k] * a.cy;
              T gx, gy;
              eps_coefs(dxx[k], MIR ? lyy - hyy : hyy - lyy, dxy[k], MIR ? lxy - hxy : hxy - lxy,
                        a.qx, a.qy, a.qxy, gx, gy);
              c.k1[k] = plain_add(ax, gx);
              c.k3[k] = plain_add(ax, -gx);
              c.k4[k] = plain_add(ay, gy);
              c.k5[k] = plain_add(ay, -gy);
              c.k6[k] = xy[k] * a.hxy;
              dg[k] = eps_diag(ax, ay);
              c.ik[k] = T(1) / dg[k];
              c.on[k] = rowok && !(v ? cur[0].d[k] : (k ? pd1 : pd0)) && (k ? in1 : in0);
            }
            own.dg[slot(rel0 + v - 1)][lane] = dg;
          }
          // rows 2m and 2m+1 are the carried rows of the next step
          own.xy[0][lane] = V2{cur[0].xy[0], cur[0].xy[1]};
          own.yy[0][lane] = V2{cur[0].yy[0], cur[0].yy[1]};
          own.xx[lane] = V2{cur[1].xx[0], cur[1].xx[1]};
          own.xy[1][lane] = V2{cur[1].xy[0], cur[1].xy[1]};
          own.yy[1][lane] = V2{cur[1].yy[0], cur[1].yy[1]};
          pd0 = cur[1].d[0];
          pd1 = cur[1].d[1];
        }
        phase();
        load_row(2 * m + 2, nxt[0]);
        load_row(2 * m + 3, nxt[1]);
        if constexpr (PROLONG) load_coarse(m + 2, c2);
        phase();
        // f minus the off-centre part of node (row 2m + o, column k)
        auto node_defect = [&](int o, int k, T f) -> T {
          const Coef<T, ST> &c = C[slot(rel0 + o)];
          const T(&mid)[2] = V[slot(rel0 + o)];
          const T(&dn)[2] = o == -2 * NU ? vb : V[slot(rel0 + o - 1)];
          const T(&up)[2] = V[slot(rel0 + o + 1)];
          const T(&lo)[2] = MIR ? up : dn;
          const T(&hi)[2] = MIR ? dn : up;
          const T sw = k ? lo[0] : below(lo[1]), se = k ? above(lo[0]) : lo[1];
          const T ww = k ? mid[0] : below(mid[1]), ee = k ? above(mid[0]) : mid[1];
          const T nw = k ? hi[0] : below(hi[1]), ne = k ? above(hi[0]) : hi[1];
          if constexpr (ST) {
            const T a9[9] = {c.a[4][k], c.a[0][k], c.a[5][k], c.a[1][k], T(0),
                             c.a[2][k], c.a[6][k], c.a[3][k], c.a[7][k]};
            return defect9(f, a9, sw, lo[k], se, ww, ee, nw, hi[k], ne);
          } else {
            return defect18(f, c.k1[k], c.k3[k], c.k4[k], c.k5[k], c.k6[k], sw, lo[k], se, ww,
                            ee, nw, hi[k], ne);
          }
        };
#pragma unroll
        for (int s = 0; s < NU; ++s)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int o = -2 * s - half;
            const V2 f = own.f[slot(rel0 + o)][lane];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const Coef<T, ST> &c = C[slot(rel0 + o)];
              const T v = relaxed(node_defect(o, k, f[k]), c.ik[k]);
              T &x = V[slot(rel0 + o)][k];
              x = c.on[k] ? v : x;
            }
            phase();
          }
        // ------------- residual, output, restriction, norm -------------
        T res[2][2] = {{T(0), T(0)}, {T(0), T(0)}};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = R0 + q, o = q - 2 * NU;
          const T(&mid)[2] = V[slot(rel0 + o)];
          const bool band = (unsigned)(r - y0) < (unsigned)(y1 - y0);
          if constexpr (RESTRICT || NORM) {
            const Coef<T, ST> &c = C[slot(rel0 + o)];
            const V2 f = own.f[slot(rel0 + o)][lane], dg = own.dg[slot(rel0 + o)][lane];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const T v = residual_of(node_defect(o, k, f[k]), dg[k], mid[k]);
              res[q][k] = c.on[k] ? v : T(0);
            }
            phase();
          }
          if (band && out) {
            T *p = a.xout + (size_t)(MIR ? ny - 1 - r : r) * nx + (unsigned)i0;
            if (in1) {
              Pair v;
              v[0] = mid[0];
              v[1] = mid[1];
              __builtin_nontemporal_store(v, reinterpret_cast<Pair *>(p));
            } else {
              __builtin_nontemporal_store(mid[0], p);
            }
            // (a node outside the grid is not relaxed: its residual is 0)
            if constexpr (NORM)
              acc += (double)(res[q][0] * res[q][0]) + (double)(res[q][1] * res[q][1]);
          }
        }
        if constexpr (RESTRICT) {
          T s[2];  // grid rows 2J-1, 2J, 2J+1 in that order
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            s[k] = MIR ? res[1][k] + T(2) * res[0][k] + rprev[k]
                       : rprev[k] + T(2) * res[0][k] + res[1][k];
            rprev[k] = res[1][k];
          }
          const T w = below(s[1]);
          const int J = R0 >> 1;
          if ((unsigned)(R0 - y0) < (unsigned)(y1 - y0) && out) {
            const int I = i0 >> 1, Jg = MIR ? a.nyc - 1 - J : J;
            // a coarse ring node is Dirichlet unless its edge is Neumann
            bool fixed = I == 0 || Jg == 0 || I == a.nxc - 1 || Jg == a.nyc - 1;
            if constexpr (ST) fixed = fixed && (!a.dirc || a.dirc[(size_t)Jg * a.nxc + I]);
            const T v = (w + T(2) * s[0] + s[1]) * T(0.0625);
            __builtin_nontemporal_store(fixed ? T(0) : v, a.bc + (size_t)Jg * a.nxc + (unsigned)I);
          }
        }
        phase();
        // the loaded rows take the slots of rows 2m-2nu and the next, which
        // stays as the row below the next residual
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          vb[k] = V[slot(rel0 + 1 - 2 * NU)][k];
          c0[k] = c1[k];
          c1[k] = c2[k];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          fix_last(nxt[q]);
          commit(q, nxt[q], c0, c1, V[slot(rel0 + 2 + q)]);
          enter(2 * m + 2 + q, slot(rel0 + 2 + q), nxt[q]);
          if constexpr (!ST) cur[q] = nxt[q];
        }
      }
    }
  }
done:
  if constexpr (NORM) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) a.partials[(size_t)by * a.nbx + bx] = acc;
  }
}

// Waves per SIMD: what the registers in flight allow.  From the tensor FP64
// takes 256 VGPRs and 20 .. 30 of the accumulation file, FP32 140 .. 150; held
// to two waves FP64 spills to scratch (a 4097^2 cycle 825 against 752 us), as
// does FP32 at four (two cycles and their refinement step 1408 against 1131
// us).  With a stored stencil it is up to 446 and 219 registers: one wave and two.
template <typename T, bool ST>
constexpr int march_waves() {
  return sizeof(T) == 8 ? 1 : (ST ? 2 : 3);
}
template <typename T, bool ST, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
__global__ __launch_bounds__(64, (march_waves<T, ST>())) void k_march(PassArgs<T> a) {
  if (a.skip && *a.skip != 0.0) return;
  int bx = blockIdx.x, by = blockIdx.y;
  if (a.xcd_order) xcd_tile(blockIdx.x, a.nbx, a.nby, bx, by);
  if (mirrored<T>(by, a.ny))
    march_body<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM, true>(a, bx, by);
  else
    march_body<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM, false>(a, bx, by);
}
template <typename T, bool ST, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
__global__ __launch_bounds__(64, (march_waves<T, ST>())) void k_march_b(BatchTab tab) {
  int bx, by;
  const PassArgs<T> a = batch_args<T>(tab, bx, by);
  if (mirrored<T>(by, a.ny))
    march_body<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM, true>(a, bx, by);
  else
    march_body<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM, false>(a, bx, by);
}

template <typename T, bool ST, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
void launch(const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (tab)
    hipLaunchKernelGGL((k_march_b<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM>), nb, 64, 0, s, *tab);
  else
    hipLaunchKernelGGL((k_march<T, ST, NU, ZERO, PROLONG, RESTRICT, NORM>),
                       a.xcd_order ? dim3(a.nbx * a.nby) : dim3(a.nbx, a.nby), 64, 0, s, a);
}
template <typename T, bool ST, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
void launch_nu(int nu, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (nu == 1)
    launch<T, ST, 1, ZERO, PROLONG, RESTRICT, NORM>(a, s, tab, nb);
  else
    launch<T, ST, 2, ZERO, PROLONG, RESTRICT, NORM>(a, s, tab, nb);
}

}  // namespace

// Gives a pass the marching form: both axes halved, at most two sweeps.  (From
// the tensor a sweep more takes some 95 registers in FP64 and 50 in FP32, with a
// stored stencil 120 .. 145 and 55: by that count only stored FP64 passes of
// three and four would not fit a wave's 512.  None are built or measured.)
template <typename T>
bool pick_march(PassArgs<T> &a, int nu, bool batch) {
  if (nu > 2 || a.ck != 0) return false;
  a.form = kFormMarch;
  a.bw = 64;
  a.W = 128 - (8 * nu + 2);
  if (batch) {
    a.CH = pick_band_batch(a.ny);
  } else {
    // As many one-wave blocks as the four SIMDs of every CU hold: half of them
    // on twice as tall bands, with fewer halo rows, leave SIMDs idle (stored
    // 2049^2 FP64 112 / 100 against 97 / 96 us, a 4097^2 cycle 760 against 741).
    static const int cus = device_cus();
    const int waves = 4 * (a.st ? march_waves<T, true>() : march_waves<T, false>());
    a.CH = pick_band(a.nx, a.ny, a.W, (long)waves * cus, 2 * nu + 3);
  }
  a.nbx = (a.nx + a.W - 1) / a.W;
  a.nby = (a.ny + a.CH - 1) / a.CH;
  a.xcd_order = !batch && a.nbx > 1 ? 1 : 0;
  return true;
}
template bool pick_march<double>(PassArgs<double> &, int, bool);
template bool pick_march<float>(PassArgs<float> &, int, bool);

template <typename T>
void march_down(int nu, bool eps, bool zero, const PassArgs<T> &a, hipStream_t s,
                const BatchTab *tab, int nb) {
  if (eps) {
    if (zero) launch_nu<T, false, true, false, true, false>(nu, a, s, tab, nb);
    else launch_nu<T, false, false, false, true, false>(nu, a, s, tab, nb);
  } else {
    if (zero) launch_nu<T, true, true, false, true, false>(nu, a, s, tab, nb);
    else launch_nu<T, true, false, false, true, false>(nu, a, s, tab, nb);
  }
}
template <typename T>
void march_up(int nu, bool eps, bool norm, const PassArgs<T> &a, hipStream_t s,
              const BatchTab *tab, int nb) {
  if (eps) {
    if (norm) launch_nu<T, false, false, true, false, true>(nu, a, s, tab, nb);
    else launch_nu<T, false, false, true, false, false>(nu, a, s, tab, nb);
  } else {
    if (norm) launch_nu<T, true, false, true, false, true>(nu, a, s, tab, nb);
    else launch_nu<T, true, false, true, false, false>(nu, a, s, tab, nb);
  }
}
template void march_down<double>(int, bool, bool, const PassArgs<double> &, hipStream_t,
                                 const BatchTab *, int);
template void march_down<float>(int, bool, bool, const PassArgs<float> &, hipStream_t,
                                const BatchTab *, int);
template void march_up<double>(int, bool, bool, const PassArgs<double> &, hipStream_t,
                               const BatchTab *, int);
template void march_up<float>(int, bool, bool, const PassArgs<float> &, hipStream_t,
                              const BatchTab *, int);

}  // namespace tomg
