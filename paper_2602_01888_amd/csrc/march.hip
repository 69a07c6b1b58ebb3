// Level-0 passes of the large levels, operator formed from the tensor
// (arXiv 2602.01888, Section 3; eq. 18): one wave marches up a band of rows,
// two columns per lane.
//
// A lane owns an even and the next odd column, so a step of two rows is one
// node of each colour per lane (quad.h's order without the quad's LDS): no
// lane idles in a colour phase.  The rows in flight -- node values and
// coefficients -- stay in registers, in rings indexed by compile-time slots,
// and a neighbour's value in the next lane comes by a one-lane wave shift
// (DPP), so a block is one wave with no LDS and no barrier.  The passes that
// kept node values in LDS, one column per thread, spent a step's time in
// eleven barrier phases with half the lanes idle.  A pass of 4097^2, those ->
// this form: FP64 239 -> 181 us (856 MB, 3.6 -> 4.7 TB/s), FP32 129 -> 105 us
// (3.4 -> 4.1 TB/s); of a batch of 256 problems of sides 65 .. 1025, FP64 39.1
// -> 34.1 ms, mixed precision 26.7 -> 23.9 ms.  What is left is the walk
// itself: a copy of the same bands streams 4.3 .. 4.7 TB/s.
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

template <typename T>
struct Row {  // one row as loaded: the lane's two columns
  T x[2], f[2], xx[2], xy[2], yy[2];
  bool d[2];
};
template <typename T>
struct Coef {  // one row's coefficients
  T k1[2], k3[2], k4[2], k5[2], k6[2], ik[2];
  bool on[2];  // the node is relaxed
};
// What a lane keeps in LDS for itself (no other lane reads it, so nothing is
// synchronised): values of the rows in flight that are read only now and
// then and would not fit the registers beside the rings.
template <typename T, int NS>
struct Own {
  typedef T V2 __attribute__((ext_vector_type(2)));
  V2 f[NS][64], dg[NS][64];         // right-hand side and diagonal
  V2 xx[64], xy[2][64], yy[2][64];  // tensor of rows 2m-2 (xy, yy) and 2m-1
};

template <typename T, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM, bool MIR>
__device__ __forceinline__ void march_body(const PassArgs<T> &a, const int bx, const int by) {
  constexpr int HL = 4 * NU + 2;
  // rows 2m+1 .. 2m-2nu are in flight in step m, and the value of the row below
  constexpr int NS = 2 * NU + 2, PER = NS / 2;  // ring slots; steps until they repeat
  typedef typename PairOf<T>::type Pair;
  __shared__ Own<T, NS> own;
  typedef typename Own<T, NS>::V2 V2;
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
  // MIR: the block marches down its band in flipped row coordinates (row r
  // is grid row ny-1-r; ny is odd, so parities and colours stay) and sums in
  // the order of the upward march
  const int ya = by * a.CH, yb = min(ny, ya + a.CH);
  const int y0 = MIR ? ny - yb : ya, y1 = MIR ? ny - ya : yb;
  const int ys = max(0, (y0 - (2 * NU + 1)) & ~1);
  const int ye = min(ny - 1, ((y1 - 1) | 1) + 2 * NU);
  // rows relaxed: those with both neighbours loaded, and the grid's edges
  // (Dirichlet rows: nothing there is relaxed)
  const int rlo = ys == 0 ? 0 : ys + 1, rn = (ye == ny - 1 ? ye : ye - 1) - rlo;
  const int m0 = ys >> 1;

  // Nodes outside the grid hold whatever their clamped loads gave: none is
  // relaxed, and only Dirichlet nodes, which are not relaxed either, have
  // such neighbours.
  auto load_row = [&](int r, Row<T> &w) {
    const int rc = min(r, ny - 1);
    const size_t at = (size_t)(MIR ? ny - 1 - rc : rc) * nx;
    auto get = [&](const T *p, T(&v)[2]) {
      const Pair q = load_pair(p + at + ib);
      v[0] = q[0];
      v[1] = q[1];
    };
    if constexpr (!ZERO) get(a.xin, w.x);
    get(a.b, w.f);
    get(a.exx, w.xx);
    get(a.exy, w.xy);
    get(a.eyy, w.yy);
    const uint8_t *d = a.dir + at + ib;
    w.d[0] = d[0] != 0;
    w.d[1] = d[1] != 0;
  };
  auto fix_last = [&](Row<T> &w) {
    if (!edge) return;
    if constexpr (!ZERO) w.x[0] = last ? w.x[1] : w.x[0];
    w.f[0] = last ? w.f[1] : w.f[0];
    w.xx[0] = last ? w.xx[1] : w.xx[0];
    w.xy[0] = last ? w.xy[1] : w.xy[0];
    w.yy[0] = last ? w.yy[1] : w.yy[0];
    w.d[0] = last ? w.d[1] : w.d[0];
  };
  auto load_coarse = [&](int J, T (&v)[2]) {  // coarse row J (flipped with the rows)
    const int j = min(J, a.nyc - 1);
    const Pair q = load_pair(a.xc + (size_t)(MIR ? a.nyc - 1 - j : j) * a.nxc + Ib);
    v[0] = q[0];  // (column nx-1 is Dirichlet: its lane's pair is not used)
    v[1] = q[1];
  };
  // value of a loaded row, with the correction of the coarse rows under row
  // r & ~1 (lo) and above it (hi)
  auto commit = [&](int q, const Row<T> &w, const T (&lo)[2], const T (&hi)[2], T (&v)[2]) {
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
  Coef<T> C[NS];
  auto slot = [](int rel) { return ((rel % NS) + NS) % NS; };
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      V[s][k] = T(0);
      C[s].k1[k] = C[s].k3[k] = C[s].k4[k] = C[s].k5[k] = C[s].k6[k] = C[s].ik[k] = T(0);
      C[s].on[k] = false;
    }
    own.f[s][lane] = own.dg[s][lane] = V2{T(0), T(0)};
  }
  own.xx[lane] = own.xy[0][lane] = own.xy[1][lane] = own.yy[0][lane] = own.yy[1][lane] =
      V2{T(0), T(0)};
  bool pd0 = true, pd1 = true;  // Dirichlet flags of row 2m-1
  T rprev[2] = {T(0), T(0)};
  double acc = 0.0;
  Row<T> cur[2], nxt[2];
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
    own.f[slot(q)][lane] = V2{cur[q].f[0], cur[q].f[1]};
  }

  for (int sb = 0;; sb += PER) {
#pragma unroll
    for (int ph = 0; ph < PER; ++ph) {
      const int m = m0 + sb + ph;
      const int R0 = 2 * (m - NU);  // first row of the residual pair
      if (R0 > y1 - 1) goto done;
      {
        const int rel0 = 2 * ph;  // ring position of row 2m
        // coefficients of rows 2m-1 (v = 0) and 2m (v = 1)
        {
          const V2 pxx = own.xx[lane], pxy = own.xy[1][lane], pyy = own.yy[1][lane];
          const V2 qxy = own.xy[0][lane], qyy = own.yy[0][lane];
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            Coef<T> &c = C[slot(rel0 - 1 + v)];
            const bool rowok = (unsigned)(2 * m - 1 + v - rlo) <= (unsigned)rn;
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
        // f minus the off-centre part at column k of row 2m + o
        auto node_defect = [&](int o, int k, T f) -> T {
          const Coef<T> &c = C[slot(rel0 + o)];
          const T(&mid)[2] = V[slot(rel0 + o)];
          const T(&dn)[2] = o == -2 * NU ? vb : V[slot(rel0 + o - 1)];
          const T(&up)[2] = V[slot(rel0 + o + 1)];
          const T(&lo)[2] = MIR ? up : dn;
          const T(&hi)[2] = MIR ? dn : up;
          if (k == 0)
            return defect18(f, c.k1[0], c.k3[0], c.k4[0], c.k5[0], c.k6[0], below(lo[1]), lo[0],
                            lo[1], below(mid[1]), mid[1], below(hi[1]), hi[0], hi[1]);
          return defect18(f, c.k1[1], c.k3[1], c.k4[1], c.k5[1], c.k6[1], lo[0], lo[1],
                          above(lo[0]), mid[0], above(mid[0]), hi[0], hi[1], above(hi[0]));
        };
#pragma unroll
        for (int s = 0; s < NU; ++s)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int o = -2 * s - half;
            const V2 f = own.f[slot(rel0 + o)][lane];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const Coef<T> &c = C[slot(rel0 + o)];
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
            const Coef<T> &c = C[slot(rel0 + o)];
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
            // the coarse ring is Dirichlet
            const bool ring = I == 0 || Jg == 0 || I == a.nxc - 1 || Jg == a.nyc - 1;
            const T v = (w + T(2) * s[0] + s[1]) * T(0.0625);
            __builtin_nontemporal_store(ring ? T(0) : v, a.bc + (size_t)Jg * a.nxc + (unsigned)I);
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
          own.f[slot(rel0 + 2 + q)][lane] = V2{nxt[q].f[0], nxt[q].f[1]};
          cur[q] = nxt[q];
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

// One wave of FP64 per SIMD, three of FP32: what the registers in flight
// allow (FP64 256 VGPRs and 20 .. 30 of the accumulation file; FP32 140 .. 150).
// Held to two waves, FP64 spills to scratch: a 4097^2 cycle 825 against 752
// us; FP32 at four 1408 against 1131 us (a refinement step of two cycles).
template <typename T, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
__global__ __launch_bounds__(64, sizeof(T) == 8 ? 1 : 3) void k_march(PassArgs<T> a) {
  if (a.skip && *a.skip != 0.0) return;
  int bx = blockIdx.x, by = blockIdx.y;
  if (a.xcd_order) xcd_tile(blockIdx.x, a.nbx, a.nby, bx, by);
  if (mirrored<T>(by, a.ny))
    march_body<T, NU, ZERO, PROLONG, RESTRICT, NORM, true>(a, bx, by);
  else
    march_body<T, NU, ZERO, PROLONG, RESTRICT, NORM, false>(a, bx, by);
}
template <typename T, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
__global__ __launch_bounds__(64, sizeof(T) == 8 ? 1 : 3) void k_march_b(BatchTab tab) {
  int bx, by;
  const PassArgs<T> a = batch_args<T>(tab, bx, by);
  if (mirrored<T>(by, a.ny))
    march_body<T, NU, ZERO, PROLONG, RESTRICT, NORM, true>(a, bx, by);
  else
    march_body<T, NU, ZERO, PROLONG, RESTRICT, NORM, false>(a, bx, by);
}

template <typename T, int NU, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
void launch(const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (tab)
    hipLaunchKernelGGL((k_march_b<T, NU, ZERO, PROLONG, RESTRICT, NORM>), nb, 64, 0, s, *tab);
  else
    hipLaunchKernelGGL((k_march<T, NU, ZERO, PROLONG, RESTRICT, NORM>),
                       a.xcd_order ? dim3(a.nbx * a.nby) : dim3(a.nbx, a.nby), 64, 0, s, a);
}
template <typename T, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
void launch_nu(int nu, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab, int nb) {
  if (nu == 1)
    launch<T, 1, ZERO, PROLONG, RESTRICT, NORM>(a, s, tab, nb);
  else
    launch<T, 2, ZERO, PROLONG, RESTRICT, NORM>(a, s, tab, nb);
}

// Blocks of a pass that fit on a CU at once.
template <typename T, bool ZERO, bool PROLONG, bool RESTRICT, bool NORM>
int blocks_per_cu(int nu) {
  const void *f = nu == 1
                      ? reinterpret_cast<const void *>(k_march<T, 1, ZERO, PROLONG, RESTRICT, NORM>)
                      : reinterpret_cast<const void *>(k_march<T, 2, ZERO, PROLONG, RESTRICT, NORM>);
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, 64, 0) != hipSuccess || nb < 1) nb = 1;
  return nb;
}

}  // namespace

// Gives a level-0 pass (operator formed from the tensor) the marching form:
// both axes halved, at most two sweeps (three sweeps' rows do not fit the
// registers).
template <typename T>
bool pick_march(PassArgs<T> &a, int nu, bool up, bool batch) {
  if (nu > 2 || a.ck != 0) return false;
  a.form = kFormMarch;
  a.bw = 64;
  a.W = 128 - (8 * nu + 2);
  if (batch) {
    a.CH = pick_band_batch(a.ny);
  } else {
    constexpr bool F64 = std::is_same<T, double>::value;
    const int nb = up ? blocks_per_cu<T, false, true, false, F64>(nu)
                      : blocks_per_cu<T, !F64, false, true, false>(nu);
    static const int cus = device_cus();
    a.CH = pick_band(a.nx, a.ny, a.W, (long)nb * cus, 2 * nu + 3);
  }
  a.nbx = (a.nx + a.W - 1) / a.W;
  a.nby = (a.ny + a.CH - 1) / a.CH;
  a.xcd_order = !batch && a.nbx > 1 ? 1 : 0;
  return true;
}
template bool pick_march<double>(PassArgs<double> &, int, bool, bool);
template bool pick_march<float>(PassArgs<float> &, int, bool, bool);

template <typename T>
void march_down(int nu, bool zero, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab,
                int nb) {
  if (zero) launch_nu<T, true, false, true, false>(nu, a, s, tab, nb);
  else launch_nu<T, false, false, true, false>(nu, a, s, tab, nb);
}
template <typename T>
void march_up(int nu, bool norm, const PassArgs<T> &a, hipStream_t s, const BatchTab *tab,
              int nb) {
  if (norm) launch_nu<T, false, true, false, true>(nu, a, s, tab, nb);
  else launch_nu<T, false, true, false, false>(nu, a, s, tab, nb);
}
template void march_down<double>(int, bool, const PassArgs<double> &, hipStream_t,
                                  const BatchTab *, int);
template void march_down<float>(int, bool, const PassArgs<float> &, hipStream_t,
                                  const BatchTab *, int);
template void march_up<double>(int, bool, const PassArgs<double> &, hipStream_t,
                                  const BatchTab *, int);
template void march_up<float>(int, bool, const PassArgs<float> &, hipStream_t,
                                  const BatchTab *, int);

}  // namespace tomg
