// The smallest levels of the V-cycle in one workgroup (arXiv 2602.01888,
// Section 3).
//
// Below a few thousand nodes per level, a level pass is bound by latency: a
// launch per pass costs more than its work.  One workgroup runs the
// sub-cycle from level lc (zero start, right-hand side from the level above)
// down to the coarsest level and back.
//
// Levels are counted from the coarsest (r = 0).  On every level above the
// coarsest a thread owns at most one 2 x 2 quad of nodes (quad.h): stencils,
// right-hand side and iterate in registers, the iterate mirrored in LDS
// planes, so a colour phase is five LDS reads, nine multiply-adds and one
// LDS write between two barriers, with every lane of an owning wave busy,
// and each stencil is read from memory once per level and cycle.  (With one
// node per thread and the stencil row streamed from L2 in every phase, half
// of the 34 us of a cycle from 33 x 33 was that streaming.)  A level of at
// most 64 quads belongs to one wave, whose phases need no barrier.  Levels
// below the first have their owners in other waves where there are enough
// of them, and keep their stencils too; the 1024-thread form has no
// registers for that and loads the stencils of its lower levels, and the
// first level's again on the way up, when they are needed.
//
// FREE: the outer ring may hold unknowns (Neumann edges; any stored level-0
// stencil).  Then quads start at node 0; otherwise at node 1, so that the
// 63 x 63 inner nodes of a 65 x 65 level are exactly 1024 quads.
// Arithmetic per node is that of the other kernels: four-colour Gauss-Seidel
// on the stored 9-point stencil, full weighting, bilinear prolongation,
// explicit coarsest inverse (staged in LDS).
#include <type_traits>

#include "quad.h"
#include "tomg_internal.h"

namespace tomg {
namespace {

constexpr int kTailWide = 1024, kTailNarrow = 512;  // threads of the two forms
constexpr int kTailMaxNodes = 65 * 65;              // per level
constexpr int kTailLdsMax = 160 * 1024 - 2 * 1024;
constexpr int kRhsThread = 128;  // first thread of the waves idle in the coarsest solve
static_assert(kSmallCoarseNodes <= kRhsThread, "a thread per node of the coarsest level");
static_assert(kMaxCoarseNodes <= kMaxCoarseUnknowns * kMaxCoarseUnknowns,
              "the coarsest solve alone keeps its right-hand side where the inverse is staged");

template <typename T, int NT, bool FREE>
__device__ __forceinline__ void tail_body(const TailArgs<T> &a, const double stop) {
  constexpr int OFF = FREE ? 0 : 1;
  constexpr bool KEEP = NT < kTailWide;  // registers for a lower level's quad beside the first's
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ double bb[kSmallCoarseNodes];
  __shared__ int ci[kSmallCoarseNodes + 1];
  double *cinv = reinterpret_cast<double *>(smem_raw);
  T *S = reinterpret_cast<T *>(cinv + kMaxCoarseUnknowns * kMaxCoarseUnknowns);
  const int t = threadIdx.x;
  const int nl = a.nl;
  auto lvl = [&](int r) -> const TailLevel<T> & { return a.lv[nl - 1 - r]; };
  // position in its quad of the nodes of colour col
  auto pos = [](int col) { return FREE ? col : 3 - col; };

  // the quad of level r that this thread owns (-1: none)
  auto owned = [&](const TailLevel<T> &v) {
    const int q = t - v.t0;
    return q >= 0 && q < v.nq ? q : -1;
  };
  // stencils of quad q of level v; nodes that are not relaxed get ik = 0
  auto load_quad = [&](const TailLevel<T> &v, int q, QuadSt<T> &Q) {
    const int u = q % v.qx, w = q / v.qx;
    const int i0 = 2 * u + OFF, j0 = 2 * w + OFF;
    const int ib = min(i0, v.nx - 2);
    const bool last = i0 > ib;  // the pair starts at the last column
    const size_t n = (size_t)v.nx * v.ny;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const size_t c = (size_t)min(j0 + b, v.ny - 1) * v.nx + ib;
#pragma unroll
      for (int z = 0; z < 9; ++z) {
        const auto p = load_pair(v.st + z * n + c);
        Q.a[2 * b][z] = last ? p[1] : p[0];
        Q.a[2 * b + 1][z] = p[1];
      }
      const int d0 = v.dir[last ? c + 1 : c], d1 = v.dir[c + 1];
      const bool row = j0 + b < v.ny - OFF;
      Q.ik[2 * b] = row && i0 < v.nx - OFF && !d0 ? T(1) / Q.a[2 * b][4] : T(0);
      Q.ik[2 * b + 1] = row && i0 + 1 < v.nx - OFF && !d1 ? T(1) / Q.a[2 * b + 1][4] : T(0);
    }
  };
  auto entry = [&](const TailLevel<T> &v, int q) {  // of quad q in a plane
    return (q / v.qx + 1) * v.pitch + q % v.qx + 1;
  };
  // `sweeps` sweeps of level v by the owners of its quads; a level of one
  // wave needs no barrier (the caller leaves out the other waves)
  auto smooth = [&](const TailLevel<T> &v, QuadSt<T> &Q, int q, int sweeps, bool one_wave) {
    T *c = S + v.xoff + (q >= 0 ? entry(v, q) : 0);
    for (int s = 0; s < sweeps; ++s)
#pragma unroll
      for (int col = 0; col < 4; ++col) {
        if (q >= 0) quad_relax<T>(Q, c, pos(col), v.ps, v.pitch);
        if (one_wave) {
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        } else {
          __syncthreads();
        }
      }
  };
  // value of coarse node (I, J) of level r
  auto coarse = [&](int r, const TailLevel<T> &v, int I, int J) -> T {
    if (r == 0) return S[v.xoff + J * v.nx + I];
    const int i = I - OFF, j = J - OFF;
    return S[v.xoff + ((i & 1) + 2 * (j & 1)) * v.ps + ((j >> 1) + 1) * v.pitch + (i >> 1) + 1];
  };
  // iterate of level v to global memory (its Dirichlet ring is zero)
  auto store = [&](const TailLevel<T> &v, const QuadSt<T> &Q, int q) {
    const int u = q % v.qx, w = q / v.qx;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = 2 * u + OFF + (k & 1), j = 2 * w + OFF + (k >> 1);
      if (i < v.nx && j < v.ny) v.x[(size_t)j * v.nx + i] = Q.x[k];
      if (!FREE) {
        if (u == 0 && (k & 1) == 0 && j < v.ny) v.x[(size_t)j * v.nx] = T(0);
        if (w == 0 && k < 2 && i < v.nx) v.x[i] = T(0);
        if (q == 0 && k == 0) v.x[0] = T(0);
      }
    }
  };

  const TailLevel<T> &top = a.lv[0], &cl = a.lv[nl - 1];
  const int nco = cl.nx * cl.ny;
  const int m = a.cidx[nco];
  if (nl == 1) {  // the coarsest solve alone (a batch; up to kMaxCoarseNodes nodes)
    if (stop != 0.0) return;
    for (int c = t; c < nco; c += NT)
      if (a.cidx[c] >= 0) cinv[a.cidx[c]] = (double)cl.b[c];
    __syncthreads();
    for (int c = t; c < nco; c += NT) {
      const int k = a.cidx[c];
      double s = 0.0;
      if (k >= 0)
        for (int q = 0; q < m; ++q) s += a.cinv[(size_t)q * m + k] * cinv[q];
      cl.x[c] = (T)s;
    }
    return;
  }
  // everything the launch reads from memory, issued together; stop, whose
  // test would cost the launch another memory latency up front, is tested after
  const int qt = owned(top);
  QuadSt<T> Q, Ql;  // the first level's quad; a lower level's
  int ql = -1, rl = -1;
  if (qt >= 0) {
    load_quad(top, qt, Q);
    const int u = qt % top.qx, w = qt / top.qx;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = min(2 * u + OFF + (k & 1), top.nx - 1);
      const int j = min(2 * w + OFF + (k >> 1), top.ny - 1);
      Q.f[k] = top.b[(size_t)j * top.nx + i];
      Q.x[k] = T(0);
    }
  }
  for (int r = nl - 2; r >= 1; --r) {
    const int q = owned(lvl(r));
    if (q >= 0) {
      ql = q;
      rl = r;
    }
  }
  if constexpr (KEEP) {
    if (ql >= 0) load_quad(lvl(rl), ql, Ql);
  }
  for (int c = t; c < a.lds; c += NT) S[c] = T(0);
  for (int c = t; c < m * m; c += NT) cinv[c] = a.cinv[c];
  if (t < nco) ci[t] = a.cidx[t];
  if (stop != 0.0) return;
  __syncthreads();

  QuadSt<T> &L = KEEP ? Ql : Q;  // registers of the lower levels
  for (int r = nl - 1; r >= 1; --r) {
    const TailLevel<T> &v = lvl(r), &cv = lvl(r - 1);
    const bool first = r == nl - 1;
    const int q = first ? qt : (rl == r ? ql : -1);
    const bool one_wave = v.nq <= 64;
    const int c0 = v.xoff + (q >= 0 ? entry(v, q) : 0);
    const int r0 = v.roff + (q >= 0 ? entry(v, q) : 0);
    T res[4] = {T(0), T(0), T(0), T(0)};
    // sweeps, then the residual into the residual planes
    auto work = [&](QuadSt<T> &P) {
      smooth(v, P, q, a.nu1, one_wave);
      if (q >= 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          res[k] = quad_resid<T>(P, S + c0, k, v.ps, v.pitch);
          S[r0 + k * v.ps] = res[k];
        }
      }
    };
    if (first) {
      if (!one_wave || t < 64) work(Q);
    } else {
      if (q >= 0) {
        if constexpr (!KEEP) load_quad(v, q, L);
        const int u = q % v.qx, w = q / v.qx;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int i = min(2 * u + OFF + (k & 1), v.nx - 1);
          const int j = min(2 * w + OFF + (k >> 1), v.ny - 1);
          L.f[k] = S[v.foff + j * v.nx + i];
          L.x[k] = T(0);
        }
      }
      if (!one_wave || (t >> 6) == (v.t0 >> 6)) work(L);
    }
    __syncthreads();
    if (q >= 0) {
      const int I = q % v.qx + OFF, J = q / v.qx + OFF;
      if (I < cv.nx - OFF && J < cv.ny - OFF) {
        T s = quad_full_weight(res, S + r0, FREE ? 0 : 3, v.ps, v.pitch);
        if (FREE) {
          const bool ring = I == 0 || J == 0 || I == cv.nx - 1 || J == cv.ny - 1;
          // a coarse ring node is Dirichlet unless its edge is Neumann
          if (ring && cv.dir[J * cv.nx + I]) s = T(0);
        }
        S[cv.foff + J * cv.nx + I] = s;
      }
    }
    __syncthreads();
  }
  {  // coarsest level: x = A^-1 b
    if (t < nco && ci[t] >= 0) bb[ci[t]] = (double)S[cl.foff + t];
    __syncthreads();
    if (t < nco) {
      const int k = ci[t];
      double s = 0.0;
      if (k >= 0)
        for (int q = 0; q < m; ++q) s += cinv[q * m + k] * bb[q];
      S[cl.xoff + t] = (T)s;
      cl.x[t] = (T)s;
    } else if (std::is_same<T, double>::value && t >= kRhsThread) {
      // right-hand sides that only LDS holds, for callers that export them, by
      // waves that have no part in the coarsest solve
      for (int r = nl - 2; r >= 0; --r) {
        const TailLevel<T> &v = lvl(r);
        for (int c = t - kRhsThread; c < v.nx * v.ny; c += NT - kRhsThread)
          v.b[c] = S[v.foff + c];
      }
    }
    __syncthreads();
  }
  for (int r = 1; r < nl; ++r) {
    const TailLevel<T> &v = lvl(r), &cv = lvl(r - 1);
    const bool first = r == nl - 1;
    const int q = first ? qt : (rl == r ? ql : -1);
    const bool one_wave = v.nq <= 64;
    auto work = [&](QuadSt<T> &P) {
      if (q >= 0) {
        const int u = q % v.qx, w = q / v.qx;
        T *c = S + v.xoff + entry(v, q);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (!KEEP && first && rl >= 0) P.x[k] = c[k * v.ps];  // registers re-used below
          if (P.ik[k] != T(0)) {
            const int i = 2 * u + OFF + (k & 1), j = 2 * w + OFF + (k >> 1);
            const int I = i >> 1, J = j >> 1;
            T e = coarse(r - 1, cv, I, J);
            if (i & 1) e = T(0.5) * (e + coarse(r - 1, cv, I + 1, J));
            if (j & 1) {
              T e1 = coarse(r - 1, cv, I, J + 1);
              if (i & 1) e1 = T(0.5) * (e1 + coarse(r - 1, cv, I + 1, J + 1));
              e = T(0.5) * (e + e1);
            }
            P.x[k] += e;
            c[k * v.ps] = P.x[k];
          }
        }
      }
      if (one_wave) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        __syncthreads();
      }
      smooth(v, P, q, a.nu2, one_wave);
      if (q >= 0) store(v, P, q);
    };
    if (first) {
      if constexpr (!KEEP) {
        if (qt >= 0 && rl >= 0) {
          load_quad(top, qt, Q);
          const int u = qt % top.qx, w = qt / top.qx;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int i = min(2 * u + OFF + (k & 1), top.nx - 1);
            const int j = min(2 * w + OFF + (k >> 1), top.ny - 1);
            Q.f[k] = top.b[(size_t)j * top.nx + i];
          }
        }
      }
      if (!one_wave || t < 64) work(Q);
    } else if (!one_wave || (t >> 6) == (v.t0 >> 6)) {
      work(L);
    }
    __syncthreads();
  }
}

template <typename T, int NT, bool FREE>
__global__ __launch_bounds__(NT) void k_tail(TailArgs<T> a) {
  const double stop = a.skip ? *a.skip : 0.0;
  tail_body<T, NT, FREE>(a, stop);
}

// Batched form: one workgroup per problem.
template <typename T, int NT, bool FREE>
__global__ __launch_bounds__(NT) void k_tail_b(BatchTab tab) {
  const TailArgs<T> &a = *static_cast<const TailArgs<T> *>(tab.e[blockIdx.x].args);
  tail_body<T, NT, FREE>(a, 0.0);
}

}  // namespace

// Number of nodes a level may have to be handled by the tail.  Alone from
// 33 x 33 down: at 65 x 65 (FP32, the 1024-thread form) the level costs more
// here than as two passes of its own (a mixed 129^2 step of two cycles 97.8
// against 90.0 us).  In a batch, where the passes' launches are shared, the
// tail takes it.  Measured alone, FP64, the tail from 33 x 33: 34 us a
// launch with one node per thread and streamed stencils, 25 us with quads
// (17 us where the stencils are still in L2: a 129^2 V-cycle 79 -> 67 us, 65^2
// 55 -> 45 us).
int tail_max_nodes(bool batch) { return batch ? kTailMaxNodes : 33 * 33; }

// Quads, LDS planes and thread ranges of the tail from level lc on; false
// when it does not fit a workgroup.
template <typename T>
static bool make_tail_args(const tomg_problem *p, int lc, TailArgs<T> &a) {
  a = TailArgs<T>{};
  const bool f32 = std::is_same<T, float>::value;
  const bool free_ring = stored_level0(p->cfg);
  const int off = free_ring ? 0 : 1;
  a.lc = lc;
  a.nl = p->L - lc;
  a.nu1 = p->cfg.nu1;
  a.nu2 = p->cfg.nu2;
  a.cinv = p->cinv;
  a.cidx = p->cidx;
  if (a.nl > kTailLevels) return false;
  int at = 0, t0 = 0, rmax = 0;
  for (int q = 0; q < a.nl; ++q) {
    const Level &v = p->lv[lc + q];
    TailLevel<T> &e = a.lv[q];
    e.nx = v.nx;
    e.ny = v.ny;
    e.st = (const T *)(f32 ? (void *)v.st32 : (void *)v.st);
    e.x = (T *)(f32 ? (void *)v.x32 : (void *)v.x);
    e.b = (T *)(f32 ? (void *)v.b32 : (void *)v.b);
    e.dir = v.dir;
    const bool coarsest = q == a.nl - 1;
    e.qx = (v.nx + 1 - off) / 2;
    const int qy = (v.ny + 1 - off) / 2;
    e.nq = e.qx * qy;
    e.pitch = e.qx + 2;
    e.ps = e.pitch * (qy + 2);
    e.xoff = at;
    at += coarsest ? v.nx * v.ny : 4 * e.ps;
    if (q > 0) {
      e.foff = at;
      at += v.nx * v.ny;
    }
    if (free_ring && !coarsest) {  // its ring of zeros is read: planes of its own
      e.roff = at;
      at += 4 * e.ps;
    } else if (!coarsest) {
      rmax = rmax > 4 * e.ps ? rmax : 4 * e.ps;
    }
    if (q > 0 && !coarsest) {
      e.t0 = t0;
      t0 = (t0 + e.nq + 63) / 64 * 64;
    }
  }
  if (!free_ring) {
    for (int q = 0; q + 1 < a.nl; ++q) a.lv[q].roff = at;
    at += rmax;
  }
  a.lds = at;
  a.shmem = (int)(kMaxCoarseUnknowns * kMaxCoarseUnknowns * sizeof(double)) + at * (int)sizeof(T);
  const int need = a.nl > 1 ? (a.lv[0].nq > t0 ? a.lv[0].nq : t0) : 1;
  a.wide = need > kTailNarrow;
  // at FP64 a quad does not fit the wide form's 128 registers per thread
  return need <= (f32 ? kTailWide : kTailNarrow) && a.shmem <= kTailLdsMax;
}

// Whether the tail can start at level l.
bool tail_fits(const tomg_problem *p, int l, bool batch) {
  if ((long)p->lv[l].nx * p->lv[l].ny > tail_max_nodes(batch)) return false;
  for (int k = l; k < p->L; ++k)
    if (p->lv[k].ck != 0) return false;
  TailArgs<double> a64;
  TailArgs<float> a32;
  return p->cfg.precision == TOMG_FP32_IR ? make_tail_args<float>(p, l, a32)
                                          : make_tail_args<double>(p, l, a64);
}

void build_tail_args(tomg_problem *p) {
  make_tail_args<double>(p, p->lc, p->hargs.tail64);
  make_tail_args<double>(p, p->lcb, p->hargs.tail64b);
  if (p->cfg.precision == TOMG_FP32_IR) {
    make_tail_args<float>(p, p->lc, p->hargs.tail32);
    make_tail_args<float>(p, p->lcb, p->hargs.tail32b);
  }
}

// Levels lc..L-1 in one workgroup.
template <typename T>
void tail_cycle(tomg_problem *p) {
  TailArgs<T> a = std::is_same<T, float>::value ? *(TailArgs<T> *)(void *)&p->hargs.tail32
                                                : *(TailArgs<T> *)(void *)&p->hargs.tail64;
  a.skip = p->skip;
  const bool fr = stored_level0(p->cfg);
  if constexpr (std::is_same<T, float>::value) {
    if (a.wide) {
      if (fr)
        hipLaunchKernelGGL((k_tail<T, kTailWide, true>), 1, kTailWide, a.shmem, p->stream, a);
      else
        hipLaunchKernelGGL((k_tail<T, kTailWide, false>), 1, kTailWide, a.shmem, p->stream, a);
      return;
    }
  }
  if (fr)
    hipLaunchKernelGGL((k_tail<T, kTailNarrow, true>), 1, kTailNarrow, a.shmem, p->stream, a);
  else
    hipLaunchKernelGGL((k_tail<T, kTailNarrow, false>), 1, kTailNarrow, a.shmem, p->stream, a);
}

template void tail_cycle<double>(tomg_problem *);
template void tail_cycle<float>(tomg_problem *);

template <typename T>
static void batch_tail_t(tomg_problem *const *probs, const int *idx, int cnt, hipStream_t s) {
  constexpr bool f32 = std::is_same<T, float>::value;
  BatchTab tab;
  for (int k0 = 0; k0 < cnt; k0 += kBatchMax) {
    tab.count = 0;
    int shmem = 0, wide = 0;
    for (int k = k0; k < cnt && k < k0 + kBatchMax; ++k) {
      tomg_problem *p = probs[idx[k]];
      BatchEntry &e = tab.e[tab.count];
      e.args = f32 ? (const void *)&p->dargs->tail32b : (const void *)&p->dargs->tail64b;
      e.phi = nullptr;
      e.role = 0;
      e.nbx = e.nby = 1;
      e.start = tab.count;
      e.slot = e.out = 0;
      const int sh = f32 ? p->hargs.tail32b.shmem : p->hargs.tail64b.shmem;
      shmem = shmem > sh ? shmem : sh;
      wide |= f32 ? p->hargs.tail32b.wide : p->hargs.tail64b.wide;
      ++tab.count;
    }
    if (!tab.count) continue;
    // a batch has one level-0 operator form, hence one kind of ring
    const bool fr = stored_level0(probs[idx[k0]]->cfg);
    if constexpr (f32) {
      if (wide) {
        if (fr)
          hipLaunchKernelGGL((k_tail_b<T, kTailWide, true>), tab.count, kTailWide, shmem, s, tab);
        else
          hipLaunchKernelGGL((k_tail_b<T, kTailWide, false>), tab.count, kTailWide, shmem, s, tab);
        continue;
      }
    }
    if (fr)
      hipLaunchKernelGGL((k_tail_b<T, kTailNarrow, true>), tab.count, kTailNarrow, shmem, s, tab);
    else
      hipLaunchKernelGGL((k_tail_b<T, kTailNarrow, false>), tab.count, kTailNarrow, shmem, s, tab);
  }
}

void batch_tail(tomg_problem *const *probs, const int *idx, int cnt, bool fp32, hipStream_t s) {
  if (fp32)
    batch_tail_t<float>(probs, idx, cnt, s);
  else
    batch_tail_t<double>(probs, idx, cnt, s);
}

}  // namespace tomg
