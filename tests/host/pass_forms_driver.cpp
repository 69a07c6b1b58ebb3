// Links the launch code of the level passes (fused.hip, tile.hip) with a
// marching form that takes no pass, and asks which problems' launch arguments
// are accepted: a pass that no kernel is built for must be refused, not left
// out of the cycle.  Host code only; no call here reaches a GPU.
#include <cstdio>

#include "tomg_internal.h"

static bool march_takes = false;

namespace tomg {
template <>
bool pick_march<double>(PassArgs<double> &a, int nu, bool) {
  if (march_takes && nu <= 2 && a.ck == 0) a.form = kFormMarch;
  return a.form == kFormMarch;
}
template <>
bool pick_march<float>(PassArgs<float> &a, int nu, bool) {
  if (march_takes && nu <= 2 && a.ck == 0) a.form = kFormMarch;
  return a.form == kFormMarch;
}
#define NO_LAUNCH(NAME, T)                                                          \
  template <>                                                                       \
  void NAME<T>(int, bool, bool, const PassArgs<T> &, hipStream_t, const BatchTab *, \
               int) {}
NO_LAUNCH(march_down, double)
NO_LAUNCH(march_down, float)
NO_LAUNCH(march_up, double)
NO_LAUNCH(march_up, float)
}  // namespace tomg

using namespace tomg;

static bool accepted(int nx, int ny, int nu1, int nu2, int precision, int neumann, int semi) {
  tomg_config c;
  tomg_config_default(&c, nx, ny, 1.0 / (nx - 1), 1.0 / (ny - 1));
  c.nu1 = nu1;
  c.nu2 = nu2;
  c.precision = precision;
  c.neumann = neumann;
  c.semi_levels = semi;
  c.semi_axis = 1;
  tomg_problem *p = new tomg_problem();
  p->cfg = c;
  if (!make_layout(c, &p->lay)) {
    std::fprintf(stderr, "no layout for %d x %d\n", nx, ny);
    delete p;
    return false;
  }
  p->L = p->lay.L;
  for (int l = 0; l < p->L; ++l) {
    p->lv[l].nx = p->lay.nx[l];
    p->lv[l].ny = p->lay.ny[l];
    p->lv[l].ck = p->lay.ck[l];
    p->lv[l].n = (size_t)p->lay.nx[l] * p->lay.ny[l];
  }
  const bool ok = build_pass_args(p) == hipSuccess;
  delete p;
  return ok;
}

int main() {
  // tiles: up to 1.2 M nodes alone and 20 thousand in a batch; a first level
  // with one axis halved (65 x 513 semi-coarsened) has the band form
  struct Grid {
    int nx, ny, semi;
    bool all_tiles_or_bands;
  };
  const Grid grids[] = {{129, 129, 0, true},    {129, 129, 1, true},   {65, 513, 1, true},
                        {257, 257, 0, false},   {257, 257, 1, false},  {1281, 1025, 0, false},
                        {1281, 1025, 1, false}};
  int bad = 0;
  for (int takes = 0; takes < 2; ++takes) {
    march_takes = takes;
    for (const Grid &g : grids)
      for (int precision = 0; precision < 2; ++precision)
        for (int neumann = 0; neumann < 2; ++neumann)
          for (int nu1 = 1; nu1 <= 4; ++nu1)
            for (int nu2 = 1; nu2 <= 4; ++nu2) {
              const bool want = takes || g.all_tiles_or_bands || (nu1 > 2 && nu2 > 2);
              const bool got = accepted(g.nx, g.ny, nu1, nu2, precision, neumann, g.semi);
              if (got == want) continue;
              std::fprintf(stderr, "%d x %d semi %d V(%d,%d) precision %d neumann %d: %d\n",
                           g.nx, g.ny, g.semi, nu1, nu2, precision, neumann, got);
              ++bad;
            }
  }
  if (bad) return 1;
  std::printf("pass forms: all checks ran\n");
  return 0;
}
