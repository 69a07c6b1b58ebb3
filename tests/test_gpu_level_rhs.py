"""Right-hand sides of the coarse levels after a V-cycle, as tomg_export gives
them: with the operator from the tensor, with Neumann edges, in the flux form
and semi-coarsened, the smallest levels in the single-workgroup tail, against
the oracle's.  Bound: a residual of level k carries the rounding of some dozens
of multiply-adds (its own nine, and those of the sweeps behind it) on terms of
at most diag_k |x_k|, and a restriction averages the levels above, so 128 ulp of
the largest such terms, summed over the levels above.  A batch of one, whose
levels take their batched kernels, leaves the same bits."""

import numpy as np
import pytest

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tomg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_01888_amd as t
    return t


def np_(t):
    return t.detach().cpu().numpy()


def _sine(nx, ny):
    return w.manufactured_sinusoidal(nx, ny=ny)


def _neumann(nx, ny):
    return w.polar_semi_annulus(nx, ny=ny, neumann=True)


CASES = {
    "tensor65": (_sine, 65, 65, {}),
    "tensor225x17": (_sine, 225, 17, {}),
    "neumann65": (_neumann, 65, 65, {}),
    "neumann97x49": (_neumann, 97, 49, {}),
    "flux33x65": (_sine, 33, 65, {"flux": True}),
    "semi49x65_x1": (_neumann, 49, 65, {"semi": 1, "semi_axis": 0}),
    "semi33x97_y2": (_sine, 33, 97, {"semi": 2, "semi_axis": 1}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_level_rhs_matches_oracle(tomg, name):
    mk, nx, ny, kw = CASES[name]
    q = mk(nx, ny)
    print(f"[level_rhs] {name}", flush=True)
    gk = {"flux": kw.get("flux", False), "semi_levels": kw.get("semi", 0),
          "semi_axis": kw.get("semi_axis", 0)}
    p, d = tomg.setup_from_grid(q, **gk)
    s = oracle.setup(q)
    mg = oracle.MG.from_setup(s, q.dx, q.dy, mask=q.mask, **kw)
    xg = d["phi0"].clone()
    p.vcycle(xg)
    xo = mg.vcycle(q.phi0, s["f"])
    free = s["dir"] == 0
    bound = 128 * np.finfo(np.float64).eps * np.max(np.abs(xo)) * 2 * (
        np.max(np.abs(s["exx"][free])) / q.dx ** 2 + np.max(np.abs(s["eyy"][free])) / q.dy ** 2)
    got = {}
    for l in range(1, mg.num_levels):
        got[l] = np_(p.export("rhs", l))
        free = mg.dirs(l) == 0
        want = mg.level_rhs(l)
        assert np.max(np.abs(want[free])) > 100 * bound, l  # the bound tells a wrong level
        assert np.max(np.abs(got[l] - want)[free]) <= bound, l
        bound += 128 * np.finfo(np.float64).eps * np.max(
            np.abs(mg.stencil(l)[4][free])) * np.max(np.abs(mg.level_x(l)))
    pb, db = tomg.setup_from_grid(q, **gk)
    phi = db["phi0"].clone()
    tomg.solve_batch([pb], [phi], rel_tol=1e-300, max_cycles=1)
    assert np.array_equal(np_(phi), np_(xg))
    for l in got:
        assert np.array_equal(np_(pb.export("rhs", l)), got[l]), l
