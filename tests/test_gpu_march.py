"""The marching passes (one wave walks up a band of rows, two columns per
lane) where their strips and bands can go wrong: 110 (118) owned columns at
two (one) sweeps, of which the last strip holds 7, 3 or 107; bands that end
inside a grid; the operator from the tensor and stored; strips wider than
the grid, in a batch.  Cycles against the oracle's at the bound of the other
V-cycle tests (1e-12): a residual's rounding error is some 4/h^2 ulp of the
iterate, 4e-10, but without order from node to node, of which the inverse
keeps 1/(20 sqrt(nodes)), under 1e-13.  A batch of several million nodes,
whose levels march where the smaller grids alone take tiles, is bitwise equal
to solving alone."""

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


def rel_err(a, b):
    return float(np.max(np.abs(np.asarray(a) - b)) / max(np.max(np.abs(b)), 1e-300))


def np_(t):
    return t.detach().cpu().numpy()


def _sine(nx, ny):
    return w.manufactured_sinusoidal(nx, ny=ny)


def _neumann(nx, ny):
    return w.polar_semi_annulus(nx, ny=ny, neumann=True)


ALONE = {
    "sine1217x1025": (_sine, 1217, 1025, 2, 2),
    "sine1537x833": (_sine, 1537, 833, 1, 1),
    "sine769x1665": (_sine, 769, 1665, 1, 2),
    "neumann1217x1025": (_neumann, 1217, 1025, 2, 2),
    "neumann1537x833": (_neumann, 1537, 833, 2, 1),
}


@pytest.mark.parametrize("name", list(ALONE))
def test_vcycles_match_oracle(tomg, name):
    mk, nx, ny, nu1, nu2 = ALONE[name]
    q = mk(nx, ny)
    print(f"[march] {name} V({nu1},{nu2})", flush=True)
    p, d = tomg.setup_from_grid(q, nu1=nu1, nu2=nu2)
    s = oracle.setup(q)
    mg = oracle.MG.from_setup(s, q.dx, q.dy, mask=q.mask, nu1=nu1, nu2=nu2)
    xg, xo = d["phi0"].clone(), q.phi0
    for _ in range(2):
        p.vcycle(xg)
        xo = mg.vcycle(xo, s["f"])
        assert rel_err(np_(xg), xo) <= 1e-12


@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("mk", [_sine, _neumann])
def test_batch_equals_alone(tomg, mk, precision, nu):
    sizes = [(161, 145), (257, 273), (1025, 1025), (1217, 1025), (833, 1025)]
    print(f"[march_batch] {mk.__name__} {precision} nu {nu}", flush=True)
    qs = [mk(nx, ny) for nx, ny in sizes]
    ps, ds = zip(*[tomg.setup_from_grid(q, precision=precision, nu1=nu, nu2=nu) for q in qs])
    phis = [d["phi0"].clone() for d in ds]
    res = tomg.solve_batch(list(ps), phis, rel_tol=1e-10, max_cycles=6)
    for q, p, d, phi, r in zip(qs, ps, ds, phis, res):
        alone = d["phi0"].clone()
        ra = p.solve(alone, rel_tol=1e-10, max_cycles=6)
        assert np.isfinite(r.rel) and r.rel < 0.1, (q.name, r)
        assert ra.cycles == r.cycles and np.array_equal(np_(alone), np_(phi)), q.name
