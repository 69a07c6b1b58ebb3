"""Tiled passes whose transfer halves one axis (each quad restricts into two
coarse nodes and takes its correction from two): ragged tiles of both sizes,
the operator from the tensor and stored, one and two sweeps, against the
oracle's cycles at the bounds of the other V-cycle tests (1e-12, 1e-11: a few
hundred roundings); and a batch large enough for the band passes, bitwise
equal to solving alone on tiles."""

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


CASES = {
    "sine145x289_x1": (_sine, 145, 289, 1, "x", 2, 2),
    "sine257x145_y1": (_sine, 257, 145, 1, "y", 1, 2),
    "sine33x97_y2": (_sine, 33, 97, 2, "y", 2, 1),
    "neumann161x145_y2": (_neumann, 161, 145, 2, "y", 2, 2),
    "neumann321x257_x2": (_neumann, 321, 257, 2, "x", 1, 1),
    "neumann49x65_x1": (_neumann, 49, 65, 1, "x", 2, 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_vcycles_match_oracle(tomg, name):
    mk, nx, ny, semi, axis, nu1, nu2 = CASES[name]
    q = mk(nx, ny)
    print(f"[semi_tiles] {name} V({nu1},{nu2})", flush=True)
    p, d = tomg.setup_from_grid(q, semi_levels=semi, semi_axis=axis, nu1=nu1, nu2=nu2)
    s = oracle.setup(q)
    mg = oracle.MG.from_setup(s, q.dx, q.dy, mask=q.mask, semi=semi,
                              semi_axis=0 if axis == "x" else 1, nu1=nu1, nu2=nu2)
    xg, xo = d["phi0"].clone(), q.phi0
    for _ in range(2):
        p.vcycle(xg)
        xo = mg.vcycle(xo, s["f"])
        assert rel_err(np_(xg), xo) <= 1e-12
    for l in range(1, mg.num_levels):
        assert rel_err(np_(p.export("x", l)), mg.level_x(l)) <= 1e-11, l


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("mk,axis", [(_sine, "y"), (_neumann, "x")])
def test_batch_equals_alone(tomg, mk, axis, precision):
    sizes = [(1025, 1025), (1025, 1025), (961, 833), (257, 129)]
    print(f"[semi_tiles_batch] {mk.__name__} {precision} {axis}", flush=True)
    qs = [mk(nx, ny) for nx, ny in sizes]
    ps, ds = zip(*[tomg.setup_from_grid(q, precision=precision, semi_levels=2, semi_axis=axis)
                   for q in qs])
    phis = [d["phi0"].clone() for d in ds]
    res = tomg.solve_batch(list(ps), phis, rel_tol=1e-10, max_cycles=6)
    for q, p, d, phi, r in zip(qs, ps, ds, phis, res):
        alone = d["phi0"].clone()
        ra = p.solve(alone, rel_tol=1e-10, max_cycles=6)
        assert np.isfinite(r.rel) and ra.cycles == r.cycles, (q.name, r)
        assert np.array_equal(np_(alone), np_(phi)), q.name
