"""The quad kernels (one thread, one 2 x 2 quad of nodes) at the sizes where
their blocking can go wrong: the single-workgroup tail with ragged, long and
minimal levels, with a Dirichlet and with a free outer ring, and the tiled
passes around their tile and threshold sizes.  Two V-cycles and
every level's correction against the oracle's at the bounds of the
other V-cycle tests (1e-12, 1e-11: a few hundred roundings), and a
batch, whose levels run in other kernels, bitwise equal to solving alone."""

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
    # tail: two levels; even coarsest sides; one wave; long and thin; 33 x 33
    "tail9": (_sine, 9, 9, 2, 2),
    "tail81x41": (_sine, 81, 41, 2, 2),
    "tail33x17": (_sine, 33, 17, 1, 3),
    "tail225x17": (_sine, 225, 17, 2, 2),
    "tail65": (_sine, 65, 65, 4, 1),
    "tail49x97": (_sine, 49, 97, 2, 2),
    # the same with free ring nodes
    "tail17_neumann": (_neumann, 17, 17, 2, 2),
    "tail65_neumann": (_neumann, 65, 65, 2, 2),
    "tail97x49_neumann": (_neumann, 97, 49, 1, 2),
    "tail33x65_neumann": (_neumann, 33, 65, 3, 3),
    # tiles: one tile wide (14 or 16 owned columns, 22 or 24 rows), one more
    # column or row than whole tiles, both tile sizes, one and two sweeps
    "tile5x9": (_sine, 5, 9, 2, 2),
    "tile17x25": (_sine, 17, 25, 2, 2),
    "tile113x89": (_sine, 113, 89, 2, 2),
    "tile129_nu1": (_sine, 129, 129, 1, 1),
    "tile257x273": (_sine, 257, 273, 2, 1),
    "tile289x577": (_sine, 289, 577, 1, 2),
    "tile161x145_neumann": (_neumann, 161, 145, 2, 2),
    "tile321x257_neumann": (_neumann, 321, 257, 1, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_vcycles_match_oracle(tomg, name):
    mk, nx, ny, nu1, nu2 = CASES[name]
    q = mk(nx, ny)
    print(f"[quads] {name} {nx}x{ny} V({nu1},{nu2})", flush=True)
    p, d = tomg.setup_from_grid(q, nu1=nu1, nu2=nu2)
    s = oracle.setup(q)
    mg = oracle.MG.from_setup(s, q.dx, q.dy, mask=q.mask, nu1=nu1, nu2=nu2)
    xg, xo = d["phi0"].clone(), q.phi0
    for _ in range(2):
        p.vcycle(xg)
        xo = mg.vcycle(xo, s["f"])
        assert rel_err(np_(xg), xo) <= 1e-12
    for l in range(1, mg.num_levels):
        assert rel_err(np_(p.export("x", l)), mg.level_x(l)) <= 1e-11, l


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
@pytest.mark.parametrize("mk", [_sine, _neumann])
def test_batch_equals_alone(tomg, mk, precision):
    qs = [mk(nx, ny) for m, nx, ny, _, _ in CASES.values() if m is mk]
    print(f"[quads_batch] {mk.__name__} {precision} {len(qs)}", flush=True)
    ps, ds = zip(*[tomg.setup_from_grid(q, precision=precision) for q in qs])
    phis = [d["phi0"].clone() for d in ds]
    # a few cycles: the long grids converge slowly
    res = tomg.solve_batch(list(ps), phis, rel_tol=1e-10, max_cycles=8)
    for q, p, d, phi, r in zip(qs, ps, ds, phis, res):
        alone = d["phi0"].clone()
        ra = p.solve(alone, rel_tol=1e-10, max_cycles=8)
        assert np.isfinite(r.rel) and r.rel < 0.1, (q.name, r)
        assert ra.cycles == r.cycles and np.array_equal(np_(alone), np_(phi)), q.name
