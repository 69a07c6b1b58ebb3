"""Three and four sweeps in an FP64 batch, whose levels below the first run on
tiles up to 65^2 (38 or 30 owned columns of 64, 18 or 14 rows of 32) where a
problem alone has bands: one tile, one column or row more than whole tiles,
the largest level, Dirichlet and free rings.  Bit for bit equal to solving
alone, which the tests of the sweep counts compare with the oracle."""

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tomg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_01888_amd as t
    return t


def _sine(nx, ny):
    return w.manufactured_sinusoidal(nx, ny=ny)


def _neumann(nx, ny):
    return w.polar_semi_annulus(nx, ny=ny, neumann=True)


SIZES = [(129, 129), (113, 89), (73, 73), (57, 113), (257, 17), (129, 49), (321, 257)]


@pytest.mark.parametrize("nu", [(3, 3), (4, 4), (3, 4), (4, 1)])
@pytest.mark.parametrize("mk", [_sine, _neumann])
def test_batch_equals_alone(tomg, mk, nu):
    print(f"[batch_sweeps] {mk.__name__} V{nu}", flush=True)
    qs = [mk(nx, ny) for nx, ny in SIZES]
    ps, ds = zip(*[tomg.setup_from_grid(q, nu1=nu[0], nu2=nu[1]) for q in qs])
    phis = [d["phi0"].clone() for d in ds]
    res = tomg.solve_batch(list(ps), phis, rel_tol=1e-10, max_cycles=5)
    for q, p, d, phi, r in zip(qs, ps, ds, phis, res):
        alone = d["phi0"].clone()
        ra = p.solve(alone, rel_tol=1e-10, max_cycles=5)
        assert np.isfinite(r.rel) and r.rel < 1.0, (q.name, r)
        assert ra.cycles == r.cycles and bool((alone == phi).all()), (q.name, r)
