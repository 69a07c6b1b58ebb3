"""The chained level-0 pass of FP32 inner cycles (the upward pass of a cycle and
the downward pass of the next in one launch): on stored stencils above the
levels that run on tiles, 2, 3 and 4 sweeps, both axes halved or one alone.  A
batch runs the same relaxations as separate passes, so its iterate is equal bit
for bit; the pass counters say that the chained launches ran."""

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


@pytest.fixture(scope="module")
def annulus():
    return w.polar_semi_annulus(1281, ny=1025, neumann=True)  # 1.3 M nodes


INNER = 3


@pytest.mark.parametrize("nu", [(1, 1), (2, 1), (1, 2), (2, 2)])
@pytest.mark.parametrize("semi,axis", [(0, "x"), (1, "x"), (1, "y"), (2, "x")])
def test_chained_equals_separate(tomg, annulus, semi, axis, nu):
    print(f"[chained] semi {semi} {axis} V{nu}", flush=True)
    kw = dict(precision="fp32_ir", nu1=nu[0], nu2=nu[1], ir_inner_cycles=INNER,
              semi_levels=semi, semi_axis=axis)
    p, d = tomg.setup_from_grid(annulus, **kw)
    phi = d["phi0"].clone()
    (rb,) = tomg.solve_batch([p], [phi], rel_tol=1e-10, max_cycles=2)
    alone = d["phi0"].clone()
    p.profile(True)
    ra = p.solve(alone, rel_tol=1e-10, max_cycles=2)
    down, up, chained = p.profile_read()[1::2]
    p.profile(False)
    assert ra.cycles == rb.cycles == 2
    assert (down, up, chained) == (2, 2, 2 * (INNER - 1))
    assert np.isfinite(rb.rel) and bool((alone == phi).all())
