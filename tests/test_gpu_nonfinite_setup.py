"""A set-up whose coarsest matrix holds a NaN.  A corner coordinate that is not
a number reaches one fine row, and through the coarse operators the diagonal of
the last of the 49 unknowns alone, so the inverse's last step finds no number
in its column.  The set-up must report the map, write nothing behind the
inverse (the unknowns' numbering lies there and the coarsest solve indexes
with it), and leave the problem fit for the next map."""

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


def _numbering(p):
    """Offset (in int32) of the coarsest 9 x 9 level's numbering in the workspace."""
    import torch
    inner = np.full((9, 9), -1, dtype=np.int32)
    inner[1:8, 1:8] = np.arange(49).reshape(7, 7)
    pat = np.append(inner.ravel(), 49).astype(np.int32)
    ws = p.workspace.view(torch.int32).cpu().numpy()
    at = [k for k in np.flatnonzero(ws == 49) - 81
          if k >= 0 and np.array_equal(ws[k:k + 82], pat)]
    assert len(at) == 1, at
    return at[0], pat


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir"])
def test_nan_in_the_last_coarse_diagonal(tomg, precision):
    import torch
    q = w.manufactured_sinusoidal(129)
    print(f"[nonfinite] {precision}", flush=True)
    p = tomg.Problem.from_grid(q, precision=precision)
    d = tomg.upload(q)
    p.setup_coeffs(d["rho"], xp=d["xp"], yp=d["yp"])
    at, pat = _numbering(p)
    ref = d["phi0"].clone()
    want = p.solve(ref)
    assert want.ok
    bad = d["xp"].clone()
    bad[-1, -1] = float("nan")
    for check in (True, False):
        with pytest.raises(tomg.TomgError) as e:
            p.setup_coeffs(d["rho"], xp=bad, yp=d["yp"], check=check)
            p.setup_check()
        assert e.value.status in (tomg.TOMG_ENONFINITE, tomg.TOMG_EGEOMETRY)
        torch.cuda.synchronize()
        got = p.workspace.view(torch.int32)[at:at + 82].cpu().numpy()
        assert np.array_equal(got, pat), check
    p.setup_coeffs(d["rho"], xp=d["xp"], yp=d["yp"])
    phi = d["phi0"].clone()
    got = p.solve(phi)
    assert got.ok and got.cycles == want.cycles and bool((phi == ref).all())
