"""The sums that bq_sync returns are those of the state it finds: mass,
energy and CFL maximum against numpy sums over the fields read back, through
states of different sums set one after the other (a state brought back before
its new sums are in it would carry those of the call before)."""
import numpy as np
import pytest

from paper_1909_04153_amd import scenarios as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_04153_amd import bq as m

    m.load()
    return m


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
@pytest.mark.parametrize("nx,ny", [(5, 4), (130, 37)])
def test_sums_are_those_of_the_present_state(bq, nx, ny, precision):
    spec = S.solitary_flat(nx=nx, ny=ny, dx=0.1, depth=0.75, x0=0.03 * nx)
    p = spec["params"]
    d = bq.Domain(p, spec["depth_c"], precision=getattr(bq, precision))
    # depth 0.75 is exact in both precisions, and so is eta = w; each side's
    # sum of n positive terms is off by at most n 2^-53 of itself
    depth, tol = 0.75, 4.0 * nx * ny * 2.0 ** -53
    seen = []
    for k, scale in enumerate((1.0, 0.25, 0.5, 0.0)):
        d.set_state(scale * spec["eta"], scale * spec["P"], scale * spec["Q"])
        for steps in (0, 3):
            d.step(steps)
            i = d.sync()
            eta, P, Q = (d.read(f) for f in ("eta", "P", "Q"))
            h = eta + depth
            mass = float(h.sum()) * p["dx"] * p["dy"]
            energy = float((0.5 * p["g"] * eta * eta + 0.5 * (P * P + Q * Q) / h).sum()) * p["dx"] * p["dy"]
            assert i.status == 0 and i.n == steps
            assert abs(i.mass - mass) <= tol * mass, (k, steps, i.mass, mass)
            assert abs(i.energy - energy) <= 4.0 * tol * energy, (k, steps, i.energy, energy)
            seen.append((i.mass, i.energy))
    assert len(set(seen[:6])) == 6      # the sums of one state are not those of another
