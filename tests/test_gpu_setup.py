"""Domain set-up on the device: the rest state a new domain starts in, and the
wavemaker's wave numbers where its column is longer than one LDS load (2048
rows)."""
import math

import numpy as np
import pytest

from oracle.oracle import OracleDomain
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


@pytest.mark.parametrize("precision", ["FP32", "FP64"])
def test_new_domain_is_the_lake_at_rest(bq, precision):
    # wet and dry cells, wavemaker and sponge sides, the run-up record
    for spec in (S.sloping_beach(nx=133, ny=21, dx=0.1, x_toe=1.0), S.conical_island(nx=90, ny=70, dx=30.0 / 90),
                 S.series_beach(nx=70, ny=13)):
        a = bq.Domain(spec["params"], spec["depth_c"], precision=getattr(bq, precision))
        b = bq.Domain(spec["params"], spec["depth_c"], precision=getattr(bq, precision))
        z = np.zeros((a.ny, a.nx))
        b.set_state(z, z, z)
        assert a.save() == b.save()
        a.step(5)
        b.step(5)
        assert a.save() == b.save()


@pytest.mark.parametrize("ny", [2047, 2048, 2049])
def test_wave_numbers_of_a_long_column(bq, ny):
    spec = S.sloping_beach(nx=12, ny=ny, dx=0.1, x_toe=0.3, slope=0.1, ramp=0.0)
    # depths that differ along the column, so that each row counts
    spec["depth_c"] = spec["depth_c"] + 0.01 * np.sin(np.arange(ny + 1))[:, None]
    o = OracleDomain(spec["params"], spec["depth_c"])
    assert o.set_state(spec["eta"], spec["P"], spec["Q"]) == 0
    g = bq.domain_from_spec(spec, precision=bq.FP64)
    assert o.step(3) == 0
    g.step(3)
    for f in ("eta", "P"):
        a, r = g.read(f), o.read(f)
        s = 0.02 * (math.sqrt(9.81 * 0.5) if f == "P" else 1.0)
        assert np.linalg.norm(a - r) <= 1e-12 * max(np.linalg.norm(r), 0.1 * s * math.sqrt(r.size)), (ny, f)
