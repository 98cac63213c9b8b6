"""Domains whose padded fields exceed 4 GiB: a channel of four columns (padded
to a tile's 64) and some millions of rows, with a wave at either end, against
a short channel that has the same ends."""
import numpy as np
import pytest

from paper_1909_04153_amd import scenarios as S

pytestmark = pytest.mark.gpu

NX, END = 4, 96     # rows compared at each end
# rows of the short channel, whose ends must not feel each other: the line
# solves' reach falls by e in about 6 rows (sqrt(2/5) d / dx)
SHORT = 232 + 1024


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_04153_amd import bq as m

    m.load()
    return m


def _spec(ny, **kw):
    """depths and waves in the last 64 rows of either end, a flat bed at rest between"""
    p = S.base_params(NX, ny, 0.1, **kw)
    rng = np.random.default_rng(3)
    d = np.full((ny + 1, NX + 1), 1.0)
    eta, P, Q = (np.zeros((ny, NX)) for _ in range(3))
    for rows in (slice(0, 64), slice(-64, None)):
        d[rows] = rng.uniform(0.8, 1.2, (64, NX + 1))
        eta[rows], P[rows], Q[rows] = (a * rng.uniform(-1.0, 1.0, (64, NX)) for a in (0.02, 0.05, 0.05))
    return dict(params=p, depth_c=d, eta=eta, P=P, Q=Q)


@pytest.mark.parametrize("precision,rows,kw", [("FP64", (1 << 22) + 232, dict(runup_delta=0.01)),
                                               ("FP32", 5592320 + 232, dict(corrector=1))])
def test_ends_of_a_long_channel(bq, precision, rows, kw):
    import torch

    prec = getattr(bq, precision)
    assert (rows - SHORT) % 16 == 0 and rows * (128 * 8 if prec == bq.FP64 else 192 * 4) > 1 << 32
    free, _ = torch.cuda.mem_get_info()
    spec = _spec(rows, **kw)
    if bq.workspace_bytes(spec["params"], prec) > free:
        pytest.skip("needs 80 GB of free device memory")
    got = []
    for s in (spec, _spec(SHORT, **kw)):
        d = bq.domain_from_spec(s, precision=prec)
        for _ in range(4):
            d.step_dt(0.004)
        i = d.sync()
        assert i.status == 0 and i.n == 4
        fields = ["eta", "P", "Q", "cfl"] + (["runup"] if "runup_delta" in kw else [])
        got.append({f: d.read(f) for f in fields})
        d.close()
        del d
        torch.cuda.empty_cache()
    # the line solves of both channels differ by what reaches END rows from
    # the other end or the middle, which is at rest: nothing above rounding
    tol = 1e-12 if prec == bq.FP64 else 1e-5
    for f in got[0]:
        a, b = got[0][f], got[1][f]
        scale = float(np.nanmax(np.abs(b)))
        for end in (slice(0, END), slice(-END, None)):
            assert np.array_equal(np.isnan(a[end]), np.isnan(b[end]))
            assert float(np.nanmax(np.abs(a[end] - b[end]))) <= tol * scale, (precision, f, end)
    rest = slice(4 * END, -4 * END)
    for f in ("eta", "P", "Q"):
        assert float(np.max(np.abs(got[0][f][rest]))) <= tol
