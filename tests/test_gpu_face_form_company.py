"""FP64 face pass: a cell's result does not depend on which cells share its
wave.  A wave whose sides are all deep takes a straight form of the pass, any
other the general one; shallow spots in a deep basin, in one row of a wave's
two, put deep rows into waves of either kind."""
import numpy as np
import pytest

from paper_1909_04153_amd import scenarios as S

pytestmark = pytest.mark.gpu

LIMIT = 0.5             # depth of the desingularisation threshold
NX, NY = 131, 21        # ends inside a tile on both axes
# one shallow cell per tile (of 64 x 8 cells), in an even or an odd row
SPOTS = [(20, 3), (104, 5), (129, 2), (40, 12), (70, 11), (128, 14), (7, 16), (90, 19), (130, 17)]


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_04153_amd import bq as m

    m.load()
    return m


def _spec(spots, theta=1.3):
    spec = S.closed_basin_hump(nx=NX, ny=NY, dx=0.1, cfl=0.125, fstar_order=1, eps_desing=LIMIT ** 4, theta=theta)
    d = np.ones((NY + 1, NX + 1))
    for i, j in spots:
        d[j:j + 2, i:i + 2] = 0.3
    rng = np.random.default_rng(7)
    eta, P, Q = (a * rng.uniform(-1.0, 1.0, (NY, NX)) for a in (0.01, 0.03, 0.03))
    return dict(spec, depth_c=d, eta=eta, P=P, Q=Q)


def _deep(d):
    """rows of each tile's 64 columns that the straight form may take, along x
    and along y (the surface moves by centimetres: face depths of 0.3, 0.65 and
    1 m stay on their side of the threshold)"""
    fx, fy = 0.5 * (d[:-1] + d[1:]), 0.5 * (d[:, :-1] + d[:, 1:])
    rows_x, rows_y = [], []
    for i0 in range(0, NX, 64):
        rows_x.append(fx[:, max(0, i0 - 1):i0 + 66].min(axis=1) > LIMIT)
        low = fy[:, i0:i0 + 64].min(axis=1) < LIMIT     # faces below cell rows 0 .. NY
        rows_y.append(np.array([not low[max(0, j - 1):j + 3].any() for j in range(NY)]))
    return rows_x, rows_y


def test_spots_mix_the_forms():
    for rows in _deep(_spec(SPOTS)["depth_c"]):
        for tile in rows:
            pairs = [(bool(tile[j]), bool(tile[j + 1])) for j in range(0, NY - 1, 2)]
            assert (True, False) in pairs or (False, True) in pairs
            assert (True, True) in pairs
    assert any((bool(t[j]), bool(t[j + 1])) == (True, False) for t in _deep(_spec(SPOTS)["depth_c"])[0]
               for j in range(0, NY - 1, 2))


@pytest.mark.parametrize("theta", [1.3, 0.0])
@pytest.mark.parametrize("shape", [(8, 16), (8, 32)])
def test_one_row_or_two_to_a_wave(bq, shape, theta):
    # alone, a wave takes one row of a tile, in a launch of over 256 tiles two
    tune = {"lanes": 1, "graph_steps": 0, "reduce_block": 256, "swizzle": 1, "reduce_segments": 1,
            "tile_y": shape[0], "chunk_x": shape[1]}
    spec = _spec(SPOTS, theta)
    got = []
    for filler in (0, 1):
        doms = [bq.domain_from_spec(spec, precision=bq.FP64)]
        if filler:
            doms.append(bq.domain_from_spec(S.solitary_flat(nx=640, ny=256, x0=5.0), precision=bq.FP64))
        b = bq.Batch(doms, lanes=1)
        b.set_tune(tune)
        out = []
        for steps in (1, 1, 10):
            b.step(steps)
            b.sync()
            assert doms[0].sync().status == 0
            out.append([doms[0].read(f) for f in ("eta", "P", "Q")])
        got.append(out)
        b.close()
    for a, r in zip(*got):
        for f, x, y in zip(("eta", "P", "Q"), a, r):
            assert np.array_equal(x, y), (shape, theta, f, np.argwhere(x != y)[:4])


def test_a_shallow_cell_in_a_deep_wave(bq):
    # the surface after one prescribed step, which no line solve has reached:
    # the same with and without the shallow cells wherever their stencil ends
    eta = []
    for spots in ([], SPOTS):
        d = bq.domain_from_spec(_spec(spots), precision=bq.FP64)
        d.step_dt(1e-3)
        assert d.sync().status == 0
        eta.append(d.read("eta"))
    far = np.ones((NY, NX), dtype=bool)
    for i, j in SPOTS:
        far[max(0, j - 3):j + 4, max(0, i - 3):i + 4] = False
    assert far.any(axis=1).all()        # every row, also a spot's own
    assert np.array_equal(eta[0][far], eta[1][far])
    assert not np.array_equal(eta[0], eta[1])
