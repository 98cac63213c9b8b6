"""The tile kernels' block widths (256, 512 or 1024 threads, by the launch's
tile count) give the same results bit for bit: a domain alone, whose launch
has few tiles, against the same domain in one launch with a large one."""
import numpy as np
import pytest

from paper_1909_04153_amd import scenarios as S

pytestmark = pytest.mark.gpu

SHAPES = {"FP32": [(16, 16), (16, 32), (8, 16), (8, 32)], "FP64": [(8, 16), (8, 32), (4, 16)]}


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_04153_amd import bq as m

    m.load()
    return m


def _specs():
    # ragged ends on both axes, shores, sponges, both F* readings, the corrector
    return [S.rip_beach_scaled(97, 61, cfl=0.125, fstar_order=1, t_end=0.0),
            S.sloping_beach(nx=133, ny=21, dx=0.1, x_toe=1.0, amp=0.05, ramp=1.0, t_end=0.0),
            S.conical_island(nx=90, ny=90, dx=30.0 / 90),
            S.closed_basin_hump(nx=65, ny=17, dx=0.1, cfl=0.25, fstar_order=2, corrector=1),
            S.solitary_flat(nx=64, ny=16, x0=1.0)]


def _set(b, shape):
    b.set_tune({"lanes": 1, "graph_steps": 0, "reduce_block": 256, "swizzle": 1, "reduce_segments": 1,
                "tile_y": shape[0], "chunk_x": shape[1]})


@pytest.mark.parametrize("precision,shape", [(p, s) for p in SHAPES for s in SHAPES[p]])
def test_block_widths_agree_bitwise(bq, precision, shape):
    prec = getattr(bq, precision)
    steps = 12
    solo = []
    for s in _specs():
        g = bq.domain_from_spec(s, precision=prec)
        b = bq.Batch([g], lanes=1)
        _set(b, shape)
        b.step(steps)
        b.sync()
        assert g.sync().status == 0
        solo.append([g.read(f) for f in ("eta", "P", "Q")])
        b.close()
    # 800 tiles of 16 rows, 1600 of 8, 3200 of 4: the narrow blocks
    doms = [bq.domain_from_spec(s, precision=prec) for s in _specs() + [S.sloping_beach(nx=1600, ny=512, t_end=0.0)]]
    b = bq.Batch(doms, lanes=1)
    _set(b, shape)
    b.step(steps)
    b.sync()
    for s, g, ref in zip(_specs(), doms, solo):
        for f, r in zip(("eta", "P", "Q"), ref):
            assert np.array_equal(g.read(f), r), (precision, shape, s["name"], f)
    b.close()
