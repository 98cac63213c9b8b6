"""The line-coupling kernel at the edges of its split of a line: 16 segments
of up to 8 chunks, panels of 128 chunks (FP64: 16 cells to an x-chunk, 8 to a
y-chunk), blocks of 16 lines.  A segment that took a wrong neighbour value
would show as an error of the size of the wave."""
import math

import numpy as np
import pytest

from oracle.oracle import OracleDomain
from paper_1909_04153_amd import scenarios as S

pytestmark = pytest.mark.gpu

# cells along the line: one chunk; a chunk per segment and one more; a full
# panel, one chunk more, and a third panel
X_CELLS = [16, 256, 257, 2048, 2049, 4112]
Y_CELLS = [8, 128, 129, 1024, 1025, 2056]


@pytest.fixture(scope="module")
def bq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_04153_amd import bq as m

    m.load()
    return m


@pytest.mark.parametrize("along,cells", [("x", n) for n in X_CELLS] + [("y", n) for n in Y_CELLS])
def test_line_coupling_at_segment_and_panel_edges(bq, along, cells):
    # 17 lines: a full block of lines and one line more
    mid = 0.5 * cells * 0.05
    if along == "x":
        spec = S.solitary_flat(nx=cells, ny=17, x0=mid)
    else:
        spec = S.transposed_solitary(nx=17, ny=cells, y0=mid)
    o = OracleDomain(spec["params"], spec["depth_c"])
    assert o.set_state(spec["eta"], spec["P"], spec["Q"]) == 0
    g = bq.domain_from_spec(spec, precision=bq.FP64)
    for _ in range(3):
        assert o.step(4) == 0
        g.step(4)
        for f in ("eta", "P", "Q"):
            a, r = g.read(f), o.read(f)
            s = 0.1 * (math.sqrt(9.81) if f != "eta" else 1.0)   # the wave's natural scale
            e = float(np.linalg.norm(a - r) / max(np.linalg.norm(r), 0.1 * s * math.sqrt(r.size)))
            assert e <= 1e-12 and float(np.max(np.abs(a - r))) <= 1e-11 * s, (along, cells, f, e)
