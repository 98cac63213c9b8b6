"""A call that waits for its stream, made while that stream is being captured,
is refused and leaves the capture as it was: the graph holds the steps alone,
and no memory that the refused calls would have written to."""
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


@pytest.mark.parametrize("call", ["sync", "read"])
def test_refused_under_capture(bq, call):
    import torch

    spec = S.solitary_flat(nx=70, ny=9, dx=0.1, x0=2.0)
    want = bq.domain_from_spec(spec)
    stream = torch.cuda.Stream()
    d = bq.domain_from_spec(spec, stream=stream)
    for x in (want, d):
        x.set_graph_steps(0)
        x.step(2)
        x.wait()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        d.step(3)
        for _ in range(70):         # more often than bq_sync has slots
            with pytest.raises(bq.BqError) as e:
                d.sync() if call == "sync" else d.read("eta")
            assert e.value.code == bq.EDEVICE
    for k in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        want.step(3)
        a, b = d.sync(), want.sync()
        assert a == b and a.n == 5 + 3 * k and a.status == 0
        for f in ("eta", "P", "Q"):
            assert np.array_equal(d.read(f), want.read(f)), (k, f)
