"""bq_sync from many threads at once: each call's state comes back through a
slot of its own, calls beyond the number of slots (64) by a copy."""
import threading

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


@pytest.mark.parametrize("threads", [1, 72])
def test_concurrent_syncs_return_their_own_state(bq, threads):
    spec = S.sloping_beach(nx=70, ny=9, dx=0.1, x_toe=1.0)
    rounds = 6

    def trace(d, k):
        out = []
        for r in range(rounds):
            d.step(1 + (k + r) % 3)           # neighbours stand at other steps
            i = d.sync()
            out.append((i.n, i.t, i.dt_last, i.smax, i.mass, i.energy, i.status))
        return out

    want = [trace(bq.domain_from_spec(spec, precision=bq.FP64), k) for k in range(3)]
    doms = [bq.domain_from_spec(spec, precision=bq.FP64) for _ in range(threads)]
    got = [None] * threads
    gate = threading.Barrier(threads)

    def run(k):
        gate.wait(60)
        got[k] = trace(doms[k], k)

    ts = [threading.Thread(target=run, args=(k,)) for k in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(threads):
        assert got[k] == want[k % 3], k
