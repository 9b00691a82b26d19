"""Launches on either side of the lines from which the number of resident workgroups is bounded, against the oracle."""
import numpy as np
import pytest
import torch

from bagua_workloads import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    assert torch.cuda.is_available()
    return b


def same(t, want):
    return np.array_equal(t.cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("k,n", [(1, (1 << 24) + 1), (2, (1 << 23) - 1), (2, (1 << 23) + 255), (3, 5592406), (5, 3355444), (8, (1 << 21) + 77), (16, (1 << 20) - 1), (16, 1 << 20)])
def test_ring_fp(bg, oracle, k, n):
    print("ring_fp k=%d n=%d" % (k, n), flush=True)
    xs = [draw("normal", n, 7 * k + i, "cpu", 0.02) for i in range(k)]
    out = [torch.full((n,), float("nan"), device="cuda") for _ in range(k)]
    bg.bagua_decentralized_avg(bg.AVG_FP, [x.cuda() for x in xs], out)
    want = oracle.ring_avg_fp([x.numpy() for x in xs])
    assert all(same(o, w) for o, w in zip(out, want))
