"""Insertion around the batch size where its resolve launch changes (65 536
links: plain atomics, then offers merged by workgroups of 1024 links) and at
half of it.  Graphs with a hub (most offers on a few slots) and without; two
batches, the table against the oracle's after each."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import compare_tables, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32767, 32768, 33001, 65535, 65536])
@pytest.mark.parametrize("hub", [False, True])
def test_insert_at_its_sizes(n, hub):
    import paper_2402_01964_amd as nlb
    rng = np.random.default_rng(n)
    N, s = 40000, 10
    g, o = nlb.Table(N, s, 0.5, 7), oracle.Oracle(N, s, 0.5, 7)
    t0 = 0
    for _ in range(2):
        src = rng.integers(0, N, n).astype(np.int32)
        dst = rng.integers(0, N, n).astype(np.int32)
        if hub:
            src[rng.random(n) < 0.7] = 5
            dst[::50] = 5                           # self-loops of the hub among them
        t = (t0 + np.sort(rng.integers(0, 1000, n))).astype(np.uint32)
        t0 = int(t[-1])
        g.insert(to_dev(src), to_dev(dst), to_dev(t))
        o.insert(src, dst, t)
        compare_tables(g, o)
    assert g.status() == nlb.NLB_OK
    g.close()
