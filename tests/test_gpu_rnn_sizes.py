"""The status update at the sizes where its launches change.

Batches on both sides of the sizes at which resolve merges in LDS (1024 links)
and both launches take larger workgroups (resolve at 16384 and 65536 links,
select past 65536 and 131072 pair rows), with statuses copied in every unit (16,
4 and 2 bytes), some on graphs so small that most rows are read as another
node's r_other while their own status is rewritten.  Two batches in a row: the winner words have to be
zero again after the first.
"""
import numpy as np
import pytest

from tests.gpu_helpers import feat_to_dev, to_dev
from tests.test_gpu_rnn import _check_batch, _log, _small_table, _weights_dev

import synth

pytestmark = pytest.mark.gpu

# (status width, type, d_time, link width, type, links, nodes)
CASES = [
    (100, "f32", 100, 0, "f32", 16384, 9000),     # merged by workgroups of 512 links from here on
    (100, "f32", 12, 0, "f32", 16385, 30000),
    (50, "f32", 20, 6, "f32", 16385, 700),        # rows of 200 bytes
    (33, "f32", 12, 5, "f32", 17001, 30000),      # rows that 16-byte units overlap in (132 bytes)
    (33, "bf16", 12, 6, "bf16", 17001, 30000),    # 2-byte units
    (128, "bf16", 100, 0, "f32", 65535, 40000),   # the most merged 512 links at a time, weight-stationary pass
    (128, "bf16", 100, 0, "f32", 65536, 500),     # merged 1024 at a time, few nodes
    (33, "bf16", 12, 6, "bf16", 257, 60),
    (20, "f32", 12, 0, "f32", 32768, 40000),      # 65 536 pair rows: the most for 256-thread select
    (20, "f32", 12, 0, "f32", 32769, 900),        # one more: 512 threads
    (20, "f32", 12, 0, "f32", 65537, 90000),      # 131 074: 1024
    (20, "f32", 12, 0, "f32", 1023, 30),          # the most that resolve without a merge
    (20, "f32", 12, 0, "f32", 1024, 30),          # merged 256 links at a time
    (20, "f32", 12, 0, "f32", 16383, 400),        # the most of these
    (3, "f32", 12, 4, "f32", 3001, 500),          # 4-byte units (rows of 12 bytes)
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}{c[1]}-t{c[2]}-e{c[3]}{c[4]}-n{c[5]}-N{c[6]}")
def test_update_at_its_sizes(case):
    d, dtype, d_time, e_dim, e_dtype, n, N = case
    rng = np.random.default_rng(n + d)
    ef = None
    if e_dim:
        ef = rng.standard_normal((2 * n - 40, e_dim)).astype(np.float32)   # the last links have no row
        if e_dtype == "bf16":
            ef = synth._to_bf16_bits(ef)
    g, fw, fb = _small_table(N, d_time, feat_to_dev(ef, e_dtype) if ef is not None else None)
    st = rng.standard_normal((N, d)).astype(np.float32)
    st = feat_to_dev(synth._to_bf16_bits(st) if dtype == "bf16" else st, dtype)
    W = synth.gru_weights_for(d, d_time, e_dim, 77 + d)
    for b in range(2):
        src = rng.integers(0, N, n).astype(np.int32)
        dst = rng.integers(0, N, n).astype(np.int32)
        t = np.sort(rng.integers(0, 10**6, n)).astype(np.uint32)
        err, frac = _check_batch(g, st, ef, W, _weights_dev(W), fw, fb, src, dst, t, b * n, f"{case} batch {b}")
        _log(f"{case} batch {b}: max err {err:.3e}, bf16 mismatches {frac:.3%}")
    assert g.status() == 0
    g.close()
