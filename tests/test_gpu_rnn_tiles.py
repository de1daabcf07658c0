"""The tiled GRU pass at the edges of its tiles and row forms.

One workgroup per CU takes 16-row blocks of the winner list, up to three as a
tile: winner counts on both sides of one, two, three and four blocks per
workgroup (256 CUs), and a few rows.  Rows in whole 16-byte units, rows that
the width cuts inside a unit, rows without a unit form; fewer unit blocks than
wavefronts (which then share row blocks), as many, and more; k-steps in whole
groups of four and not.  Every node is touched once, so the winners are 2n.
"""
import numpy as np
import pytest

import paper_2402_01964_amd as nlb
import synth
from tests.gpu_helpers import feat_to_dev, to_dev
from tests.test_gpu_rnn import _check_batch, _log, _small_table, _weights_dev

pytestmark = pytest.mark.gpu

# (status width, type, d_time, link width, type, links)
CASES = [
    (100, "f32", 100, 172, "f32", 2048),    # 4096 winners: one full block per workgroup
    (100, "f32", 100, 186, "bf16", 2049),   # one row of a second
    (100, "f32", 12, 0, "f32", 6144),       # three each
    (100, "f32", 12, 5, "f32", 6145),       # four: two tiles of two
    (33, "f32", 1, 7, "f32", 4097),         # cut units, four unit blocks' wavefronts share row blocks
    (17, "f32", 30, 0, "f32", 6200),        # two unit blocks
    (5, "f32", 9, 4, "f32", 2100),          # one unit block
    (34, "bf16", 20, 10, "bf16", 4099),     # cut bf16 units
    (33, "bf16", 20, 6, "bf16", 4099),      # no unit form
    (50, "f32", 100, 6, "bf16", 2100),      # link rows without one
    (130, "bf16", 64, 64, "f32", 6150),     # nine unit blocks: a wavefront's second
    (50, "f32", 20, 40, "bf16", 8195),      # workgroups of 256 threads
    (200, "f32", 33, 8, "bf16", 2050),      # thirteen
    (100, "f32", 100, 172, "f32", 1),
    (128, "f32", 0, 16, "f32", 9),          # no time encoding
]


def _ids(c):
    return f"d{c[0]}{c[1]}-t{c[2]}-e{c[3]}{c[4]}-n{c[5]}"


@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_update_tiles(case):
    _check_tiles(case)


# bf16 statuses without a time encoding: no column of the input has a second
# bf16 term (no link rows, or bf16 ones), or the link rows' columns alone.
# One, two, four, five and seven k-steps of the status; a few rows and more
# than one tile per workgroup.
BARE = [(d, "bf16", 0, e, et, n) for d, n in ((8, 3), (34, 2100), (64, 6146), (128, 2049), (160, 40), (200, 2050))
        for e, et in ((0, "f32"), (10, "bf16"), (7, "f32"), (4, "bf16"), (3, "f32"))]


@pytest.mark.parametrize("case", BARE, ids=_ids)
def test_update_tiles_without_time_encoding(case):
    _check_tiles(case)


# Rows without a unit form, at more row blocks than CUs: a workgroup per tile of
# one 16-row block, of two from 32 768 pair rows on; remainders of a tile.
ANY = [
    (33, "bf16", 12, 5, "f32", 2053),
    (33, "bf16", 40, 0, "f32", 16385),
    (101, "f32", 20, 3, "f32", 2050),
    (72, "bf16", 33, 4, "bf16", 2049),
    (128, "f32", 100, 6, "bf16", 16390),
    (200, "f32", 0, 2, "f32", 2055),        # no time encoding
    (160, "bf16", 0, 2, "bf16", 16387),
    (6, "bf16", 0, 0, "f32", 2100),
    (3, "f32", 5, 12, "bf16", 16400),
    (1, "bf16", 0, 0, "f32", 1),
]


@pytest.mark.parametrize("case", ANY, ids=_ids)
def test_update_rows_without_unit_form(case):
    _check_tiles(case)


# Batches large enough for a workgroup per tile, rows in piece forms: from 3 row
# blocks per CU (five, nine and ten unit blocks) and from 9.
LARGE = [
    (72, "f32", 33, 10, "bf16", 6150),
    (68, "bf16", 20, 12, "f32", 6149),
    (144, "f32", 100, 0, "f32", 6145),
    (160, "bf16", 100, 24, "bf16", 6146),
    (100, "f32", 100, 0, "f32", 18433),
    (172, "f32", 40, 6, "bf16", 18440),
    (144, "bf16", 0, 0, "f32", 18435),      # no time encoding
    (144, "bf16", 0, 8, "f32", 16386),
    (34, "bf16", 100, 172, "f32", 18434),
]


@pytest.mark.parametrize("case", LARGE, ids=_ids)
def test_update_tiles_of_large_batches(case):
    _check_tiles(case)


@pytest.mark.parametrize("case", [(144, "f32", 100, 0, "f32", 6145), (33, "bf16", 12, 5, "f32", 2053)], ids=_ids)
def test_update_tiles_captured_and_without_allocation(case):
    """Three updates in a row: eager, from the static array, and as replays of
    one HIP graph with other work of the program between them -- bit for bit
    the same statuses."""
    import torch
    d, dtype, d_time, e_dim, e_dtype, n = case
    rng = np.random.default_rng(n)
    N = 2 * n + 5
    ef = rng.standard_normal((n, e_dim)).astype(np.float32) if e_dim else None
    g, _, _ = _small_table(N, d_time, feat_to_dev(ef, e_dtype) if e_dim else None)
    st = rng.standard_normal((N, d)).astype(np.float32)
    st = feat_to_dev(synth._to_bf16_bits(st) if dtype == "bf16" else st, dtype)
    W = _weights_dev(synth.gru_weights_for(d, d_time, e_dim, 5))
    ends = rng.permutation(N)[:2 * n].astype(np.int32)
    args = [to_dev(np.ascontiguousarray(x)) for x in (ends[:n], ends[n:], np.sort(rng.integers(0, 10**6, n)).astype(np.uint32))]
    eager, fixed, graph = st.clone(), st.clone(), st.clone()
    g.rnn_update(*args, 0, W, eager)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured, stream=stream):
        g.rnn_update(*args, 0, W, graph)
    for k in range(3):
        if k:
            g.rnn_update(*args, 0, W, eager)
        g.rnn_update(*args, 0, W, fixed, noalloc=True)
        torch.cuda.synchronize()
        captured.replay()
        torch.cuda.synchronize()
        assert torch.equal(fixed, eager) and torch.equal(graph, eager), f"update {k}"
    assert not torch.equal(eager, st) and g.status() == 0
    g.close()


def _check_tiles(case):
    d, dtype, d_time, e_dim, e_dtype, n = case
    rng = np.random.default_rng(n + d)
    N = 2 * n + 5
    ef = None
    if e_dim:
        ef = rng.standard_normal((max(1, 2 * n - 3), e_dim)).astype(np.float32)   # the last links have no row
        if e_dtype == "bf16":
            ef = synth._to_bf16_bits(ef)
    g, fw, fb = _small_table(N, d_time, feat_to_dev(ef, e_dtype) if ef is not None else None)
    st = rng.standard_normal((N, d)).astype(np.float32)
    st = feat_to_dev(synth._to_bf16_bits(st) if dtype == "bf16" else st, dtype)
    W = synth.gru_weights_for(d, d_time, e_dim, 77 + d)
    for b in range(2):
        ends = rng.permutation(N)[:2 * n].astype(np.int32)
        t = np.sort(rng.integers(0, 10**6, n)).astype(np.uint32)
        err, frac = _check_batch(g, st, ef, W, _weights_dev(W), fw, fb, np.ascontiguousarray(ends[:n]),
                                 np.ascontiguousarray(ends[n:]), t, b * n, f"{case} batch {b}")
        _log(f"{case} batch {b}: max err {err:.3e}, bf16 mismatches {frac:.3%}")
    assert g.status() == 0
    assert g.info()["rnn_form"] == nlb.RNN_FORM_TILED
    g.close()
