"""Eq. (4) aggregation for row types and widths without an instance of their own.

Such launches take the kernel whose widths are run-time values: node rows of
up to 128 and link rows of up to 192 values, fp32 or bf16, at 4-byte
alignment, tables of up to 64 slots, one or two heads.  The cases sit at its
edges: the narrowest and widest rows, widths that cut a 16-byte unit, rows
that start 4 bytes off a 16-byte boundary, no rows of one kind or of both, no
time encoding, one slot and 64, groups of one query and partial last groups,
links past the link table and query nodes out of range.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_helpers import feat_to_dev, to_dev
from tests.test_gpu_parity import AGG_TOL, _agg_dev, agg_error

pytestmark = pytest.mark.gpu

# (node width, type, link width, type, d_time, s, heads)
CASES = [
    (100, "f32", 172, "f32", 100, 20, 1),
    (77, "f32", 191, "f32", 97, 16, 2),
    (4, "f32", 5, "f32", 1, 1, 1),
    (128, "f32", 192, "bf16", 128, 64, 2),
    (126, "bf16", 10, "bf16", 33, 17, 1),
    (128, "bf16", 131, "f32", 100, 10, 2),
    (8, "bf16", 0, "f32", 128, 33, 2),
    (0, "f32", 7, "f32", 0, 10, 1),
    (0, "f32", 0, "f32", 100, 20, 2),
    (127, "f32", 190, "bf16", 101, 12, 1),
    (50, "f32", 0, "f32", 100, 10, 1),
]


def _ids(c):
    n, nt, e, et, d, s, h = c
    return f"{nt}node{n}-{et}edge{e}-t{d}-s{s}-h{h}"


def _off16(t):
    """The same tensor starting 4 bytes past a 16-byte boundary."""
    import torch
    k = 4 // t.element_size()
    flat = torch.empty(t.numel() + k, dtype=t.dtype, device=t.device)
    flat[k:] = t.reshape(-1)
    out = flat[k:].view(t.shape)
    assert out.data_ptr() % 16 == 4
    return out


@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_any_width_aggregation_matches_oracle(case):
    _check_against_oracle(case, _off16)


# Wide link rows without node rows, at 16-byte alignment: the per-query kernel
# or this one by the number of queries (none, or two and more, per wavefront).
WIDE = [(0, "f32", 172, "f32", 100, 20, 1), (0, "f32", 164, "f32", 100, 10, 2),
        (0, "f32", 186, "bf16", 100, 20, 2), (0, "f32", 172, "f32", 100, 64, 1),
        (0, "f32", 172, "f32", 100, 65, 1)]


@pytest.mark.parametrize("case", WIDE, ids=_ids)
def test_wide_link_rows_match_oracle(case):
    _check_against_oracle(case, lambda t: t)


# Around the number of queries up to which narrow rows stay with the tiled
# kernel (1152 on 256 CUs, fewer for wider rows or more slots).
SMALL = [((16, "f32", 16, "f32", 16, 10, 2), (1152, 1153)), ((64, "f32", 30, "f32", 100, 3, 1), (1152, 1153)),
         ((8, "bf16", 9, "f32", 8, 12, 1), (124, 125)), ((0, "f32", 8, "bf16", 0, 3, 1), (99, 100)),
         ((0, "f32", 20, "f32", 20, 4, 2), (424, 425)), ((16, "f32", 0, "f32", 8, 7, 1), (174, 175)),
         ((5, "f32", 6, "f32", 7, 33, 1), (24, 1152))]


@pytest.mark.parametrize("case,nqs", SMALL, ids=[_ids(c) for c, _ in SMALL])
def test_small_launches_match_oracle(case, nqs):
    _check_against_oracle(case, lambda t: t, nqs)


def _check_against_oracle(case, place, nqs=(1, 37, 5003, 40001)):
    import paper_2402_01964_amd as nlb
    dn, nt, de, et, d_time, s, heads = case
    base = synth.workload(1)
    w = dataclasses.replace(synth.scaled(base, 12 * base.batch), node_dim=dn, node_dtype=nt, edge_dim=de,
                            edge_dtype=et, d_time=d_time, s=s)
    src, dst, t, neg = synth.host_links(w)
    ef = synth.host_features(w, "edge") if de else None
    nf = synth.host_features(w, "node") if dn else None
    if ef is not None:
        ef = ef[:w.links - 300]                     # the last links have no row
    fw, fb = synth.time_params(w) if d_time else (np.zeros(0, np.float32),) * 2
    g = nlb.Table(w.num_nodes, s, w.alpha, w.table_seed,
                  time_w=to_dev(fw) if d_time else None, time_b=to_dev(fb) if d_time else None,
                  edge_feat=place(feat_to_dev(ef, et)) if ef is not None else None,
                  node_feat=place(feat_to_dev(nf, nt)) if nf is not None else None)
    o = oracle.Oracle(w.num_nodes, s, w.alpha, w.table_seed)
    g.insert(to_dev(src), to_dev(dst), to_dev(t))
    o.insert(src, dst, t)
    W = synth.agg_weights(w)
    rng = np.random.default_rng(11 * dn + de)
    ends = np.concatenate([src, dst, neg])
    worst = 0.0
    for nq in nqs:
        q = ends[rng.integers(0, len(ends), nq)].astype(np.int32)
        tq = rng.integers(0, int(t[-1]) + 2, nq).astype(np.uint32)
        tq[-1] = int(t[-1]) + 1
        tq[3::9] = 0                                # no valid slot
        gz = g.aggregate(to_dev(q), to_dev(tq), _agg_dev(W), heads=heads).cpu().numpy()
        pos = np.unique(np.append(rng.choice(nq, min(nq, 400), replace=False), nq - 1))
        oz = o.aggregate(q[pos], tq[pos], fw, fb, ef, nf, W, heads=heads)
        worst = max(worst, agg_error(gz[pos], oz))
    print(f"aggregate {_ids(case)}: max scaled error {worst:.3e}", flush=True)
    assert worst <= AGG_TOL
    assert g.status() == nlb.NLB_OK
    # an out-of-range query node: no slots and a zero row, flagged
    qr = np.array([w.num_nodes, int(src[0]), -1], np.int32)
    tr = np.full(3, int(t[-1]) + 1, np.uint32)
    gz = g.aggregate(to_dev(qr), to_dev(tr), _agg_dev(W), heads=heads).cpu().numpy()
    assert g.status() == nlb.NLB_ERANGE
    oz = o.aggregate(qr[1:2], tr[1:2], fw, fb, ef, nf, W, heads=heads)
    assert agg_error(gz[1:2], oz) <= AGG_TOL
    np.testing.assert_array_equal(gz[0], gz[2])
    g.close()


@pytest.mark.parametrize("heads", [1, 2])
def test_an_infinite_feature_stays_with_its_own_queries(heads):
    """Rows of several queries share a block: a neighbour with an infinite
    feature must not reach queries that do not hold it (bit for bit the
    results without it), whatever its own queries get."""
    import torch

    import paper_2402_01964_amd as nlb
    base = synth.workload(1)
    w = dataclasses.replace(synth.scaled(base, 12 * base.batch), node_dim=30, node_dtype="bf16", edge_dim=0)
    src, dst, t, _ = synth.host_links(w)
    nf = feat_to_dev(synth.host_features(w, "node"), "bf16")
    fw, fb = synth.time_params(w)
    g = nlb.Table(w.num_nodes, w.s, w.alpha, w.table_seed, time_w=to_dev(fw), time_b=to_dev(fb), node_feat=nf)
    g.insert(to_dev(src), to_dev(dst), to_dev(t))
    q = to_dev(np.arange(w.num_nodes, dtype=np.int32))
    tq = to_dev(np.full(w.num_nodes, int(t[-1]) + 1, np.uint32))
    W = _agg_dev(synth.agg_weights(w))
    ids = g.sample(q, tq, want=("nbr",))["nbr"]
    bad = int(src[len(src) // 2])
    holds = ((ids == bad).any(1) | (q == bad)).cpu().numpy()
    assert 0 < holds.sum() < w.num_nodes // 2
    for nq in (w.num_nodes, 40):                    # groups of one query; a short launch
        plain = g.aggregate(q[:nq], tq[:nq], W, heads=heads).clone()
        keep = nf[bad].clone()
        nf[bad, 29] = float("inf")
        nf[bad, 3] = float("-inf")
        got = g.aggregate(q[:nq], tq[:nq], W, heads=heads).clone()
        nf[bad] = keep
        rest = torch.from_numpy(~holds[:nq]).to(q.device)
        assert torch.equal(got[rest], plain[rest])
    many = 40 * w.num_nodes                         # groups of 16 queries
    q40, tq40 = q.repeat(40), tq.repeat(40)
    plain = g.aggregate(q40, tq40, W, heads=heads).clone()
    nf[bad, 29] = float("inf")
    got = g.aggregate(q40, tq40, W, heads=heads)
    rest = torch.from_numpy(~np.tile(holds, 40)).to(q.device)
    assert got.shape[0] == many and torch.equal(got[rest], plain[rest])
    g.close()
