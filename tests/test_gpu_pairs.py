"""Node sizes counted from the indices alone (2^22 indices or more, 2^20 above
128 ranks, where few indices have two entries; the other reduce tests
reach the tile pass's): every number of slots a wave, streams shared by
several waves, several tiles a chunk, more indices held twice than a round of
rows takes (shared supports), entries crowded into a part of the range, a range
with an offset, unaligned and empty streams, and a root union in
(thr / 2, thr].  Against the oracle: sizes and representation of every node and
the root's indices equal."""
import numpy as np
import pytest

import oracle
from paper_1802_08021_amd import inputs
from gpu_util import assert_values, say, to_dev, to_np

pytestmark = pytest.mark.gpu

N22 = 1 << 22
CASES = [
    # P, N, range, entries a stream, shape, qbits, delta ("band": 1.5 unions)
    (2, N22, None, 30_000, "ragged", 0, 0.001),
    (3, N22 + 1, None, 200_001, "uniform", 4, 0.9),
    (5, N22 + 5, None, 60_000, "crowded", 0, 0.02),
    (8, N22, None, 90_000, "shared", 0, "band"),
    (16, N22 + 3, (3, N22), 9_000, "ragged", 2, 0.9),
    (24, N22, None, 3_000, "uniform", 0, 0.001),
    (33, N22 + 77, None, 20_000, "crowded", 0, "band"),
    (64, N22, None, 6_000, "shared", 8, 0.9),
    (64, 40_000_001, None, 20_000, "ragged", 0, 0.9),
    (100, N22, None, 5_000, "uniform", 4, 0.001),
    (128, N22 + 1, None, 300, "ragged", 0, "band"),
    (129, 1 << 20, None, 1_500, "uniform", 0, 0.9),
    (150, 3_000_001, (100_000, 1_290_001), 1_500, "crowded", 0, 0.01),
    (256, 1_100_003, None, 5_000, "shared", 0, "band"),
    (256, 1_000_003, None, 6_000, "uniform", 4, 0.001),
]


@pytest.mark.parametrize("P,N,rng_,k,shape,qbits,delta", CASES)
def test_pairs(P, N, rng_, k, shape, qbits, delta):
    import torch
    from paper_1802_08021_amd import sparcml as S
    rng = np.random.default_rng(P * 15485863 + N)
    lo, hi = rng_ or (0, N)
    R = hi - lo
    same = inputs.uniform_subset(rng, R, k)

    def draw(r):
        if shape == "shared":
            return same
        if shape == "crowded":
            return (R // 4 + inputs.uniform_subset(rng, max(k, R // 16), k)).astype(np.uint32)
        return inputs.uniform_subset(rng, R, int(rng.integers(0, k + 1)) if shape == "ragged" else k)

    idx = [(draw(r) + np.uint32(lo)).astype(np.uint32) for r in range(P)]
    val = [inputs.normal(rng, a.size) for a in idx]
    say(f"[pairs] P={P} N={N} range={rng_} k={k} {shape} qbits={qbits} delta={delta}")
    if delta == "band":
        delta = 1.5 * np.unique(np.concatenate(idx)).size / R
    ti = [to_dev(np.concatenate([np.zeros(r % 3, np.uint32), a]))[r % 3:] for r, a in enumerate(idx)]
    kw = dict(vals=[to_dev(v) for v in val])
    if qbits:
        q, scale, val = oracle.quantize(val, qbits, seed=P)
        kw = dict(codes=[to_dev(a if a.size else np.zeros(1, np.uint8)) for a in q], scales=to_dev(scale), qbits=qbits)
    o = oracle.sparse_reduce_range(idx, val, N, lo, hi, delta)
    if rng_:
        kw.update(lo=lo, hi=hi)
    for info in (True, False):
        c = S.ReduceCall(ti, N, delta, node_info=info, **kw)
        for _ in range(2):  # the second on counters that the first has used
            c.run_async()
        torch.cuda.synchronize()
        nnz, dense = c.result_header()
        assert (nnz, bool(dense)) == (o["nnz"], bool(o["dense"])), info
        if dense:
            assert_values(to_np(c.out_val), o["val"], f"info={info}")
        else:
            np.testing.assert_array_equal(to_np(c.out_idx[:nnz], np.uint32), o["idx"])
            assert_values(to_np(c.out_val[:nnz]), o["val"], f"info={info}")
        if info:
            np.testing.assert_array_equal(to_np(c.node_nnz).astype(np.uint64), o["node_nnz"].astype(np.uint64))
            np.testing.assert_array_equal(to_np(c.node_dense).astype(np.uint8), o["node_dense"].astype(np.uint8))


@pytest.mark.parametrize("P,N,k", [(128, N22 - 1, 900), (129, (1 << 20) - 1, 400)])
def test_below(P, N, k):
    """Just below the rule's sizes, by the tile pass."""
    test_pairs(P, N, None, k, "uniform", 0, 0.001)
