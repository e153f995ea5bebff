"""The tile pass where many windows of some streams end in one tile: one, a
few, five to eight and all of a wave's slots continued, with runs of indices
that no one, some and all ranks share (heavy indices by the thousand, in rounds
of rows), wide tiles and narrow, codes that do not start at a word, more than
128 ranks.  Against the oracle: indices, sizes and representation equal, values
bitwise."""
import numpy as np
import pytest

import oracle
from paper_1802_08021_amd import inputs
from gpu_util import assert_values, say, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [
    # P, N, streams with runs, length of a run, runs, shared, entries of the others, qbits, delta
    (2, 200_003, 2, 9_001, 2, False, 0, 0, 0.01),
    (8, 300_001, 3, 5_000, 3, True, 900, 4, 0.01),
    (16, 1_000_003, 16, 3_001, 4, True, 0, 0, 0.01),
    (16, 1_000_003, 5, 700, 9, False, 4_000, 2, 0.9),
    (33, 2_000_003, 7, 2_500, 5, True, 300, 0, 0.0001),
    (64, 1_500_001, 64, 4_097, 3, True, 0, 8, 0.01),
    (64, 1_500_001, 21, 1_111, 6, False, 2_000, 0, 0.5),
    (128, 700_001, 128, 2_049, 2, True, 0, 4, 0.001),
    (128, 3_000_017, 6, 20_000, 1, True, 500, 0, 0.001),
    (128, 1_000_003, 40, 300, 20, False, 1_000, 0, 0.9),
    (150, 400_003, 150, 900, 3, True, 0, 0, 0.001),
    (256, 500_009, 11, 3_000, 2, True, 700, 4, 0.01),
    (256, 300_007, 256, 1_025, 1, True, 0, 0, 0.9),
]


def _runs(rng, N, length, n):
    at = np.sort(rng.integers(0, N - length, n))
    return np.unique(np.concatenate([np.arange(a, a + length) for a in at])).astype(np.uint32)


@pytest.mark.parametrize("P,N,nrun,length,n,shared,k,qbits,delta", CASES)
def test_clusters(P, N, nrun, length, n, shared, k, qbits, delta):
    import torch
    from paper_1802_08021_amd import sparcml as S
    rng = np.random.default_rng(P * 7919 + N)
    one = _runs(rng, N, length, n)
    which = set(rng.permutation(P)[:nrun].tolist())
    idx = []
    for r in range(P):
        a = (one if shared else _runs(rng, N, length, n)) if r in which else np.zeros(0, np.uint32)
        idx.append(np.union1d(a, inputs.uniform_subset(rng, N, int(rng.integers(0, k + 1)))).astype(np.uint32))
    val = [inputs.normal(rng, a.size) for a in idx]
    for v in val:
        v[::9] = 0.0
        v[4::13] = -0.0
    say(f"[clusters] P={P} N={N} {nrun} streams of {n} x {length} shared={shared} qbits={qbits} delta={delta}")
    kw = dict(vals=[to_dev(v) for v in val])
    if qbits:
        q, scale, val = oracle.quantize(val, qbits, seed=P)
        kw = dict(codes=[to_dev(a if a.size else np.zeros(1, np.uint8)) for a in q], scales=to_dev(scale), qbits=qbits)
    o = oracle.sparse_reduce(idx, val, N, delta)
    ti = [to_dev(a) for a in idx]
    for info in (False, True):
        c = S.ReduceCall(ti, N, delta, node_info=info, **kw)
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


# Entries far from even over the range, so that the workgroups take ranges of
# equal weight: P, N, range, entries a stream, shape, qbits, delta
UNEVEN = [
    (2, 1_000_003, None, 150_000, "layer", 0, 0.01),
    (7, 1_000_003, (130_000, 900_001), 9_000, "low", 4, 0.9),
    (16, 3_000_001, None, 30_000, "end", 0, 0.9),
    (17, 200_001, None, 5_000, "one", 2, 0.001),
    (24, 2_000_003, (5, 2_000_003), 40_000, "layer", 8, 0.001),
    (40, 1_000_003, None, 60_000, "low", 0, 0.9),
    (64, 1_500_001, (64, 1_400_000), 20_000, "layer", 0, 0.02),
    (128, 1_000_003, None, 10_000, "low", 4, 0.001),
    (128, 1_000_003, None, 128, "end", 4, 0.9),
    (128, 70_000, None, 3_000, "layer", 0, 0.01),
    (200, 600_001, None, 4_000, "layer", 0, 0.9),
    (256, 500_001, (99_999, 300_001), 3_000, "low", 2, 0.001),
]


@pytest.mark.parametrize("P,N,rng_,k,shape,qbits,delta", UNEVEN)
def test_uneven(P, N, rng_, k, shape, qbits, delta):
    import torch
    from paper_1802_08021_amd import sparcml as S
    rng = np.random.default_rng(P * 104729 + N)
    lo, hi = rng_ or (0, N)
    R = hi - lo

    def draw(r):
        if shape == "one" and r != P // 2:
            return inputs.uniform_subset(rng, R, 3)
        if shape == "low":
            a = np.unique((R * rng.random(2 * k) ** 6).astype(np.uint32))
            return np.sort(rng.choice(a, min(k, a.size), replace=False)).astype(np.uint32)
        width = max(k, R // 20) if shape == "layer" else k
        at = R - width if shape == "end" else R // 3
        return (at + inputs.uniform_subset(rng, width, min(width, k))).astype(np.uint32)

    idx = [(draw(r) + np.uint32(lo)).astype(np.uint32) for r in range(P)]
    val = [inputs.normal(rng, a.size) for a in idx]
    say(f"[uneven] P={P} N={N} range={rng_} k={k} {shape} qbits={qbits} delta={delta}")
    kw = dict(vals=[to_dev(v) for v in val])
    if qbits:
        q, scale, val = oracle.quantize(val, qbits, seed=P)
        kw = dict(codes=[to_dev(a) for a in q], scales=to_dev(scale), qbits=qbits)
    o = oracle.sparse_reduce_range(idx, val, N, lo, hi, delta)
    if rng_:
        kw.update(lo=lo, hi=hi)
    ti = [to_dev(a) for a in idx]
    for info in (False, True):
        c = S.ReduceCall(ti, N, delta, node_info=info, **kw)
        c.run_async()
        torch.cuda.synchronize()
        nnz, dense = c.result_header()
        assert (nnz, bool(dense)) == (o["nnz"], bool(o["dense"])), info
        if dense:
            assert_values(to_np(c.out_val), o["val"], f"info={info}")
        else:
            np.testing.assert_array_equal(to_np(c.out_idx[:nnz], np.uint32), o["idx"])
            assert_values(to_np(c.out_val[:nnz]), o["val"], f"info={info}")
        if info and P > 1:
            np.testing.assert_array_equal(to_np(c.node_nnz).astype(np.uint64), o["node_nnz"].astype(np.uint64))
            np.testing.assert_array_equal(to_np(c.node_dense).astype(np.uint8), o["node_dense"].astype(np.uint8))
