"""The tile pass of the sparse reduce without node sizes (the other reduce
tests ask for them) and with, at the edges of its parts: P classes of slots a
wave, tile and chunk widths, windows continued past 64 entries, more than two
entries of a block at an index (uniform, shared by all ranks, runs), streams
shorter than a window or a code word, unaligned arrays, and a root union in
(thr / 2, thr], where the node sizes decide after a dense guess.  Against the
oracle: indices, sizes and representation equal, values bitwise (additions in
the oracle's association)."""
import numpy as np
import pytest

import oracle
from paper_1802_08021_amd import inputs
from gpu_util import assert_values, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _supports(rng, P, N, k, kind):
    if kind == "shared":
        base = inputs.uniform_subset(rng, N, min(N, k))
        return [base] * P
    if kind == "zipf":  # low indices in most ranks
        u = [np.unique((N * rng.random(2 * k) ** 6).astype(np.uint32)) for _ in range(P)]
        return [np.sort(rng.choice(a, min(k, a.size), replace=False)).astype(np.uint32) for a in u]
    if kind == "runs":  # consecutive indices, tiles apart
        at = [int(rng.integers(0, max(1, N - k))) // 4096 * 4096 for _ in range(P)]
        return [np.arange(a, min(N, a + k), dtype=np.uint32) for a in at]
    ks = [int(rng.integers(0, k + 1)) if kind == "ragged" else min(N, k) for _ in range(P)]
    return [inputs.uniform_subset(rng, N, n) for n in ks]


def _unaligned(a, lead):
    t = to_dev(np.concatenate([np.zeros(lead, a.dtype), a, np.zeros(8, a.dtype)]))
    return t[lead:lead + a.size]


CASES = [
    # P, N, k, support, qbits, delta ("band": 1.5 unions)
    (2, 4097, 4097, "uniform", 0, 0.1),
    (3, 100_003, 9_000, "ragged", 4, 0.01),
    (16, 63, 5, "ragged", 2, 1e-9),
    (16, 1 << 20, 20_000, "uniform", 8, 0.05),
    (17, 300_001, 3, "ragged", 4, 1e-9),
    (24, 3_000_017, 7_001, "ragged", 0, 0.25),
    (33, 700_001, 6_000, "zipf", 2, 0.001),
    (48, 1_000_003, 17_000, "ragged", 0, 0.25),
    (64, 2_097_152, 10_000, "zipf", 0, 0.1),
    (64, 500_000, 9_000, "shared", 0, "band"),
    (100, 400_001, 300, "runs", 4, 1e-6),
    (128, 1_048_576, 10_485, "uniform", 4, 0.1),
    (128, 1_048_577, 30_000, "uniform", 0, 0.1),
    (128, 60_000, 1_000, "shared", 8, "band"),
    (128, 5_000_011, 200, "uniform", 4, 1e-9),
    (129, 80_000, 700, "uniform", 2, "band"),
    (256, 262_144, 1_500, "uniform", 0, 0.1),
    (256, 262_144, 9_000, "uniform", 4, 0.1),
    (256, 2_000_003, 900, "shared", 2, 0.01),
]


@pytest.mark.parametrize("P,N,k,kind,qbits,delta", CASES)
def test_tile_pass(P, N, k, kind, qbits, delta):
    import torch
    from paper_1802_08021_amd import sparcml as S
    rng = np.random.default_rng(P * 1_000_003 + N + k)
    idx = _supports(rng, P, N, k, kind)
    val = [inputs.normal(rng, a.size) for a in idx]
    for v in val:
        v[::7] = 0.0
        v[3::11] = -0.0
    say(f"[accum] P={P} N={N} k={k} {kind} qbits={qbits} delta={delta}")
    if delta == "band":
        delta = 1.5 * np.unique(np.concatenate(idx)).size / N
    ti = [_unaligned(a, r % 4) for r, a in enumerate(idx)]
    kw = dict(vals=[_unaligned(v, 1 + r % 3) for r, v in enumerate(val)])
    if qbits:
        q, scale, val = oracle.quantize(val, qbits, seed=P)
        kw = dict(codes=[_unaligned(a if a.size else np.zeros(1, np.uint8), r % 5) for r, a in enumerate(q)],
                  scales=to_dev(scale), qbits=qbits)
    o = oracle.sparse_reduce(idx, val, N, delta)
    for info in (False, True):
        c = S.ReduceCall(ti, N, delta, node_info=info, **kw)
        for rep in range(2):
            if rep:  # a dense output that is not 16-byte aligned
                c.out_val = torch.empty(N + 1, dtype=torch.float32, device=c.dev)[1:]
                c.out.val = c.out_val.data_ptr()
            c.run_async()
            torch.cuda.synchronize()
            nnz, dense = c.result_header()
            label = f"info={info} run {rep}"
            assert (nnz, bool(dense)) == (o["nnz"], bool(o["dense"])), label
            if dense:
                assert_values(to_np(c.out_val), o["val"], label)
            else:
                np.testing.assert_array_equal(to_np(c.out_idx[:nnz], np.uint32), o["idx"], err_msg=label)
                assert_values(to_np(c.out_val[:nnz]), o["val"], label)
            if info and P > 1:
                np.testing.assert_array_equal(to_np(c.node_nnz).astype(np.uint64), o["node_nnz"].astype(np.uint64))
                np.testing.assert_array_equal(to_np(c.node_dense).astype(np.uint8), o["node_dense"].astype(np.uint8))
