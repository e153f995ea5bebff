"""QSGD with dequantized copies: streams around the edges of a thread's words
and a workgroup's share (1024 and 4096 elements at 8 bits), values and copies
that are not 16-byte aligned, streams without a copy, and descriptor tables in
the launch's arguments (up to 96 streams) or uploaded; against the oracle,
bitwise.  Words around every copy keep what they held."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1802_08021_amd import inputs
from paper_1802_08021_amd import sparcml as S
from gpu_util import say, to_dev, to_np, torch_dev

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 3, 4, 5, 1023, 1025, 4095, 4096, 4097, 8193, 12289]
MARK = 12345.0


def _run(vals, bits, seed, bucket, off_v, off_d, skip):
    torch, dev = torch_dev()
    P, per = len(vals), 8 // bits
    tv = [to_dev(np.concatenate([np.zeros(off_v, np.float32), v, np.zeros(1, np.float32)])) for v in vals]
    td = [torch.full((off_d + v.size + 4,), MARK, device=dev) for v in vals]
    tq = [torch.zeros((v.size + per - 1) // per + 1, dtype=torch.uint8, device=dev) for v in vals]
    arr = (S.Stream * P)()
    for r, v in enumerate(vals):
        arr[r] = S.Stream(None, tv[r].data_ptr() + 4 * off_v, None, None, v.size, 0, 0)
    q = (ctypes.c_void_p * P)(*[c.data_ptr() for c in tq])
    d = (ctypes.c_void_p * P)(*[None if r in skip else t.data_ptr() + 4 * off_d for r, t in enumerate(td)])
    nscale = sum((v.size + bucket - 1) // bucket for v in vals) if bucket else P
    scale = torch.empty(nscale, device=dev)
    op = S.OP_QUANTIZE_BUCKETED if bucket else S.OP_QUANTIZE
    ws = S.alloc_workspace(S.workspace_size(op, P, 1, 0 if bucket else max(v.size for v in vals)), dev)
    tail = (ctypes.cast(q, ctypes.c_void_p), ctypes.c_void_p(scale.data_ptr()), ctypes.cast(d, ctypes.c_void_p),
            ctypes.c_void_p(ws.data_ptr()), ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    if bucket:
        rc = S.lib().sparcml_quantize_bucketed(P, arr, bits, bucket, seed, *tail)
    else:
        rc = S.lib().sparcml_quantize(P, arr, bits, seed, *tail)
    assert rc == 0
    torch.cuda.synchronize()
    return [to_np(c) for c in tq], to_np(scale), [to_np(t) for t in td]


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("last,bucket", [(32768, 0), (40007, 0), (40007, 64), (40007, 4096)])
@pytest.mark.parametrize("off_v,off_d,more", [(0, 0, 0), (1, 0, 83), (0, 3, 84), (2, 1, 0)])
def test_quantize_copies(bits, last, bucket, off_v, off_d, more):
    rng = np.random.default_rng(1000 * bits + last % 100 + bucket)
    vals = [inputs.laplace(rng, 1e-3, n) for n in SIZES + [last] + [17] * more]
    skip = {2, 8}
    seed = 0xFACE_0000 + bits
    say(f"[quant] copies: bits={bits} last={last} bucket={bucket} off={off_v},{off_d} streams={len(vals)}")
    oq, osc, od = oracle.quantize(vals, bits, seed, bucket)
    gq, gsc, gd = _run(vals, bits, seed, bucket, off_v, off_d, skip)
    np.testing.assert_array_equal(gsc.view(np.uint32), osc[: gsc.size].view(np.uint32))
    for r, v in enumerate(vals):
        nb = (v.size * bits + 7) // 8
        np.testing.assert_array_equal(gq[r][:nb], oq[r][:nb], err_msg=f"codes {r}")
        assert gq[r][nb] == 0
        got = gd[r]
        want = np.full(got.size, MARK, np.float32)
        if r not in skip:
            want[off_d: off_d + v.size] = od[r][: v.size]
        np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32), err_msg=f"copy {r}")
