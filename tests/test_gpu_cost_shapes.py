"""What a call costs must follow from the entries it moves, whatever their
shape: a call on indices of one shape is timed against one on as many entries
of an even shape, both on this device, in turn.  The bounds lie at about the
geometric mean of the ratios with and without the code that each case is for
(both stated there, measured on one MI355X)."""
import pytest

from gpu_util import say, torch_dev

pytestmark = pytest.mark.gpu


def _time(*calls):
    """Least time of a call (us), five rounds of the calls in turn."""
    torch, _ = torch_dev()
    best = [float("inf")] * len(calls)
    for _ in range(6):
        for i, c in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(3):
                c()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / 3)
    return best


def _uniform(N, k, r):
    torch, dev = torch_dev()
    g = torch.Generator(device=dev)
    g.manual_seed(1000 + r)
    a = torch.unique(torch.randint(N, (k + k // 4 + 64,), generator=g, device=dev))
    return a[torch.randperm(a.numel(), generator=g, device=dev)[:k]].sort().values


def _reduce(N, idx, info=False, delta=0.01):
    from paper_1802_08021_amd import sparcml as S
    torch, dev = torch_dev()
    idx = [a.to(torch.int32) for a in idx]
    vals = [torch.ones(a.numel(), device=dev) for a in idx]
    return S.ReduceCall(idx, N, delta, vals=vals, node_info=info).run_async


def _comb(N, k, run):
    """Runs of consecutive indices, evenly spread."""
    torch, dev = torch_dev()
    n = k // run
    return ((torch.arange(n, device=dev) * (N // n))[:, None] + torch.arange(run, device=dev)).reshape(-1)


# Runs that all ranks share, the same number of them in every part of the
# range: the tiles they fill hold 64 windows a stream and nothing but heavy
# indices.  One window at a time, and all of them again for every round of
# rows: 27.7, 35 and 15.8 times the uniform call; windows in batches, each
# round its own part: 7.8, 10.9 and 3.5 times.
@pytest.mark.parametrize("P,bound", [(64, 15.0), (128, 20.0), (256, 7.5)])
def test_reduce_shared_runs(P, bound):
    N, k = 1 << 23, 1 << 17
    even = _reduce(N, [_uniform(N, k, r) for r in range(P)])
    runs = _reduce(N, [_comb(N, k, 4096)] * P)
    t0, t1 = _time(even, runs)
    say(f"[cost] shared runs P={P}: {t1:.1f} us, uniform {t0:.1f} us")
    assert t1 < bound * t0


# Entries that crowd into a part of the range, 128 ranks: with a workgroup for
# every part of the range alike, a few of them do all the work, 46, 159 and 62
# times the uniform call; with ranges of equal weight 9.7, 5.3 and 9.2 times.
@pytest.mark.parametrize("shape,bound", [("layer", 17.0), ("run", 45.0), ("low", 20.0)])
def test_reduce_crowded(shape, bound):
    torch, dev = torch_dev()
    P, N, k = 128, 1 << 22, (1 << 22) // 100

    def crowd(r):
        if shape == "run":
            return torch.arange(N // 5, N // 5 + k, device=dev)
        if shape == "layer":
            return N // 3 + _uniform(N // 20, k, r)
        g = torch.Generator(device=dev)
        g.manual_seed(50 + r)
        return torch.unique((N * torch.rand(2 * k, generator=g, device=dev, dtype=torch.float64) ** 6).long())[:k]

    even = _reduce(N, [_uniform(N, k, r) for r in range(P)])
    t0, t1 = _time(even, _reduce(N, [crowd(r) for r in range(P)]))
    say(f"[cost] crowded {shape}: {t1:.1f} us, uniform {t0:.1f} us")
    assert t1 < bound * t0


# Few ranks, one entry in ten indices against one in 160: with tiles that hold
# one window of a stream the denser call takes 6.8, 6.9 and 4.5 times as long
# (its tiles are narrow, and most waves idle); with eight windows 3.0, 3.3 and
# 3.2 times.
@pytest.mark.parametrize("P,bound", [(2, 4.6), (4, 4.8), (8, 3.9)])
def test_reduce_few_dense_ranks(P, bound):
    N = 1 << 24
    thin = _reduce(N, [_uniform(N, N // 160, r) for r in range(P)], delta=1e-3)
    thick = _reduce(N, [_uniform(N, N // 10, r) for r in range(P)], delta=1e-3)
    t0, t1 = _time(thin, thick)
    say(f"[cost] few ranks P={P}: {t1:.1f} us, a sixteenth of the entries {t0:.1f} us")
    assert t1 < bound * t0


# Node sizes where few indices have two entries, against the call without
# them.  In the tile pass, whose tiles are narrow there, 5.1, 2.3 and 1.9 times
# as long; from the indices alone 1.2, 1.3 and 1.4 times.
@pytest.mark.parametrize("P,k,bound", [(256, 1 << 14, 2.5), (128, 1 << 14, 1.7), (64, 1 << 15, 1.65)])
def test_reduce_node_sizes(P, k, bound):
    N = 1 << 24
    idx = [_uniform(N, k, r) for r in range(P)]
    t0, t1 = _time(_reduce(N, idx), _reduce(N, idx, info=True))
    say(f"[cost] node sizes P={P}: {t1:.1f} us, without {t0:.1f} us")
    assert t1 < bound * t0


# Just more entries an index, where the tile pass cuts the ranks into more
# blocks: its tiles narrow to a quarter.  With the same rule for every number of
# ranks 1.3 to 1.5 times the entries cost 1.6, 2.3 and 2.1 times the time; with
# its own above 128 ranks and at 8 and 16 1.3, 1.3 and 1.1 times.
@pytest.mark.parametrize("P,low,high,bound", [(256, 0.38, 0.48, 1.45), (16, 0.38, 0.5, 1.6), (8, 0.24, 0.36, 1.5)])
def test_reduce_blocks(P, low, high, bound):
    N = 1 << 24
    t0, t1 = _time(*[_reduce(N, [_uniform(N, int(N * m / P), r) for r in range(P)]) for m in (low, high)])
    say(f"[cost] blocks P={P}: {t1:.1f} us, a little fewer entries {t0:.1f} us")
    assert t1 < bound * t0


# Top-k of many short rows, ten times the entries against ten times fewer (which
# come from one gather).  With a window of keys, whose histograms are larger than
# the rows, 2.2, 1.06 and 1.8 times as long; with passes over the rows 0.54, 0.68
# and 0.61 times.
@pytest.mark.parametrize("P,N,bound", [(4096, 4096, 1.1), (64, 4096, 0.85), (512, 16384, 1.05)])
def test_topk_short_rows(P, N, bound):
    from paper_1802_08021_amd import sparcml as S
    torch, dev = torch_dev()
    g = torch.Generator(device=dev)
    g.manual_seed(P)
    x = torch.randn(P, N, generator=g, device=dev)
    t0, t1 = _time(S.TopkCall(x, N // 1000).run, S.TopkCall(x, N // 100).run)
    say(f"[cost] top-k of {P} x {N}: {t1:.1f} us, a tenth of the entries {t0:.1f} us")
    assert t1 < bound * t0


# Rows whose selection ends among equal keys, more than a window's units take:
# read for the window in vain, then by the passes: 1.35 times as long as the
# passes at once (which take over where a fourth is selected, and cost much the
# same whatever the count); with the sample's count of them 1.13 times.
def test_topk_ties():
    from paper_1802_08021_amd import sparcml as S
    torch, dev = torch_dev()
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    x = (torch.rand(64, 1 << 20, generator=g, device=dev) - 0.5).sign() * 0.25
    t0, t1 = _time(S.TopkCall(x, (1 << 18) + 100).run, S.TopkCall(x, (1 << 20) // 100).run)
    say(f"[cost] top-k of equal magnitudes: {t1:.1f} us, a fourth of them {t0:.1f} us")
    assert t1 < 1.24 * t0
