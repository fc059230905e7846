"""The end of a classify under the static schedule (the last n mod 16
addresses, the histogram's last workgroup): grids of one workgroup and more, with and without
a remainder, whole-XCD masks, every number of masks, two calls in a row (the
accumulators and the arrival counters are clear again) and a queued launch
between them.  Bit-exact against the oracle."""
import sys

import numpy as np
import pytest

import synth
import paper_2407_13996_amd as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,K,cus", [(0, 3, None), (7, 1, None), (16, 2, None), (4096, 4, None),
                                     (4111, 5, range(32)), (40001, 6, None), (300007, 7, range(64, 128)),
                                     (2100011, 8, None)])
@pytest.mark.parametrize("hist", [False, True])
def test_last_workgroup(ctx, orc, n, K, cus, hist):
    print(f"classify {n} addresses, K {K}, hist {hist}, CUs {cus}", file=sys.stderr, flush=True)
    masks = synth.xor_masks(K, seed=K, min_bit=12)
    addrs = synth.page_addresses(max(n, 1), seed=n)[:n]
    ref, ref_hist = orc.classify(addrs, masks)
    d_addrs = torch.from_numpy(addrs.view(np.int64)).to(DEV)
    for mask in (cus, range(20), cus):
        d_col = torch.full((n + 32,), 0xEE, dtype=torch.uint8, device=DEV)
        d_hist = torch.full((1 << K,), 9, dtype=torch.int64, device=DEV) if hist else None
        sg.set_cu_mask(ctx, None, mask)
        sg.colour_classify(ctx, masks, d_addrs, d_col, d_hist)
        assert ctx.last_schedule() == ("queue" if mask == range(20) else "static")
        sg.set_cu_mask(ctx, None, None)
        got = d_col.cpu().numpy()
        assert (got[:n] == ref).all() and (got[n:] == 0xEE).all()
        if hist:
            assert (d_hist.cpu().numpy().astype(np.uint64) == ref_hist).all()


def test_overlapping_replays_without_histogram(ctx, orc):
    """Two classifies without a histogram, captured on one stream and replayed
    on two at once: the launches share no state, so every replay colours its
    last n mod 16 addresses, and the stream's next histogram is right."""
    n, K, rounds = (1 << 20) + 5, 6, 24
    masks = synth.xor_masks(K, seed=K, min_bit=12)
    cap = torch.cuda.Stream()
    jobs = []
    for seed in (1, 2):
        addrs = synth.page_addresses(n, seed=seed)
        ref, ref_hist = orc.classify(addrs, masks)
        d_addrs = torch.from_numpy(addrs.view(np.int64)).to(DEV)
        col = torch.full((n,), 0xEE, dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=cap):
            sg.colour_classify(ctx, masks, d_addrs, col)
        assert ctx.last_schedule(cap) == "static"
        jobs.append((g, d_addrs, col, ref, ref_hist, torch.empty(rounds, 5, dtype=torch.uint8, device=DEV),
                     torch.cuda.Stream()))
    torch.cuda.synchronize()
    print(f"{rounds} replays of two captured classifies of {n} addresses on two streams", file=sys.stderr, flush=True)
    for r in range(rounds):
        for g, _, col, _, _, tails, st in jobs:
            with torch.cuda.stream(st):
                g.replay()
                tails[r].copy_(col[-5:])
                col[-5:].fill_(0xEE)
    torch.cuda.synchronize()
    for g, d_addrs, col, ref, ref_hist, tails, _ in jobs:
        assert (col[:-5].cpu().numpy() == ref[:-5]).all()
        assert (tails.cpu().numpy() == ref[-5:]).all()
        d_hist = torch.full((1 << K,), 9, dtype=torch.int64, device=DEV)
        sg.colour_classify(ctx, masks, d_addrs, col, d_hist, cap)
        torch.cuda.synchronize()
        assert (d_hist.cpu().numpy().astype(np.uint64) == ref_hist).all()
    del jobs, g
    torch.cuda.synchronize()
    sg.stream_release(ctx, cap)
