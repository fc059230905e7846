"""Classify's last workgroup under the static schedule (the last n mod 16
addresses, the histogram): grids of one workgroup and more, with and without
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
