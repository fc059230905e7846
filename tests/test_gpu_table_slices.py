"""Classify through colour tables around the size from which the table is
gathered slice by slice (6 MiB, and 2^22 addresses), whole and ragged last
slices, under the static schedule and the queues, with addresses below and
past the table, and through an empty table; and there with addresses in order,
in runs, in one slice, outside the table, and tiles that begin in order and go on
at random.  Bit-exact against the oracle."""
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


N = 1 << 22


@pytest.mark.parametrize("entries,n,cus", [
    (1 << 22, N, None), ((1 << 22) + 1, N, None), ((1 << 22) + 1, N - 1, None),
    ((6 << 20) - 5, N + 4096 + 17, None), ((6 << 20) - 5, N + 15, range(64)),
    (6 << 20, N, None), ((6 << 20) - 1, N, None), ((6 << 20) + 5, N + 4096 + 17, None), ((6 << 20) + 5, N + 15, range(64)),
    ((4 << 21) + 16, N + 16, "spread"), (1 << 24, N, None), ((1 << 24) + 1, N, None), (0, 5000, None)])
@pytest.mark.parametrize("hist", [False, True])
def test_table_slices(ctx, orc, entries, n, cus, hist):
    print(f"table of {entries} partitions, {n} addresses, hist {hist}, CUs {cus}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(entries + n)
    origin, shift = 1 << 35, 10
    lut = rng.integers(0, 256, size=max(entries, 1), dtype=np.uint8)[:entries]
    span = max(entries, 64) << shift
    addrs = (origin + rng.integers(-(span >> 5), span + (span >> 5), size=n)).astype(np.uint64)
    addrs[:4] = [origin - 1, origin, origin + (entries << shift), (1 << 48) - 1]
    if entries:
        addrs[4] = origin + (entries << shift) - 1
    check(ctx, orc, addrs, lut, origin, shift, cus, hist)


@pytest.mark.parametrize("order", ["lines", "partitions", "runs", "one slice", "strided", "outside", "mixed"])
@pytest.mark.parametrize("cus", [None, "spread"])
def test_table_slices_address_orders(ctx, orc, order, cus):
    print(f"table slices, addresses: {order}, CUs {cus}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(3)
    entries, n, origin, shift = (5 << 21) + 77, N + 4096 + 33, 1 << 35, 10
    lut = rng.integers(0, 256, size=entries, dtype=np.uint8)
    span = entries << shift
    i = np.arange(n, dtype=np.int64)
    at = rng.integers(0, span, size=n)
    if order == "lines":
        off = i * 64
    elif order == "partitions":
        off = i << shift
    elif order == "runs":
        off = (at[i // 64] & ~0xFFFF) + ((i % 64) << shift)
    elif order == "one slice":
        off = (3 << (21 + shift)) + at % (1 << (21 + shift))
    elif order == "strided":
        off = i << 16
    elif order == "outside":
        off = np.where(i % 3 == 0, span + at, -1 - at)
    else:  # in order for the first 0 to 4095 addresses of each tile, then anywhere
        off = np.where(i % 4096 < i // 4096 * 5 % 4096, i << shift, at - 5000)
    if order in ("lines", "partitions", "runs", "strided"):
        off = off % span
    check(ctx, orc, (origin + off).astype(np.uint64), lut, origin, shift, cus, True)


def check(ctx, orc, addrs, lut, origin, shift, cus, hist):
    n = len(addrs)
    ref, ref_hist = orc.classify_lut(addrs, lut, origin, shift)
    t = sg.colour_table(torch.from_numpy(lut).to(DEV), origin, shift)
    d_addrs = torch.from_numpy(addrs.view(np.int64)).to(DEV)
    d_col = torch.full((n + 32,), 0xEE, dtype=torch.uint8, device=DEV)
    d_hist = torch.full((256,), 7, dtype=torch.int64, device=DEV) if hist else None
    if cus == "spread":
        cus = synth.random_cu_subset(ctx.num_cus, 100, seed=2)
    sg.set_cu_mask(ctx, None, cus)
    try:
        for _ in range(2):
            sg.colour_classify_table(ctx, t, d_addrs, d_col, d_hist)
    finally:
        sg.set_cu_mask(ctx, None, None)
    got = d_col.cpu().numpy()
    assert (got[:n] == ref).all() and (got[n:] == 0xEE).all()
    if hist:
        assert (d_hist.cpu().numpy().astype(np.uint64) == ref_hist).all()
    assert ctx.device_error() & ~sg.DEVFLAG_GATE_FALLBACK == 0
