"""Batch 1-2 GEMV under the static schedule (the ring kernel: the next rows'
loads stay in flight) against the oracle and, bit for bit, against the queue
schedule (a partial mask; the tile loop): every ring length, rows that cross a
page end, row and slice remainders, more and fewer tiles than workgroups, fewer
rows than a tile, small pages of one or a few whole rows, tables of more than
2048 entries, and page-table entries outside the pool.  Rows of 4 KiB or less
take the tile loop on every mask."""
import sys

import numpy as np
import pytest

import gemv_cases as gc
import paper_2407_13996_amd as sg
import synth
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
BF16, F16, F32 = sg.BF16, sg.F16, sg.F32


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("M,K,B,dt,shift", gc.RING)
def test_ring_equals_oracle_and_queue(ctx, orc, M, K, B, dt, shift):
    print(f"gemv ring {M}x{K} B={B} dtype {dt} pages 2^{shift}", file=sys.stderr, flush=True)
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, dt, shift, range(48), M + K, 1, 6)
    xb = tp.x_bits(dt, B * K, M)
    ref, absdot = orc.gemv(pool, pt, dt, M, K, xb, dt, B, shift)
    ys = []
    for cus in gc.RING_MASKS:
        n = ctx.num_cus if cus is None else len(cus)
        y = tp.launch_gemv(ctx, d_pool, d_pt, pool_pages, M, K, B, dt, dt, tp.to_dev(xb), shift, cus)
        schedule = ctx.last_schedule()
        assert schedule == gc.schedule(n)
        form, loads = sg.gemv_form(n, schedule, dt, M, K, dt, B, shift)
        row = K * (4 if dt == F32 else 2)
        want = ("ring", -(-row // 4096)) if schedule == "static" and row > 4096 else ("tiles", loads)
        assert (form, loads) == want
        tp.gemv_check(ctx, y, ref, absdot, M, K, B, dt, dt, cus, tag="ring")
        ys.append(y.view(np.uint32))
    assert all((y == ys[0]).all() for y in ys[1:])


@pytest.mark.parametrize("bad", [0, 1, 2])
def test_ring_skips_a_bad_page(ctx, orc, bad):
    """Rows on a page outside the pool read as zeros and raise the flag, the
    same bits as the queue schedule's."""
    M, K, shift = 300, 4096, 20
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, BF16, shift, range(48), 9, 1, 6)
    assert len(pt) == 3
    d_bad = d_pt.clone()
    d_bad[bad] = pool_pages
    xb = tp.to_dev(tp.x_bits(BF16, K, 5))
    ys = []
    for cus in (None, list(range(40))):
        y = torch.full((M,), 7.0, device=DEV)
        ctx.device_error()
        sg.set_cu_mask(ctx, None, cus)
        sg.colored_gemv(ctx, sg.paged(d_pool, d_bad, pool_pages), BF16, M, K, xb, BF16, 1, y, shift)
        sg.set_cu_mask(ctx, None, None)
        assert ctx.device_error() & sg.DEVERR_PT_RANGE
        ys.append(y.cpu().numpy().view(np.uint32))
    assert (ys[0] == ys[1]).all()
    rows = np.arange(M) * 2 * K >> shift
    assert (ys[0][rows == bad][:-1] == 0).all() and (ys[0][rows != bad] != 0).any()


def test_ring_skips_bad_small_pages(ctx, orc):
    """The same with a row a page: each page's entry is some wavefront's own."""
    M, K, shift = 2060, 4096, 13
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, BF16, shift, range(48), 9, 1, 6)
    assert len(pt) == M
    xb = tp.to_dev(tp.x_bits(BF16, K, 5))
    for bad in (0, 1, 4, 1027, M - 1):
        d_bad = d_pt.clone()
        d_bad[bad] = pool_pages
        ys = []
        for cus in (None, list(range(40))):
            y = torch.full((M,), 7.0, device=DEV)
            ctx.device_error()
            sg.set_cu_mask(ctx, None, cus)
            sg.colored_gemv(ctx, sg.paged(d_pool, d_bad, pool_pages), BF16, M, K, xb, BF16, 1, y, shift)
            sg.set_cu_mask(ctx, None, None)
            assert ctx.device_error() & sg.DEVERR_PT_RANGE
            ys.append(y.cpu().numpy())
        assert (ys[0].view(np.uint32) == ys[1].view(np.uint32)).all()
        assert ys[0][bad] == 0 and (np.delete(ys[0], bad) != 0).all()
