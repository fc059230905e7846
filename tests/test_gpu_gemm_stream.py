"""Batch 3-8 GEMM under the static schedule with several tiles per workgroup
(chunk loads that run on over tile ends) against the oracle and, bit for bit,
against the queue schedule (a partial mask; tile by tile): both tile heights,
four and eight x rows, x for the whole K in LDS, odd and even chunk counts,
rows shorter than a chunk, a ragged last tile, tiles that span pages, and a
page-table entry outside the pool."""
import sys

import numpy as np
import pytest

import gemv_cases as gc
import paper_2407_13996_amd as sg
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("M,K,B,dt,shift", gc.STREAM)
def test_stream_equals_oracle_and_queue(ctx, orc, M, K, B, dt, shift):
    print(f"gemm stream {M}x{K} B={B} dtype {dt} pages 2^{shift}", file=sys.stderr, flush=True)
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, dt, shift, range(48), M + K, 1, 6)
    xb = tp.x_bits(dt, B * K, M)
    ref, absdot = orc.gemv(pool, pt, dt, M, K, xb, dt, B, shift)
    ys = []
    for cus in gc.STREAM_MASKS:
        n = ctx.num_cus if cus is None else len(cus)
        y = tp.launch_gemv(ctx, d_pool, d_pt, pool_pages, M, K, B, dt, dt, tp.to_dev(xb), shift, cus)
        schedule = ctx.last_schedule()
        assert schedule == gc.schedule(n)
        form, _ = sg.gemv_form(n, schedule, dt, M, K, dt, B, shift)
        if cus is gc.STREAM_MASKS[0]:
            assert form == "stream"
        tp.gemv_check(ctx, y, ref, absdot, M, K, B, dt, dt, cus, tag="stream")
        ys.append(y.view(np.uint32))
    assert all((y == ys[0]).all() for y in ys[1:])


@pytest.mark.parametrize("bad", [0, 2, 4])
def test_stream_skips_a_bad_page(ctx, orc, bad):
    M, K, B, shift = 1280, 4096, 8, 21
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, sg.BF16, shift, range(48), 9, 1, 6)
    assert len(pt) == 5
    d_bad = d_pt.clone()
    d_bad[bad] = pool_pages
    xb = tp.to_dev(tp.x_bits(sg.BF16, B * K, 5))
    ys = []
    for cus in (list(range(32)), list(range(20))):
        y = torch.full((B, M), 7.0, device=DEV)
        ctx.device_error()
        sg.set_cu_mask(ctx, None, cus)
        sg.colored_gemv(ctx, sg.paged(d_pool, d_bad, pool_pages), sg.BF16, M, K, xb, sg.BF16, B, y, shift)
        sg.set_cu_mask(ctx, None, None)
        assert ctx.device_error() & sg.DEVERR_PT_RANGE
        ys.append(y.cpu().numpy().view(np.uint32))
    assert (ys[0] == ys[1]).all()
    rows = np.arange(M) * 2 * K >> shift
    assert (ys[0][:, rows == bad] == 0).all() and (ys[0][:, rows != bad] != 0).any()
