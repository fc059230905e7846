"""Vector-path GEMV at batch 3-8: one slice in flight per lane (more tiles than
allowed CUs) and two (fewer), row and slice remainders, against the oracle and
bit for bit against each other."""
import sys

import numpy as np
import pytest

import paper_2407_13996_amd as sg
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
BF16, F16, F32 = sg.BF16, sg.F16, sg.F32


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("M,K,B,wd,xd", [(515, 2056, 5, BF16, F32), (401, 1024, 8, F32, F32), (262, 3080, 3, F16, F32),
                                         (300, 8, 4, BF16, F32), (259, 2048, 8, F16, BF16), (601, 520, 7, F32, BF16)])
def test_wide_batches(ctx, orc, M, K, B, wd, xd):
    print(f"gemv wide {M}x{K} B={B} w {wd} x {xd}", file=sys.stderr, flush=True)
    shift = 16
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, wd, shift, range(48), M + K, 1, 6)
    xb = tp.x_bits(xd, B * K, M)
    ref, absdot = orc.gemv(pool, pt, wd, M, K, xb, xd, B, shift)
    ys, loads = [], set()
    for cus in (None, range(32), range(50), range(200)):
        n = ctx.num_cus if cus is None else len(cus)
        loads.add(sg.gemv_plan(n, wd, M, K, xd, B)["loads"])
        y = tp.launch_gemv(ctx, d_pool, d_pt, pool_pages, M, K, B, wd, xd, tp.to_dev(xb), shift, cus)
        tp.gemv_check(ctx, y, ref, absdot, M, K, B, wd, xd, cus, tag="wide")
        ys.append(y.view(np.uint32))
    assert loads == {1, 2}
    assert all((y == ys[0]).all() for y in ys[1:])
