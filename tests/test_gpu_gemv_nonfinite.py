"""GEMV with infinities and NaN in x: the static schedule's kernels (the ring,
also on rows that cross a page end, the streaming GEMM, the wide vector
kernel) against the oracle's classes and, outside NaN bit for bit, against the
queue schedule's tile loops."""
import sys

import numpy as np
import pytest

import paper_2407_13996_amd as sg
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
BF16, F16, F32 = sg.BF16, sg.F16, sg.F32
INF = {BF16: 0x7F80, F16: 0x7C00, F32: 0x7F800000}
NAN = {BF16: 0x7FC0, F16: 0x7E00, F32: 0x7FC00000}
SIGN = {BF16: 0x8000, F16: 0x8000, F32: 0x80000000}


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


# (M, K, batch, w dtype, x dtype, page shift, whole-XCD mask): the ring with rows
# that cross page ends (both tile heights, both batches, all types), the
# stream kernel at both x forms, one slice in flight
CASES = [(513, 11008, 1, BF16, BF16, 21, None), (1031, 2056, 1, F16, F16, 18, None),
         (300, 5120, 1, F32, F32, 20, None), (700, 6136, 2, F16, F16, 19, None),
         (1301, 4096, 8, BF16, BF16, 17, range(32)), (2900, 4096, 4, BF16, BF16, 21, range(32)),
         (515, 2056, 5, BF16, F32, 16, range(32))]


@pytest.mark.parametrize("kind", ["+inf", "-inf", "both", "nan"])
@pytest.mark.parametrize("M,K,B,wd,xd,shift,whole", CASES)
def test_nonfinite_x(ctx, orc, M, K, B, wd, xd, shift, whole, kind):
    print(f"gemv {M}x{K} B={B} w {wd} x {xd} pages 2^{shift}, {kind} in x", file=sys.stderr, flush=True)
    pool, pt, d_pool, d_pt, pool_pages = tp.upload_w(orc, M, K, wd, shift, range(48), M + K, 1, 6)
    xb = tp.x_bits(xd, B * K, M).copy()
    # in the first batch row only: the others stay finite
    at = {"+inf": [(K // 3, INF[xd])], "-inf": [(K - 1, INF[xd] | SIGN[xd])],
          "both": [(0, INF[xd]), (K // 2, INF[xd] | SIGN[xd])], "nan": [(K // 5, NAN[xd])]}[kind]
    for i, bits in at:
        xb[i] = bits
    with np.errstate(invalid="ignore"):
        ref, absdot = orc.gemv(pool, pt, wd, M, K, xb, xd, B, shift)
    finite = np.isfinite(ref)
    assert not finite[0].any() and finite[1:].all()
    ys = []
    for cus, schedule in ((whole, "static"), (range(100), "queue")):
        y = tp.launch_gemv(ctx, d_pool, d_pt, pool_pages, M, K, B, wd, xd, tp.to_dev(xb), shift, cus)
        assert ctx.last_schedule() == schedule
        bad = np.nonzero((np.isnan(y) != np.isnan(ref)) | (np.isposinf(y) != np.isposinf(ref))
                         | (np.isneginf(y) != np.isneginf(ref)))
        assert bad[0].size == 0, (schedule, bad[1][:8], y[bad][:8], ref[bad][:8])
        depth = sg.gemv_plan(ctx.num_cus if cus is None else len(cus), wd, M, K, xd, B)["sum_depth"]
        err = np.abs(y[1:].astype(np.float64) - ref[1:])
        assert np.all(err <= 2 * depth * 2.0 ** -24 * absdot[1:] + 1e-30)
        ys.append(np.where(np.isnan(y), np.float32(0), y).view(np.uint32))
    assert (ys[0] == ys[1]).all()
