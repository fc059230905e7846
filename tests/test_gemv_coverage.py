"""CPU check: every GEMV kernel variant a benchmark configuration launches
is launched by some GPU parity test as well.  The variant comes from the
library's host-only queries (colored_gemv_plan, colored_gemv_form), the same
functions colored_gemv launches by."""
import pytest

import gemv_cases as gc

sg = pytest.importorskip("paper_2407_13996_amd")


def _variant(case, schedule):
    M, K, B, wd, xd, shift, cus = case
    n = gc.NUM_CUS if cus is None else cus
    p = sg.gemv_plan(n, wd, M, K, xd, B)
    form, loads = sg.gemv_form(n, schedule, wd, M, K, xd, B, shift)
    esize = 4 if wd == gc.F32 else 2
    # (the tile loops) table staged once per workgroup
    whole = form != "tiles" or -(-(M * K * esize) // (1 << shift)) <= 256
    return (schedule, p["path"], form, p["rows"], loads, p["batch_cols"], p["x_once"], wd, xd, whole)


def test_every_benchmarked_gemv_variant_is_gpu_tested():
    tested = {_variant(c, gc.schedule(c[-1])) for c in gc.gpu_cases()}
    timed = [(c, gc.schedule(c[-1])) for c in gc.bench_cases()] + [(c, "queue") for c in gc.bench_spread_cases()]
    missing = {}
    for c, schedule in timed:
        v = _variant(c, schedule)
        if v not in tested:
            missing[v] = c
    assert not missing, f"benchmarked GEMV variants no GPU test reaches: {missing}"


def test_form_rules():
    """Which form of a plan's kernel a launch takes: the ring for batch 1-2, rows
    of two loads per lane or more in one round, one type, pages of 32 rows or of
    whole rows; the streaming MFMA kernel for rows that divide the page and more
    than two tiles per CU (four with x in LDS); both under the static schedule
    only."""
    def form(cus, M, K, B, shift=21, wd=gc.BF16, xd=None, schedule="static"):
        return sg.gemv_form(cus, schedule, wd, M, K, wd if xd is None else xd, B, shift)
    for cus in (64, 128, 192, 256):
        assert form(cus, 4096, 11008, 1) == ("ring", 6)
        assert form(cus, 11008, 4096, 1) == ("ring", 2) == form(cus, 11008, 4096, 2)
        assert form(cus, 4096, 11008, 2) == ("tiles", 3)                   # two rounds
        assert form(cus, 4096, 2048, 1) == ("tiles", 2)                    # one load per lane
        assert form(cus, 4096, 2056, 1) == ("ring", 2)
        assert form(cus, 4096, 11008, 1, xd=gc.F32)[0] == "tiles"
        assert form(cus, 4096, 11008, 1, schedule="queue") == ("tiles", 6)
        assert form(cus, 11008, 4096, 8)[0] == "stream"
        assert form(cus, 11008, 4096, 8, schedule="queue")[0] == "tiles"
        assert form(cus, 4096, 11008, 8)[0] == "tiles"                     # rows cross pages
    assert form(256, 3000, 6000, 1, shift=16)[0] == "tiles"                # 64 KiB: under 32 rows
    assert form(256, 3000, 8192, 1, shift=14) == ("ring", 4)               # one whole row a page
    assert [form(c, 11008, 4096, 4)[0] for c in (64, 128, 192)] == ["stream", "stream", "tiles"]
    assert form(64, 16 * 128, 4096, 8)[0] == "tiles" and form(64, 16 * 128 + 1, 4096, 8)[0] == "stream"


def test_wide_batch_slices():
    """Slices in flight of the vector path at batch 3-8: one above two four-row
    tiles per CU (8 columns, or 4 with x wider than W), above one for fp32 x beside
    16-bit W at 8 columns."""
    def loads(tiles, wd, xd, B):
        return sg.gemv_plan(64, wd, 4 * tiles - 3, 4096, xd, B)["loads"]
    for wd, xd, B, line in ((gc.F32, gc.F32, 8, 128), (gc.F32, gc.BF16, 5, 128), (gc.BF16, gc.F16, 6, 128),
                            (gc.BF16, gc.F32, 8, 64), (gc.F16, gc.F32, 5, 64), (gc.BF16, gc.F32, 4, 128),
                            (gc.F16, gc.F32, 3, 128)):
        assert (loads(line, wd, xd, B), loads(line + 1, wd, xd, B)) == (2, 1), (wd, xd, B)
    assert loads(1000, gc.F32, gc.F32, 4) == 2 == loads(1000, gc.BF16, gc.F16, 3)


def test_form_rejects_bad_arguments():
    L = sg.lib()
    import ctypes
    f, n = ctypes.c_uint32(), ctypes.c_uint32()
    ok = (64, 1, gc.BF16, 16, 16, gc.BF16, 1, 16)
    assert L.colored_gemv_form(*ok, ctypes.byref(f), ctypes.byref(n)) == sg.OK
    assert L.colored_gemv_form(*ok, None, ctypes.byref(n)) == sg.EINVAL
    assert L.colored_gemv_form(*ok, ctypes.byref(f), None) == sg.EINVAL
    for i, bad in ((0, 0), (0, 257), (1, 2), (2, 3), (4, 12), (6, 9), (7, 9), (7, 40)):
        args = ok[:i] + (bad,) + ok[i + 1:]
        assert L.colored_gemv_form(*args, ctypes.byref(f), ctypes.byref(n)) == sg.EINVAL, args


def test_plan_matches_the_c3_sweep_expectations():
    """The two LS layers (4096x11008, 11008x4096) at batch 1 and 8 on 256 CUs: the vector path with
    two-row tiles for 4096 x 11008 batch 1 (six loads per lane: one round
    over a 22 KB row), MFMA from batch 3 on, and a summation depth far below
    the 1e-3 criterion's K."""
    p = sg.gemv_plan(256, gc.BF16, 4096, 11008, gc.BF16, 1)
    assert (p["path"], p["rows"], p["loads"]) == ("valu", 2, 6)
    assert p["tiles"] == 2048
    q = sg.gemv_plan(256, gc.BF16, 11008, 4096, gc.BF16, 8)
    assert q["path"] == "mfma" and q["tiles"] == 11008 // q["rows"]
    for r in (p, q):
        assert 0 < r["sum_depth"] < 200


def test_plan_rejects_bad_arguments():
    with pytest.raises(sg.SgdrcError):
        sg.gemv_plan(0, gc.BF16, 16, 16, gc.BF16, 1)
    with pytest.raises(sg.SgdrcError):
        sg.gemv_plan(257, gc.BF16, 16, 16, gc.BF16, 1)
    with pytest.raises(sg.SgdrcError):
        sg.gemv_plan(64, gc.BF16, 16, 12, gc.BF16, 1)     # K * 2 not a multiple of 16
    with pytest.raises(sg.SgdrcError):
        sg.gemv_plan(64, gc.BF16, 16, 16, gc.BF16, 9)


def test_plan_x_once_rules():
    """Which launches load x once per workgroup: vector path when one round
    of loads covers a row and x is half a tile's bytes (W and x of one
    type); MFMA path at batch 3-4 with rows of at most 8 KiB."""
    for cus in (64, 128, 192, 256):
        p = sg.gemv_plan(cus, gc.BF16, 4096, 11008, gc.BF16, 1)
        assert (p["path"], p["rows"], p["loads"], p["x_once"]) == ("valu", 2, 6, True), (cus, p)
        assert not sg.gemv_plan(cus, gc.BF16, 4096, 11008, gc.F32, 1)["x_once"]
        assert not sg.gemv_plan(cus, gc.BF16, 11008, 4096, gc.BF16, 1)["x_once"]   # x a quarter
        assert sg.gemv_plan(cus, gc.BF16, 11008, 4096, gc.BF16, 2)["x_once"]
        assert not sg.gemv_plan(cus, gc.BF16, 4096, 11008, gc.BF16, 2)["x_once"]   # two rounds
        q = sg.gemv_plan(cus, gc.BF16, 11008, 4096, gc.BF16, 4)
        assert q["path"] == "mfma" and q["batch_cols"] == 4 and q["x_once"], (cus, q)
        assert not sg.gemv_plan(cus, gc.BF16, 4096, 11008, gc.BF16, 4)["x_once"]   # 22 KB rows
        assert not sg.gemv_plan(cus, gc.BF16, 11008, 4096, gc.BF16, 8)["x_once"]   # eight x rows
    # rows longer than six loads per lane cover keep per-tile x
    assert not sg.gemv_plan(256, gc.BF16, 512, 16384, gc.BF16, 1)["x_once"]
