"""Triad, relayout and batched relayout at the sizes where their tiles and
schedule change (16 KiB tiles up to one 64 KiB tile per allowed CU, the static
schedule up to 32, the queue beyond and on partial masks), with remainders of
1 to 15 bytes.  Bit-exact against the oracle; every byte outside the
destination's pages and length stays as it was; every tile is taken once."""
import sys

import numpy as np
import pytest

import synth
import paper_2407_13996_amd as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
T64 = 65536


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = sg.Context(0)
    yield c
    c.close()


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def up(a):
    return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).to(DEV)


# (CUs, bytes, schedule, tile bytes); None: all 256 CUs
PLANS = [(None, 0, "static", 16384), (None, 15, "static", 16384), (None, 16, "static", 16384),
         (None, 16384 + 4, "static", 16384), (None, 256 * T64, "static", 16384),
         (None, 256 * T64 + 20, "static", T64), (None, 3 * 256 * T64 + 12, "static", T64),
         (range(32), 32 * T64 + 8, "static", 16384), (range(32), 32 * T64 + 16, "static", T64),
         (list(range(64, 96)) + list(range(224, 256)), 64 * T64 - 4, "static", 16384),
         (range(32), 32 * 32 * T64, "static", T64), (range(32), 32 * 32 * T64 + 16, "queue", T64),
         ([7], 4 * T64 + 4, "queue", T64), (range(40), 3 * T64 + 8, "queue", T64)]


class Logged:
    """The work log and CU mask of one launch."""

    def __init__(self, ctx, cus):
        self.ctx, self.cus = ctx, cus

    def __enter__(self):
        self.cu = torch.zeros(self.ctx.num_cus, dtype=torch.int32, device=DEV)
        self.tile = torch.zeros(4096, dtype=torch.int32, device=DEV)
        sg.set_cu_mask(self.ctx, None, self.cus)
        self.ctx.set_worklog(self.cu, self.tile)
        return self

    def __exit__(self, *exc):
        self.tiles, self.schedule = self.ctx.last_tiles(), self.ctx.last_schedule()
        self.ctx.set_worklog(None, None)
        sg.set_cu_mask(self.ctx, None, None)

    def check(self, n_bytes, schedule, tile):
        n = -(-(n_bytes & ~15) // tile)
        assert (self.tiles, self.schedule) == (n, schedule)
        seen = self.tile.cpu().numpy()
        assert (seen[:n] == 1).all() and (seen[n:] == 0).all()
        worked = np.nonzero(self.cu.cpu().numpy())[0].tolist()
        if self.cus is not None:
            assert set(worked) <= set(self.cus)


@pytest.mark.parametrize("cus,n_bytes,schedule,tile", PLANS)
@pytest.mark.parametrize("shift", [11, 16])
def test_relayout_and_batch(ctx, orc, cus, n_bytes, schedule, tile, shift):
    extra = 7 if n_bytes % 16 else 0   # relayouts are byte-granular
    n_bytes += extra - (extra and n_bytes % 16 > 8) * 7
    say(f"relayout {n_bytes} bytes, pages 2^{shift}, CUs {cus}")
    pages = max(1, -(-n_bytes >> shift))
    pool = pages + 5
    src = synth.random_bytes(pool << shift, seed=1)
    dst = synth.random_bytes(pool << shift, seed=2)
    pt_s, pt_d = (synth.random_permutation(pool, seed=s)[:pages].astype(np.uint32) for s in (3, 4))
    ref = dst.copy()
    orc.relayout(ref, pt_d, src, pt_s, n_bytes, shift)
    d_src, d_ps, d_pd = up(src), up(pt_s), up(pt_d)
    for batch in (False, True):
        d_dst = up(dst)
        a, b = sg.paged(d_dst, d_pd, pool), sg.paged(d_src, d_ps, pool)
        with Logged(ctx, cus) as log:
            if batch:
                sg.bimodal_relayout_batch(ctx, [(a, b, n_bytes, shift)])
            else:
                sg.bimodal_relayout(ctx, a, b, n_bytes, shift)
        assert (d_dst.cpu().numpy() == ref).all(), batch
        log.check(n_bytes, schedule, tile)
    assert ctx.device_error() & ~sg.DEVFLAG_GATE_FALLBACK == 0


@pytest.mark.parametrize("cus,n_bytes,schedule,tile", PLANS)
def test_triad(ctx, orc, cus, n_bytes, schedule, tile):
    shift, n = 16, n_bytes // 4
    say(f"triad {n} elements, CUs {cus}")
    pages = max(1, -(-4 * n >> shift))
    pool = pages + 3
    data = [synth.uniform_f32(pool << (shift - 2), seed=s) for s in (1, 2, 3)]
    pts = [synth.random_permutation(pool, seed=s)[:pages].astype(np.uint32) for s in (4, 5, 6)]
    d = [up(x) for x in data]
    d_pt = [up(p) for p in pts]
    ref = data[0].copy()
    orc.triad(ref, pts[0], data[1], pts[1], data[2], pts[2], 3.0, n, shift)
    with Logged(ctx, cus) as log:
        sg.colored_stream(ctx, *[sg.paged(x, p, pool) for x, p in zip(d, d_pt)], 3.0, n, shift)
    assert (d[0].cpu().numpy().view(np.uint32) == ref.view(np.uint32)).all()
    log.check(4 * n, schedule, tile)


def test_bad_page_in_small_and_static_launches(ctx):
    """An entry past the pool is skipped and flagged, the tail's too."""
    shift, pool = 16, 300
    for n_bytes in (3 * T64 + 8, 290 * T64 + 8):
        pages = -(-n_bytes >> shift)
        for bad in (0, pages - 1):
            pt = torch.arange(pages, dtype=torch.int32, device=DEV)
            pt_bad = pt.clone()
            pt_bad[bad] = pool
            src = torch.randint(0, 255, (pool << shift,), dtype=torch.uint8, device=DEV)
            dst = torch.full_like(src, 0xEE)
            ctx.device_error()
            sg.bimodal_relayout(ctx, sg.paged(dst, pt, pool), sg.paged(src, pt_bad, pool), n_bytes, shift)
            assert ctx.device_error() & sg.DEVERR_PT_RANGE
            lo, hi = bad << shift, min((bad + 1) << shift, n_bytes)
            assert bool((dst[lo:hi] == 0xEE).all()) and bool((dst[n_bytes:] == 0xEE).all())
            assert torch.equal(dst[:lo], src[:lo]) and torch.equal(dst[hi:n_bytes], src[hi:n_bytes])


# the static schedule's last size and the queue's first on five, six and all eight XCDs
@pytest.mark.parametrize("triad,cus,per_cu", [(True, 160, 12), (True, 192, 12), (True, 256, 28), (False, 160, 32),
                                              (False, 192, 16), (True, 128, 32), (False, 256, 32)])
def test_schedule_line_by_mask(ctx, triad, cus, per_cu):
    shift = 16
    for tiles, schedule in ((per_cu * cus, "static"), (per_cu * cus + 1, "queue")):
        say(f"{'triad' if triad else 'relayout'} of {tiles} tiles on {cus} CUs")
        ident = torch.arange(tiles, dtype=torch.int32, device=DEV)
        b, c = (torch.randint(-1000, 1000, (tiles << shift - 2,), device=DEV).float() for _ in range(2))
        a = torch.full_like(b, -1.0)
        pa, pb, pc = (sg.paged(t, ident, tiles) for t in (a, b, c))
        sg.set_cu_mask(ctx, None, range(cus))
        if triad:
            sg.colored_stream(ctx, pa, pb, pc, 3.0, b.numel(), shift)
        else:
            sg.bimodal_relayout(ctx, pa, pb, 4 * b.numel(), shift)
        assert (ctx.last_schedule(), ctx.last_tiles()) == (schedule, tiles)
        sg.set_cu_mask(ctx, None, None)
        assert torch.equal(a, b + 3 * c if triad else b)   # (whole numbers: exact either way)
