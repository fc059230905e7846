"""The page-table builds where their paths part: runs of pages that hold
equal counts (one launch) against hashes and colour tables that take the
counting and the emitting pass, at pool sizes around a run, a round and a
chunk, origins inside a run, pages of fewer and more partitions, and pools
that reach past either end of the table.  Bit-exact against the oracle."""
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


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def check(build, ref, found, n):
    """``build(n, pt)`` against the oracle's table (of the whole pool)."""
    pt = torch.full((n + 8,), -1, dtype=torch.int32, device=DEV)
    if found >= n:
        assert build(n, pt) == found
    else:
        with pytest.raises(sg.SgdrcError) as e:
            build(n, pt)
        assert e.value.code == sg.ENOMEM and e.value.n_found == found
    got = pt.cpu().numpy().view(np.uint32)
    k = min(n, found)
    assert (got[:k] == ref[:k]).all() and (got[k:] == 0xFFFFFFFF).all()


# the runs' equal counts come from the masks' lowest bits: full rank there
# (one launch), rank reached by page-number bit 11 only (runs of 4096 pages),
# never reached (single high bits; a zero mask), and bits inside the page
HASHES = {"low": lambda s: synth.xor_masks(6, seed=3, min_bit=s),
          "eight": lambda s: synth.xor_masks(8, seed=4, min_bit=s),
          "bit11": lambda s: [1 << s, 1 << (s + 11)],
          "high": lambda s: [1 << (s + 12), (1 << (s + 13)) | (1 << s)],
          "zero": lambda s: [0, 1 << (s + 1)],
          "inside": lambda s: [1 << (s - 1), 1 << s, 1 << (s + 2)]}


@pytest.mark.parametrize("pool,offset", [(1, 0), (1023, 1), (1024, 0), (1025, 1023), (4097, 4095),
                                         (70001, 12345), (600001, 7)])
@pytest.mark.parametrize("name", sorted(HASHES))
def test_xor_builds(ctx, orc, name, pool, offset):
    shift = 12
    masks = HASHES[name](shift)
    origin = (1 << 34) + (offset << shift)
    colours = 1 << len(masks)
    for S in ([0], list(range(colours // 2)), list(range(colours))):
        ref, found = orc.pagetable(masks, origin, shift, pool, synth.colour_set_bits(S), pool)
        for n in sorted({0, 1, max(1, found // 3), max(1, found), min(pool, found + 1)}):
            say(f"page table {name}: pool {pool} from page {offset}, |S|={len(S)}, need {n} of {found}")

            def build(n, pt):
                return sg.colour_alloc_pagetable(ctx, masks, origin, shift, pool, S, n, pt)

            def build_noalloc(n, pt):
                d = torch.full((1,), -1, dtype=torch.int64, device=DEV)
                sg.colour_alloc_pagetable_noalloc(ctx, masks, origin, shift, pool, S, n, pt, d)
                if int(d) < n:   # the caller's own comparison
                    raise sg.SgdrcError(sg.ENOMEM, "", int(d))
                return int(d)
            check(build, ref, found, n)
            check(build_noalloc, ref, found, n)


def test_xor_builds_at_the_end_of_the_address_space(ctx, orc):
    shift, pool = 20, 3000
    origin = (1 << 48) - (pool << shift)
    for masks in (synth.xor_masks(4, seed=5, min_bit=shift), [1 << 47, 1 << 35]):
        ref, found = orc.pagetable(masks, origin, shift, pool, synth.colour_set_bits([1]), pool)
        check(lambda n, pt: sg.colour_alloc_pagetable(ctx, masks, origin, shift, pool, [1], n, pt),
              ref, found, max(1, found))


@pytest.mark.parametrize("entries", [1, 15, 16, 17, 4099, 70003, 600011])
@pytest.mark.parametrize("page_shift", [10, 11, 12, 13, 14, 15, 16, 17])
def test_table_builds(ctx, orc, page_shift, entries):
    lut_shift = 11
    rng = np.random.default_rng(entries + page_shift)
    # long stretches of one colour, so that pages of many partitions qualify
    lut = np.repeat(rng.integers(0, 8, size=entries // 40 + 1), 40)[:entries].astype(np.uint8)
    lut[rng.random(entries) < 0.002] = 255
    origin = 1 << 34
    d_lut = torch.from_numpy(lut).to(DEV)
    t = sg.colour_table(d_lut, origin, lut_shift)
    P = 1 << page_shift
    # from the table's start, from before it, and (small pages) inside a partition
    for start in (0, -3 * P, 5 * P):
        pool = max(1, ((entries << lut_shift) - start) // P + 2)
        S = [0, 1, 2, 5]
        ref, found = orc.pagetable_lut(lut, origin, lut_shift, origin + start, page_shift, pool,
                                       synth.colour_set_bits(S), pool)
        for n in sorted({0, 1, max(1, found // 2), max(1, found), min(pool, found + 1)}):
            say(f"table build: {entries} partitions, pages 2^{page_shift} from {start}, need {n} of {found}")
            check(lambda n, pt: sg.colour_alloc_pagetable_table(ctx, t, origin + start, page_shift,
                                                                pool, S, n, pt), ref, found, n)
