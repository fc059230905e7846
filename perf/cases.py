"""The work that a program has this library do, as cases that can be timed.

Each case is one call, or the few calls that belong together, through the
package's public functions: colouring addresses, building page tables,
streaming and moving paged tensors, the memory-bound layer, the change of
co-location state, and the co-located pair itself.  Sizes are those of the
benchmark and the tests, or generic ones between and around them.

All inputs come from a seed.  Pool addresses are synthetic (``ORIGIN``), so
that page tables do not depend on where the allocator put a pool.
"""
import math
import random

import torch

import paper_2407_13996_amd as sg

ORIGIN = 1 << 36
DTYPES = {"f32": (sg.F32, torch.float32), "bf16": (sg.BF16, torch.bfloat16),
          "f16": (sg.F16, torch.float16)}
DEV = "cuda"
_CTX = None
_STREAMS = {}


def listed():
    return [
        # the plumbing case: a small pool's addresses are coloured and counted
        {"name": "classify-64k-hist", "kind": "classify", "n": 65536, "k": 4, "hist": True},
        # colouring a whole address population, as when a pool map is made
        {"name": "classify-64m", "kind": "classify", "n": 1 << 26, "k": 6, "hist": False},
        # a non-linear hash's table over 16 GiB in 1 KiB partitions: colour
        # addresses through it, then list the sectors of a colour set
        {"name": "table-16m", "kind": "table", "entries": 1 << 24, "n": 1 << 24, "need": 1 << 20},
        # the page tables of three 1 GiB arrays on 8 of 64 colours
        {"name": "pagetable-400k", "kind": "pagetable", "pool": 409600, "shift": 16, "k": 6,
         "colours": 8, "need": 49152, "noalloc": False},
        # a best-effort stream over three 1 GiB arrays on 16 of 64 colours
        {"name": "triad-1g", "kind": "triad", "n": 1 << 28, "shift": 16, "colours": 16, "cus": 256},
        # an odd-sized small stream on 2 KiB sectors
        {"name": "triad-3m-sectors", "kind": "triad", "n": 3000001, "shift": 11, "colours": 32,
         "cus": 256},
        # moving one large half-precision tensor to its restricted pages
        {"name": "relayout-1g", "kind": "relayout", "bytes": 1 << 30, "shift": 16, "colours": 16,
         "to_part": True, "cus": 256},
        # a change of co-location state and back, with one layer's matrices
        {"name": "switch-layer", "kind": "switch", "hidden": 4096, "inner": 11008, "shift": 21},
        # the smallest layer: one fp32 matrix that fits in the caches
        {"name": "gemv-1k-f32-b1", "kind": "gemv", "m": 1024, "k": 1024, "w": "f32", "x": "f32",
         "batch": 1, "cus": 256, "spread": False, "shift": 16, "layers": 1},
        # single-sequence decoding through the down projections of four layers
        {"name": "gemv-down-bf16-b1", "kind": "gemv", "m": 4096, "k": 11008, "w": "bf16",
         "x": "bf16", "batch": 1, "cus": 256, "spread": False, "shift": 21, "layers": 4},
        # eight sequences through the up projections of four layers
        {"name": "gemv-up-bf16-b8", "kind": "gemv", "m": 11008, "k": 4096, "w": "bf16",
         "x": "bf16", "batch": 8, "cus": 256, "spread": False, "shift": 21, "layers": 4},
        # the co-located pair: latency-sensitive layers on 192 CUs beside a
        # best-effort stream on the other 64
        {"name": "corun", "kind": "corun", "m": 4096, "k": 11008, "calls": 32, "layers": 8,
         "n": 1 << 27},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["classify", "table", "pagetable", "triad", "relayout", "switch", "gemv",
                       "gemv", "gemv", "corun"])
    if kind == "classify":
        return {"kind": kind, "n": _log(rng, 4096, 1 << 26), "k": rng.randint(1, 8),
                "hist": rng.random() < 0.5}
    if kind == "table":
        entries = _log(rng, 1 << 16, 1 << 24)
        return {"kind": kind, "entries": entries, "n": _log(rng, 1 << 16, 1 << 24),
                "need": max(1, entries // rng.randint(8, 64))}
    if kind == "pagetable":
        pool, colours = _log(rng, 1024, 1 << 22), rng.choice([8, 16, 32, 48, 64])
        most = pool // 256 * 4 * colours
        return {"kind": kind, "pool": pool, "shift": rng.choice([10, 12, 16, 21]), "k": 6,
                "colours": colours, "need": rng.randint(max(1, most // 4), most),
                "noalloc": rng.random() < 0.5}
    if kind == "triad":
        return {"kind": kind, "n": _log(rng, 1000, 1 << 28), "shift": rng.choice([10, 11, 12, 16, 21]),
                "colours": rng.choice([16, 32, 48, 64]), "cus": rng.choice([64, 128, 192, 256, 256])}
    if kind == "relayout":
        return {"kind": kind, "bytes": _log(rng, 10000, 1 << 30), "shift": rng.choice([10, 12, 16, 21]),
                "colours": rng.choice([16, 32, 48, 64]), "to_part": rng.random() < 0.5,
                "cus": rng.choice([64, 128, 192, 256, 256])}
    if kind == "switch":
        hidden = 8 * _log(rng, 64, 512)
        return {"kind": kind, "hidden": hidden, "inner": 8 * _log(rng, hidden // 8, 1376),
                "shift": rng.choice([16, 21])}
    if kind == "gemv":
        m, k = _log(rng, 256, 11008), 8 * _log(rng, 32, 1376)
        w = rng.choice(["bf16", "bf16", "f16", "f32"])
        x = w if rng.random() < 0.8 else "f32"
        return {"kind": kind, "m": m, "k": k, "w": w, "x": x, "batch": rng.choice([1, 1, 2, 3, 4, 5, 8, 8]),
                "cus": rng.choice([64, 128, 192, 256, 256]), "spread": rng.random() < 0.25,
                "shift": rng.choice([16, 21]), "layers": rng.randint(1, 4)}
    return {"kind": kind, "m": _log(rng, 2048, 4096), "k": 8 * _log(rng, 512, 1376),
            "calls": rng.randint(16, 32), "layers": 8, "n": _log(rng, 1 << 26, 1 << 27)}


# ---------------------------------------------------------------- inputs

def _ctx():
    global _CTX
    if _CTX is None:
        _CTX = sg.Context(0)
    return _CTX


def _stream(name):
    if name not in _STREAMS:
        _STREAMS[name] = torch.cuda.Stream()
    return _STREAMS[name]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rank(vectors):
    basis = []
    for v in vectors:
        for b in basis:
            v = min(v, v ^ b)
        if v:
            basis = sorted(basis + [v], reverse=True)
    return len(basis)


def _masks(k, lo):
    """k random masks on address bits lo..40, of full rank also on their k + 2
    lowest bits, so that every aligned run of 2^(k+2) pages holds all colours
    alike."""
    rng = random.Random(1)
    window = ((1 << (k + 2)) - 1) << lo
    while True:
        masks = [rng.getrandbits(41 - lo) << lo for _ in range(k)]
        if _rank(masks) == k and _rank([m & window for m in masks]) == k:
            return masks


def _table(shift, pool_pages, colours, need):
    """The first ``need`` pool pages with colours below ``colours`` of 64."""
    pt = torch.empty(need, dtype=torch.int32, device=DEV)
    sg.colour_alloc_pagetable(_ctx(), _masks(6, shift), ORIGIN, shift, pool_pages, range(colours),
                              need, pt)
    return pt


def _pages_for(need, colours):
    """Pool pages that hold ``need`` pages of ``colours`` of 64 colours."""
    return -(-need // (4 * colours)) * 256


def _cus(n, spread):
    if n == 256:
        return None
    return [x * 32 + i for x in range(8) for i in range(n // 8)] if spread else range(n)


def _scatter(pool, pt, shift, flat):
    """Puts the bytes of ``flat`` (a whole number of 4-byte words) on the pool's pages ``pt``."""
    words = (1 << shift) // 4
    pages = pool.view(torch.int32).view(-1, words)
    w = flat.view(torch.int32)
    whole = w.numel() // words
    pages[pt[:whole].long()] = w[:whole * words].view(whole, words)
    if w.numel() > whole * words:
        pages[int(pt[whole]), :w.numel() - whole * words] = w[whole * words:]


def _classify_inputs(case, seed):
    return torch.randint(0, 1 << 36, (case["n"],), generator=_gen(seed), device=DEV) << 12


def _table_inputs(case, seed):
    g = _gen(seed)
    lut = torch.randint(0, 64, (case["entries"],), generator=g, device=DEV, dtype=torch.uint8)
    # one address in 32 lies past the table and has no colour
    span = case["entries"] + case["entries"] // 31
    addrs = ORIGIN + torch.randint(0, span << 10, (case["n"],), generator=g, device=DEV)
    return lut, addrs


def _triad_inputs(case, seed):
    g = _gen(seed)
    return [torch.rand(case["n"], generator=g, device=DEV).mul_(2).sub_(1) for _ in range(2)]


def _relayout_inputs(case, seed):
    n = -(-case["bytes"] // 4)
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=_gen(seed), device=DEV, dtype=torch.int32)


def _weights(m, k, dtype, layers, seed):
    g = _gen(seed)
    return [torch.randn(m, k, generator=g, device=DEV).mul_(0.02).to(dtype) for _ in range(layers)]


def _acts(batch, k, dtype, count, seed):
    g = _gen(seed + 1000003)
    return [torch.randn(batch, k, generator=g, device=DEV).to(dtype) for _ in range(count)]


def _paged_weights(ws, shift):
    """The matrices on colours 0..47 of 64 of one pool, with their tables."""
    per = -(-ws[0].numel() * ws[0].element_size() >> shift)
    pages = _pages_for(per * len(ws), 48)
    pool = torch.zeros(pages << shift, dtype=torch.uint8, device=DEV)
    pt = _table(shift, pages, 48, per * len(ws))
    out = []
    for i, w in enumerate(ws):
        mine = pt[i * per:(i + 1) * per]
        _scatter(pool, mine, shift, w.view(-1))
        out.append(sg.paged(pool, mine, pages))
    return out


def _paged_triad(case, seed):
    n, shift = case["n"], case["shift"]
    per = -(-4 * n >> shift)
    pages = _pages_for(3 * per, case["colours"])
    pool = torch.zeros(pages << shift, dtype=torch.uint8, device=DEV)
    pt = _table(shift, pages, case["colours"], 3 * per)
    b, c = _triad_inputs(case, seed)
    _scatter(pool, pt[per:2 * per], shift, b)
    _scatter(pool, pt[2 * per:], shift, c)
    # the pages up to the last of a: a's tables entries ascend, b's come after
    last = int(pt[per - 1])
    return {"abc": [sg.paged(pool, pt[i * per:(i + 1) * per], pages) for i in range(3)],
            "a": pool[:(last + 1) << shift].view(torch.float32)}


def prepare(case, seed):
    ctx, kind = _ctx(), case["kind"]
    st = {"case": case, "ctx": ctx}
    sg.set_cu_mask(ctx, None, _cus(case.get("cus", 256), case.get("spread", False)))
    if kind == "classify":
        st["masks"] = _masks(case["k"], 12)
        st["addrs"] = _classify_inputs(case, seed)
        st["colours"] = torch.zeros(case["n"], dtype=torch.uint8, device=DEV)
        st["hist"] = torch.zeros(1 << case["k"], dtype=torch.int64, device=DEV) if case["hist"] else None
    elif kind == "table":
        lut, st["addrs"] = _table_inputs(case, seed)
        st["table"] = sg.colour_table(lut, ORIGIN, 10)
        st["colours"] = torch.zeros(case["n"], dtype=torch.uint8, device=DEV)
        st["hist"] = torch.zeros(256, dtype=torch.int64, device=DEV)
        st["pt"] = torch.zeros(case["need"], dtype=torch.int32, device=DEV)
    elif kind == "pagetable":
        # another seed is another place in the address space
        st["masks"] = _masks(case["k"], case["shift"])
        st["origin"] = _origin(case, seed)
        st["pt"] = torch.zeros(case["need"], dtype=torch.int32, device=DEV)
        st["found"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    elif kind == "triad":
        st.update(_paged_triad(case, seed))
    elif kind == "relayout":
        shift = case["shift"]
        per = -(-case["bytes"] >> shift)
        pages = _pages_for(per, case["colours"])
        part_pt = _table(shift, pages, case["colours"], per)
        all_pt = torch.arange(per, dtype=torch.int32, device=DEV)
        part = torch.zeros(pages << shift, dtype=torch.uint8, device=DEV)
        every = torch.zeros(per << shift, dtype=torch.uint8, device=DEV)
        flat = _relayout_inputs(case, seed)
        if case["to_part"]:
            _scatter(every, all_pt, shift, flat)
        else:
            _scatter(part, part_pt, shift, flat)
        forms = [sg.paged(every, all_pt, per), sg.paged(part, part_pt, pages)]
        st["src"], st["dst"] = forms if case["to_part"] else forms[::-1]
        st["out"] = (part if case["to_part"] else every).view(torch.int16)
    elif kind == "switch":
        st["bm"] = sg.Bimodal(ctx)
        st["out"] = []
        for every, ws in _switch_inputs(case, seed):
            shift = case["shift"]
            per = -(-ws.numel() * 2 >> shift)
            pages = _pages_for(per, 48)
            part = torch.zeros(pages << shift, dtype=torch.uint8, device=DEV)
            part_pt = _table(shift, pages, 48, per)
            st["bm"].register(sg.BM_LS_TENSOR, sg.paged(every, torch.arange(per, dtype=torch.int32, device=DEV), per),
                              sg.paged(part, part_pt, pages), ws.numel() * 2, shift)
            st["out"] += [every.view(torch.int16), part.view(torch.int16)]
    elif kind == "gemv":
        w, x = DTYPES[case["w"]], DTYPES[case["x"]]
        st["w"] = _paged_weights(_weights(case["m"], case["k"], w[1], case["layers"], seed), case["shift"])
        st["x"] = _acts(case["batch"], case["k"], x[1], case["layers"], seed)
        st["y"] = [torch.zeros(case["batch"], case["m"], device=DEV) for _ in range(case["layers"])]
    else:
        ls, be = _stream("ls"), _stream("be")
        sg.set_cu_mask(ctx, ls, range(192))
        sg.set_cu_mask(ctx, be, range(192, 256))
        st.update(_paged_triad({"n": case["n"], "shift": 16, "colours": 16}, seed))
        st["w"] = _paged_weights(_weights(case["m"], case["k"], torch.bfloat16, case["layers"], seed), 21)
        st["x"] = _acts(1, case["k"], torch.bfloat16, case["calls"], seed)
        st["y"] = [torch.zeros(1, case["m"], device=DEV) for _ in range(case["calls"])]
    return st


def _origin(case, seed):
    return ORIGIN + ((seed % 4096) * 256 << case["shift"])


def _switch_inputs(case, seed):
    """Up and down projection of one layer, whole pages each."""
    out = []
    for i, (m, k) in enumerate(((case["inner"], case["hidden"]), (case["hidden"], case["inner"]))):
        w = _weights(m, k, torch.bfloat16, 1, seed + i)[0].view(-1)
        per = -(-w.numel() * 2 >> case["shift"])
        every = torch.zeros(per << case["shift"], dtype=torch.uint8, device=DEV)
        every[:w.numel() * 2] = w.view(torch.uint8)
        out.append((every, w))
    return out


# ------------------------------------------------------------------ calls

def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "classify":
        sg.colour_classify(ctx, st["masks"], st["addrs"], st["colours"], st["hist"])
        return {"colours": st["colours"], "hist": st["hist"]}
    if kind == "table":
        sg.colour_classify_table(ctx, st["table"], st["addrs"], st["colours"], st["hist"])
        found = sg.colour_alloc_pagetable_table(ctx, st["table"], ORIGIN, 10, case["entries"],
                                                range(16), case["need"], st["pt"])
        return {"colours": st["colours"], "hist": st["hist"], "pt": st["pt"], "found": found}
    if kind == "pagetable":
        build = (ctx, st["masks"], st["origin"], case["shift"], case["pool"], range(case["colours"]),
                 case["need"], st["pt"])
        if case["noalloc"]:
            sg.colour_alloc_pagetable_noalloc(*build, st["found"])
            return {"pt": st["pt"], "found": st["found"]}
        return {"pt": st["pt"], "found": sg.colour_alloc_pagetable(*build)}
    if kind == "triad":
        sg.colored_stream(ctx, *st["abc"], 3.0, case["n"], case["shift"])
        return st["a"]
    if kind == "relayout":
        sg.bimodal_relayout(ctx, st["dst"], st["src"], case["bytes"], case["shift"])
        return st["out"]
    if kind == "switch":
        st["bm"].set_state(sg.BM_COLOCATED)
        st["bm"].set_state(sg.BM_MONOPOLY)
        return st["out"]
    if kind == "gemv":
        w, x = DTYPES[case["w"]][0], DTYPES[case["x"]][0]
        for i in range(case["layers"]):
            sg.colored_gemv(ctx, st["w"][i], w, case["m"], case["k"], st["x"][i], x, case["batch"],
                            st["y"][i], case["shift"])
        return st["y"]
    ls, be, cur = _stream("ls"), _stream("be"), torch.cuda.current_stream()
    ls.wait_stream(cur)
    be.wait_stream(cur)
    sg.colored_stream(ctx, *st["abc"], 3.0, case["n"], 16, be)
    for i in range(case["calls"]):
        sg.colored_gemv(ctx, st["w"][i % case["layers"]], sg.BF16, case["m"], case["k"], st["x"][i],
                        sg.BF16, 1, st["y"][i], 21, ls)
    cur.wait_stream(ls)
    cur.wait_stream(be)
    return {"y": st["y"], "a": st["a"]}


def work(case):
    kind = case["kind"]
    if kind == "classify":
        return {"bytes": 9 * case["n"] + (8 << case["k"] if case["hist"] else 0), "flops": 0}
    if kind == "table":
        return {"bytes": 9 * case["n"] + 2 * case["entries"] + 4 * case["need"] + 2048, "flops": 0}
    if kind == "pagetable":
        return {"bytes": 4 * case["need"] + 8, "flops": 0}
    if kind == "triad":
        return {"bytes": 12 * case["n"], "flops": 2 * case["n"]}
    if kind == "relayout":
        return {"bytes": 2 * case["bytes"], "flops": 0}
    if kind == "switch":
        return {"bytes": 2 * 2 * 2 * 2 * case["hidden"] * case["inner"], "flops": 0}
    if kind == "gemv":
        m, k, b = case["m"], case["k"], case["batch"]
        ws, xs = (DTYPES[case[d]][1].itemsize for d in ("w", "x"))
        return {"bytes": case["layers"] * (m * k * ws + b * k * xs + 4 * b * m),
                "flops": case["layers"] * 2 * b * m * k}
    m, k = case["m"], case["k"]
    return {"bytes": case["calls"] * (2 * m * k + 2 * k + 4 * m) + 12 * case["n"],
            "flops": case["calls"] * 2 * m * k + 2 * case["n"]}


def tolerance(case):
    if case["kind"] in ("gemv", "corun"):
        # fp32 sums of up to 11008 products, whose order is free: up to 1.4e-7
        # from the 64-bit sums here
        return {"rel": 1e-6, "max": 1e-5}
    # colours, tables and copies are whole numbers; the triad has one rounding
    return "exact"


# ----------------------------------------------------- 64-bit references

def _parity(v):
    for s in (32, 16, 8, 4, 2, 1):
        v = v ^ (v >> s)
    return v & 1


def _colours(masks, addrs):
    c = torch.zeros_like(addrs)
    for i, m in enumerate(masks):
        c |= _parity(addrs & m) << i
    return c


def _exact_table(masks, origin, shift, pool, colours):
    pages = torch.arange(pool, device=DEV)
    return torch.nonzero(_colours(masks, origin + (pages << shift)) < colours).view(-1)


def _exact_triad(case, seed):
    n, shift = case["n"], case["shift"]
    per = -(-4 * n >> shift)
    pt = _exact_table(_masks(6, shift), ORIGIN, shift, _pages_for(3 * per, case["colours"]),
                      case["colours"])[:per]
    b, c = _triad_inputs(case, seed)
    a = 3.0 * c.double() + b.double()
    words = (1 << shift) // 4
    out = torch.zeros(int(pt[-1]) + 1, words, dtype=torch.float64, device=DEV)
    out[pt] = torch.nn.functional.pad(a, (0, per * words - n)).view(per, words)
    return out.view(-1)


def _exact_gemv(w, x):
    return x.double() @ w.double().t()


def exact(case, seed):
    kind = case["kind"]
    if kind == "classify":
        c = _colours(_masks(case["k"], 12), _classify_inputs(case, seed))
        return {"colours": c.to(torch.uint8),
                "hist": torch.bincount(c, minlength=1 << case["k"]) if case["hist"] else None}
    if kind == "table":
        lut, addrs = _table_inputs(case, seed)
        i = (addrs - ORIGIN) >> 10
        inside = i < case["entries"]
        c = torch.where(inside, lut[i.clamp(max=case["entries"] - 1)].long(), 255)
        pages = torch.nonzero(lut < 16).view(-1)
        return {"colours": c.to(torch.uint8), "hist": torch.bincount(c, minlength=256),
                "pt": pages[:case["need"]].to(torch.int32), "found": pages.numel()}
    if kind == "pagetable":
        pages = _exact_table(_masks(case["k"], case["shift"]), _origin(case, seed), case["shift"],
                             case["pool"], case["colours"])
        found = torch.tensor([pages.numel()]) if case["noalloc"] else pages.numel()
        return {"pt": pages[:case["need"]].to(torch.int32), "found": found}
    if kind == "triad":
        return _exact_triad(case, seed)
    if kind == "relayout":
        shift = case["shift"]
        per = -(-case["bytes"] >> shift)
        flat = _relayout_inputs(case, seed).view(torch.uint8)[:case["bytes"]]
        pages = torch.nn.functional.pad(flat, (0, (per << shift) - case["bytes"])).view(per, -1)
        if not case["to_part"]:
            return pages.reshape(-1).view(torch.int16)
        pool = _pages_for(per, case["colours"])
        out = torch.zeros(pool, 1 << shift, dtype=torch.uint8, device=DEV)
        out[_exact_table(_masks(6, shift), ORIGIN, shift, pool, case["colours"])[:per]] = pages
        return out.view(-1).view(torch.int16)
    if kind == "switch":
        outs, shift = [], case["shift"]
        for every, _ in _switch_inputs(case, seed):
            per = every.numel() >> shift
            pool = _pages_for(per, 48)
            part = torch.zeros(pool, 1 << shift, dtype=torch.uint8, device=DEV)
            part[_exact_table(_masks(6, shift), ORIGIN, shift, pool, 48)[:per]] = every.view(per, -1)
            outs += [every.view(torch.int16), part.view(-1).view(torch.int16)]
        return outs
    if kind == "gemv":
        ws = _weights(case["m"], case["k"], DTYPES[case["w"]][1], case["layers"], seed)
        xs = _acts(case["batch"], case["k"], DTYPES[case["x"]][1], case["layers"], seed)
        return [_exact_gemv(w, x) for w, x in zip(ws, xs)]
    ws = _weights(case["m"], case["k"], torch.bfloat16, case["layers"], seed)
    xs = _acts(1, case["k"], torch.bfloat16, case["calls"], seed)
    return {"y": [_exact_gemv(ws[i % case["layers"]], x) for i, x in enumerate(xs)],
            "a": _exact_triad({"n": case["n"], "shift": 16, "colours": 16}, seed)}
