"""The work that the framework's performance is measured on.

Each case goes through the package's public entry points (views, `llama_copy`, `llama_pack`, `llama_unpack`, batches,
the n-body step and its energy) on device blobs, over the sizes that such programs have: a few thousand records up to
the 64 Mi particles of the benchmark, on the 16-byte and 128-byte grids and off them.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs, views and batches on the GPU
  run(state)           one pass; returns the destination blobs (and the energy)
  work(case)           bytes and operations that one pass cannot do without
  exact(case, seed)    the computed outputs in 64 bits, from plain torch
"""
import math

import torch

import paper_2302_08251_amd as lm

DEV = "cuda"
SIZE = {"u8": 1, "i8": 1, "u16": 2, "i16": 2, "f16": 2, "bf16": 2, "u32": 4, "i32": 4, "f32": 4, "u64": 8, "i64": 8, "f64": 8}
TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32, "f64": torch.float64,
         "i8": torch.int8, "i16": torch.int16, "i32": torch.int32, "i64": torch.int64}

LAYOUTS = {
    "aos": {"kind": "aos"},
    "soa_sb": {"kind": "soa_sb"},
    "soa_mb": {"kind": "soa_mb"},
    "aosoa32": {"kind": "aosoa", "lanes": 32},
    "aosoa64": {"kind": "aosoa", "lanes": 64},
    "bytesplit": {"kind": "bytesplit", "inner": {"kind": "soa_sb"}},
}
RING = ("aos", "soa_sb", "soa_mb", "aosoa32", "aosoa64", "bytesplit", "aos")
PAIRS = [(a, b) for a in LAYOUTS for b in LAYOUTS if a != b]

# records of leaves of several sizes: an event with a flag, a time, a channel and an amplitude; a detector hit
MIXED = {
    "event": ["u8", "f64", "i16", "f32"],
    "hit": ["u32", "u16", "u8", "u8", "f32", "f32", "f64"],
}

# ways that values are stored, and stored again in another form
REENCODE = {
    # integer samples: kept as 16-bit values, archived at 12 bits, read back
    "i32_i16_b12": ("i32", 12, [{"kind": "soa_mb"}, {"kind": "changetype", "to": "i16", "inner": {"kind": "soa_mb"}},
                                {"kind": "bitpack_int", "bits": 12}, {"kind": "changetype", "to": "i16", "inner": {"kind": "aosoa", "lanes": 32}},
                                {"kind": "aos"}]),
    # 64-bit identifiers: kept as 32-bit values, archived at 40 bits, read back
    "i64_i32_b40": ("i64", 31, [{"kind": "aos"}, {"kind": "changetype", "to": "i32", "inner": {"kind": "soa_sb"}},
                                {"kind": "bitpack_int", "bits": 40}, {"kind": "aos"}]),
    # particles kept at 24 bits, archived at 16, read back
    "f32_e8m15_e5m10": ("f32", 0, [{"kind": "aos"}, {"kind": "bitpack_float", "exp": 8, "man": 15},
                                   {"kind": "bitpack_float", "exp": 5, "man": 10}, {"kind": "soa_mb"}]),
}


def listed():
    return [
        # one small set of particles converted between two steps of a program: launch and host latency
        {"name": "copy_small", "kind": "ring", "scalar": "f64", "n": 4096, "ring": "aos,soa_mb"},
        # the whole particle set of the benchmark taken through every layout
        {"name": "copy_layouts", "kind": "ring", "scalar": "f32", "n": 64 << 20, "ring": ",".join(RING)},
        # the same round with a record count off every grid, as particle counts in real runs are
        {"name": "copy_ragged", "kind": "ring", "scalar": "f32", "n": 3000017, "ring": ",".join(RING)},
        # particles written to and read back from 24-bit float codes
        {"name": "pack_floats", "kind": "pack_float", "n": 4000037, "fields": 7, "exp": 8, "man": 15, "round": "trunc", "layout": "aos"},
        # one long column of integers packed to 11 bits and read back
        {"name": "pack_ints", "kind": "pack_int", "n": 256 << 20, "fields": 1, "bits": 11, "layout": "soa_mb"},
        # double precision particles stored in single precision, and read back
        {"name": "changetype", "kind": "changetype", "n": 16 << 20, "user": "f64", "stored": "f32", "layout": "aos", "inner": "soa_mb"},
        # records of mixed leaf sizes taken apart into columns, divided between two mappings, and put together again
        {"name": "mixed_records", "kind": "mixed", "record": "event", "n": 5000011, "at": 2},
        # values already stored in one computed form stored in another
        {"name": "reencode", "kind": "reencode", "chain": "i32_i16_b12", "fields": 3, "n": 3000017},
        # a three-dimensional field handed from a row-major program to a column-major one, and back
        {"name": "transpose", "kind": "transpose", "scalar": "f32", "fields": 3, "e0": 301, "e1": 256, "e2": 203, "src": "aos", "dst": "soa_mb"},
        # many views of uneven sizes and mixed layout pairs in one launch
        {"name": "batch", "kind": "batch", "views": 256, "mix": 0},
        # steps of the all-pairs consumer through the benchmark's storage form, with the energy check after them
        {"name": "nbody", "kind": "nbody", "n": 65536, "steps": 2, "layout": "aosoa32", "user": "f64"},
        # a copy with access counters on both sides
        {"name": "heatmap", "kind": "heatmap", "n": 16 << 20, "granularity": 128, "src": "aos", "dst": "soa_sb"},
    ]


def _log(rng, lo, hi):
    """A size spread over the logarithm of its range; odd, round and 128-grid ones."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    how = rng.randrange(3)
    n = n if how == 0 else (n | 1) if how == 1 else max(128, n // 128 * 128)
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(["ring", "ring", "pack_float", "pack_int", "changetype", "mixed", "reencode", "transpose", "batch", "nbody", "heatmap"])
    c = {"kind": kind}
    if kind == "ring":
        c["scalar"] = rng.choice(["f32", "f32", "f64", "u16"])
        k = rng.randrange(2, 5)
        ring = [rng.choice(list(LAYOUTS))]
        while len(ring) < k:
            ring.append(rng.choice([x for x in LAYOUTS if x != ring[-1]]))
        c["ring"] = ",".join(ring)
        c["n"] = _log(rng, 1000, 16 << 20)
    elif kind == "pack_float":
        e, m = rng.choice([(8, 15), (5, 10), (8, 7), (8, 23), (5, 2), (4, 3), (6, 13), (8, 10)])
        c.update(fields=rng.choice([1, 3, 7]), exp=e, man=m, round=rng.choice(["trunc", "trunc", "rne"]), layout=rng.choice(["aos", "soa_mb", "aosoa32", "soa_sb"]))
        c["n"] = _log(rng, 1000, (64 << 20) // c["fields"])
    elif kind == "pack_int":
        c.update(fields=rng.choice([1, 3]), bits=rng.randrange(3, 32), layout=rng.choice(["aos", "soa_mb", "aosoa32", "soa_sb"]))
        c["n"] = _log(rng, 1000, (64 << 20) // c["fields"])
    elif kind == "changetype":
        c["user"], c["stored"] = rng.choice([("f64", "f32"), ("f32", "f16"), ("f32", "bf16"), ("f64", "bf16")])
        c.update(layout=rng.choice(["aos", "soa_mb", "aosoa32"]), inner=rng.choice(["aos", "soa_mb", "soa_sb", "aosoa64"]))
        c["n"] = _log(rng, 1000, 8 << 20)
    elif kind == "mixed":
        c["record"] = rng.choice(list(MIXED))
        c["at"] = rng.randrange(1, len(MIXED[c["record"]]))
        c["n"] = _log(rng, 1000, 8 << 20)
    elif kind == "reencode":
        c["chain"] = rng.choice(list(REENCODE))
        c["fields"] = rng.choice([1, 3, 7])
        c["n"] = _log(rng, 1000, (12 << 20) // c["fields"])
    elif kind == "transpose":
        c["scalar"] = rng.choice(["f32", "f32", "f64", "u16"])
        c["fields"] = rng.choice([1, 3, 7])
        e = [_log(rng, 16, 384) for _ in range(3)]
        if rng.randrange(2):
            e = [e[0] * 8 + rng.randrange(8), e[1], 1]
        c["e0"], c["e1"], c["e2"] = e
        c["src"], c["dst"] = rng.choice(list(LAYOUTS)[:5]), rng.choice(list(LAYOUTS)[:5])
    elif kind == "batch":
        c["views"] = _log(rng, 8, 256)
        c["mix"] = rng.randrange(1, 1 << 20)
    elif kind == "nbody":
        c.update(steps=rng.randrange(1, 5), layout=rng.choice(["aos", "soa_mb", "aosoa32"]), user=rng.choice(["f32", "f64"]))
        c["n"] = _log(rng, 300, 32768)
    else:
        c.update(granularity=rng.choice([1, 16, 64, 128, 4096]), src=rng.choice(["aos", "soa_sb", "soa_mb", "aosoa32"]), dst=rng.choice(["aos", "soa_sb", "soa_mb", "aosoa32"]))
        c["n"] = _log(rng, 1000, (2 << 20) if c["granularity"] == 1 else (16 << 20))
    return c


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _bits(g, nbytes):
    """Uniform random bytes: every NaN payload, infinity and denormal."""
    n = (max(nbytes, 16) + 7) // 8
    return torch.randint(-(1 << 63), (1 << 63) - 1, (n,), generator=g, device=DEV, dtype=torch.int64).view(torch.uint8)


def _particles(g, n, dtype):
    """pos ~ U[-1, 1], vel ~ N(0, 0.1), mass ~ U[0.5, 1], drawn field by field."""
    p = [torch.rand(n, generator=g, device=DEV, dtype=dtype) * 2 - 1 for _ in range(3)]
    p += [torch.randn(n, generator=g, device=DEV, dtype=dtype) * 0.1 for _ in range(3)]
    p.append(torch.rand(n, generator=g, device=DEV, dtype=dtype) * 0.5 + 0.5)
    return p


def _specials(g, x):
    """About 1 % each of infinities, quiet NaNs and values that the narrower formats hold as subnormals or drop."""
    u = torch.rand(x.shape, generator=g, device=DEV, dtype=torch.float32)
    x = torch.where(u < 0.01, torch.copysign(torch.full_like(x, math.inf), x), x)
    x = torch.where((u >= 0.01) & (u < 0.02), torch.full_like(x, math.nan), x)
    return torch.where((u >= 0.02) & (u < 0.03), x * 2.0 ** -20, x)


def _floats(case, seed):
    """The values of a float case, field by field."""
    g = _gen(seed)
    dt = TORCH[case.get("user", "f32")]
    return [_specials(g, p) for p in _particles(g, case["n"], dt)[:case.get("fields", 7)]]


def _ints(case, scalar, bits, seed):
    g = _gen(seed)
    lo, hi = -(1 << (bits - 1)), (1 << (bits - 1)) - 1
    return [torch.randint(lo, hi + 1, (case["n"],), generator=g, device=DEV, dtype=torch.int64).to(TORCH[scalar]) for _ in range(case["fields"])]


def _planes_view(rec, planes, extents):
    """The planes as they are: a view with one blob per field."""
    blobs = []
    for p in planes:
        b = p.view(torch.uint8)
        blobs.append(b if b.numel() >= 16 else torch.cat([b, b.new_zeros(16)]))
    return lm.View(rec, {"kind": "soa_mb"}, extents, blobs=blobs)


def _loaded(rec, spec, planes, extents):
    """A view of mapping `spec` that holds the planes' values."""
    src = _planes_view(rec, planes, extents)
    if spec["kind"] == "soa_mb" and not spec.get("col_major"):
        return src
    dst = lm.View(rec, spec, extents, fill=0)
    lm.llama_copy(src, dst)
    torch.cuda.synchronize()
    return dst


def _blobs(view, dtype=torch.uint8):
    return [b[:s].view(dtype) if s % torch.empty(0, dtype=dtype).element_size() == 0 else b[:s] for b, s in zip(view.blobs, view.sizes)]


def _chain(case):
    """Record, value bits and mappings of a re-encoding."""
    scalar, bits, chain = REENCODE[case["chain"]]
    nf = case["fields"]
    out = []
    for m in chain:
        m = dict(m)
        if m["kind"] == "changetype":
            m = {"kind": "changetype", "stored": [m["to"]] * nf, "inner": m["inner"]}
        out.append(m)
    return scalar, bits, [scalar] * nf, out


def _split(at, a, b):
    return {"kind": "split", "at": at, "parts": [a, b]}


def _batch_views(case):
    """Record counts log-uniform in [1e3, 4e6] and layout pairs, as the benchmark's batch draws them."""
    g = torch.Generator().manual_seed(1000003 + case["mix"])
    u = torch.rand(case["views"], generator=g, dtype=torch.float64)
    ns = torch.exp(math.log(1e3) + u * (math.log(4e6) - math.log(1e3))).round().to(torch.int64).tolist()
    ps = torch.randint(0, len(PAIRS), (case["views"],), generator=g).tolist()
    return [(n, PAIRS[p]) for n, p in zip(ns, ps)]


def _extents(case):
    return [e for e in (case["e0"], case["e1"], case["e2"]) if e > 1]


# ---------------------------------------------------------------- the program's state

def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind == "ring":
        names = case["ring"].split(",")
        rec = [case["scalar"]] * 7
        views = [lm.View(rec, LAYOUTS[k], case["n"], fill=0) for k in names]
        for b in views[0].blobs:
            b.copy_(_bits(g, b.numel())[:b.numel()])
        return {"copies": list(zip(views, views[1:])), "out": [b for v in views[1:] for b in _blobs(v)]}
    if kind in ("pack_float", "pack_int", "changetype"):
        if kind == "pack_float":
            rec = ["f32"] * case["fields"]
            spec = {"kind": "bitpack_float", "exp": case["exp"], "man": case["man"]}
            if case["round"] == "rne":
                spec["round"] = "rne"
            planes, layout = _floats(case, seed), case["layout"]
        elif kind == "pack_int":
            rec = ["i32"] * case["fields"]
            spec = {"kind": "bitpack_int", "bits": case["bits"]}
            planes, layout = _ints(case, "i32", case["bits"], seed), case["layout"]
        else:
            rec = [case["user"]] * 7
            spec = {"kind": "changetype", "stored": [case["stored"]] * 7, "inner": LAYOUTS[case["inner"]]}
            planes, layout = _floats(case, seed), case["layout"]
        src = _loaded(rec, LAYOUTS[layout], planes, case["n"])
        code = lm.View(rec, spec, case["n"], fill=0)
        back = lm.View(rec, LAYOUTS[layout], case["n"], fill=0)
        return {"pack": (src, code), "unpack": (code, back), "out": [_blobs(code), _blobs(back, TORCH[rec[0]])]}
    if kind == "mixed":
        rec = MIXED[case["record"]]
        n, at = case["n"], case["at"]
        aos = lm.View(rec, LAYOUTS["aos"], n, fill=0)
        for b in aos.blobs:
            b.copy_(_bits(g, b.numel())[:b.numel()])
        cols = lm.View(rec, LAYOUTS["soa_mb"], n, fill=0)
        parts = lm.View(rec, _split(at, LAYOUTS["aosoa32"], {"kind": "aos", "packed": True}), n, fill=0)
        back = lm.View(rec, LAYOUTS["aos"], n, fill=0)
        return {"copies": [(aos, cols), (cols, parts), (parts, back)], "out": [b for v in (cols, parts, back) for b in _blobs(v)]}
    if kind == "reencode":
        scalar, bits, rec, maps = _chain(case)
        planes = _floats(case, seed) if scalar == "f32" else _ints(case, scalar, bits, seed)
        views = [_loaded(rec, maps[0], planes, case["n"])] + [lm.View(rec, m, case["n"], fill=0) for m in maps[1:]]
        out = [b for v in views[1:-1] for b in _blobs(v)]
        return {"copies": list(zip(views, views[1:])), "out": [out, _blobs(views[-1], TORCH[scalar])]}
    if kind == "transpose":
        ext = _extents(case)
        rec = [case["scalar"]] * case["fields"]
        a = lm.View(rec, LAYOUTS[case["src"]], ext, fill=0)
        for b in a.blobs:
            b.copy_(_bits(g, b.numel())[:b.numel()])
        b = lm.View(rec, dict(LAYOUTS[case["dst"]], col_major=True), ext, fill=0)
        c = lm.View(rec, LAYOUTS[case["src"]], ext, fill=0)
        return {"copies": [(a, b), (b, c)], "out": [x for v in (b, c) for x in _blobs(v)]}
    if kind == "batch":
        # sources and destinations in two arenas, every blob on a 256-byte boundary
        rec = ["f32"] * 7
        todo = _batch_views(case)
        sizes = [[lm.blob_sizes(rec, LAYOUTS[p[side]], n) for n, p in todo] for side in (0, 1)]
        room = [sum(-(-s // 256) * 256 for v in part for s in v) for part in sizes]
        arena = [_bits(g, room[0]), torch.zeros(room[1], dtype=torch.uint8, device=DEV)]
        views = [[], []]
        for side in (0, 1):
            at = 0
            for (n, p), part in zip(todo, sizes[side]):
                blobs = []
                for s in part:
                    blobs.append(arena[side][at:at + s])
                    at += -(-s // 256) * 256
                views[side].append(lm.View(rec, LAYOUTS[p[side]], n, blobs=blobs))
        batch = lm.Batch(views[0], views[1])
        return {"batch": batch, "views": views, "out": arena[1]}
    if kind == "nbody":
        dt = TORCH["f64"]
        planes = [p.to(TORCH[case["user"]]) for p in _particles(g, case["n"], dt)]
        rec = [case["user"]] * 7
        spec = LAYOUTS[case["layout"]]
        if case["user"] == "f64":
            spec = {"kind": "changetype", "stored": ["f32"] * 7, "inner": spec}
        v = lm.View(rec, spec, case["n"], fill=0)
        lm.llama_copy(_planes_view(rec, planes, case["n"]), v)
        torch.cuda.synchronize()
        return {"particles": v, "steps": case["steps"], "out": _blobs(v, torch.float32)}
    rec = ["f32"] * 7
    views = [lm.View(rec, {"kind": "heatmap", "granularity": case["granularity"], "inner": LAYOUTS[case[k]]}, case["n"], fill=0) for k in ("src", "dst")]
    for v in views:
        v.data = len(v.blobs) // 2
    for b in views[0].blobs[:views[0].data]:
        b.copy_(_bits(g, b.numel())[:b.numel()])
    out = _blobs(views[1])[:views[1].data] + [x.view(torch.int64) for v in views for x in _blobs(v)[v.data:]]
    return {"copies": [tuple(views)], "out": out}


# time step and softening, as the 32-bit numbers that cross the interface
DT, EPS2 = (float(torch.tensor(x, dtype=torch.float32)) for x in (1e-4, 0.01))


def run(state):
    if "copies" in state:
        for a, b in state["copies"]:
            lm.llama_copy(a, b)
    elif "batch" in state:
        state["batch"].launch()
    elif "particles" in state:
        lm.nbody_step(state["particles"], state["steps"], DT, EPS2)
        return state["out"], lm.nbody_energy(state["particles"], EPS2)
    else:
        lm.llama_pack(*state["pack"])
        lm.llama_unpack(*state["unpack"])
    return state["out"]


# ---------------------------------------------------------------- what a pass cannot do without

def _stored(rec, spec, n):
    """Bytes of n records as mapping `spec` stores them, padding not counted."""
    k = spec["kind"]
    if k == "bitpack_int":
        return len(rec) * ((n * spec["bits"] + 7) // 8)
    if k == "bitpack_float":
        return len(rec) * ((n * (1 + spec["exp"] + spec["man"]) + 7) // 8)
    return n * sum(SIZE[t] for t in spec.get("stored", rec))


def work(case):
    kind = case["kind"]
    if kind == "ring":
        return {"bytes": 2 * 7 * SIZE[case["scalar"]] * case["n"] * case["ring"].count(","), "flops": 0}
    if kind == "pack_float":
        n = case["n"] * case["fields"]
        return {"bytes": 2 * (4 * n + n * (1 + case["exp"] + case["man"]) // 8), "flops": 0}
    if kind == "pack_int":
        n = case["n"] * case["fields"]
        return {"bytes": 2 * (4 * n + n * case["bits"] // 8), "flops": 0}
    if kind == "changetype":
        return {"bytes": 2 * 7 * case["n"] * (SIZE[case["user"]] + SIZE[case["stored"]]), "flops": 0}
    if kind == "mixed":
        return {"bytes": 3 * 2 * case["n"] * sum(SIZE[t] for t in MIXED[case["record"]]), "flops": 0}
    if kind == "reencode":
        _, _, rec, maps = _chain(case)
        b = [_stored(rec, m, case["n"]) for m in maps]
        return {"bytes": sum(x + y for x, y in zip(b, b[1:])), "flops": 0}
    if kind == "transpose":
        return {"bytes": 2 * 2 * case["e0"] * case["e1"] * case["e2"] * case["fields"] * SIZE[case["scalar"]], "flops": 0}
    if kind == "batch":
        return {"bytes": 2 * 28 * sum(n for n, _ in _batch_views(case)), "flops": 0}
    if kind == "nbody":
        # 20 operations for each ordered pair and step, 12 for each unordered pair of the energy
        n = case["n"]
        return {"bytes": 28 * n * (2 * case["steps"] + 1), "flops": 20 * n * n * case["steps"] + 6 * n * n}
    counters = 2 * (-(-28 * case["n"] // case["granularity"]))
    return {"bytes": 2 * 28 * case["n"] + 16 * counters, "flops": 0}


# ---------------------------------------------------------------- 64-bit results

def _quantize(x, E, M, rne):
    """x (float64, holding f32 values) as the float code of E exponent and M mantissa bits holds it."""
    bias = (1 << (E - 1)) - 1
    a = x.abs()
    fin = torch.isfinite(x)
    _, e = torch.frexp(torch.where(fin, a, torch.zeros_like(a)))
    q = torch.clamp(e - 1, min=1 - bias).to(torch.float64) - M
    t = torch.where(fin, a, torch.zeros_like(a)) * torch.exp2(-q)
    t = (torch.round(t) if rne else torch.floor(t)) * torch.exp2(q)
    t = torch.where(t >= 2.0 ** (bias + 1), torch.full_like(t, math.inf), t)
    return torch.copysign(torch.where(fin, t, a), x)


def _as_blobs(planes, layout):
    """The planes in the order that a view of `layout` keeps them, one tensor per blob."""
    if layout == "soa_mb":
        return planes
    if layout == "soa_sb":
        return [torch.cat(planes)]
    m = torch.stack(planes, 1)
    if layout == "aos":
        return [m.reshape(-1)]
    lanes = LAYOUTS[layout]["lanes"]
    pad = -m.shape[0] % lanes
    m = torch.cat([m, m.new_zeros(pad, m.shape[1])])
    return [m.view(-1, lanes, m.shape[1]).transpose(1, 2).reshape(-1)]


def _forces(pos, mass):
    """Softened accelerations and twice the (negative) potential energy, in 64 bits, a block of rows at a time."""
    acc, pot = torch.empty_like(pos), 0.0
    for i in range(0, pos.shape[0], 1024):
        d = [pos[:, k][None, :] - pos[i:i + 1024, k][:, None] for k in range(3)]
        inv = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + EPS2).rsqrt_()
        pot += float(((inv * mass[None, :]).sum(1) * mass[i:i + 1024]).sum())
        w = inv * inv * inv * mass[None, :]
        for k in range(3):
            acc[i:i + 1024, k] = (d[k] * w).sum(1)
    return acc, pot - float((mass * mass).sum()) * EPS2 ** -0.5


def exact(case, seed):
    kind = case["kind"]
    if kind == "pack_float":
        planes = [_quantize(p.double(), case["exp"], case["man"], case["round"] == "rne") for p in _floats(case, seed)]
        return [[None] * case["fields"], _as_blobs(planes, case["layout"])]
    if kind == "changetype":
        planes = [p.to(TORCH[case["stored"]]).double() for p in _floats(case, seed)]
        n_code = 7 if case["inner"] == "soa_mb" else 1
        return [[None] * n_code, _as_blobs(planes, case["layout"])]
    if kind == "reencode" and REENCODE[case["chain"]][0] == "f32":
        planes = [_quantize(_quantize(p.double(), 8, 15, False), 5, 10, False) for p in _floats(case, seed)]
        return [[None] * (2 * case["fields"]), planes]
    if kind == "nbody":
        p = [x.float().double() for x in _particles(_gen(seed), case["n"], torch.float64)]
        pos, vel, mass = torch.stack(p[:3], 1), torch.stack(p[3:6], 1), p[6]
        for _ in range(case["steps"]):
            vel = vel + DT * _forces(pos, mass)[0]
            pos = pos + DT * vel
        pot = _forces(pos, mass)[1]
        energy = float(0.5 * (mass * (vel * vel).sum(1)).sum()) - 0.5 * pot
        planes = [pos[:, k].contiguous() for k in range(3)] + [vel[:, k].contiguous() for k in range(3)] + [mass]
        return _as_blobs(planes, case["layout"]), energy
    return None
