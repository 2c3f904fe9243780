"""The work a program gives this library, as cases that can be timed and compared.

A case is one call sequence of a domain-parallel program on the GPU that holds
one shard:

  conv   one convolution layer: `pass` "fwd" is the halo exchange's local half
         (pack the faces to send, unpack the received slabs) and the forward;
         "bwd" the input gradient, the reverse exchange's local half and the
         weight gradient; "train" both. `fold` reads the halo from the received
         slabs instead of unpacking it (forward as interior then boundary, the
         way the exchange is overlapped).
  halo   the local half of the exchange alone, over every sharded axis.
  norm   group normalisation: the shard's sums, then the normalised interior.
  attn   ring attention: one device's steps over `blocks` key/value blocks.

Spatial extents are the shard's interior, "DxHxW" outermost first. `shard` has a
letter per axis: "-" the axis is whole on this GPU, "m" it is split and this
shard has neighbours on both sides, "e" it is split and this shard lies at the
domain's low edge (its low margin is zero padding).
"""
from __future__ import annotations

import math

import torch

from paper_2605_11111_amd import shardconv as sc

DTYPES = {"f32": (torch.float32, 4), "bf16": (torch.bfloat16, 2)}


def conv_case(name, dtype, n, cin, cout, ext, k, s, shard, what, fold=False):
    c = {"kind": "conv", "dtype": dtype, "n": n, "cin": cin, "cout": cout, "ext": ext, "k": k, "s": s,
         "shard": shard, "pass": what, "fold": fold}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small 2D field split in two: the shard that fits a GPU many times over, where launches and
        # latency are all there is
        conv_case("train_2d_f32_c8_small", "f32", 1, 8, 8, "32x64", 3, 1, "e-", "train"),
        # a 4096 x 4096 field split four ways along H, 64 channels: the largest 2D layer of the benchmark
        conv_case("train_2d_bf16_c64", "bf16", 1, 64, 64, "1024x4096", 3, 1, "m-", "train"),
        # a 512^3 volume split four ways along D, 32 channels: the benchmark's default layer, and the largest
        conv_case("train_3d_bf16_c32", "bf16", 1, 32, 32, "128x512x512", 3, 1, "m--", "train"),
        # the backward of the first, wide-kernel layer of a 256^3 volume split over two axes
        conv_case("bwd_3d_bf16_c16_k5", "bf16", 1, 16, 64, "128x128x256", 5, 1, "ee-", "bwd"),
        # a strided layer in full precision on a 384^3 volume split eight ways, forward (inference) ...
        conv_case("fwd_3d_f32_c64_s2", "f32", 1, 64, 128, "48x384x384", 3, 2, "m--", "fwd"),
        # ... and its backward
        conv_case("bwd_3d_f32_c64_s2", "f32", 1, 64, 128, "48x384x384", 3, 2, "m--", "bwd"),
        # the same kind of downsampling layer in mixed precision, further down a network
        conv_case("train_3d_bf16_c32_s2", "bf16", 1, 32, 64, "64x128x128", 3, 2, "m--", "train"),
        # a wide 2D layer at odd, ragged sizes with a small batch
        conv_case("train_2d_bf16_c128_ragged", "bf16", 2, 128, 128, "253x381", 3, 1, "m-", "train"),
        # a 3D layer split over two axes at odd sizes, exchange overlapped with the interior
        conv_case("train_3d_bf16_c32_fold", "bf16", 1, 32, 32, "61x117x123", 3, 1, "mm-", "train", True),
        # the normalisation after a layer, at odd sizes
        {"name": "norm_3d_bf16_c32", "kind": "norm", "dtype": "bf16", "n": 1, "c": 32, "ext": "48x131x157",
         "halo": 1, "groups": 8},
        # a ring of four devices, an odd local sequence: four block steps
        {"name": "attn_ring_d128", "kind": "attn", "b": 1, "h": 16, "sq": 2044, "sk": 2044, "d": 128, "blocks": 4},
        # the exchange of a volume split over all three axes (faces that are not contiguous)
        {"name": "halo_3d_f32_c32", "kind": "halo", "dtype": "f32", "n": 1, "c": 32, "ext": "96x128x160", "width": 1,
         "shard": "mmm"},
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv"] * 7 + ["norm", "attn", "halo"])
    if kind == "attn":
        sq = log_int(rng, 128, 6000)
        return {"kind": "attn", "b": rng.choice([1, 1, 2]), "h": rng.choice([4, 8, 16]), "sq": sq,
                "sk": sq if rng.random() < 0.5 else log_int(rng, 128, 6000), "d": rng.choice([64, 128]),
                "blocks": rng.choice([1, 2, 4])}
    if kind in ("norm", "halo"):
        nd = rng.choice([2, 3])
        dtype, n = rng.choice(["f32", "bf16", "bf16"]), rng.choice([1, 1, 2])
        c = rng.choice([8, 16, 32, 64, 96, 128])
        vox = log_int(rng, 4096, (1 << 28) // c)
        ext = extents(rng, nd, vox)
        if kind == "norm":
            return {"kind": "norm", "dtype": dtype, "n": n, "c": c, "ext": ext, "halo": rng.choice([0, 1, 2]),
                    "groups": rng.choice([g for g in (1, 4, 8, c) if c % g == 0])}
        return {"kind": "halo", "dtype": dtype, "n": n, "c": c, "ext": ext, "width": rng.choice([1, 1, 2]),
                "shard": shard_letters(rng, nd)}
    nd = rng.choice([2, 2, 3, 3, 3])
    dtype, n = rng.choice(["f32", "bf16", "bf16"]), rng.choice([1, 1, 2])
    cin = rng.choice([3, 8, 16, 24, 32, 32, 48, 64, 64, 96, 128])
    cout = rng.choice([8, 16, 32, 32, 48, 64, 64, 96, 128])
    k = rng.choice([1, 3, 3, 3, 3, 3, 5, 7] if nd == 2 else [1, 3, 3, 3, 3, 3, 5])
    s = rng.choice([1, 1, 1, 2])
    what = rng.choice(["fwd", "bwd", "train"])
    # up to 50 GFLOP a direction (the largest listed case takes 1855)
    flops_vox = 2.0 * cin * cout * k ** nd / s ** nd
    vox = log_int(rng, 1500, min(5e10 / flops_vox, 3e7) / n)
    return conv_case(None, dtype, n, cin, cout, extents(rng, nd, vox), k, s, shard_letters(rng, nd), what,
                     rng.random() < 0.25)


def extents(rng, nd, vox):
    """Extents of about `vox` voxels in all, none below 8, most of them odd or ragged."""
    f = [rng.uniform(0.6, 1.6) for _ in range(nd)]
    side = (vox / math.prod(f)) ** (1.0 / nd)
    return "x".join(str(max(8, int(round(side * v)))) for v in f)


def shard_letters(rng, nd):
    s = [rng.choice("me")] + [rng.choice("--me") for _ in range(nd - 1)]
    return "".join(s)


# --- geometry, as the library's caller knows it --------------------------------------

def axes_of(case):
    return [int(v) for v in case["ext"].split("x")]


def placement(case):
    """(global extent, shard offset) per axis: three equal shards, or two for a shard at the low edge."""
    g, off = [], []
    for e, l in zip(axes_of(case), case["shard"]):
        g.append(e if l == "-" else 3 * e if l == "m" else 2 * e)
        off.append(e if l == "m" else 0)
    return g, off


def plain_geometry(ext, off, k, s, sharded):
    """halo_lo, halo_hi, pad_lo, out_ext of one axis, from the definitions: "same" padding of (k - 1) / 2, output j
    belongs to the shard that holds input row j s."""
    p = (k - 1) // 2
    j0, j1 = -(-off // s), -(-(off + ext) // s)
    if not sharded:
        return 0, 0, p, j1 - j0
    if j1 <= j0:
        return 0, 0, 0, 0
    lo = max(0, off - (j0 * s - p))
    hi = max(0, (j1 - 1) * s - p + k - 1 - (off + ext - 1))
    return lo, hi, off - lo + p - j0 * s, j1 - j0


def geometry(case):
    """Per axis: halo_lo, halo_hi, pad_lo, out_ext, and the widths the low and high neighbours ask for."""
    _, off = placement(case)
    rows = []
    for e, o, l in zip(axes_of(case), off, case["shard"]):
        me = plain_geometry(e, o, case["k"], case["s"], l != "-")
        below = plain_geometry(e, o - e, case["k"], case["s"], True)[1] if l == "m" else 0
        above = plain_geometry(e, o + e, case["k"], case["s"], True)[0] if l in "me" else 0
        rows.append(me + (below, above))
    return [list(v) for v in zip(*rows)]


def slab_shape(n, c, ext, lo, hi, axis, width):
    return [n] + [lo[b] + ext[b] + hi[b] if b < axis else width if b == axis else ext[b] for b in range(len(ext))] + [c]


def randn(gen, shape, dtype, std=1.0):
    return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)


def field(gen, n, c, dims, dtype):
    """A field of the domain, channels last: smooth over a few voxels, with noise on it (unit variance)."""
    coarse = [max(2, -(-d // 6)) for d in dims]
    mode = {1: "linear", 2: "bilinear", 3: "trilinear"}[len(dims)]
    out = torch.empty([n] + list(dims) + [c], dtype=dtype, device="cuda")
    for ch in range(c):  # one channel at a time: the intermediates stay small
        z = torch.randn([n, 1] + coarse, generator=gen, device="cuda")
        z = torch.nn.functional.interpolate(z, size=list(dims), mode=mode, align_corners=False)[:, 0]
        z = z * 1.4 + 0.3 * torch.randn(z.shape, generator=gen, device="cuda")
        out[..., ch] = z.to(dtype)
    return out


def inside(t, lo, ext):
    """The interior of a padded channels-last tile."""
    for a, (l, e) in enumerate(zip(lo, ext)):
        t = t.narrow(1 + a, l, e)
    return t


def conv_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = DTYPES[case["dtype"]][0]
    ext, nd = axes_of(case), len(axes_of(case))
    lo, hi, pad, out, below, above = geometry(case)
    n, cin, cout, k = case["n"], case["cin"], case["cout"], case["k"]
    d = {"x": field(gen, n, cin, ext, dt), "w": randn(gen, [cout, cin] + [k] * nd, dt, 1 / math.sqrt(cin * k ** nd))}
    d["dy"] = randn(gen, [n] + out + [cout], dt) if case["pass"] != "fwd" else None
    d["slabs"], d["grads"] = {}, {}
    for a in range(nd):
        for side, width, there in ((0, lo[a], case["shard"][a] == "m"), (1, hi[a], case["shard"][a] != "-")):
            if there and width:
                d["slabs"][a, side] = field(gen, n, cin, slab_shape(n, cin, ext, lo, hi, a, width)[1:-1], dt)
        for side, width in ((0, below[a]), (1, above[a])):
            if width and case["pass"] != "fwd":
                d["grads"][a, side] = randn(gen, slab_shape(n, cin, ext, lo, hi, a, width), dt)
    return d


def prepare_conv(case, seed):
    d = conv_inputs(case, seed)
    dt, code = DTYPES[case["dtype"]][0], sc.SHARD_F32 if case["dtype"] == "f32" else sc.SHARD_BF16
    ext, nd = axes_of(case), len(axes_of(case))
    n, cin, cout = case["n"], case["cin"], case["cout"]
    K, S = [case["k"]] * nd, [case["s"]] * nd
    g_ext, off = placement(case)
    g = sc.shard_conv_geometry(g_ext, off, ext, K, S, [int(l != "-") for l in case["shard"]])
    lo, hi, out = g["halo_lo"], g["halo_hi"], g["out_ext"]
    below, above = geometry(case)[4:]
    tile = torch.zeros([n] + [a + b + c for a, b, c in zip(lo, ext, hi)] + [cin], dtype=dt, device="cuda")
    inside(tile, lo, ext).copy_(d.pop("x"))
    desc = sc.tile_desc(n, cin, ext, lo, hi)

    def ws(op):
        return torch.empty(max(16, sc.shard_conv_workspace_bytes(op, desc, code, cout, K, S, out)), dtype=torch.uint8,
                           device="cuda")

    st = dict(d, case=case, desc=desc, tile=tile, K=K, S=S, pad=g["pad_lo"], out=out)
    st["widths"] = [(below[a], above[a]) for a in range(nd)]
    st["send"] = {(a, side): torch.empty(slab_shape(n, cin, ext, lo, hi, a, w), dtype=dt, device="cuda")
                  for a in range(nd) for side, w in enumerate((below[a], above[a])) if w}
    st["axes"] = [a for a in range(nd) if case["shard"][a] != "-"]
    if case["pass"] != "bwd":
        st["y"] = torch.empty([n] + out + [cout], dtype=dt, device="cuda")
        st["ws0"] = ws(0)
    else:
        # the forward has filled the margins
        for a in st["axes"]:
            sc.shard_halo_unpack_pair(desc, tile, a, d["slabs"].get((a, 0)), d["slabs"].get((a, 1)))
    if case["pass"] != "fwd":
        st["dtile"] = torch.empty_like(tile)
        st["dw"] = torch.empty([cout, cin] + K, dtype=torch.float32, device="cuda")
        st["ws1"], st["ws2"] = ws(1), ws(2)
        st["back"] = {k: torch.empty_like(v) for k, v in d["slabs"].items()}
    return st


def run_conv(st):
    case, desc, tile = st["case"], st["desc"], st["tile"]
    K, S, pad, out, cout = st["K"], st["S"], st["pad"], st["out"], st["case"]["cout"]
    slabs, res = st["slabs"], {}
    if case["pass"] != "bwd":
        for a in st["axes"]:
            wl, wh = st["widths"][a]
            sc.shard_halo_pack_pair(desc, tile, a, wl, st["send"].get((a, 0)), wh, st["send"].get((a, 1)))
            if not case["fold"]:
                sc.shard_halo_unpack_pair(desc, tile, a, slabs.get((a, 0)), slabs.get((a, 1)))
        if case["fold"]:
            for region in (sc.SHARD_REGION_INTERIOR, sc.SHARD_REGION_BOUNDARY):
                sc.shard_conv_fwd_folded(desc, tile, slabs, region, st["w"], cout, K, S, pad, out, st["y"], st["ws0"])
        else:
            sc.shard_conv_fwd(desc, tile, st["w"], cout, K, S, pad, out, st["y"], st["ws0"])
        # a folded exchange packs from a tile whose margins are never filled: its slabs' corners hold nothing
        if not case["fold"]:
            res["send"] = [st["send"][k] for k in sorted(st["send"])]
        res["y"] = st["y"]
    if case["pass"] != "fwd":
        sc.shard_conv_dgrad(desc, st["dy"], st["w"], cout, K, S, pad, out, st["dtile"], st["ws2"])
        for a in reversed(st["axes"]):
            sc.shard_halo_pack_margin_pair(desc, st["dtile"], a, st["back"].get((a, 0)), st["back"].get((a, 1)))
            wl, wh = st["widths"][a]
            sc.shard_halo_accumulate_pair(desc, st["dtile"], a, wl, st["grads"].get((a, 0)), wh,
                                          st["grads"].get((a, 1)))
        if case["fold"]:
            sc.shard_conv_wgrad_folded(desc, tile, slabs, st["dy"], cout, K, S, pad, out, st["dw"], st["ws1"])
        else:
            sc.shard_conv_wgrad(desc, tile, st["dy"], cout, K, S, pad, out, st["dw"], st["ws1"])
        res["dtile"], res["dw"] = st["dtile"], st["dw"]
        res["back"] = [st["back"][k] for k in sorted(st["back"])]
    return res


def taps_of(k, nd):
    return [(())] if nd == 0 else [(t,) + r for t in range(k) for r in taps_of(k, nd - 1)]


def chunks(n, most):
    return [(i, min(n, i + most)) for i in range(0, n, most)]


def fill_margins(tile, slabs, lo, hi, ext):
    """The received slabs written into a padded tile's margins, axis by axis."""
    for a in range(len(ext)):
        for side in (0, 1):
            v = slabs.get((a, side))
            if v is None:
                continue
            t = tile.narrow(1 + a, 0 if side == 0 else lo[a] + ext[a], v.shape[1 + a])
            for b in range(a + 1, len(ext)):
                t = t.narrow(1 + b, lo[b], ext[b])
            t.copy_(v)


def exact_conv(case, seed):
    d = conv_inputs(case, seed)
    ext, nd = axes_of(case), len(axes_of(case))
    lo, hi, pad, out, below, above = geometry(case)
    n, cin, cout, k, s = case["n"], case["cin"], case["cout"], case["k"], case["s"]
    P = [a + b + c for a, b, c in zip(lo, ext, hi)]
    w = d["w"].double()
    # the tile inside a frame of zeros wide enough for every tap
    f_lo = [max(0, p) for p in pad]
    f_hi = [max(0, (o - 1) * s - p + k - q) for o, p, q in zip(out, pad, P)]
    frame = torch.zeros([n] + [a + b + c for a, b, c in zip(f_lo, P, f_hi)] + [cin], dtype=torch.float64, device="cuda")
    tile = inside(frame, f_lo, P)
    inside(tile, lo, ext).copy_(d.pop("x"))
    res = {}
    if case["pass"] != "bwd":
        send = {}
        for a in range(nd):
            for side, width in ((0, below[a]), (1, above[a])):
                if width:
                    t = tile.narrow(1 + a, lo[a] if side == 0 else lo[a] + ext[a] - width, width)
                    for b in range(a + 1, nd):
                        t = t.narrow(1 + b, lo[b], ext[b])
                    send[a, side] = t.clone()
            fill_margins(tile, {key: v for key, v in d["slabs"].items() if key[0] == a}, lo, hi, ext)
        if not case["fold"]:
            res["send"] = [send[key] for key in sorted(send)]
        del send
    else:
        fill_margins(tile, d["slabs"], lo, hi, ext)

    def window(t, tap, p0, p1):
        """Rows a tap meets for the outputs [p0, p1) of axis 0, on a framed tensor."""
        for a in range(nd):
            j0, j1 = (p0, p1) if a == 0 else (0, out[a])
            first = j0 * s - pad[a] + tap[a] + f_lo[a]
            t = t.narrow(1 + a, first, (j1 - j0 - 1) * s + 1)
            t = t[(slice(None),) * (1 + a) + (slice(None, None, s),)]
        return t

    per_row = n * math.prod(out[1:])
    rows = chunks(out[0], max(1, (1 << 22) // max(1, per_row)))  # output rows of axis 0 at a time
    if case["pass"] != "bwd":
        y = torch.empty([n] + out + [cout], dtype=torch.float64, device="cuda")
        for p0, p1 in rows:
            acc = torch.zeros([per_row * (p1 - p0), cout], dtype=torch.float64, device="cuda")
            for tap in taps_of(k, nd):
                wt = w[(slice(None), slice(None)) + tap].t().contiguous()
                acc.addmm_(window(frame, tap, p0, p1).reshape(-1, cin), wt)
            y[:, p0:p1] = acc.view([n, p1 - p0] + out[1:] + [cout])
        res["y"] = y
    if case["pass"] != "fwd":
        dframe = torch.zeros_like(frame)
        dw = torch.zeros([cout, cin] + [k] * nd, dtype=torch.float64, device="cuda")
        for p0, p1 in rows:
            dy = d["dy"][:, p0:p1].double().reshape(-1, cout)
            m = dy.shape[0]
            step = min(m, 2048)
            whole = m // step * step
            dyt = dy[:whole].view(-1, step, cout).transpose(1, 2).contiguous()
            for tap in taps_of(k, nd):
                xv = window(frame, tap, p0, p1).reshape(-1, cin)
                part = torch.bmm(dyt, xv[:whole].view(-1, step, cin)).sum(0)
                if whole < m:
                    part += dy[whole:].t().contiguous() @ xv[whole:]
                dw[(slice(None), slice(None)) + tap] += part
                dx = window(dframe, tap, p0, p1)
                dx += (dy @ w[(slice(None), slice(None)) + tap].contiguous()).view(dx.shape)
        dtile = inside(dframe, f_lo, P).clone()
        back = {}
        for a in reversed(range(nd)):
            for side in (0, 1):
                v = d["slabs"].get((a, side))
                if v is not None:
                    t = dtile.narrow(1 + a, 0 if side == 0 else lo[a] + ext[a], v.shape[1 + a])
                    for b in range(a + 1, nd):
                        t = t.narrow(1 + b, lo[b], ext[b])
                    back[a, side] = t.clone()
            for side, width in ((0, below[a]), (1, above[a])):
                if width:
                    t = dtile.narrow(1 + a, lo[a] if side == 0 else lo[a] + ext[a] - width, width)
                    for b in range(a + 1, nd):
                        t = t.narrow(1 + b, lo[b], ext[b])
                    t += d["grads"][a, side].double()
        res["dtile"], res["dw"] = dtile, dw
        res["back"] = [back[key] for key in sorted(back)]
    return res


def work_conv(case):
    ext, nd = axes_of(case), len(axes_of(case))
    lo, hi, _, out, below, above = geometry(case)
    n, cin, cout, esz = case["n"], case["cin"], case["cout"], DTYPES[case["dtype"]][1]
    weights = cout * cin * case["k"] ** nd
    inner = n * math.prod(ext) * cin * esz
    tile = n * math.prod(a + b + c for a, b, c in zip(lo, ext, hi)) * cin * esz
    y = n * math.prod(out) * cout * esz
    faces = sum(math.prod(slab_shape(n, cin, ext, lo, hi, a, w)) for a in range(nd) for w in (below[a], above[a])) * esz
    halo = tile - inner  # what the received slabs hold, corners once
    flops = 2.0 * n * math.prod(out) * weights
    fwd = faces + halo + y  # faces written, slabs read, outputs written
    bwd = y + tile + 4 * weights + halo + faces  # dy read; gradient, dw and margin slabs written; returned slabs read
    both = inner + weights * esz  # read by either pass
    return {"bytes": both + (fwd if case["pass"] != "bwd" else 0) + (bwd if case["pass"] != "fwd" else 0),
            "flops": flops * {"fwd": 1, "bwd": 2, "train": 3}[case["pass"]]}


# --- the exchange alone --------------------------------------------------------------

def halo_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = DTYPES[case["dtype"]][0]
    ext, w = axes_of(case), case["width"]
    m = [0 if l == "-" else w for l in case["shard"]]
    x = field(gen, case["n"], case["c"], ext, dt)
    slabs = {}
    for a, l in enumerate(case["shard"]):
        for side in (0, 1):
            if l == "m" or (l == "e" and side == 1):
                slabs[a, side] = randn(gen, slab_shape(case["n"], case["c"], ext, m, m, a, w), dt)
    return x, slabs, m


def prepare_halo(case, seed):
    x, slabs, m = halo_inputs(case, seed)
    ext = axes_of(case)
    tile = torch.zeros([case["n"]] + [2 * a + b for a, b in zip(m, ext)] + [case["c"]], dtype=x.dtype, device="cuda")
    inside(tile, m, ext).copy_(x)
    return {"case": case, "desc": sc.tile_desc(case["n"], case["c"], ext, m, m), "tile": tile, "slabs": slabs,
            "send": {k: torch.empty_like(v) for k, v in slabs.items()}}


def run_halo(st):
    w, tile, desc = st["case"]["width"], st["tile"], st["desc"]
    for a, l in enumerate(st["case"]["shard"]):
        if l != "-":
            sc.shard_halo_pack_pair(desc, tile, a, w if l == "m" else 0, st["send"].get((a, 0)), w, st["send"][a, 1])
            sc.shard_halo_unpack_pair(desc, tile, a, st["slabs"].get((a, 0)), st["slabs"][a, 1])
    return {"tile": tile, "send": [st["send"][k] for k in sorted(st["send"])]}


def exact_halo(case, seed):
    x, slabs, m = halo_inputs(case, seed)
    ext = axes_of(case)
    tile = torch.zeros([case["n"]] + [2 * a + b for a, b in zip(m, ext)] + [case["c"]], dtype=torch.float64,
                       device="cuda")
    inside(tile, m, ext).copy_(x)
    send = {}
    for a in range(len(ext)):
        for side in (0, 1):
            if (a, side) in slabs:
                t = tile.narrow(1 + a, m[a] if side == 0 else ext[a], case["width"])
                for b in range(a + 1, len(ext)):
                    t = t.narrow(1 + b, m[b], ext[b])
                send[a, side] = t.clone()
        fill_margins(tile, {k: v for k, v in slabs.items() if k[0] == a}, m, m, ext)
    return {"tile": tile, "send": [send[k] for k in sorted(send)]}


def work_halo(case):
    ext, w, esz = axes_of(case), case["width"], DTYPES[case["dtype"]][1]
    m = [0 if l == "-" else w for l in case["shard"]]
    moved = 0
    for a, l in enumerate(case["shard"]):
        one = math.prod(slab_shape(case["n"], case["c"], ext, m, m, a, w)) * esz
        # a face packed and a slab unpacked are each read and written; a zero-filled margin is written
        moved += {"-": 0, "m": 8, "e": 5}[l] * one
    return {"bytes": moved, "flops": 0}


# --- normalisation -------------------------------------------------------------------

def norm_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = field(gen, case["n"], case["c"], axes_of(case), DTYPES[case["dtype"]][0])
    gamma = 1 + 0.1 * torch.randn(case["c"], generator=gen, device="cuda")
    beta = 0.1 * torch.randn(case["c"], generator=gen, device="cuda")
    return x, gamma, beta


def prepare_norm(case, seed):
    x, gamma, beta = norm_inputs(case, seed)
    ext = axes_of(case)
    m = [case["halo"]] + [0] * (len(ext) - 1)
    tile = torch.zeros([case["n"]] + [2 * a + b for a, b in zip(m, ext)] + [case["c"]], dtype=x.dtype, device="cuda")
    inside(tile, m, ext).copy_(x)
    desc = sc.tile_desc(case["n"], case["c"], ext, m, m)
    code = sc.SHARD_F32 if case["dtype"] == "f32" else sc.SHARD_BF16
    ws = torch.empty(max(16, sc.shard_norm_workspace_bytes(desc, code, case["groups"])), dtype=torch.uint8,
                     device="cuda")
    sums = torch.empty([case["n"], case["groups"], 2], dtype=torch.float64, device="cuda")
    return {"case": case, "desc": desc, "tile": tile, "gamma": gamma, "beta": beta, "ws": ws, "sums": sums,
            "out": torch.zeros_like(tile), "count": math.prod(ext) * case["c"] // case["groups"]}


def run_norm(st):
    g = st["case"]["groups"]
    sc.shard_norm_stats(st["desc"], st["tile"], g, st["sums"], st["ws"])
    sc.shard_norm_apply(st["desc"], st["tile"], st["sums"], st["count"], 1e-5, g, st["gamma"], st["beta"], st["out"],
                        st["ws"])
    return {"sums": st["sums"], "out": st["out"]}


def exact_norm(case, seed):
    x, gamma, beta = norm_inputs(case, seed)
    ext, n, c, g = axes_of(case), case["n"], case["c"], case["groups"]
    v = x.double().view(n, -1, g, c // g)
    s1, s2 = v.sum((1, 3)), (v * v).sum((1, 3))
    count = math.prod(ext) * c // g
    mean = s1 / count
    rstd = 1 / torch.sqrt((s2 / count - mean * mean).clamp_min(0) + 1e-5)
    y = ((v - mean[:, None, :, None]) * rstd[:, None, :, None]).view([n] + ext + [c]) * gamma.double() + beta.double()
    m = [case["halo"]] + [0] * (len(ext) - 1)
    out = torch.zeros([n] + [2 * a + b for a, b in zip(m, ext)] + [c], dtype=torch.float64, device="cuda")
    inside(out, m, ext).copy_(y)
    return {"sums": torch.stack([s1, s2], -1), "out": out}


def work_norm(case):
    b = case["n"] * math.prod(axes_of(case)) * case["c"] * DTYPES[case["dtype"]][1]
    # the sums have to be complete before the first element can be normalised: the interior is read twice
    return {"bytes": 3 * b, "flops": 0}


# --- ring attention ------------------------------------------------------------------

def attn_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    b, h, d = case["b"], case["h"], case["d"]
    q = randn(gen, [b, h, case["sq"], d], torch.bfloat16)
    kv = [(randn(gen, [b, h, case["sk"], d], torch.bfloat16), randn(gen, [b, h, case["sk"], d], torch.bfloat16))
          for _ in range(case["blocks"])]
    return q, kv


def prepare_attn(case, seed):
    q, kv = attn_inputs(case, seed)
    return {"q": q, "kv": kv, "o": torch.empty(q.shape, dtype=torch.float32, device="cuda"),
            "lse": torch.empty(q.shape[:3], dtype=torch.float32, device="cuda"), "scale": 1 / math.sqrt(case["d"])}


def run_attn(st):
    for i, (k, v) in enumerate(st["kv"]):
        sc.shard_attn_block(st["q"], k, v, st["o"], st["lse"], st["scale"], i == 0)
    return {"o": st["o"], "lse": st["lse"]}


def exact_attn(case, seed):
    q, kv = attn_inputs(case, seed)
    scale = 1 / math.sqrt(case["d"])
    o = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device="cuda")
    for b in range(case["b"]):
        for h in range(case["h"]):
            k = torch.cat([x[0][b, h] for x in kv]).double()
            v = torch.cat([x[1][b, h] for x in kv]).double()
            s = (q[b, h].double() @ k.t().contiguous()) * scale
            lse[b, h] = torch.logsumexp(s, 1)
            o[b, h] = torch.softmax(s, 1) @ v
    return {"o": o, "lse": lse}


def work_attn(case):
    bh, d, sq, keys = case["b"] * case["h"], case["d"], case["sq"], case["sk"] * case["blocks"]
    return {"bytes": bh * (sq * d * 2 + keys * d * 4 + sq * d * 4 + sq * 4), "flops": 4.0 * bh * sq * keys * d}


KINDS = {"conv": (prepare_conv, exact_conv, work_conv), "halo": (prepare_halo, exact_halo, work_halo),
         "norm": (prepare_norm, exact_norm, work_norm), "attn": (prepare_attn, exact_attn, work_attn)}


def prepare(case, seed):
    return dict(KINDS[case["kind"]][0](case, seed), kind=case["kind"])


def run(state):
    return {"conv": run_conv, "halo": run_halo, "norm": run_norm, "attn": run_attn}[state["kind"]](state)


def exact(case, seed):
    return KINDS[case["kind"]][1](case, seed)


def work(case):
    return KINDS[case["kind"]][2](case)


def tolerance(case):
    # about four times the error against 64 bits that the cases show
    if case["kind"] == "halo":
        return "exact"
    if case["kind"] == "attn":
        # probabilities rounded to bf16 against a reference maximum that an implementation may choose: 1.7e-3
        return {"rel": 7e-3, "max": 4e-2}
    if case["dtype"] == "f32":
        # binary32 sums: 1.5e-7 to 2.1e-6 over the sizes here, five times that at the largest
        return {"rel": 1e-5, "max": 6e-5}
    # bf16 outputs of binary32 sums: 1.7e-3, at most half a step of the last place (2e-3 to 3.9e-3)
    return {"rel": 7e-3, "max": 1.6e-2}
