"""Performance cases of the neural-texture decode library.

Each case is work that a program using this library has it do through its public
entry points (``paper_2608_27888_amd.ntc``): binning and decoding a frame, the
decode in stream order, the latent gather alone, the divergence measurements,
and the clustering of textures into shared decoders.  Sizes are those of the
library's own workloads (tiny, single, divergent, clustered4k, wide_trilinear,
k_per_wave) and of its timing study; ``draw`` varies them over the same ranges.

Inputs are drawn on the GPU from the seed alone: latents ~ N(0, 1) in fp16,
Kaiming-uniform weights and biases U(-0.1, 0.1) in fp16, screen-coherent or
random texture coordinates, and one of five material layouts:

  one      texture 0 everywhere, uv over the whole screen
  tiles    one texture per 8x8 pixel tile, drawn uniformly
  regions  a Voronoi map of seeded sites (2,000 at 3840x2160, in proportion to
           the area elsewhere), each with its own texture, uv offset and scale
  lanes    every 64-query wave holds every texture once in turn
  random   texture and uv drawn per query, without coherence

Each drawn seed gives other latents, weights, maps, layouts and coordinates.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2608_27888_amd import ntc

DEV = "cuda"
PAD = -1  # NTC_PAD as int32
SITES_AT_4K = 2000


def _decode(name, op, **kw):
    """A case that samples latents; the defaults are the clustered frame's shape."""
    c = {"name": name, "op": op, "width": 1920, "height": 1080, "spp": 1, "layout": "regions",
         "textures": 512, "decoders": 16, "map": "zipf", "base": 256, "levels": 2, "channels": 16,
         "hidden": 64, "hidden_layers": 1, "out": 8, "mip": False, "pe": 0, "slope": 0.0,
         "rows": "f32", "engine": "mfma"}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: 65,536 incoherent queries over 4 small textures and 2
        # decoders, as a tool or a texture-space pass issues it; launches and
        # latency count.
        _decode("tiny_64k", "frame", width=256, height=256, layout="random", textures=4,
                decoders=2, map="equal", base=64, channels=8),
        # A 1080p frame of one material: one decoder, nothing to sort.
        _decode("single_1080p", "frame", layout="one", textures=1, decoders=1, map="equal",
                base=512),
        # A 1080p frame whose 8x8 tiles all differ in material, a decoder each: the
        # divergent frame the paper starts from, at its binning limit.
        _decode("divergent_1080p", "frame", layout="tiles", textures=64, decoders=64,
                map="equal"),
        # The ordinary 4K frame: 512 textures clustered into 16 shared decoders.
        _decode("clustered_4k", "frame", width=3840, height=2160),
        # The same frame with a decoder per texture (nothing clustered).
        _decode("per_texture_4k", "frame", width=3840, height=2160, decoders=512, map="equal"),
        # The largest: 4 samples a pixel at 4K, 3 latent levels blended by mip, a
        # 48-128-128-128-8 decoder.
        _decode("wide_trilinear_4k", "frame", width=3840, height=2160, spp=4, decoders=8,
                map="equal", base=512, levels=3, hidden=128, hidden_layers=2, mip=True),
        # The decoder of the paper's own training setup: positional encoding,
        # LeakyReLU, RGB rows in fp16, an odd-sized frame.
        _decode("setup_rgb_1440p", "frame", width=2559, height=1439, out=3, pe=4, slope=0.01,
                rows="f16"),
        # A frame decoded in stream order, without binning: what a renderer calls
        # when it cannot afford the sort, and the paper's baseline.
        _decode("stream_1080p", "stream"),
        # The timing study's image with ten decoders in every wave, on the per-lane
        # vector engine.
        _decode("lanes10_fma_1024", "stream", width=1024, height=1024, layout="lanes",
                textures=10, decoders=10, map="equal", engine="fma"),
        # Feature vectors alone, for a decoder outside the library (a program's own
        # MLP, training-side checks).
        _decode("gather_1080p", "gather", rows="f16"),
        # Both divergence measurements of a 4K frame: per 64-query wave and per 8x8
        # screen block.
        _decode("divergence_4k", "divergence", width=3840, height=2160, block=8),
        # 512 textures' embeddings clustered into 16 decoder groups.
        {"name": "cluster_512", "op": "kmeans", "points": 512, "groups": 16, "dim": 512,
         "spread": 0.35, "max_iter": 100},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _screen(rng, lo, hi):
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    aspect = rng.uniform(1.0, 2.0)
    w = max(1, int(math.sqrt(n * aspect)))
    return w, max(1, int(n / w))


def draw(rng):
    op = rng.choice(["frame"] * 6 + ["stream", "stream", "gather", "divergence", "kmeans"])
    if op == "kmeans":
        n = _log_int(rng, 64, 1024)
        return {"op": op, "points": n, "groups": _log_int(rng, 2, min(40, n)),
                "dim": _log_int(rng, 16, 512), "spread": round(rng.uniform(0.2, 0.9), 2),
                "max_iter": 100}
    c = _decode("", op)
    del c["name"]
    c["width"], c["height"] = _screen(rng, 1 << 14, (1 << 23) if op != "stream" else (1 << 21))
    if rng.random() < 0.2 and c["width"] * c["height"] < (1 << 21):
        c["spp"] = rng.choice([2, 4])
    c["layout"] = rng.choice(["one", "tiles", "regions", "regions", "regions", "lanes", "random"])
    if c["layout"] == "one":
        c["textures"] = c["decoders"] = 1
    elif c["layout"] == "lanes":
        c["textures"] = c["decoders"] = rng.randint(2, 10)
    elif c["layout"] == "random":  # incoherent: a few small textures
        c["textures"] = rng.randint(2, 16)
        c["decoders"] = rng.randint(1, min(4, c["textures"]))
    else:
        c["textures"] = _log_int(rng, 4, 512)
        c["decoders"] = (c["textures"] if rng.random() < 0.25
                         else _log_int(rng, 1, min(64, c["textures"])))
    c["map"] = rng.choice(["zipf", "equal"]) if c["decoders"] < c["textures"] else "equal"
    if c["layout"] == "random":
        c["base"] = 64
    else:
        c["base"] = rng.choice([64, 100, 128, 256, 256, 512 if c["textures"] <= 128 else 256])
    if op == "divergence":
        c["block"] = rng.choice([4, 8, 8, 16, 5])
        c["spp"] = 1
        return c
    c["levels"], c["channels"] = rng.choice([(2, 8), (2, 16), (2, 16), (3, 16)])
    c["rows"] = rng.choice(["f32", "f32", "f16"])
    c["mip"] = rng.random() < 0.25
    if op == "gather":
        return c
    c["hidden"] = rng.choice([64, 64, 64, 128])
    c["hidden_layers"] = rng.choice([1, 1, 2])
    c["out"] = rng.choice([8, 8, 3, 4, rng.randint(1, 16)])
    c["slope"] = rng.choice([0.0, 0.0, 0.01, 0.2])
    if c["levels"] == 2 and c["hidden"] == 64 and c["hidden_layers"] == 1 and not c["mip"]:
        c["pe"] = rng.choice([0, 0, 4, 8])
    if op == "stream" and c["hidden"] == 64 and not c["mip"] and rng.random() < 0.3:
        c["engine"], c["out"] = "fma", rng.choice([8, 16])
    return c


# ------------------------------------------------------------------------- sizes


def _res(case):
    return [max(2, case["base"] >> k) for k in range(case["levels"])]


def _dims(case):
    f = case["levels"] * case["channels"] + 4 * case["pe"]
    return [f] + [case["hidden"]] * (1 + case["hidden_layers"]) + [case["out"]]


def _n(case):
    return case["width"] * case["height"] * case["spp"]


def _mlp_flops(case):
    d = _dims(case)
    return sum(2 * a * b for a, b in zip(d[:-1], d[1:]))


def _latent_bytes(case):
    """Latent texels that the queries touch, each once, without the rims of the
    touched areas (a lower estimate)."""
    n, total = _n(case), 0.0
    for r in _res(case):
        every = case["textures"] * r * r
        if case["layout"] == "one" or case["layout"] == "tiles":
            touched = r * r  # every screen position once, in whichever texture
        elif case["layout"] == "regions":
            touched = r * r * 3.79  # mean of scale^2, scale = 2^U(-1, 2)
        else:
            touched = every
        total += min(every, touched, 4.0 * n) * case["channels"] * 2
    return total


def work(case):
    if case["op"] == "kmeans":
        # two assignments at the least: one that moves labels, one that finds no move
        n, m, d = case["points"], case["groups"], case["dim"]
        return {"bytes": 4 * n * d + 8 * m * d + 4 * n + 4 * m, "flops": 2 * 3 * n * m * d}
    n = _n(case)
    if case["op"] == "divergence":
        blocks = -(-case["width"] // case["block"]) * -(-case["height"] // case["block"])
        return {"bytes": 2 * 4 * n + 4 * (n // 64) + 4 * blocks, "flops": 0}
    es = 4 if case["rows"] == "f32" else 2
    per = 4 + 8 + (4 if case["mip"] else 0)  # texture id, uv, mip
    if case["op"] == "gather":
        per += case["levels"] * case["channels"] * es
        return {"bytes": n * per + _latent_bytes(case), "flops": 0}
    per += case["out"] * es + (4 if case["op"] == "frame" else 0)  # row; permutation entry
    d = _dims(case)
    params = 2 * case["decoders"] * sum(b * (a + 1) for a, b in zip(d[:-1], d[1:]))
    return {"bytes": n * per + _latent_bytes(case) + params, "flops": n * _mlp_flops(case)}


def tolerance(case):
    if case["op"] == "divergence":
        return "exact"
    if case["op"] == "kmeans":
        return {"rel": 1e-12, "max": 1e-11}
    # About four times the distance of the fp16 path from float64 (relative 1.9e-4 for
    # fp32 rows, 2.8e-4 for fp16 rows, largest single value 2.3e-3; feature rows 3.9e-4
    # and 3.2e-3).
    if case["op"] == "gather":
        return {"rel": 1.6e-3, "max": 1.3e-2}
    return {"rel": 8e-4 if case["rows"] == "f32" else 1.2e-3, "max": 9e-3}


# ------------------------------------------------------------------------ inputs


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _map(case, g):
    """texture -> decoder, int32 [textures]."""
    T, D = case["textures"], case["decoders"]
    if D == T:
        return torch.arange(T, dtype=torch.int32, device=DEV)
    order = torch.randperm(T, generator=g, device=DEV)
    if case["map"] == "equal":
        sizes = torch.full((D,), T // D, dtype=torch.int64)
        sizes[: T % D] += 1
    else:
        w = torch.arange(1, D + 1, dtype=torch.float64) ** -1.1
        q = T * w / w.sum()
        sizes = q.floor().to(torch.int64)
        rest = torch.argsort(q - q.floor(), descending=True, stable=True)
        sizes[rest[: T - int(sizes.sum())]] += 1
    labels = torch.repeat_interleave(torch.arange(D, dtype=torch.int32), sizes).to(DEV)
    m = torch.empty(T, dtype=torch.int32, device=DEV)
    m[order] = labels
    return m


def _pixels(case):
    i = torch.arange(_n(case), dtype=torch.int64, device=DEV) // case["spp"]
    return i % case["width"], i // case["width"]


def _regions(case, g):
    """Index of the nearest of the seeded sites, per pixel (int64 [height * width])."""
    W, H = case["width"], case["height"]
    sites = max(4, round(SITES_AT_4K * W * H / (3840 * 2160)))
    at = torch.rand((sites, 2), generator=g, device=DEV) * torch.tensor([W, H], device=DEV)
    half = (at * at).sum(1) / 2
    out = torch.empty(W * H, dtype=torch.int64, device=DEV)
    step = max(1, (1 << 28) // sites)
    for a in range(0, W * H, step):
        i = torch.arange(a, min(W * H, a + step), device=DEV)
        x, y = (i % W).float() + 0.5, torch.div(i, W, rounding_mode="floor").float() + 0.5
        d = torch.addcmul(half[None, :] - x[:, None] * at[None, :, 0], y[:, None],
                          at[None, :, 1], value=-1)
        out[a:a + step] = d.argmin(1)
    return out, sites


def _queries(case, g):
    """(tex_id int32 [n], uv float32 [n, 2], mip float32 [n] or None)."""
    n, T, W, H = _n(case), case["textures"], case["width"], case["height"]
    uv = torch.rand((n, 2), generator=g, device=DEV)  # the jitter inside a pixel
    if case["layout"] == "random":
        tex = torch.randint(0, T, (n,), generator=g, device=DEV, dtype=torch.int32)
    else:
        x, y = _pixels(case)
        u = (x + uv[:, 0].double()) / W
        v = (y + uv[:, 1].double()) / H
        if case["layout"] == "one":
            tex = torch.zeros(n, dtype=torch.int32, device=DEV)
        elif case["layout"] == "tiles":
            tw, th = -(-W // 8), -(-H // 8)
            tiles = torch.randint(0, T, (th * tw,), generator=g, device=DEV, dtype=torch.int32)
            tex = tiles[(y // 8) * tw + x // 8]
        elif case["layout"] == "lanes":
            tex = (torch.arange(n, device=DEV) % 64 % T).to(torch.int32)
        else:
            region, sites = _regions(case, g)
            region = torch.repeat_interleave(region, case["spp"]) if case["spp"] > 1 else region
            pick = torch.randint(0, T, (sites,), generator=g, device=DEV, dtype=torch.int32)
            off = torch.rand((sites, 2), generator=g, device=DEV).double()
            scale = 2.0 ** (torch.rand(sites, generator=g, device=DEV).double() * 3 - 1)
            tex = pick[region]
            u = torch.remainder(off[region, 0] + scale[region] * u, 1.0)
            v = torch.remainder(off[region, 1] + scale[region] * v, 1.0)
        uv = torch.stack([u, v], 1).float().clamp_(0.0, 1.0 - 2.0 ** -24)
    mip = None
    if case["mip"]:
        mip = torch.rand(n, generator=g, device=DEV) * 2.0
    return tex.contiguous(), uv.contiguous(), mip


def _model(case, g):
    T, res, ch = case["textures"], _res(case), case["channels"]
    stride = sum(r * r * ch for r in res)
    latents = torch.empty((T, stride), dtype=torch.float16, device=DEV)
    step = max(1, (1 << 28) // stride)
    for t in range(0, T, step):
        latents[t:t + step].normal_(generator=g)
    dims, D = _dims(case), case["decoders"]
    parts = []
    for a, b in zip(dims[:-1], dims[1:]):
        bound = math.sqrt(6.0 / a)
        parts.append((torch.rand((D, b * a), generator=g, device=DEV) * 2 - 1) * bound)
        parts.append((torch.rand((D, b), generator=g, device=DEV) * 2 - 1) * 0.1)
    params = torch.cat(parts, 1).half().contiguous()
    return ntc.DeviceModel(T, res, [ch] * case["levels"], latents.view(torch.int16).reshape(-1), D,
                           dims, params.view(torch.int16).reshape(-1), _map(case, g),
                           case["pe"])


def _points(case, seed, g):
    """Unit feature vectors around group centres with Zipf(1.1) sizes, and seeds."""
    n, m, d = case["points"], case["groups"], case["dim"]
    centres = torch.randn((m, d), generator=g, device=DEV)
    centres /= centres.norm(dim=1, keepdim=True)
    w = torch.arange(1, m + 1, device=DEV, dtype=torch.float64) ** -1.1
    u = torch.rand(n, generator=g, device=DEV).double()
    group = torch.searchsorted(torch.cumsum(w / w.sum(), 0), u).clamp_(max=m - 1)
    f = centres[group] + torch.randn((n, d), generator=g, device=DEV) * (
        case["spread"] / math.sqrt(d))
    f /= f.norm(dim=1, keepdim=True)
    init = np.sort(np.random.default_rng(int(seed)).choice(n, size=m, replace=False))
    return f.contiguous(), init.astype(np.uint32)


def prepare(case, seed):
    g = _generator(seed)
    if case["op"] == "kmeans":
        f, init = _points(case, seed, g)
        return SimpleNamespace(case=case, features=f, init=init)
    if case["op"] == "divergence":
        tex, _, _ = _queries(case, g)
        return SimpleNamespace(case=case, tex=tex, tex_to_dec=_map(case, g))
    model = _model(case, g)
    queries = ntc.DeviceQueries(*_queries(case, g))
    half = case["rows"] == "f16"
    width = sum(model.channels) if case["op"] == "gather" else case["out"]
    out = torch.zeros((queries.n, width), dtype=torch.float16 if half else torch.float32,
                      device=DEV)
    bins = None
    if case["op"] == "frame":
        bins = ntc.alloc_bins(queries.n, case["decoders"], 64, DEV)
        bins.perm.fill_(PAD)  # entries past the last bin are left untouched
    return SimpleNamespace(case=case, model=model, queries=queries, out=out, bins=bins)


def run(s):
    c = s.case
    if c["op"] == "kmeans":
        k = ntc.kmeans(s.features, s.init, c["max_iter"])
        return {"assign": k.assign, "centroids": k.centroids, "counts": k.counts,
                "iterations": k.iterations, "converged": k.converged}
    if c["op"] == "divergence":
        per, tot = ntc.divergence_stats(s.tex, s.tex_to_dec, c["decoders"])
        dmap, hist, mtot = ntc.divergence_map(s.tex, c["width"], c["height"], s.tex_to_dec,
                                              c["decoders"], 1, c["block"], c["block"])
        return {"per_wave": per, "totals": tot, "map": dmap, "histogram": hist,
                "map_totals": mtot}
    if c["op"] == "gather":
        return {"rows": ntc.gather_features(s.model, s.queries, s.out, s.out.dtype)}
    slope = c["slope"] or None
    if c["op"] == "stream":
        return {"rows": ntc.decode(s.model, s.queries, None, out=s.out, leaky_slope=slope,
                                   out_dtype=s.out.dtype, engine=c["engine"])}
    ntc.build_bins(s.queries.tex_id, s.model.tex_to_dec, c["decoders"], bins=s.bins)
    rows = ntc.decode(s.model, s.queries, s.bins, out=s.out, leaky_slope=slope,
                      out_dtype=s.out.dtype)
    return {"rows": rows, "bin_count": s.bins.bin_count, "bin_offset": s.bins.bin_offset,
            "perm": s.bins.perm}


# ------------------------------------------------------------------------- exact


def _bilinear(table, base, res, uv, rows):
    """Bilinear samples, clamp to edge, in float64.  table: fp16 [texels, channels]."""
    x, y = uv[:, 0] * res - 0.5, uv[:, 1] * res - 0.5
    x0, y0 = torch.floor(x), torch.floor(y)
    fx, fy = (x - x0)[:, None], (y - y0)[:, None]
    xi = [(x0 + k).clamp(0, res - 1).long() for k in (0, 1)]
    yi = [(y0 + k).clamp(0, res - 1).long() for k in (0, 1)]
    base = base + rows

    def tap(j, i):
        return table[base + yi[j] * res + xi[i]].double()

    top = tap(0, 0) * (1 - fx) + tap(0, 1) * fx
    low = tap(1, 0) * (1 - fx) + tap(1, 1) * fx
    return top * (1 - fy) + low * fy


def _features(case, model, tex, uv, mip):
    """float64 feature rows of the queries (latents, then positional encoding)."""
    res, ch = _res(case), case["channels"]
    table = model.latents.view(torch.float16).view(-1, ch)
    texels = sum(r * r for r in res)
    first = np.cumsum([0] + [r * r for r in res])
    base, uv = tex.long() * texels, uv.double()
    parts = []
    if mip is None:
        parts = [_bilinear(table, base, r, uv, int(o)) for r, o in zip(res, first)]
    else:
        levels = [_bilinear(table, base, r, uv, int(o)) for r, o in zip(res, first)]
        stack = torch.stack(levels)
        top = case["levels"] - 1
        m = mip.double().clamp(0, top)
        at = torch.arange(tex.numel(), device=DEV)
        for k in range(case["levels"]):
            lod = m.clamp(min=k)
            k0 = lod.floor().long()
            k1 = (k0 + 1).clamp(max=top)
            t = (lod - k0)[:, None]
            parts.append(stack[k0, at] * (1 - t) + stack[k1, at] * t)
    for k in range(case["pe"]):
        for c in (0, 1):
            a = uv[:, c:c + 1] * (math.pi * 2 ** k)
            parts += [torch.sin(a), torch.cos(a)]
    return torch.cat(parts, 1)


def _kmeans64(f, init, max_iter):
    x = f.double()
    c = x[torch.from_numpy(init.astype(np.int64)).to(DEV)].clone()
    labels, m = None, c.shape[0]
    for it in range(max_iter):
        d = torch.stack([((x - c[j]) ** 2).sum(1) for j in range(m)], 1)
        new = d.argmin(1)
        if labels is not None and torch.equal(new, labels):
            return c
        labels = new
        for j in range(m):
            mine = x[labels == j]
            if mine.shape[0]:
                c[j] = mine.sum(0) / mine.shape[0]
    return c


def exact(case, seed):
    if case["op"] == "divergence":
        return None  # counts: no rounding
    if case["op"] == "kmeans":
        f, init = _points(case, seed, _generator(seed))
        return {"assign": None, "centroids": _kmeans64(f, init, case["max_iter"]), "counts": None,
                "iterations": None, "converged": None}
    n = _n(case)
    if n * _mlp_flops(case) > 4e14 and case["op"] != "gather":
        return None  # too long in float64
    s = prepare(case, seed)
    tex, uv, mip = s.queries.tex_id, s.queries.uv, s.queries.mip
    width = s.out.shape[1]
    rows = torch.empty((n, width), dtype=torch.float64, device=DEV)
    dims = _dims(case)
    stride = sum(b * (a + 1) for a, b in zip(dims[:-1], dims[1:]))
    params = s.model.params.view(torch.float16).view(-1, stride).double()
    dec = s.model.tex_to_dec.long()[tex.long()]
    slope = float(np.float16(case["slope"]))
    groups = [0] if case["op"] == "gather" else range(case["decoders"])
    for d in groups:
        of = torch.arange(n, device=DEV) if case["op"] == "gather" else (dec == d).nonzero()[:, 0]
        for q in of.split(1 << 20):
            h = _features(case, s.model, tex[q], uv[q], None if mip is None else mip[q])
            if case["op"] != "gather":
                at = 0
                for i, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
                    w = params[d, at:at + a * b].view(b, a)
                    z = h @ w.t() + params[d, at + a * b:at + a * b + b]
                    at += a * b + b
                    last = i == len(dims) - 2
                    h = torch.sigmoid(z) if last else torch.maximum(z, slope * z)
            rows[q] = h
    if case["op"] == "frame":
        return {"rows": rows, "bin_count": None, "bin_offset": None, "perm": None}
    return {"rows": rows}
