"""The workloads whose speed this repository watches.

Each case is one call of the public entry points (`paper_1812_07607_amd.ops`)
on data that is on the GPU already, at sizes taken from the repository's own
workloads (`paper_1812_07607_amd/synth.py`, `bench.py`): the near-duplicate
join of 100,000 patch histograms, joins of unit-norm embeddings from a few
thousand to a million rows, top-k joins, small and large requests against a
resident store, and the featurisers that fill the relations.

Two kinds of relation are drawn, as the workloads have them: rows of a
Gaussian mixture on the unit sphere (embeddings), and 8 x 8 x 8 colour
histograms of palette patches (their squared distances are exact in binary).
"""
import math

import torch

from paper_1812_07607_amd import ops

PALETTE = 16      # base colours of the synthetic patches
PIXEL_SIGMA = 20.0
MIX_SIGMA = 0.05  # spread of a mixture component around its centre
BASE = 11         # seed of the point sets


# ------------------------------------------------------------------- cases
def listed():
    return [
        # a small on-line join (the 2,000 x 2,000 workload): latency and launches
        {"name": "eps_2k_d64", "kind": "eps", "n_r": 2000, "n_s": 2000, "d": 64, "self": False, "prec": "bf16",
         "centres": 20, "k_eps": 10},
        # deduplication of an embedding table of an odd size, half precision
        {"name": "eps_self_60k_d100_fp16", "kind": "eps", "n_r": 60001, "n_s": 60001, "d": 100, "self": True,
         "prec": "fp16", "centres": 300, "k_eps": 10},
        # the large eps-join, 10^6 x 10^6 unit vectors
        {"name": "eps_1m_d128", "kind": "eps", "n_r": 1000000, "n_s": 1000000, "d": 128, "self": False,
         "prec": "bf16", "centres": 1000, "k_eps": 10},
        # deduplication of 100,000 patch histograms: all pairs, and with the index built in the call
        {"name": "dedup_hist_100k_fp16", "kind": "hist_eps", "n": 100000, "side": 32, "prec": "fp16", "indexed": False},
        {"name": "dedup_hist_100k_indexed", "kind": "hist_eps", "n": 100000, "side": 32, "prec": "fp16",
         "indexed": True},
        # the same kind of join with float32 candidates, as that workload states it
        {"name": "eps_fp32_30k_d128", "kind": "eps", "n_r": 30000, "n_s": 40000, "d": 128, "self": False,
         "prec": "fp32", "centres": 64, "k_eps": 10},
        # closest images: top-10 of 200,000 x 200,000
        {"name": "topk_200k_d128", "kind": "topk", "n_r": 200000, "n_s": 200000, "d": 128, "k": 10, "prec": "bf16",
         "centres": 1000},
        # a batch of queries against a resident FP8 store, top-32
        {"name": "store_topk_20k_1m_d256_fp8", "kind": "store_topk", "n_r": 20000, "n_s": 1000000, "d": 256, "k": 32,
         "prec": "fp8", "centres": 1024},
        # one small request against a large resident store, each mode (serving latency)
        {"name": "store_topk_37_4m_d128", "kind": "store_topk", "n_r": 37, "n_s": 4000000, "d": 128, "k": 10,
         "prec": "bf16", "centres": 1000},
        {"name": "store_eps_900_2m_d128", "kind": "store_eps", "n_r": 900, "n_s": 2000000, "d": 128, "prec": "bf16",
         "centres": 1000, "k_eps": 10},
        # featurisation: cut patches, and ragged boxes over video frames
        {"name": "featurize_100k_32x32", "kind": "featurize", "n": 100000, "h": 32, "w": 32},
        {"name": "crops_20k_720p", "kind": "crops", "frames": 64, "height": 720, "width": 1280, "boxes": 20000,
         "max_side": 96},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["eps", "eps", "eps_self", "eps_fp32", "hist_eps", "topk", "store_topk", "store_eps",
                       "featurize", "crops"])
    if kind in ("eps", "eps_self", "eps_fp32"):
        fp32 = kind == "eps_fp32"
        n_s = _log_int(rng, 500, 40000 if fp32 else 600000)
        n_r = n_s if kind == "eps_self" else _log_int(rng, 500, 40000 if fp32 else 600000)
        return {"kind": "eps", "n_r": n_r, "n_s": n_s, "d": rng.choice([32, 64, 96, 100, 128, 200, 256]),
                "self": kind == "eps_self", "prec": "fp32" if fp32 else rng.choice(["bf16", "bf16", "fp16", "fp8"]),
                "centres": max(4, n_s // rng.choice([100, 200, 1000])), "k_eps": rng.choice([2, 5, 10])}
    if kind == "hist_eps":
        return {"kind": "hist_eps", "n": _log_int(rng, 1000, 100000), "side": rng.choice([16, 32]), "prec": "fp16",
                "indexed": rng.random() < 0.5}
    if kind == "topk":
        return {"kind": "topk", "n_r": _log_int(rng, 500, 200000), "n_s": _log_int(rng, 2000, 300000),
                "d": rng.choice([64, 100, 128, 256]), "k": rng.choice([1, 10, 32, 50]),
                "prec": rng.choice(["bf16", "fp16"]), "centres": rng.choice([100, 1000])}
    if kind in ("store_topk", "store_eps"):
        case = {"kind": kind, "n_r": _log_int(rng, 1, 20000), "n_s": _log_int(rng, 100000, 4000000),
                "d": rng.choice([64, 128]), "prec": rng.choice(["bf16", "fp16"]), "centres": 1000}
        if kind == "store_topk":
            return dict(case, k=rng.choice([1, 10, 32]))
        return dict(case, k_eps=10)
    if kind == "featurize":
        h, w = rng.choice([(32, 32), (16, 48), (31, 33), (64, 64), (20, 20)])
        return {"kind": "featurize", "n": _log_int(rng, 100, 60000), "h": h, "w": w}
    return {"kind": "crops", "frames": rng.choice([8, 64]), "height": 720, "width": 1280,
            "boxes": _log_int(rng, 50, 40000), "max_side": rng.choice([64, 96, 200])}


# ------------------------------------------------------------------ inputs
def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _mixture(n, d, centres, seed, stream):
    """n unit rows around `centres` random directions (shared by the streams,
    so two streams give two relations of one mixture); the seed orders the
    rows and turns the space (coordinates permuted and mirrored)."""
    g = _gen(BASE, 1)
    mu = torch.randn(centres, d, device="cuda", generator=g)
    mu /= mu.norm(dim=1, keepdim=True)
    g = _gen(BASE, 2 + stream)
    out = torch.empty(n, d, device="cuda")
    step = 1 << 20
    for lo in range(0, n, step):
        m = min(step, n - lo)
        x = torch.randn(m, d, device="cuda", generator=g).mul_(MIX_SIGMA)
        x += mu[torch.randint(centres, (m,), device="cuda", generator=g)]
        out[lo:lo + m] = x / x.norm(dim=1, keepdim=True)
    if seed is None:
        return out
    g = _gen(seed, 3)
    turn = torch.randperm(d, device="cuda", generator=g)
    mirror = torch.randint(2, (d,), device="cuda", generator=g).float() * 2 - 1
    order = torch.randperm(n, device="cuda", generator=_gen(seed, 20 + stream))
    for lo in range(0, n, step):  # in place, through columns: no second relation
        out[lo:lo + step] = out[lo:lo + step][:, turn] * mirror
    return out[order]


def _radius(case):
    """Median k-th neighbour distance of some rows (a self-join's own row aside)."""
    R, S = _relations(case, None)
    k, self_join = case["k_eps"], case.get("self", False)
    q = R[:: max(1, R.shape[0] // 128)][:128]
    d2 = (q * q).sum(1, keepdim=True) + (S * S).sum(1)[None, :] - 2 * (q @ S.T)
    k = min(k + (1 if self_join else 0), S.shape[0])
    kth = torch.topk(d2, k, dim=1, largest=False).values[:, -1].clamp_min(0)
    return float(kth.double().sqrt().median())


def _patches(n, h, w, seed):
    """uint8 RGB patches: one of 16 base colours plus Gaussian noise per pixel and channel."""
    g = _gen(seed, 5)
    base = torch.randint(0, 256, (PALETTE, 3), device="cuda", generator=g).float()
    out = torch.empty(n, h, w, 3, dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 24) // (h * w))
    for lo in range(0, n, step):
        m = min(step, n - lo)
        c = torch.randint(PALETTE, (m,), device="cuda", generator=g)
        z = torch.randn(m, h, w, 3, device="cuda", generator=g).mul_(PIXEL_SIGMA)
        z += base[c][:, None, None, :]
        out[lo:lo + m] = z.round_().clamp_(0, 255).to(torch.uint8)
    return out


def _frames_and_boxes(case, seed):
    """Frames in large flat coloured areas with noise, and boxes with log-uniform sides."""
    g = _gen(seed, 6)
    nf, hh, ww, m = case["frames"], case["height"], case["width"], case["boxes"]
    base = torch.randint(0, 256, (nf, hh // 40 + 1, ww // 40 + 1, 3), device="cuda", generator=g).float()
    frames = torch.empty(nf, hh, ww, 3, dtype=torch.uint8, device="cuda")
    ys, xs = torch.arange(hh, device="cuda") // 40, torch.arange(ww, device="cuda") // 40
    for f in range(nf):
        z = torch.randn(hh, ww, 3, device="cuda", generator=g).mul_(PIXEL_SIGMA)
        z += base[f][ys][:, xs]
        frames[f] = z.round_().clamp_(0, 255).to(torch.uint8)
    lo, hi = math.log(4.0), math.log(float(case["max_side"]))
    u = torch.rand(m, 4, device="cuda", generator=g, dtype=torch.float64)
    w = torch.exp(lo + (hi - lo) * u[:, 0]).round().long()
    h = torch.exp(lo + (hi - lo) * u[:, 1]).round().long()
    x0 = (u[:, 2] * (ww - w + 1)).long()
    y0 = (u[:, 3] * (hh - h + 1)).long()
    f = torch.randint(nf, (m,), device="cuda", generator=g)
    return frames, torch.stack([f, x0, y0, x0 + w, y0 + h], 1).to(torch.int32)


def _bins(px):
    """Cell of each pixel in the 8 x 8 x 8 colour cube."""
    p = px.long() >> 5
    return (p[..., 0] * 8 + p[..., 1]) * 8 + p[..., 2]


def _counts(patches):
    n = patches.shape[0]
    out = torch.zeros(n, 512, dtype=torch.int32, device="cuda")
    step = max(1, (1 << 24) // (patches.shape[1] * patches.shape[2]))
    for lo in range(0, n, step):
        b = _bins(patches[lo:lo + step]).reshape(-1, patches.shape[1] * patches.shape[2])
        out[lo:lo + step].scatter_add_(1, b, torch.ones_like(b, dtype=torch.int32))
    return out


def _histograms(case, seed):
    h = _counts(_patches(case["n"], case["side"], case["side"], BASE))
    if seed is not None:
        g = _gen(seed, 8)
        channels = torch.randperm(3, device="cuda", generator=g).tolist()
        inverted = [c + 1 for c in range(3) if int(torch.randint(2, (1,), device="cuda", generator=g))]
        h = h.reshape(-1, 8, 8, 8).permute(0, *(c + 1 for c in channels)).flip(inverted).reshape(-1, 512)
        h = h[torch.randperm(case["n"], device="cuda", generator=g)]
    return h.float() / (case["side"] * case["side"])


def _hist_radius(case):
    """The 0.01% quantile of the distances of 200,000 random pairs (the lower order statistic)."""
    H = _histograms(case, None)
    g = _gen(BASE, 7)
    i = torch.randint(H.shape[0], (200000,), device="cuda", generator=g)
    j = torch.randint(H.shape[0] - 1, (200000,), device="cuda", generator=g)
    j += j >= i
    d2 = torch.cat([((H[a] - H[b]).double() ** 2).sum(1) for a, b in zip(i.split(50000), j.split(50000))])
    return math.sqrt(float(d2.sort().values[19]))


def _relations(case, seed):
    R = _mixture(case["n_r"], case["d"], case["centres"], seed, 0)
    return R, R if case.get("self") else _mixture(case["n_s"], case["d"], case["centres"], seed, 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "featurize":
        return {"case": case, "patches": _patches(case["n"], case["h"], case["w"], seed)}
    if kind == "crops":
        frames, boxes = _frames_and_boxes(case, seed)
        return {"case": case, "frames": frames, "boxes": boxes}
    if kind == "hist_eps":
        H = _histograms(case, seed)
        return {"case": case, "R": H, "eps": _hist_radius(case)}
    R, S = _relations(case, seed)
    state = {"case": case, "R": R, "S": S}
    if "k_eps" in case:
        state["eps"] = _radius(case)
    if kind.startswith("store"):
        state["store"] = ops.Store(S, case["prec"])
    return state


# --------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "featurize":
        return ops.featurize_rgb8(state["patches"], 8)
    if kind == "crops":
        return ops.featurize_crops_rgb8(state["frames"], state["boxes"], 8)
    if kind == "topk":
        r = ops.join_topk(state["R"], state["S"], case["k"], prec=case["prec"])
        return r.j, r.dist
    if kind == "store_topk":
        r = state["store"].join_topk(state["R"], case["k"])
        return r.j, r.dist
    if kind == "store_eps":
        r = state["store"].join_eps(state["R"], state["eps"])
    elif kind == "hist_eps" and case["indexed"]:
        r, _ = ops.join_eps_indexed(state["R"], None, state["eps"], prec=case["prec"])
    elif kind == "hist_eps" or case["self"]:
        r = ops.join_eps(state["R"], None, state["eps"], prec=case["prec"])
    else:
        r = ops.join_eps(state["R"], state["S"], state["eps"], prec=case["prec"])
    return r.i, r.j, r.dist


def work(case):
    """Inputs read once, outputs written once (about ten pairs of 12 bytes a
    row), and one multiply-add per pair and coordinate."""
    kind = case["kind"]
    if kind == "featurize":
        px = case["n"] * case["h"] * case["w"]
        return {"bytes": 3 * px + 2048 * case["n"], "flops": px}
    if kind == "crops":
        # mean of the square of a log-uniform side
        mean = (case["max_side"] - 4) / math.log(case["max_side"] / 4)
        px = int(case["boxes"] * mean * mean)
        return {"bytes": 3 * px + 2048 * case["boxes"], "flops": px}
    if kind == "hist_eps":
        n = case["n"]
        pairs = n * n // 2 // (PALETTE if case["indexed"] else 1)  # patches of one colour, with the index
        return {"bytes": 4 * 512 * n, "flops": 2 * 512 * pairs}
    n_r, n_s, d = case["n_r"], case["n_s"], case["d"]
    out = 8 * n_r * case["k"] if "k" in case else 12 * 10 * n_r
    if case.get("self"):
        return {"bytes": 4 * d * n_r + out, "flops": d * n_r * n_r}
    elem = {"fp8": 1, "fp32": 4}.get(case["prec"], 2) if kind.startswith("store") else 4  # a store holds its copy
    return {"bytes": 4 * d * n_r + elem * d * n_s + out, "flops": 2 * d * n_r * n_s}


# ------------------------------------------------- the results in 64 bits
def _d2_of(R, S, i, j):
    step = max(1, (1 << 27) // R.shape[1])
    return torch.cat([((R[a].double() - S[b].double()) ** 2).sum(1) for a, b in zip(i.split(step), j.split(step))]) \
        if i.numel() else torch.empty(0, dtype=torch.float64, device="cuda")


def _pairs64(R, S, eps, self_join):
    """(i, j, distance) with distance <= eps: a float32 product finds every
    pair near the radius or inside it, the float64 differences decide."""
    nr, ns = (R * R).sum(1), (S * S).sum(1)
    slack = 1e-4 * float(nr.max() + ns.max())
    step = max(1, (1 << 30) // S.shape[0])
    out = []
    for lo in range(0, R.shape[0], step):
        g = R[lo:lo + step] @ S.T
        g.mul_(-2).add_(ns[None, :])
        hit = (g <= (eps * eps + slack - nr[lo:lo + step])[:, None]).nonzero()
        i, j = hit[:, 0] + lo, hit[:, 1]
        if self_join:
            i, j = i[i < j], j[i < j]
        d = _d2_of(R, S, i, j).sqrt()
        keep = d <= eps
        out.append((i[keep], j[keep], d[keep]))
    i, j, d = (torch.cat(x) for x in zip(*out))
    return i.to(torch.int32), j.to(torch.int32), d


def _topk64(R, S, k):
    nr, ns = (R * R).sum(1), (S * S).sum(1)
    want, spare = min(k, S.shape[0]), min(k + 16, S.shape[0])
    step = max(1, (1 << 29) // S.shape[0])
    js, ds = [], []
    for lo in range(0, R.shape[0], step):
        q = R[lo:lo + step]
        g = (q @ S.T).mul_(-2).add_(ns[None, :])
        j = torch.topk(g, spare, dim=1, largest=False).indices.sort(dim=1).values
        i = torch.arange(q.shape[0], device="cuda").repeat_interleave(spare)
        d2 = _d2_of(q, S, i, j.reshape(-1)).reshape(j.shape)
        d2, at = d2.sort(dim=1, stable=True)
        js.append(j.gather(1, at)[:, :want])
        ds.append(d2[:, :want].sqrt())
    return torch.cat(js).to(torch.int32), torch.cat(ds)


def exact(case, seed):
    kind = case["kind"]
    if kind == "featurize":
        return _counts(_patches(case["n"], case["h"], case["w"], seed)).double() / (case["h"] * case["w"])
    if kind == "crops":
        frames, boxes = _frames_and_boxes(case, seed)
        b = boxes.long()
        w, h = b[:, 3] - b[:, 1], b[:, 4] - b[:, 2]
        out = torch.empty(b.shape[0], 512, dtype=torch.float64, device="cuda")
        for lo in range(0, b.shape[0], 4000):
            q, ww, hh = b[lo:lo + 4000], w[lo:lo + 4000], h[lo:lo + 4000]
            area = ww * hh
            own = torch.repeat_interleave(torch.arange(q.shape[0], device="cuda"), area)
            at = torch.arange(own.numel(), device="cuda") - (area.cumsum(0) - area)[own]
            px = frames[q[own, 0], q[own, 2] + at // ww[own], q[own, 1] + at % ww[own]]
            c = torch.bincount(own * 512 + _bins(px), minlength=512 * q.shape[0]).reshape(-1, 512)
            out[lo:lo + 4000] = c.double() / area[:, None]
        return out
    if kind == "hist_eps":
        H = _histograms(case, seed)
        return _pairs64(H, H, _hist_radius(case), True)
    R, S = _relations(case, seed)
    if "k_eps" in case:
        return _pairs64(R, S, _radius(case), case.get("self", False))
    return _topk64(R, S, case["k"])
