"""The workloads on which this framework's speed is watched.

Each case is one call that a program using the package makes, over inputs that
are made on the GPU from a seed:

  depth    lf_depth on one light field: the whole method, into a kept workspace
  plan     a captured batch plan over several light fields of mixed sizes
  initial  lf_initial_disparity: Census, initial SGM, fusion, borders
  cost     lf_cost_volume_bounded: the matching cost on given per-pixel ranges
  sgm      lf_sgm_aggregate on a bounded cost volume
  wta      lf_wta_subpixel on aggregated costs

The scenes are a slanted background with slanted elliptical planes before it,
under smooth noise with some pixel noise: the family of the `paper` workload of
lfsynth, rendered here with torch so that a light field takes milliseconds.
"""
import ctypes
import math
import random

import torch
import torch.nn.functional as F

from paper_1907_13449_amd import lf

# Method parameters of the two parameter sets in use: that of the small 8-bit
# light fields and that of the full-size ones (lfsynth.workload).
SMALL = dict(win_h=5, win_w=5, P1_init=10, P2_init=120, P1_final=10, P2_final=120, lam=2,
             edge_tau=math.inf)
FULL = dict(win_h=7, win_w=9, P1_init=21, P2_init=45, P1_final=17, P2_final=35, lam=3,
            edge_tau=128.0)


def _field(kind, S, T, H, W, N, span, dtype="f32", C=1, npaths=8, sum_bits=32, cost="l2",
           lam=3, window="7x9", raw=False):
    return dict(kind=kind, S=S, T=T, H=H, W=W, N=N, span=span, dtype=dtype, C=C, npaths=npaths,
                sum_bits=sum_bits, cost=cost, lam=lam, window=window, raw=raw)


def listed():
    named = {
        # the smallest whole call: a 5x5 patch of 8-bit views, bound by launches
        "depth_small_u8": _field("depth", 5, 5, 96, 96, 32, 4.0, dtype="u8", sum_bits=16, lam=2,
                                 window="5x5"),
        # the benchmark light field
        "depth_9x9_f32": _field("depth", 9, 9, 512, 512, 100, 8.0),
        # the same size without bounds (every pixel keeps the full range)
        "depth_boundless": _field("depth", 9, 9, 512, 512, 100, 8.0, lam=-1),
        # the paper's own setting: 8-bit colour views, 16 paths, a sparse 7x7 window
        "depth_rgb_u8_16paths": _field("depth", 9, 9, 512, 512, 100, 8.0, dtype="u8", C=3,
                                       npaths=16, window="sparse"),
        # a moving-stage light field, the largest image
        "depth_stage_u8": _field("depth", 11, 1, 1080, 1920, 96, 24.0, dtype="u8"),
        # many light fields of mixed sizes run as one captured batch
        "plan_mixed": dict(kind="plan", count=12, mix=0),
        # odd sizes through the initial stage alone
        "initial_ragged": _field("initial", 7, 7, 331, 449, 77, 6.0),
        # the bounded l2 cost: plenoptic views (with the raw sums), and 8-bit ones
        "cost_plenoptic_f32": _field("cost", 15, 15, 434, 625, 64, 3.0, raw=True),
        "cost_u8": _field("cost", 9, 9, 512, 512, 100, 8.0, dtype="u8"),
        # the Census final cost
        "cost_census": _field("cost", 7, 7, 384, 384, 64, 6.0, cost="census"),
        # aggregation over many hypotheses with 16-bit sums
        "sgm_wide": _field("sgm", 9, 9, 375, 450, 200, 8.0, sum_bits=16, npaths=16, lam=6),
        # winner, sub-pixel step and median of a large map
        "wta_large": _field("wta", 11, 1, 1080, 1920, 96, 24.0),
    }
    return [dict(c, name=n) for n, c in named.items()]


GRIDS = ((3, 3), (5, 5), (7, 7), (9, 9), (9, 9), (15, 15), (11, 1), (1, 9), (7, 3))


def draw(rng):
    top = max(_load(c) for c in listed())
    while True:
        kind = rng.choice(("depth", "depth", "depth", "depth", "initial", "cost", "cost", "sgm",
                           "wta", "plan"))
        if kind == "plan":
            c = dict(kind="plan", count=rng.randint(2, 12), mix=rng.randint(1, 1 << 20))
        else:
            S, T = rng.choice(GRIDS)
            small = rng.random() < 0.25
            c = _field(kind, S, T,
                       H=round(math.exp(rng.uniform(math.log(24), math.log(1080)))),
                       W=round(math.exp(rng.uniform(math.log(24), math.log(1920)))),
                       N=round(math.exp(rng.uniform(math.log(12), math.log(224)))),
                       span=round(rng.uniform(2.0, 24.0 if 1 in (S, T) else 8.0), 2),
                       dtype=rng.choice(("u8", "f32", "f32")), C=rng.choice((1, 1, 1, 3)),
                       npaths=rng.choice((8, 8, 8, 16)), sum_bits=16 if small else 32,
                       cost="census" if rng.random() < 0.15 else "l2",
                       lam=-1 if rng.random() < 0.1 else rng.randint(1, 6),
                       window="5x5" if small else rng.choice(("7x9", "7x9", "sparse", "5x7")),
                       raw=kind == "cost" and rng.random() < 0.5)
        if _load(c) <= top and _elements(c) <= 100_000_000:
            return c


# ------------------------------------------------------------------- sizes
def _members(case):
    """The light fields of a batch: square ones of three shapes in turn (mix 0, the
    batched workload's), or of drawn shapes."""
    rng = random.Random(case["mix"])
    shapes = ((5, 256, 256), (7, 384, 384), (9, 512, 512))
    out = []
    for i in range(case["count"]):
        S, H, W = shapes[i % 3]
        if case["mix"]:
            S = rng.choice((3, 5, 7, 9))
            H, W = rng.randint(64, 512), rng.randint(64, 512)
        out.append(_field("depth", S, S, H, W, rng.randint(32, 128), 8.0))
    return out


def _elements(c):
    return max(_elements(m) for m in _members(c)) if c["kind"] == "plan" else \
        c["S"] * c["T"] * c["C"] * c["H"] * c["W"]


def _cross(c):
    return (2 if c["S"] > 1 else 0) + (2 if c["T"] > 1 else 0)


def _bits(c):
    return {"5x5": 24, "5x7": 34, "7x9": 62, "sparse": 24}[c["window"]]


def _cells(c):
    """Cells of the bounded volume: about an eighth of the pixels keep every hypothesis."""
    HW, w = c["H"] * c["W"], min(2 * c["lam"] + 1, c["N"])
    full = HW if c["lam"] < 0 else _full_pixels(c)
    return full * c["N"] + (HW - full) * w


def work(case):
    """Inputs read once, outputs written once.  Operations: one compare per Census
    bit; per cell and path direction of Eq. (8)-(9) two additions of P1, four minima,
    the cost, the minimum and the sum (9); a Hamming distance per cell (2); the l2
    cost 9 per channel, view and cell and 2 for the sum; 3 per cell for the WTA."""
    if case["kind"] == "plan":
        parts = [work(m) for m in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    c, kind = case, case["kind"]
    HW, cells, N = c["H"] * c["W"], _cells(c), c["N"]
    views = c["S"] * c["T"]
    image = HW * c["C"] * (1 if c["dtype"] == "u8" else 4)
    sums = c["sum_bits"] // 8
    initial = (1 + _cross(c)) * HW * c["C"] * _bits(c) + \
        _cross(c) * HW * N * (2 * c["C"] + 9 * c["npaths"])
    if c["cost"] == "l2":
        cost = cells * (views - 1) * (9 * c["C"] + 2)
    else:
        cost = views * c["C"] * (HW * _bits(c) + 2 * cells)
    sgm, wta = 9 * c["npaths"] * cells, 3 * cells
    if kind == "initial":
        return dict(bytes=(1 + _cross(c)) * image + HW * 2 * (_cross(c) + 3), flops=initial)
    if kind == "cost":
        return dict(bytes=views * image + 12 * HW + cells * (6 if c["raw"] else 2), flops=cost)
    if kind == "sgm":
        return dict(bytes=12 * HW + cells * (2 + sums), flops=sgm)
    if kind == "wta":
        return dict(bytes=18 * HW + cells * sums, flops=wta)
    return dict(bytes=views * image + 6 * HW,
                flops=(initial if c["lam"] >= 0 else 0) + cost + sgm + wta)


def _load(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def _params(c):
    small = c["window"] == "5x5"
    p = dict(SMALL if small else FULL, npaths=c["npaths"], lam=c["lam"], phi=3, fill_passes=2,
             alpha=1.0 if c["dtype"] == "u8" else 255.0, sum_bits=c["sum_bits"],
             cost_kind=lf.LF_COST_L2 if c["cost"] == "l2" else lf.LF_COST_CENSUS, median=3)
    if c["window"] == "5x7":
        p.update(win_h=5, win_w=7)
    if c["window"] == "sparse":          # the even-sum pixels of a 7x7 window
        p.update(win_h=7, win_w=7, census_offsets=[
            (i, j) for i in range(-3, 4) for j in range(-3, 4)
            if (i + j) % 2 == 0 and (i, j) != (0, 0)])
    return p


# ------------------------------------------------------------------ scenes
def _range(c):
    """Smallest disparity: 3-D light fields of a moving stage start at zero."""
    return (0.0, c["span"]) if 1 in (c["S"], c["T"]) else (-c["span"] / 2, c["span"] / 2)


def _planes(c, rng):
    """(a, b, cc, uc, vc, ax, ay): d = a + b (u - uc) + cc (v - vc) inside an ellipse."""
    H, W = c["H"], c["W"]
    lo, hi = _range(c)
    span, scale = hi - lo, max(min(H, W) / 512.0, 0.05)
    a = lo + span * rng.uniform(0.1, 0.25)
    slope = min(a - lo, hi - a) / (W + H)
    out = [(a, slope * rng.uniform(-1, 1), slope * rng.uniform(-1, 1), W / 2, H / 2, 1e9, 1e9)]
    for _ in range(11):
        ax, ay = (scale * rng.uniform(20, 100) for _ in range(2))
        a = rng.uniform(lo, hi)
        b, cc = (0.0025 * span * rng.uniform(-1, 1) for _ in range(2))
        reach, room = abs(b) * ax + abs(cc) * ay, min(a - lo, hi - a)
        f = min(1.0, room / reach) if reach > 0 else 1.0
        out.append((a, b * f, cc * f, rng.uniform(0, W), rng.uniform(0, H), ax, ay))
    return out


def _texture(C, h, w, rng, gen, dev):
    """Four octaves of smooth noise and a little pixel noise, in [0, 1]."""
    sigma = rng.uniform(16, 64)
    tex = torch.zeros(1, C, h, w, device=dev)
    for o in range(4):
        n = [max(4, round(x * 2 ** o / sigma) + 3) for x in (h, w)]
        grid = torch.rand(1, C, *n, device=dev, generator=gen) * 2 - 1
        tex += F.interpolate(grid, size=(h, w), mode="bicubic", align_corners=True) * 0.5 ** o
    tex = 0.5 + 0.3 * tex / 1.875 + 0.15 * (torch.rand(1, C, h, w, device=dev, generator=gen) - 0.5)
    return tex.clamp_(0, 1)


def _scene(c, seed, textured=True):
    """Views [T][S]([C])[H][W] (None without textures) and the disparity of the middle one."""
    dev = torch.device("cuda")
    rng = random.Random(seed)
    gen = torch.Generator(dev).manual_seed(seed)
    S, T, H, W, C = c["S"], c["T"], c["H"], c["W"], c["C"]
    planes = _planes(c, rng)
    m = math.ceil(max(S, T) / 2 * max(abs(x) for x in _range(c))) + 2
    h, w = H + 2 * m, W + 2 * m
    s, t = (torch.arange(S, device=dev), torch.arange(T, device=dev)) if textured else \
        (torch.full((1,), (S - 1) // 2, device=dev), torch.full((1,), (T - 1) // 2, device=dev))
    cs = ((S - 1) // 2 - s).float().repeat(len(t)).view(-1, 1, 1)
    ct = ((T - 1) // 2 - t).float().repeat_interleave(len(s)).view(-1, 1, 1)
    V = cs.shape[0]
    y = torch.arange(H, device=dev, dtype=torch.float32).view(1, H, 1)
    x = torch.arange(W, device=dev, dtype=torch.float32).view(1, 1, W)
    best = torch.full((V, H, W), -1e9, device=dev)
    img = torch.zeros((C, V * H, W), device=dev) if textured else None
    for a, b, cc, uc, vc, ax, ay in planes:
        k0 = a - b * uc - cc * vc
        m00, m01, m10, m11 = 1 + cs * b, cs * cc, ct * b, 1 + ct * cc
        det = m00 * m11 - m01 * m10
        rx, ry = x - cs * k0, y - ct * k0
        u, v = (m11 * rx - m01 * ry) / det, (m00 * ry - m10 * rx) / det
        d = k0 + b * u + cc * v
        take = ((u - uc) / ax) ** 2 + ((v - vc) / ay) ** 2 <= 1
        take &= d > best
        best = torch.where(take, d, best)
        if textured:
            grid = torch.stack(((u + m) * (2 / (w - 1)) - 1, (v + m) * (2 / (h - 1)) - 1), -1)
            tex = F.grid_sample(_texture(C, h, w, rng, gen, dev), grid.view(1, V * H, W, 2),
                                mode="bilinear", padding_mode="border", align_corners=True)
            img = torch.where(take.view(1, V * H, W), tex[0], img)
    mid = ((T - 1) // 2) * S + (S - 1) // 2 if textured else 0
    if not textured:
        return None, best[0]
    img = img.view(C, T, S, H, W).permute(1, 2, 0, 3, 4)
    img = (img * 255).round_().to(torch.uint8) if c["dtype"] == "u8" else img
    return (img[:, :, 0] if C == 1 else img).contiguous(), best[mid]


def _hypotheses(c):
    lo, hi = _range(c)
    k = torch.arange(c["N"], dtype=torch.float64)
    return (lo + k * (hi - lo) / (c["N"] - 1)).float().cuda()


def _full_pixels(c):
    return round(0.12 * c["H"] * c["W"])


def _bounds(c, disparity, seed):
    """Per-pixel ranges as the borders step leaves them: a window of 2 lam + 1 around
    the true index (moved inside at the ends of the range), all hypotheses for an
    eighth of the pixels, beside occlusions first and then in patches.  The number of
    cells depends on the sizes alone."""
    lo, hi = _range(c)
    N, H, W = c["N"], c["H"], c["W"]
    k = ((disparity - lo) * ((N - 1) / (hi - lo))).round().clamp(0, N - 1)
    if c["lam"] < 0 or 2 * c["lam"] + 1 >= N:
        return torch.zeros_like(k, dtype=torch.int16), torch.full_like(k, N - 1, dtype=torch.int16)
    k4 = k.view(1, 1, H, W)
    jump = F.max_pool2d(k4, 3, 1, 1) + F.max_pool2d(-k4, 3, 1, 1) > 4
    gen = torch.Generator("cuda").manual_seed(seed + 1)
    rough = torch.rand(1, 1, H // 4 + 2, W // 4 + 2, device="cuda", generator=gen)
    rough = F.interpolate(rough, size=(H, W), mode="bicubic", align_corners=True)
    order = torch.sort((rough + 10.0 * jump).flatten(), descending=True, stable=True).indices
    full = torch.zeros(H * W, dtype=torch.bool, device="cuda")
    full[order[:_full_pixels(c)]] = True
    full = full.view(H, W)
    mid = k.clamp(c["lam"], N - 1 - c["lam"])
    d_lo = torch.where(full, torch.zeros_like(k), mid - c["lam"])
    d_hi = torch.where(full, torch.full_like(k, N - 1), mid + c["lam"])
    return d_lo.to(torch.int16), d_hi.to(torch.int16)


def _cell_grid(d_lo, d_hi):
    """CSR offsets [H*W + 1] and each cell's pixel and hypothesis."""
    widths = (d_hi.long() - d_lo.long() + 1).flatten()
    off = torch.zeros(widths.numel() + 1, dtype=torch.int64, device=widths.device)
    torch.cumsum(widths, 0, out=off[1:])
    pix = torch.repeat_interleave(torch.arange(widths.numel(), device=widths.device), widths)
    k = torch.arange(pix.numel(), device=widths.device) - off[pix] + d_lo.long().flatten()[pix]
    return off, pix, k


# ------------------------------------------------------------ prepare, run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "plan":
        items = []
        for i, m in enumerate(_members(case)):
            st = prepare(m, seed * 64 + i)
            items.append((st["views"], st["hyp"], st["params"], st["out"], st["d_index"]))
        plan = lf.Plan(items)
        plan.capture()
        return dict(kind=kind, plan=plan, out=[(it[3], it[4]) for it in items])
    c, params, hyp = case, _params(case), _hypotheses(case)
    S, T, H, W, N, C = (c[k] for k in ("S", "T", "H", "W", "N", "C"))
    st = dict(kind=kind, params=params, hyp=hyp)
    views, disparity = _scene(c, seed, textured=kind in ("depth", "initial", "cost"))
    st["views"] = views
    if kind == "depth":
        st["ws"] = lf.workspace(lf.depth_workspace_bytes(S, T, H, W, N, params, C), "cuda")
        st["out"] = torch.empty((H, W), dtype=torch.float32, device="cuda")
        st["d_index"] = torch.empty((H, W), dtype=torch.int16, device="cuda")
        return st
    prm = lf.make_params(params)
    if kind == "initial":
        st["ws"] = lf.workspace(lf.lib.lf_initial_workspace_size(S, T, C, H, W, N, ctypes.byref(prm)),
                                "cuda")
        return st
    d_lo, d_hi = _bounds(c, disparity, seed)
    off, pix, k = _cell_grid(d_lo, d_hi)
    st.update(d_lo=d_lo, d_hi=d_hi, off=off, cells=pix.numel(), raw=c["raw"])
    if kind == "cost":
        st["ws"] = lf.workspace(lf.lib.lf_cost_workspace_size(S, T, C, H, W, N, ctypes.byref(prm)),
                                "cuda")
        return st
    # costs that grow away from the true index, at a pixel's own contrast
    lo, hi = _range(c)
    gen = torch.Generator("cuda").manual_seed(seed + 2)
    true = ((disparity - lo) * ((N - 1) / (hi - lo))).flatten()
    contrast = torch.rand(H * W, device="cuda", generator=gen) * 1200 + 60
    away = (k - true[pix]).abs()
    cost = contrast[pix] * (away / (away + 0.15 * N)) * \
        (0.6 + 0.8 * torch.rand(k.numel(), device="cuda", generator=gen))
    cap = lf.cost_cap(params["P2_final"], c["npaths"], c["sum_bits"])
    per_path = cost.round().clamp(max=cap).to(torch.int32)
    if kind == "sgm":
        # the volume has its worst-case capacity, as lf_cost_volume_bounded returns it
        st["cost"] = torch.zeros(H * W * N, dtype=torch.int16, device="cuda")
        st["cost"][:k.numel()] = per_path.to(torch.int16)
        st["ws"] = lf.workspace(lf.lib.lf_sgm_workspace_size(H, W, N, c["npaths"]), "cuda")
        st["csum"] = torch.empty(H * W * N, dtype=torch.int16 if c["sum_bits"] == 16
                                 else torch.int32, device="cuda")
    else:
        sums = torch.zeros(H * W * N, dtype=torch.int32, device="cuda")
        sums[:k.numel()] = per_path * c["npaths"] + \
            torch.randint(0, 64, (k.numel(),), device="cuda", generator=gen)
        if c["sum_bits"] == 16:          # 16-bit sums, kept as the bits of int16
            sums = sums.clamp_(max=65535).to(torch.int16)
        st["csum"] = sums
        st["ws"] = lf.workspace(lf.lib.lf_wta_workspace_size(H, W), "cuda")
    return st


def run(state):
    st, kind = state, state["kind"]
    if kind == "depth":
        lf.lf_depth(st["views"], st["hyp"], st["params"], ws=st["ws"], out=st["out"],
                    d_index=st["d_index"])
        return dict(disparity=st["out"], d_index=st["d_index"])
    if kind == "plan":
        st["plan"].run()
        return st["out"]
    if kind == "initial":
        r = lf.lf_initial_disparity(st["views"], st["hyp"], st["params"], ws=st["ws"])
        return {k: r[k] for k in ("maps", "d_init", "d_lo", "d_hi")}
    if kind == "cost":
        r = lf.lf_cost_volume_bounded(st["views"], st["hyp"], st["params"], st["d_lo"], st["d_hi"],
                                      want_f32=st["raw"], ws=st["ws"])
        out = dict(offsets=r["offsets"], cost=r["cost"][:st["cells"]])
        if st["raw"]:
            out["cost_f32"] = r["cost_f32"][:st["cells"]]
        return out
    p = st["params"]
    if kind == "sgm":
        csum = lf.lf_sgm_aggregate(st["cost"], st["off"], st["d_lo"], st["d_hi"],
                                   st["hyp"].shape[0], p["P1_final"], p["P2_final"], p["npaths"],
                                   p["sum_bits"], csum=st["csum"], ws=st["ws"])
        return dict(csum=csum[:st["cells"]])
    return lf.lf_wta_subpixel(st["csum"], p["sum_bits"], st["off"], st["d_lo"], st["d_hi"],
                              st["hyp"], ws=st["ws"])


# ------------------------------------------------------------------- exact
def exact(case, seed):
    """The computed numbers in float64: the raw l2 sums, and the refined disparities
    of given sums.  The other outputs are integers, or follow from the whole
    method's integer decisions."""
    if case["kind"] == "cost" and case["raw"] and case["cost"] == "l2":
        return _exact_cost(case, prepare(case, seed))
    if case["kind"] == "wta":
        return _exact_wta(case, prepare(case, seed))
    return None


def _exact_cost(c, st):
    S, T, H, W, C = (c[k] for k in ("S", "T", "H", "W", "C"))
    views = st["views"].view(T, S, C, H * W).double()
    _, pix, k = _cell_grid(st["d_lo"], st["d_hi"])
    u, v, d = pix % W, pix // W, st["hyp"].double()[k]
    ref = views[(T - 1) // 2, (S - 1) // 2][:, pix]
    acc = torch.zeros_like(d)
    for t in range(T):
        for s in range(S):
            x, y = u + ((S - 1) // 2 - s) * d, v + ((T - 1) // 2 - t) * d
            x0, y0 = x.floor(), y.floor()
            fx, fy = x - x0, y - y0
            x0, y0 = x0.long(), y0.long()
            xa, xb = x0.clamp(0, W - 1), (x0 + 1).clamp(0, W - 1)
            ya, yb = y0.clamp(0, H - 1) * W, (y0 + 1).clamp(0, H - 1) * W
            img = views[t, s]
            val = (1 - fy) * ((1 - fx) * img[:, ya + xa] + fx * img[:, ya + xb]) + \
                fy * ((1 - fx) * img[:, yb + xa] + fx * img[:, yb + xb])
            acc += (ref - val).square().sum(0).sqrt()
    return dict(offsets=None, cost=None, cost_f32=acc)


def _exact_wta(c, st):
    N, H, W = c["N"], c["H"], c["W"]
    off, pix, k = _cell_grid(st["d_lo"], st["d_hi"])
    sums = st["csum"][:k.numel()].long()
    if c["sum_bits"] == 16:
        sums = sums & 0xFFFF
    key = torch.full((H * W,), 1 << 62, dtype=torch.int64, device=sums.device)
    key.scatter_reduce_(0, pix, sums * 256 + k, "amin")
    best = key % 256
    lo, hi = st["d_lo"].long().flatten(), st["d_hi"].long().flatten()
    fine = (best > lo) & (best < hi) & (hi - lo >= 4)
    at = off[:-1] + best - lo
    cm, c0, cp = (sums[(at + o).clamp(0, k.numel() - 1)].double() for o in (-1, 0, 1))
    hyp = st["hyp"].double()
    den = 2 * (cm + cp - 2 * c0)
    o = torch.where(fine & (den > 0), (cm - cp) / den.clamp(min=1), torch.zeros_like(cm))
    up = hyp[(best + 1).clamp(max=N - 1)] - hyp[best]
    down = hyp[best] - hyp[(best - 1).clamp(min=0)]
    disp = (hyp[best] + o * torch.where(o >= 0, up, down)).view(1, 1, H, W)
    win = F.unfold(F.pad(disp, (1, 1, 1, 1), mode="replicate"), 3)
    return dict(d_index=best.view(H, W), disparity=win.median(1).values.view(H, W))
