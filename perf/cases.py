"""The work that a user of this library has it do, as timed cases.

Every case goes through the Python binding (paper_2106_07927_amd/sgm.py) with
the buffers, workspaces and plans a program keeps between frames.  Sizes are
those of the library's own workloads (datagen.CONFIGS, the batch and served
mixes) and ragged ones between them.

kinds:
  frame      StereoSGM.run, the streamlined form: census, cost, aggregation
             fused with the selection (a camera or dataset frame)
  four_call  StereoSGM.run with fused=False, which also keeps S_bar
  ncc        the NCC cost volume, then the streamlined aggregation with the
             wide penalties that go with it
  subpixel   streamlined aggregation with subpixel refinement, from a cost
             volume
  exact_lr   the whole path with the exact consistency check
  select     disparity selection alone, from an S_bar volume a program holds
  volume     census of both images and the matching-cost volume
  batch      a plan of pairs of mixed sizes, one graph launch
"""
import json
import random

import torch
import torch.nn.functional as F

from paper_2106_07927_amd import sgm

SIZES = ((320, 240), (640, 512), (1242, 375), (1920, 1080))     # datagen.BATCH_SIZES
NDISP = (64, 128, 256)                                          # datagen.BATCH_NDISP
MAX_ELEMS = 1920 * 1080 * 256                                   # the largest listed volume


def _case(name, kind, w, h, nd, win=9, npaths=8, p1=10, p2=120, lr=1, median=True, **more):
    c = {"kind": kind, "w": w, "h": h, "nd": nd, "win": win, "npaths": npaths, "p1": p1, "p2": p2,
         "lr": lr, "median": median, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest workload: quarter-VGA, 5x5 census, 4 paths, plain WTA;
        # one small frame at a time, where launches and latency count
        _case("frame_320x240_d64_r4", "frame", 320, 240, 64, win=5, npaths=4, p1=7, p2=86, lr=-1,
              median=False),
        # a served camera stream's frame
        _case("frame_640x512_d128", "frame", 640, 512, 128),
        # the headline workload: a KITTI-sized frame
        _case("frame_1242x375_d128", "frame", 1242, 375, 128),
        # the large frame
        _case("frame_1920x1080_d256", "frame", 1920, 1080, 256),
        # a cropped image and a disparity range that is no multiple of 16:
        # the streamlined call's general form
        _case("frame_803x397_d100", "frame", 803, 397, 100),
        # the four calls, by a program that reads S_bar itself
        _case("four_call_1242x375_d128", "four_call", 1242, 375, 128),
        # the NCC cost with its penalties (P2 = 880: 16-bit path values)
        _case("ncc5_1242x375_d128", "ncc", 1242, 375, 128, win=5, p1=90, p2=880),
        # subpixel disparities of a VGA frame, 4 paths
        _case("subpixel_640x480_d64_r4", "subpixel", 640, 480, 64, npaths=4),
        # exact consistency check of a VGA frame
        _case("exact_lr_640x480_d128", "exact_lr", 640, 480, 128),
        # selection from a held S_bar volume
        _case("select_1242x375_d128", "select", 1242, 375, 128),
        # census and cost volume of the large frame
        _case("volume_1920x1080_d128", "volume", 1920, 1080, 128),
        # many pairs of mixed sizes and ranges in one graph launch
        _case("batch_24_mixed", "batch", 0, 0, 0, pairs=24, mix=2109),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "four_call", "ncc", "subpixel", "exact_lr", "select",
                       "volume", "batch"])
    if kind == "batch":
        return _case(None, "batch", 0, 0, 0, npaths=rng.choice((4, 8)), pairs=rng.randint(2, 20),
                     mix=rng.randrange(1 << 20))
    while True:
        w, h = _log_int(rng, 160, 1920), _log_int(rng, 120, 1080)
        nd = rng.choice((16, 32, 48, 64, 80, 96, 128, 160, 192, 256, 256, rng.randint(8, 256),
                         rng.randint(8, 256)))
        if w > nd // 2 and w * h * nd <= MAX_ELEMS // (2 if kind in ("exact_lr", "ncc", "four_call") else 1):
            break
    npaths = rng.choice((4, 8, 8))
    win = rng.choice((5, 9))
    p1, p2 = rng.choice(((10, 120), (10, 120), (7, 86), (11, 110), (20, 160)))
    if kind == "ncc":
        p1, p2 = 90, 880
    lr = rng.choice((1, 1, 2, -1))
    return _case(None, kind, w, h, nd, win=win, npaths=npaths, p1=p1, p2=p2, lr=lr,
                 median=rng.choice((True, True, False)))


# ---------------------------------------------------------------------------
# inputs: a textured left image, a piecewise-planar disparity map, the right
# image warped from the left one, holes and noise (datagen's recipe, on the
# GPU so that they are quick to make)
# ---------------------------------------------------------------------------
def _texture(g, h, w, dev):
    n = torch.rand((1, 1, h + 6, w + 6), generator=g, device=dev) * 255.0
    t = torch.arange(-3, 4, device=dev, dtype=torch.float32)
    k = torch.exp(-0.5 * t * t)
    k = k / k.sum()
    s = F.conv2d(F.conv2d(n, k.view(1, 1, 1, 7)), k.view(1, 1, 7, 1))[0, 0]
    return (s - s.mean()) * (0.6 * 73.6 / s.std()) + 127.5


def _pair(w, h, nd, seed, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    r = random.Random(seed)
    xs = torch.arange(w, device=dev, dtype=torch.float32)[None, :]
    ys = torch.arange(h, device=dev, dtype=torch.float32)[:, None]
    left = _texture(g, h, w, dev) + r.uniform(-48, 48) * (xs / w - 0.5) + r.uniform(-48, 48) * (ys / h - 0.5)
    left = left.round().clamp(0, 255)
    best = torch.full((h, w), float("inf"), device=dev)
    disp = torch.zeros((h, w), device=dev)
    for _ in range(r.randint(8, 16)):
        cx, cy, a = r.uniform(0, w), r.uniform(0, h), r.uniform(0, nd - 1)
        b, c = r.uniform(-0.05, 0.05), r.uniform(-0.05, 0.05)
        dist = (xs - cx) ** 2 + (ys - cy) ** 2
        near = dist < best
        best = torch.where(near, dist, best)
        disp = torch.where(near, a + b * (xs - cx) + c * (ys - cy), disp)
    disp = disp.round().clamp(0, nd - 1).long()
    # forward warp, the larger disparity in front
    xr = xs.long() - disp
    flat = (ys.long() * w + xr.clamp(min=0)).reshape(-1)
    d = torch.where(xr >= 0, disp, torch.full_like(disp, -1)).reshape(-1)
    front = torch.full((h * w,), -1, device=dev, dtype=torch.long).scatter_reduce(0, flat, d, "amax")
    front = front.view(h, w)
    src = (xs.long() + front).clamp(0, w - 1)
    right = torch.where(front >= 0, left.gather(1, src), _texture(g, h, w, dev))
    for _ in range(10):                                          # occluding blobs, about 5 % of the frame
        rad = 0.04 * (w * h) ** 0.5 * r.uniform(0.6, 1.4) + 2
        blob = (xs - r.uniform(0, w)) ** 2 + (ys - r.uniform(0, h)) ** 2 <= rad * rad
        right = torch.where(blob, _texture(g, h, w, dev), right)
    right = right + 2.0 * torch.randn((h, w), generator=g, device=dev)
    return left.to(torch.uint8), right.round().clamp(0, 255).to(torch.uint8)


def _mix(case):
    r = random.Random(case["mix"])
    return [(*r.choice(SIZES), r.choice(NDISP)) for _ in range(case["pairs"])]


def _params(case, nd=None):
    win = (5, 5) if case["win"] == 5 else (9, 7)
    return sgm.Params(win_w=win[0], win_h=win[1], ndisp=case["nd"] if nd is None else nd,
                      npaths=case["npaths"], p1=case["p1"], p2=case["p2"], lr_tolerance=case["lr"],
                      median3x3=case["median"])


def _images(case, seed):
    return _pair(case["w"], case["h"], case["nd"], seed)


def prepare(case, seed):
    kind, w, h, nd = case["kind"], case["w"], case["h"], case["nd"]
    dev = "cuda"
    if kind == "batch":
        specs = _mix(case)
        pairs = [_pair(pw, ph, pd, seed * 1000 + i) for i, (pw, ph, pd) in enumerate(specs)]
        plan = sgm.BatchPlan([p[0] for p in pairs], [p[1] for p in pairs], [s[2] for s in specs],
                             _params(case), tune_table=json.dumps({}), want_right=True)
        torch.cuda.synchronize()
        return {"kind": kind, "plan": plan}
    p = _params(case)
    left, right = _images(case, seed)
    s = {"kind": kind, "p": p, "left": left, "right": right}
    out16 = lambda: torch.empty((h, w), dtype=torch.uint16, device=dev)  # noqa: E731
    if kind in ("frame", "four_call"):
        s["eng"] = sgm.StereoSGM(w, h, p, device=dev, fused=kind == "frame")
    elif kind == "ncc":
        s["cost"] = sgm._empty((h, w, nd), torch.uint8, torch.device(dev))
        s["work"] = sgm._aligned_bytes(sgm.aggregate_select_work_bytes(w, h, nd, p.npaths, p.p2), dev)
        s["disp"], s["disp_right"] = out16(), out16()
    elif kind == "subpixel":
        cl, cr = sgm.sgm_census_pair(left, right, p.win_w, p.win_h)
        s["cost"] = sgm.sgm_cost(cl, cr, nd)
        s["work"] = sgm._aligned_bytes(sgm.aggregate_select_subpixel_work_bytes(w, h, nd, p.npaths, p.p2), dev)
        s["disp"], s["disp_right"] = torch.empty((h, w), dtype=torch.float32, device=dev), out16()
    elif kind == "exact_lr":
        s["work"] = sgm._aligned_bytes(sgm.disparity_exact_lr_work_bytes(w, h, p), dev)
        s["disp"], s["disp_right"] = out16(), out16()
    elif kind == "select":
        cl, cr = sgm.sgm_census_pair(left, right, p.win_w, p.win_h)
        s["agg"] = sgm.sgm_aggregate(sgm.sgm_cost(cl, cr, nd), p.npaths, p.p1, p.p2)
        s["work"] = sgm._empty((sgm.wta_lrc_work_elems(w, h),), torch.uint16, torch.device(dev))
        s["disp"], s["disp_right"] = out16(), out16()
    elif kind == "volume":
        s["cl"] = torch.empty((h, w), dtype=torch.uint64, device=dev)
        s["cr"] = torch.empty((h, w), dtype=torch.uint64, device=dev)
        s["cost"] = sgm._empty((h, w, nd), torch.uint8, torch.device(dev))
    return s


def run(s):
    kind = s["kind"]
    if kind == "batch":
        s["plan"].run()
        return {"disp": s["plan"].disp, "disp_right": s["plan"].disp_right}
    p = s["p"]
    if kind in ("frame", "four_call"):
        e = s["eng"]
        e.run(s["left"], s["right"])
        out = {"disp": e.disp, "disp_right": e.disp_right}
        if kind == "four_call":
            out["agg"] = e.agg.view(torch.int16)                 # S_bar stays below 2^15 here
        return out
    if kind == "ncc":
        sgm.sgm_cost_ncc(s["left"], s["right"], p.win_w, p.ndisp, out=s["cost"])
        sgm.sgm_aggregate_select(s["cost"], p.npaths, p.p1, p.p2, p.lr_tolerance, p.median3x3, out=s["disp"],
                                 out_right=s["disp_right"], work=s["work"])
        return {"cost": s["cost"], "disp": s["disp"], "disp_right": s["disp_right"]}
    if kind == "subpixel":
        sgm.sgm_aggregate_select_subpixel(s["cost"], p.npaths, p.p1, p.p2, p.lr_tolerance, p.median3x3,
                                          out=s["disp"], out_right=s["disp_right"], work=s["work"])
    elif kind == "exact_lr":
        sgm.sgm_disparity_exact_lr(s["left"], s["right"], p, out=s["disp"], out_right=s["disp_right"],
                                   work=s["work"])
    elif kind == "select":
        sgm.sgm_wta_lrc(s["agg"], p.lr_tolerance, p.median3x3, out=s["disp"], out_right=s["disp_right"],
                        work=s["work"])
    else:
        sgm.sgm_census_pair(s["left"], s["right"], p.win_w, p.win_h, out_left=s["cl"], out_right=s["cr"])
        sgm.sgm_cost(s["cl"], s["cr"], p.ndisp, out=s["cost"])
        return {"census_left": s["cl"], "census_right": s["cr"], "cost": s["cost"]}
    return {"disp": s["disp"], "disp_right": s["disp_right"]}


def work(case):
    """Bytes: every input read once, every output written once; the volumes a
    case takes or returns are among them, those it makes on the way are not.
    Operations: two integer operations per window comparison; xor and count of
    a descriptor pair (2); a step of the path recursion (8: four minima, two
    sums, the difference, the path sum); selection (2 minima per element); an
    NCC cost (2 win + 10)."""
    def frame(w, h, nd):
        n, v = w * h, w * h * nd
        kind = case["kind"]
        maps = 4 * n                                             # D and D^R
        census = 2 * n * (24 if case["win"] == 5 else 62) * 2
        path = 8 * case["npaths"] * v
        if kind in ("frame", "batch"):
            return 2 * n + maps, census + 2 * v + path + 2 * v
        if kind == "four_call":
            return 2 * n + maps + 2 * v, census + 2 * v + path + 2 * v
        if kind == "ncc":
            return 2 * n + maps + v, (2 * case["win"] + 10) * v + path + 2 * v
        if kind == "subpixel":
            return v + 6 * n, path + 2 * v
        if kind == "exact_lr":
            return 2 * n + maps, 2 * (census + 2 * v + path + v)
        if kind == "select":
            return 2 * v + maps, 2 * v
        return 2 * n + 16 * n + v, census + 2 * v                # volume
    shapes = _mix(case) if case["kind"] == "batch" else [(case["w"], case["h"], case["nd"])]
    got = [frame(*s) for s in shapes]
    return {"bytes": sum(g[0] for g in got), "flops": sum(g[1] for g in got)}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64-bit throughout
# ---------------------------------------------------------------------------
def _x_census(img, ww, wh):
    h, w = img.shape
    rx, ry = ww // 2, wh // 2
    pad = F.pad(img.long(), (rx, rx, ry, ry))
    out = torch.zeros((h, w), dtype=torch.int64, device=img.device)
    for dy in range(wh):
        for dx in range(ww):
            if dy != ry or dx != rx:
                out = (out << 1) | (pad[dy:dy + h, dx:dx + w] < img.long()).long()
    return out


def _x_bits(v):
    n = torch.zeros_like(v)
    for k in range(62):
        n += (v >> k) & 1
    return n


def _x_cost(cl, cr, nd):
    h, w = cl.shape
    c = torch.full((h, w, nd), 255, dtype=torch.uint8, device=cl.device)
    for d in range(min(nd, w)):
        c[:, d:, d] = _x_bits(cl[:, d:] ^ cr[:, :w - d]).to(torch.uint8)
    return c


def _x_ncc(left, right, win, nd):
    h, w = left.shape
    n = win * win
    box = torch.ones((1, 1, win, win), dtype=torch.float64, device=left.device)

    def total(v):
        return F.conv2d(v[None, None], box, padding=win // 2)[0, 0]

    a, b = left.double(), right.double()
    sa, sb = total(a), total(b)
    va, vb = n * total(a * a) - sa * sa, n * total(b * b) - sb * sb
    c = torch.full((h, w, nd), 255, dtype=torch.uint8, device=left.device)
    ap, pad = F.pad(a, (win, win)), win
    for d in range(min(nd, w)):
        shifted = F.pad(b, (win, win)).roll(d, 1)
        shifted[:, :d] = 0
        slr = total(ap * shifted)[:, pad + d:pad + w]
        vl, vr = va[:, d:], vb[:, :w - d]
        num = n * slr - sa[:, d:] * sb[:, :w - d]
        ok = (vl > 0) & (vr > 0)
        phi = num / torch.where(ok, (vl * vr).sqrt(), torch.ones_like(vl))
        v = (255.0 * (1.0 - phi.clamp(min=0))).round().clamp(0, 255)
        c[:, d:, d] = torch.where(ok, v, torch.full_like(v, 255.0)).to(torch.uint8)
    return c


def _x_aggregate(cost, npaths, p1, p2):
    h, w, nd = cost.shape
    big = 1 << 40
    total = torch.zeros((h, w, nd), dtype=torch.int64, device=cost.device)

    def step(prev, c):
        m = prev.min(-1, keepdim=True).values
        p = F.pad(prev, (1, 1), value=big)
        best = torch.minimum(torch.minimum(prev, m + p2), torch.minimum(p[..., :-2], p[..., 2:]) + p1)
        return c + best - m

    dirs = [(1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, -1), (-1, 1), (1, -1)][:npaths]
    for dx, dy in dirs:
        if dy == 0:
            prev = None
            for x in (range(w) if dx > 0 else range(w - 1, -1, -1)):
                c = cost[:, x].long()
                prev = c if prev is None else step(prev, c)
                total[:, x] += prev
        else:
            prev = None
            for y in (range(h) if dy > 0 else range(h - 1, -1, -1)):
                c = cost[y].long()
                if prev is None:
                    cur = c
                else:
                    cur = c.clone()
                    lo, hi = max(0, dx), w + min(0, dx)
                    if hi > lo:
                        cur[lo:hi] = step(prev[lo - dx:hi - dx], c[lo:hi])
                prev = cur
                total[y] += prev
    return total


def _x_right(s):
    h, w, nd = s.shape
    best = torch.full((h, w), 1 << 40, dtype=torch.int64, device=s.device)
    arg = torch.zeros((h, w), dtype=torch.int64, device=s.device)
    for d in range(min(nd, w)):
        v = s[:, d:, d]
        less = v < best[:, :w - d]
        best[:, :w - d] = torch.where(less, v, best[:, :w - d])
        arg[:, :w - d] = torch.where(less, torch.full_like(v, d), arg[:, :w - d])
    return arg


def _x_wta(s):
    nd = s.shape[-1]
    return (s * 256 + torch.arange(nd, device=s.device)).min(-1).values & 255


def _x_finish(dl, dr, value, lr, median, bad):
    """LR check on the integer maps, then the median of `value` (float64)."""
    h, w = dl.shape
    xs = torch.arange(w, device=dl.device)[None, :]
    v = value.double()
    if lr >= 0:
        xr = xs - dl
        ok = (xr >= 0) & ((dl - dr.gather(1, xr.clamp(min=0))).abs() <= lr)
        v = torch.where(ok, v, torch.full_like(v, float("inf")))
    if median:
        p = F.pad(v[None, None], (1, 1, 1, 1), value=float("inf"))[0, 0]
        nine = torch.stack([p[dy:dy + h, dx:dx + w] for dy in range(3) for dx in range(3)])
        v = torch.where(torch.isinf(v), v, nine.median(0).values)
    return torch.where(torch.isinf(v), torch.full_like(v, bad), v)


def _x_maps(s, lr, median):
    dl, dr = _x_wta(s), _x_right(s)
    return {"disp": _x_finish(dl, dr, dl, lr, median, 65535.0).long(), "disp_right": dr}


def exact(case, seed):
    kind, nd = case["kind"], case["nd"]
    if kind == "batch":                                          # tens of frames: too long in plain torch
        return None
    p = _params(case)
    left, right = _images(case, seed)
    if kind == "ncc":
        c = _x_ncc(left, right, p.win_w, nd)
        return {"cost": c, **_x_maps(_x_aggregate(c, p.npaths, p.p1, p.p2), p.lr_tolerance, p.median3x3)}
    cl, cr = _x_census(left, p.win_w, p.win_h), _x_census(right, p.win_w, p.win_h)
    c = _x_cost(cl, cr, nd)
    if kind == "volume":
        return {"census_left": cl, "census_right": cr, "cost": c}
    s = _x_aggregate(c, p.npaths, p.p1, p.p2)
    if kind == "exact_lr":
        fl, fr = right.flip(1), left.flip(1)
        c = _x_cost(_x_census(fl, p.win_w, p.win_h), _x_census(fr, p.win_w, p.win_h), nd)
        dl, dr = _x_wta(s), _x_wta(_x_aggregate(c, p.npaths, p.p1, p.p2)).flip(1)
        return {"disp": _x_finish(dl, dr, dl, p.lr_tolerance, p.median3x3, 65535.0).long(), "disp_right": dr}
    if kind == "subpixel":
        dl, dr = _x_wta(s), _x_right(s)
        at = dl.clamp(1, max(1, nd - 2))[..., None]
        a, b, e = (s.gather(-1, (at + k).clamp(0, nd - 1))[..., 0].double() for k in (-1, 0, 1))
        den = a - 2 * b + e
        off = torch.where(den > 0, (a - e) / (2 * den.clamp(min=1)), torch.zeros_like(den))
        off = torch.where((dl > 0) & (dl < nd - 1), off, torch.zeros_like(off))
        return {"disp": _x_finish(dl, dr, dl.double() + off, p.lr_tolerance, p.median3x3, -1.0),
                "disp_right": dr}
    maps = _x_maps(s, p.lr_tolerance, p.median3x3)
    return {**maps, "agg": s.to(torch.int16)} if kind == "four_call" else maps
