"""Performance cases of the library: what its users have it do, at the sizes
they have it done.

Each case is one pass through a public entry point of the Python binding.
``listed()`` holds the fixed cases, ``draw()`` gives further ones of the same
kinds and ranges. Sizes are those of the benchmark (256x256, 4096x4096,
planar RGB at 1080p, the 512-image batch, the 2048x2048 quad mesh, 256 MiB
of bytes) and generic image sizes between 64 and 4096 a side, odd ones among
them. Pixels, weights and edge values are drawn as the benchmark draws them:
uniform pixels, normalised Gaussian taps, int8 weights in -8..8 with a shift
of 6, standard-normal edge values.

Every program that cares for speed loads the tuned table once at its start,
as the benchmark does; ``prepare`` does the same.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_1302_5586_amd as pf

TABLE = os.path.join(os.path.dirname(os.path.abspath(pf.__file__)), "tune_mi355x.json")
BORDERS = ("clamp", "zero", "reflect", "mirror")  # PF_BORDER_* in order
ALIGN = 64                                        # elements, as pack_batch
SERVER_BYTES = 2 << 30


def listed():
    return [
        # A thumbnail or one tile of a viewer, smoothed on its own: the
        # smallest call, whose time is the launch and the host's part of it.
        {"name": "filter2d 256 r1", "kind": "2d", "h": 256, "w": 256, "r": 1, "exact": False},
        # Smoothing a whole large image: streaming work, one read and one
        # write of every pixel.
        {"name": "filter2d 4096 r2", "kind": "2d", "h": 4096, "w": 4096, "r": 2, "exact": False},
        # A wide non-separable kernel (a matched or learnt filter) over a
        # photograph of odd size: arithmetic dominates.
        {"name": "filter2d 1533x2047 r7", "kind": "2d", "h": 1533, "w": 2047, "r": 7, "exact": False},
        # A wide Gaussian over a UHD frame in the bit-reproducible mode, as
        # pipelines that check themselves against the C program run it.
        {"name": "sep 2160x3840 r6 exact", "kind": "sep", "h": 2160, "w": 3840, "r": 6, "exact": True},
        # A video frame: planar RGB at 1080p through a 7x7 integer filter.
        {"name": "u8 rgb 1080p r3", "kind": "u8", "c": 3, "h": 1080, "w": 1920, "r": 3, "shift": 6},
        # A grey camera frame whose rows are not a multiple of four bytes.
        {"name": "u8 grey 719x1277 r2", "kind": "u8", "c": 1, "h": 719, "w": 1277, "r": 2, "shift": 6},
        # A data set in one launch: 512 images of uneven sizes, radii 1..4,
        # separable Gaussians, replayed from the plan's graph.
        {"name": "batch 512", "kind": "batch", "n": 512, "sizes": 3, "share_2d": 0.0, "exact": False},
        # Iterated smoothing (diffusion steps): four 3x3 passes, fused.
        {"name": "chain 4096 r1 x4", "kind": "chain", "h": 4096, "w": 4096, "r": 1, "passes": 4, "border": "clamp",
         "exact": False},
        # Mean and total of a large image, reproducible.
        {"name": "sum 16M", "kind": "sum", "n": 4096 * 4096},
        # Histogram of a large byte volume.
        {"name": "hist 256MiB", "kind": "hist", "n": 1 << 28},
        # One flux step of an unstructured mesh code: edges add into cells.
        {"name": "inc quads 2048", "kind": "inc", "nx": 2048, "ny": 2048},
        # A burst of requests to the server, images already on the device.
        {"name": "serve 48", "kind": "serve", "n": 48, "sizes": 40},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: a kind, then sizes spread over the logarithm of its range."""
    kind = rng.choice(("2d", "2d", "2d", "sep", "sep", "sep", "u8", "u8", "u8", "chain", "chain", "batch", "sum", "hist",
                       "inc", "serve"))
    if kind in ("2d", "sep"):
        return {"kind": kind, "h": _log_int(rng, 64, 4096), "w": _log_int(rng, 64, 4096), "r": rng.randint(0, pf.PF_R_MAX),
                "exact": rng.random() < 0.3}
    if kind == "u8":
        # Half of the widths are multiples of four, as camera and video rows are.
        w = _log_int(rng, 64, 3840)
        if rng.random() < 0.5:
            w = max(64, w // 4 * 4)
        return {"kind": kind, "c": rng.choice((1, 3)), "h": _log_int(rng, 64, 2160), "w": w,
                "r": rng.randint(0, pf.PF_R_MAX), "shift": rng.randint(4, 8)}
    if kind == "chain":
        r = rng.choice((1, 1, 1, 2, 2, 3, 4))
        return {"kind": kind, "h": _log_int(rng, 64, 4096), "w": _log_int(rng, 64, 4096), "r": r,
                "passes": rng.randint(1, min(8, pf.CHAIN_HALO_MAX // r)), "border": rng.choice(BORDERS),
                "exact": rng.random() < 0.3}
    if kind == "batch":
        return {"kind": kind, "n": _log_int(rng, 16, 384), "sizes": rng.randint(100, 999),
                "share_2d": rng.choice((0.0, 0.0, 0.25)), "exact": rng.random() < 0.3}
    if kind == "sum":
        return {"kind": kind, "n": _log_int(rng, 1 << 12, 1 << 27)}
    if kind == "hist":
        return {"kind": kind, "n": _log_int(rng, 1 << 14, 1 << 28)}
    if kind == "inc":
        return {"kind": kind, "nx": _log_int(rng, 64, 2048), "ny": _log_int(rng, 64, 2048)}
    return {"kind": kind, "n": _log_int(rng, 8, 96), "sizes": rng.randint(100, 999)}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gaussian(r, sigma):
    i = np.arange(-r, r + 1, dtype=np.float64)
    g = np.exp(-(i * i) / (2.0 * sigma * sigma))
    return (g / g.sum()).astype(np.float32)


def _gaussian_2d(r, sigma):
    g = _gaussian(r, sigma).astype(np.float64)
    return (g[:, None] * g[None, :]).astype(np.float32)


def _image_set(n, sizes):
    """Sizes (log-uniform in 64..2048), radii 1..4 and arena offsets of n
    images; the same for the same ``sizes``."""
    rng = np.random.default_rng(sizes)

    def side():
        v = np.rint(np.exp(rng.uniform(math.log(64), math.log(2048), n)))
        return np.clip(v, 64, 2048).astype(np.int64)

    w, h = side(), side()
    r = rng.integers(1, 5, n).astype(np.int64)
    room = (h * w + ALIGN - 1) // ALIGN * ALIGN
    off = np.concatenate([[0], np.cumsum(room)[:-1]]).astype(np.int64)
    return h, w, r, off, int(room.sum())


def _batch_kinds(case):
    """The first ``share_2d`` of the images carry full 2D filters."""
    n2 = int(round(case["share_2d"] * case["n"]))
    return [pf.KIND_2D] * n2 + [pf.KIND_SEP] * (case["n"] - n2)


def _batch_filters(r, kinds, seed):
    rng = np.random.default_rng(seed)
    sigma = rng.uniform(0.5, 2.0, len(r))
    out = []
    for rr, k, s in zip(r, kinds, sigma):
        g = _gaussian(int(rr), float(s))
        out.append(_gaussian_2d(int(rr), float(s)).ravel() if k == pf.KIND_2D else np.concatenate([g, g]))
    return out


def _mesh(nx, ny, seed):
    """Edge-to-cell map of an nx x ny quad mesh with cells and edges numbered
    at random, as an int32 tensor on the GPU."""
    g = _gen(seed)
    ids = torch.randperm(nx * ny, generator=g, device="cuda").reshape(ny, nx)
    horiz = torch.stack([ids[:, :-1].reshape(-1), ids[:, 1:].reshape(-1)], 1)
    vert = torch.stack([ids[:-1, :].reshape(-1), ids[1:, :].reshape(-1)], 1)
    e2c = torch.cat([horiz, vert])
    e2c = e2c[torch.randperm(len(e2c), generator=g, device="cuda")]
    flip = torch.rand(len(e2c), generator=g, device="cuda") < 0.5
    return torch.where(flip[:, None], e2c.flip(1), e2c).to(torch.int32).contiguous()


def _inputs(case, seed):
    """Everything ``prepare`` and ``exact`` draw from the seed."""
    g, k = _gen(seed), case["kind"]
    sigma = float(np.random.default_rng(seed).uniform(0.5, 2.0))
    if k in ("2d", "sep", "chain"):
        x = torch.rand((case["h"], case["w"]), generator=g, device="cuda")
        taps = _gaussian(case["r"], sigma) if k == "sep" else _gaussian_2d(case["r"], sigma)
        return {"x": x, "f": torch.from_numpy(taps).cuda()}
    if k == "u8":
        d = 2 * case["r"] + 1
        x = torch.randint(0, 256, (case["c"], case["h"], case["w"]), generator=g, device="cuda", dtype=torch.uint8)
        return {"x": x, "f": torch.randint(-8, 9, (d, d), generator=g, device="cuda", dtype=torch.int8)}
    if k == "sum":
        return {"x": torch.rand(case["n"], generator=g, device="cuda")}
    if k == "hist":
        return {"x": torch.randint(0, 256, (case["n"],), generator=g, device="cuda", dtype=torch.uint8)}
    if k == "inc":
        e2c = _mesh(case["nx"], case["ny"], seed)
        edge = torch.randn(len(e2c), generator=g, device="cuda", dtype=torch.float64)
        cell = torch.randn(case["nx"] * case["ny"], generator=g, device="cuda", dtype=torch.float64)
        return {"e2c": e2c, "edge": edge, "cell": cell}
    h, w, r, off, npix = _image_set(case["n"], case["sizes"])
    kinds = _batch_kinds(case) if k == "batch" else [pf.KIND_SEP] * case["n"]
    return {"h": h, "w": w, "r": r, "off": off, "npix": npix, "kinds": kinds, "filters": _batch_filters(r, kinds, seed),
            "x": torch.rand(npix, generator=g, device="cuda")}


def _views(arena, s):
    return [arena[o:o + h * w].view(int(h), int(w)) for o, h, w in zip(s["off"], s["h"], s["w"])]


def prepare(case, seed):
    pf.tune_load(TABLE)
    s = _inputs(case, seed)
    s["case"], k = case, case["kind"]
    if k == "batch":
        foff = np.concatenate([[0], np.cumsum([f.size for f in s["filters"]])[:-1]])
        fil = np.concatenate(s["filters"])
        s["f"] = torch.from_numpy(fil).cuda()
        s["out"] = torch.zeros_like(s["x"])
        s["plan"] = pf.BatchPlan(s["h"], s["w"], s["r"], s["kinds"], s["off"], foff, s["npix"], fil.size,
                                 exact=case["exact"])
    elif k == "serve":
        s["out"] = torch.zeros_like(s["x"])
        s["images"], s["outs"] = _views(s["x"], s), _views(s["out"], s)
        s["server"] = pf.Server(SERVER_BYTES, n_streams=3, max_batch=256)
    elif k == "inc":
        s["plan"] = pf.IncPlan(case["nx"] * case["ny"], s.pop("e2c").cpu().numpy())
    return s


def run(s):
    case, k = s["case"], s["case"]["kind"]
    if k == "2d":
        return pf.filter2d(s["x"], s["f"], exact=case["exact"])
    if k == "sep":
        return pf.filter_sep(s["x"], s["f"], s["f"], exact=case["exact"])
    if k == "u8":
        return pf.filter2d_u8(s["x"], s["f"], case["shift"])
    if k == "chain":
        return pf.filter_chain(s["x"], s["f"], case["passes"], BORDERS.index(case["border"]), exact=case["exact"])
    if k == "batch":
        return s["plan"].run(s["x"], s["f"], s["out"])
    if k == "sum":
        return pf.sum_f32(s["x"])
    if k == "hist":
        return pf.hist256_u8(s["x"])
    if k == "inc":
        return s["plan"].run(s["edge"], s["cell"])  # accumulates, as a time step does
    srv, tickets = s["server"], []
    for x, r, f in zip(s["images"], s["r"], s["filters"]):
        tickets.append(srv.submit(x, int(r), pf.KIND_SEP, f))
    for t, o in zip(tickets, s["outs"]):
        srv.wait(t)
        srv.result(t, o.shape[0], o.shape[1], out=o)
    return s["out"]


def work(case):
    k = case["kind"]
    if k in ("2d", "sep", "chain"):
        n, d = case["h"] * case["w"], 2 * case["r"] + 1
        taps = 2 * d if k == "sep" else d * d * case.get("passes", 1)
        return {"bytes": 8 * n, "flops": 2 * taps * n}
    if k == "u8":
        n = case["c"] * case["h"] * case["w"]
        return {"bytes": 2 * n, "flops": 2 * (2 * case["r"] + 1) ** 2 * n}
    if k == "sum":
        return {"bytes": 4 * case["n"], "flops": case["n"]}
    if k == "hist":
        return {"bytes": case["n"], "flops": case["n"]}
    if k == "inc":
        nc, ne = case["nx"] * case["ny"], 2 * case["nx"] * case["ny"] - case["nx"] - case["ny"]
        return {"bytes": 16 * ne + 16 * nc, "flops": 2 * ne}
    h, w, r, _, _ = _image_set(case["n"], case["sizes"])
    kinds = _batch_kinds(case) if k == "batch" else [pf.KIND_SEP] * case["n"]
    taps = [(2 * rr + 1) ** 2 if kk == pf.KIND_2D else 2 * (2 * rr + 1) for rr, kk in zip(r, kinds)]
    return {"bytes": int((8 * h * w).sum()), "flops": int((2 * h * w * np.array(taps)).sum())}


# ------------------------------------------- the same in 64 bits, plain torch

def _index(n, r, border):
    """Source index of positions -r .. n+r-1 of an axis of n elements; -1
    reads zero."""
    i = torch.arange(-r, n + r, device="cuda")
    if border == "clamp":
        return i.clamp(0, n - 1)
    if border == "zero":
        return torch.where((i >= 0) & (i < n), i, -1)
    if border == "reflect":
        m = i % (2 * n)
        return torch.where(m < n, m, 2 * n - 1 - m)
    p = max(2 * n - 2, 1)
    m = i % p
    return torch.where(m < n, m, p - m)


def _extend(x, r, border, axis):
    i = _index(x.shape[axis], r, border)
    y = x.index_select(axis, i.clamp(min=0))
    if border == "zero":
        shape = [1] * x.dim()
        shape[axis] = -1
        y = y * (i >= 0).to(y.dtype).view(shape)
    return y


def _correlate(x, taps, border="clamp"):
    """x [..., H, W] with the taps [a, b]: sums over the extended image."""
    a, b = len(taps), len(taps[0])
    y = _extend(_extend(x, a // 2, border, -2), b // 2, border, -1)
    h, w = x.shape[-2:]
    out = torch.zeros_like(x)
    for i in range(a):
        for j in range(b):
            out.add_(y[..., i:i + h, j:j + w], alpha=taps[i][j])
    return out


def _sep64(x, f):
    f = [float(v) for v in f]
    return _correlate(_correlate(x.double(), [f]), [[v] for v in f])


def exact(case, seed):
    s, k = _inputs(case, seed), case["kind"]
    if k == "2d":
        return _correlate(s["x"].double(), s["f"].double().tolist())
    if k == "sep":
        return _sep64(s["x"], s["f"].tolist())
    if k == "u8":
        y = _correlate(s["x"].long(), s["f"].long().tolist())
        return (y >> case["shift"]).clamp_(0, 255).to(torch.uint8)
    if k == "chain":
        y, f = s["x"].double(), s["f"].double().tolist()
        for _ in range(case["passes"]):
            y = _correlate(y, f, case["border"])
        return y
    if k == "sum":
        t = s["x"].double().sum()
        return torch.stack([t, t / case["n"]])
    if k == "hist":
        return torch.stack([(s["x"] == v).sum() for v in range(256)])
    if k == "inc":
        at = s["e2c"].long()
        return s["cell"].index_add(0, at[:, 1], s["edge"]).index_add(0, at[:, 0], s["edge"])
    out = torch.zeros(s["npix"], dtype=torch.float64, device="cuda")
    for x, o, r, kd, f in zip(_views(s["x"], s), _views(out, s), s["r"], s["kinds"], s["filters"]):
        d = 2 * int(r) + 1
        if kd == pf.KIND_2D:
            o.copy_(_correlate(x.double(), f.reshape(d, d).astype(np.float64).tolist()))
        else:
            o.copy_(_sep64(x, f[:d]))
    return out
