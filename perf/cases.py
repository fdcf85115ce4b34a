"""What the library is timed on: the calls a two-stage detector makes of it.

A case is a dict of plain values.  `prepare` makes its inputs on the GPU from a seed and
the buffers a training or serving loop keeps (outputs, gradient pyramid, plan workspace);
`run` is one pass through the public entry points; `exact` is the same result in 64 bits
by plain torch (dense interpolation matrices or per-sample gathers, the sample positions
in the binary32 steps of the operator's definition).

Kinds of case:
  align    plan, RoIAlign forward and, in training, backward on one FPN pyramid
  extract  the same through `roi_extract` and torch.autograd
  heads    box and mask head of one batch: both forwards in one call, both backwards in one
  pool     RoI max pooling forward and backward
  deform   modulated deformable RoI pooling forward and backward
  nms      greedy NMS of a batch's proposals (`box_nms`, the image as category)
  select   per-category selection (`box_nms_batched`), greedy or Soft-NMS
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1906_07155_amd as rex
from paper_1906_07155_amd import workloads as W

STRIDES = (4, 8, 16, 32)
GAMMA = 0.1                     # scale of the deformable offsets
FINEST = 56.0


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _roi_case(kind, images, per_image, **kw):
    case = {"kind": kind, "images": images, "per_image": per_image, "channels": 256,
            "height": 800, "width": 1344, "levels": 4, "out": 7, "sampling": 2,
            "dtype": "f32", "layout": "cl", "backward": True, "lo": 8.0, "hi": 800.0}
    case.update(kw)
    return case


def listed():
    return [
        # A detector without FPN (one stride-16 map), 128 sampled RoIs: the smallest call.
        dict(_roi_case("align", 1, 128, levels=1, height=800, width=1088, lo=16.0, hi=512.0,
                       backward=False), name="single_level_infer_f32"),
        # Serving an FPN detector in bf16: 1000 proposals of one image.
        dict(_roi_case("extract", 1, 1000, dtype="bf16", backward=False),
             name="fpn_infer_bf16"),
        # The box head of a training step, 512 sampled RoIs on each of two images.
        dict(_roi_case("align", 2, 512), name="box_train_f32"),
        # The mask head of the same step: the positive RoIs, 14x14.
        dict(_roi_case("align", 2, 128, out=14, lo=32.0, hi=512.0), name="mask_train_f32"),
        # A whole Mask R-CNN step at batch 16 in bf16, both heads on one pyramid: the largest.
        dict(_roi_case("heads", 16, 512, mask_per_image=128, dtype="bf16"),
             name="heads_train_b16_bf16"),
        # The box head on the neck's default layout (contiguous NCHW), both directions.
        dict(_roi_case("align", 2, 512, layout="nchw"), name="box_train_nchw_f32"),
        # Adaptive sampling (as many samples as a bin has pixels) through autograd, on
        # images whose maps end in partial tiles and an odd number of RoIs.
        dict(_roi_case("extract", 3, 171, height=608, width=1056, sampling=0),
             name="box_train_adaptive_f32"),
        # Fast R-CNN's RoI max pooling in training.
        dict(_roi_case("pool", 2, 512), name="pool_train_f32"),
        # A deformable (modulated) box head in training.
        dict(_roi_case("deform", 2, 512), name="deform_train_f32"),
        # Proposal NMS over the best boxes of two images.
        {"kind": "nms", "images": 2, "per_image": 4096, "iou": 0.7, "max_keep": 8192,
         "name": "nms_8192"},
        # The proposal step of a batch of 16 images: 2000 scored boxes each, 1000 kept.
        {"kind": "select", "categories": 16, "per_category": 2000, "method": "hard", "iou": 0.7,
         "score_threshold": -1.0, "score_power": 1.0, "max_keep": 1000, "name": "select_16x2000"},
        # Test-time selection of 80 classes by Soft-NMS: 1000 boxes scored for every class,
        # most of them under the score threshold.
        {"kind": "select", "categories": 80, "per_category": 1000, "method": "linear",
         "iou": 0.3, "score_threshold": 0.05, "score_power": 8.0, "max_keep": 100,
         "name": "soft_80x1000"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["align", "align", "align", "extract", "extract", "heads", "pool", "deform",
                       "nms", "select", "select"])
    if kind == "nms":
        images = rng.randint(1, 4)
        n = max(1, _log_int(rng, 500, 8192) // images)
        return {"kind": kind, "images": images, "per_image": n,
                "iou": rng.choice([0.5, 0.6, 0.7, 0.8]),
                "max_keep": rng.choice([n * images, 1000, 2000])}
    if kind == "select":
        method = rng.choice(["hard", "hard", "linear", "gaussian"])
        if rng.random() < 0.5:      # proposals of a batch: the image is the category
            cats, per, power, thr = rng.randint(1, 16), _log_int(rng, 200, 2000), 1.0, -1.0
        else:                       # classes of a few images
            cats, per, power, thr = rng.randint(20, 160), _log_int(rng, 100, 1000), 8.0, 0.05
        keep = 100 if method != "hard" else rng.choice([100, 300, 1000])
        if method != "hard":
            thr = max(thr, 0.001)
        return {"kind": kind, "categories": cats, "per_category": per, "method": method,
                "iou": rng.choice([0.3, 0.5, 0.7]), "score_threshold": thr,
                "score_power": power, "max_keep": keep}
    height, width = 32 * rng.randint(15, 25), 32 * rng.randint(20, 42)
    channels = rng.choice([256, 256, 256, 128, 192, 96])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "heads":
        images = _log_int(rng, 2, 16)
        return _roi_case(kind, images, _log_int(rng, 64, 512),
                         mask_per_image=_log_int(rng, 16, 128), height=height, width=width,
                         channels=channels, dtype=dtype if images <= 4 else "bf16")
    images = _log_int(rng, 1, 4)
    per = _log_int(rng, 32, 1024 // images)
    kw = dict(height=height, width=width, channels=channels, dtype=dtype)
    if kind in ("align", "extract"):
        kw["backward"] = rng.random() < 0.6
        if rng.random() < 0.3:
            kw["out"] = 14
            per = max(1, per // 4)
        if kind == "align" and rng.random() < 0.35:
            kw["layout"] = "nchw"
        if kind == "extract" and rng.random() < 0.6:
            # the adaptive grid multiplies the samples of a bin: a small batch
            kw["sampling"] = 0
            images = min(images, 3)
            per = min(per, 513 // images)
    return _roi_case(kind, images, per, **kw)


# ---------------------------------------------------------------------------
# Inputs and buffers
# ---------------------------------------------------------------------------

def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _shapes(case):
    """(level sizes, scales) of the case's maps."""
    strides = STRIDES if case["levels"] == 4 else (16,)
    return ([(case["height"] // s, case["width"] // s) for s in strides],
            [1.0 / s for s in strides])


def _pyramid(case, make):
    n, c = case["images"], case["channels"]
    maps = []
    for h, w in _shapes(case)[0]:
        if case["layout"] == "cl":      # [N, H, W, C] in memory
            maps.append(make((n, h, w, c)).permute(0, 3, 1, 2))
        else:
            maps.append(make((n, c, h, w)))
    return maps


def _rois(case, seed, stream, per_image):
    rng = np.random.default_rng([int(seed), stream])
    r = W.draw_rois(rng, case["images"], per_image, (case["height"], case["width"]),
                    (case["lo"], case["hi"]))
    if case["kind"] == "heads":         # sampled training RoIs crowd around the objects
        r = W.add_duplicates(rng, r, 0.2, 2.0, (case["height"], case["width"]))
    return torch.from_numpy(r).cuda()


def prepare(case, seed):
    st = {"case": dict(case)}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = _dtype(case) if "dtype" in case else torch.float32

    def randn(shape, dtype=dt):
        return torch.randn(shape, generator=gen, dtype=dtype, device="cuda")

    kind = case["kind"]
    if kind in ("nms", "select"):
        rng = np.random.default_rng([int(seed), 7])
        groups = case["images"] if kind == "nms" else case["categories"]
        per = case["per_image"] if kind == "nms" else case["per_category"]
        boxes, scores, cats = W.draw_proposals(rng, groups, per)
        scores = (scores.astype(np.float64) ** case.get("score_power", 1.0)).astype(np.float32)
        st["boxes"], st["scores"], st["cats"] = (torch.from_numpy(np.ascontiguousarray(x)).cuda()
                                                 for x in (boxes, scores, cats))
        n, dev = boxes.shape[0], st["boxes"].device
        if kind == "nms":
            st["keep"] = torch.empty(max(1, min(n, case["max_keep"])), dtype=torch.int32,
                                     device=dev)
            st["num"] = torch.empty(1, dtype=torch.int32, device=dev)
        else:
            shape = (groups, case["max_keep"])
            st["keep"] = torch.empty(shape, dtype=torch.int32, device=dev)
            st["kept_scores"] = torch.empty(shape, dtype=torch.float32, device=dev)
            st["num"] = torch.empty(groups, dtype=torch.int32, device=dev)
        return st

    c, p = case["channels"], case["out"]
    st["scales"] = _shapes(case)[1]
    st["feats"] = _pyramid(case, randn)
    heads = [(case["per_image"], p)]
    if kind == "heads":
        heads.append((case["mask_per_image"], 14))
    st["heads"] = []
    for i, (per, grid) in enumerate(heads):
        rois = _rois(case, seed, 1 + i, per)
        k = rois.shape[0]
        h = {"rois": rois, "out_size": (grid, grid)}
        if kind != "extract":           # a loop's own buffers
            h["levels"] = torch.empty(k, dtype=torch.int32, device="cuda")
            h["ws"] = torch.empty(rex.workspace_size(st["feats"], st["scales"], k),
                                  dtype=torch.uint8, device="cuda")
            h["out"] = torch.empty((k, c, grid, grid), dtype=dt, device="cuda")
        if case["backward"]:
            h["gout"] = randn((k, c, grid, grid))
        st["heads"].append(h)
    k = st["heads"][0]["rois"].shape[0]
    if case["backward"]:
        if kind == "extract":
            for f in st["feats"]:
                f.requires_grad_(True)
        else:
            st["grads"] = _pyramid(case, lambda s: torch.empty(s, dtype=torch.float32,
                                                               device="cuda"))
    if kind == "pool":
        st["argmax"] = torch.empty((k, c, p, p), dtype=torch.int32, device="cuda")
    if kind == "deform":
        st["offset"] = randn((k, 2, p, p), torch.float32) * 0.3
        st["mask"] = torch.sigmoid(randn((k, p, p), torch.float32))
        st["grad_offset"] = torch.empty_like(st["offset"])
        st["grad_mask"] = torch.empty_like(st["mask"])
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "nms":
        keep, num = rex.box_nms(st["boxes"], st["scores"], case["iou"], st["cats"],
                                case["max_keep"], keep=st["keep"], num_keep=st["num"])
        return {"keep": keep, "num": num}
    if kind == "select":
        keep, scores, num = rex.box_nms_batched(
            st["boxes"], st["scores"], st["cats"], case["categories"], case["method"],
            case["iou"], 0.5, case["score_threshold"], case["max_keep"], keep=st["keep"],
            kept_scores=st["kept_scores"], num_keep=st["num"])
        return {"keep": keep, "scores": scores, "num": num}

    feats, scales, h = st["feats"], st["scales"], st["heads"][0]
    size, s = h["out_size"], case["sampling"]
    if kind == "extract":
        if not case["backward"]:
            with torch.no_grad():
                return {"out": rex.roi_extract(feats, scales, h["rois"], size, s)}
        out = rex.roi_extract(feats, scales, h["rois"], size, s)
        return {"out": out.detach(), "grads": list(torch.autograd.grad(out, feats, h["gout"]))}

    for q in st["heads"]:
        rex.plan(feats, scales, q["rois"], FINEST, levels_out=q["levels"], workspace=q["ws"])
    if kind == "heads":
        heads = [{"rois": q["rois"], "roi_levels": q["levels"], "out_size": q["out_size"],
                  "workspace": q["ws"], "out": q["out"], "grad_out": q["gout"]}
                 for q in st["heads"]]
        outs = rex.roi_align_fwd_multi(feats, scales, heads)
        rex.roi_align_bwd_multi(heads, st["grads"], scales, zero_init=True)
        return {"outs": outs, "grads": st["grads"]}
    if kind == "align":
        rex.roi_align_fwd(feats, scales, h["rois"], h["levels"], size, s, True,
                          workspace=h["ws"], out=h["out"])
        if not case["backward"]:
            return {"levels": h["levels"], "out": h["out"]}
        rex.roi_align_bwd(h["gout"], h["rois"], h["levels"], size, s, True, st["grads"], scales,
                          zero_init=True, workspace=h["ws"])
        return {"levels": h["levels"], "out": h["out"], "grads": st["grads"]}
    if kind == "pool":
        rex.roi_pool_fwd(feats, scales, h["rois"], h["levels"], size, workspace=h["ws"],
                         out=h["out"], argmax=st["argmax"])
        rex.roi_pool_bwd(h["gout"], st["argmax"], h["rois"], h["levels"], st["grads"], scales,
                         workspace=h["ws"])
        return {"out": h["out"], "argmax": st["argmax"], "grads": st["grads"]}
    rex.deform_roi_pool_fwd(feats, scales, h["rois"], h["levels"], size, st["offset"],
                            st["mask"], GAMMA, s, workspace=h["ws"], out=h["out"])
    rex.deform_roi_pool_bwd(h["gout"], feats, h["rois"], h["levels"], st["offset"], st["mask"],
                            st["grads"], scales, GAMMA, s, grad_offset=st["grad_offset"],
                            grad_mask=st["grad_mask"], workspace=h["ws"])
    return {"out": h["out"], "grads": st["grads"], "grad_offset": st["grad_offset"],
            "grad_mask": st["grad_mask"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how close two correct results are
# ---------------------------------------------------------------------------

def work(case):
    if case["kind"] in ("nms", "select"):
        groups = case["images"] if case["kind"] == "nms" else case["categories"]
        per = case["per_image"] if case["kind"] == "nms" else case["per_category"]
        n = groups * per
        # candidates over the score threshold; each meets the kept boxes before it
        share = 1.0 - max(0.0, case.get("score_threshold", 0.0)) ** (1.0 / case.get("score_power", 1.0))
        cand = per * share
        keep = min(cand, case["max_keep"])
        return {"bytes": n * 24 + groups * min(per, case["max_keep"]) * 8,
                "flops": groups * cand * keep * 16 / 2}
    size = 2 if case["dtype"] == "bf16" else 4
    c, n = case["channels"], case["images"]
    pixels = n * sum(h * w for h, w in _shapes(case)[0])
    heads = [(n * case["per_image"], case["out"])]
    if case["kind"] == "heads":
        heads.append((n * case["mask_per_image"], 14))
    nbytes, flops = 0.0, 0.0
    # features: every pixel at most once, and no more than one pixel per sample position
    nbytes += min(pixels, sum(k * (2 * p) ** 2 for k, p in heads)) * c * size
    for k, p in heads:
        block = k * c * p * p
        nbytes += block * size + k * 20                  # output, RoIs
        flops += block * 4 * 8                           # four samples of four taps
        if case["kind"] == "pool":
            nbytes += block * 4                          # argmax written (and read below)
        if case["kind"] == "deform":
            nbytes += k * p * p * 12
        if case["backward"]:
            nbytes += block * size                       # upstream gradient
            flops += block * 4 * 8
            if case["kind"] == "pool":
                nbytes += block * 4
            if case["kind"] == "deform":
                nbytes += k * p * p * 12
    if case["backward"]:
        nbytes += pixels * c * (size if case["kind"] == "extract" else 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] in ("nms", "select"):
        return "exact"                  # the definition fixes every decision bit for bit
    if case["dtype"] == "bf16":
        # binary32 sums rounded once to bf16: another order of the sums moves a few values
        # to the neighbouring bf16 number, 2^-7 of the value at most (measured: 2e-5, 7e-3)
        return {"rel": 2e-4, "max": 1.6e-2, "differ": 0.0}
    # binary32 sums: two orders differ by 6e-8 .. 1e-7 (largest difference 2.4e-6), and are
    # as far from the 64-bit result
    return {"rel": 5e-7, "max": 1.2e-5, "differ": 0.0}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _levels_of(case, rois):
    """The FPN level rule in binary32."""
    num = len(_shapes(case)[0])
    area = (rois[:, 3] - rois[:, 1]) * (rois[:, 4] - rois[:, 2])
    lvl = torch.zeros(rois.shape[0], dtype=torch.int64, device=rois.device)
    for j in range(1, num):
        lvl += (area >= float(np.float32(FINEST * 2 ** j) ** 2)).long()
    return lvl


def _axis(c1, c2, scale, p, sampling):
    """(start, bin, samples per bin, length) of one axis, binary32, aligned boxes."""
    start = c1 * scale - 0.5
    length = (c2 * scale - 0.5) - start
    # (a tensor divisor: torch multiplies by the reciprocal of a scalar one)
    bins = length / torch.full_like(length, float(p))
    if sampling > 0:
        grid = torch.full_like(bins, float(sampling))
    else:
        grid = torch.where(bins > 0, torch.ceil(bins), torch.zeros_like(bins)).clamp(max=64.0)
    return start, bins, grid, length


def _positions(start, bins, grid, p, shift=None):
    """[k, p, g] binary32 sample positions and whether each exists."""
    g = max(1, int(grid.max().item()) if grid.numel() else 1)
    i = torch.arange(g, device=start.device, dtype=torch.float32)
    q = torch.arange(p, device=start.device, dtype=torch.float32)
    base = start[:, None] + q[None] * bins[:, None]
    within = ((i[None] + 0.5) * bins[:, None]) / grid.clamp(min=1.0)[:, None]
    if shift is None:
        pos = base[:, :, None] + within[:, None, :]
    else:
        pos = (base[:, :, None] + shift)[..., None] + within[:, None, None, :]
    return pos, i[None] < grid[:, None]


def _taps(pos, size):
    """(valid, lo, hi, fraction, clamped) of positions on a map of `size` pixels."""
    valid = (pos >= -1.0) & (pos <= float(size))
    v = torch.where(valid, pos, torch.zeros_like(pos)).clamp(min=0.0)
    lo = v.floor().long()
    edge = lo >= size - 1
    lo = torch.where(edge, torch.full_like(lo, size - 1), lo)
    frac = torch.where(edge, torch.zeros_like(v), v - lo.float()).double()
    hi = torch.where(edge, lo, lo + 1)
    return valid, lo, hi, frac, edge | (pos < 0)


def _matrix(c1, c2, scale, p, sampling, size):
    """[k, p, size] interpolation weights of one axis, divided by the samples per bin."""
    start, bins, grid, _ = _axis(c1, c2, scale, p, sampling)
    pos, there = _positions(start, bins, grid, p)
    valid, lo, hi, frac, _ = _taps(pos, size)
    keep = (valid & there[:, None, :]).double() / grid.clamp(min=1.0).double()[:, None, None]
    m = torch.zeros(pos.shape[0], p, size, dtype=torch.float64, device=pos.device)
    m.scatter_add_(2, lo, (1.0 - frac) * keep)
    m.scatter_add_(2, hi, frac * keep)
    return m


def _groups(case, rois, chunk):
    """Runs of RoIs on one level and image: (level, image, their indices)."""
    lvl = _levels_of(case, rois)
    img = rois[:, 0].long()
    for l in range(len(_shapes(case)[0])):
        for b in range(case["images"]):
            idx = torch.nonzero((lvl == l) & (img == b)).flatten()
            for part in idx.split(chunk):
                if part.numel():
                    yield l, b, part


def _exact_align(case, st):
    feats, scales, c = st["feats"], st["scales"], case["channels"]
    grads = [torch.zeros(f.shape[0], f.shape[2], f.shape[3], c, dtype=torch.float64,
                         device="cuda") for f in feats] if case["backward"] else None
    outs = []
    for h in st["heads"]:
        rois, p = h["rois"], h["out_size"][0]
        out = torch.zeros(rois.shape[0], c, p, p, dtype=torch.float64, device="cuda")
        for l, b, idx in _groups(case, rois, 48):
            fm = feats[l].detach()[b]
            hh, ww = fm.shape[1:]
            r = rois[idx]
            my = _matrix(r[:, 2], r[:, 4], scales[l], p, case["sampling"], hh)
            mx = _matrix(r[:, 1], r[:, 3], scales[l], p, case["sampling"], ww)
            rows = my.reshape(-1, hh)
            f64 = fm.permute(1, 2, 0).double().reshape(hh, ww * c)
            t = (rows @ f64).reshape(-1, p, ww, c)
            out[idx] = torch.matmul(mx[:, None], t).permute(0, 3, 1, 2)
            if grads is not None:
                g = h["gout"][idx].double().permute(0, 2, 3, 1).contiguous()
                t = torch.matmul(mx.transpose(1, 2).contiguous()[:, None], g)
                grads[l][b] += (rows.t().contiguous() @ t.reshape(-1, ww * c)).reshape(hh, ww, c)
        outs.append(out)
    if grads is not None:
        grads = [g.permute(0, 3, 1, 2) for g in grads]
    return outs, grads


def _exact_pool(case, st):
    feats, scales, c = st["feats"], st["scales"], case["channels"]
    h = st["heads"][0]
    rois, p = h["rois"], h["out_size"][0]
    out = torch.zeros(rois.shape[0], p * p, c, dtype=torch.float64, device="cuda")
    grads = [torch.zeros(f.shape[0], f.shape[2] * f.shape[3], c, dtype=torch.float64,
                         device="cuda") for f in feats]

    def edges(c1, c2, scale, size):
        def half_away(x):
            return torch.where(x >= 0, torch.floor(x.double() + 0.5), torch.ceil(x.double() - 0.5))
        s, e = half_away(c1 * scale).float(), half_away(c2 * scale).float()
        length = (e - s + 1.0).clamp(min=1.0)
        bins = length / torch.full_like(length, float(p))       # binary32, as defined
        q = torch.arange(p, device="cuda", dtype=torch.float32)
        lo = torch.floor(q[None] * bins[:, None]) + s[:, None]
        hi = torch.ceil((q[None] + 1) * bins[:, None]) + s[:, None]
        return lo.clamp(0, size).long(), hi.clamp(0, size).long()

    for l, b, idx in _groups(case, rois, 16):
        fm = feats[l][b]
        hh, ww = fm.shape[1:]
        f64 = fm.permute(1, 2, 0).double().reshape(hh * ww, c)
        r = rois[idx]
        y0, y1 = edges(r[:, 2], r[:, 4], scales[l], hh)
        x0, x1 = edges(r[:, 1], r[:, 3], scales[l], ww)
        ny, nx = int((y1 - y0).max().item()), int((x1 - x0).max().item())
        if ny <= 0 or nx <= 0:
            continue
        ys = y0[:, :, None] + torch.arange(ny, device="cuda")
        xs = x0[:, :, None] + torch.arange(nx, device="cuda")
        ok = (ys < y1[:, :, None])[:, :, None, :, None] & (xs < x1[:, :, None])[:, None, :, None, :]
        pix = ys.clamp(max=hh - 1)[:, :, None, :, None] * ww + \
            xs.clamp(max=ww - 1)[:, None, :, None, :]
        ok, pix = (v.expand(-1, p, p, ny, nx).reshape(-1, p * p, ny * nx) for v in (ok, pix))
        best = torch.full((idx.numel(), p * p, c), -math.inf, dtype=torch.float64, device="cuda")
        where = torch.full(best.shape, -1, dtype=torch.int64, device="cuda")
        for j in range(ny * nx):        # row-major: a later pixel wins only if larger
            v = f64[pix[:, :, j]]
            new = ok[:, :, j, None] & (v > best)
            best = torch.where(new, v, best)
            where = torch.where(new, pix[:, :, j, None].expand_as(where), where)
        out[idx] = torch.where(where >= 0, best, torch.zeros_like(best))
        g = h["gout"][idx].double().reshape(-1, c, p * p).permute(0, 2, 1)
        g = torch.where(where >= 0, g, torch.zeros_like(g))
        grads[l][b].scatter_add_(0, where.clamp(min=0).reshape(-1, c), g.reshape(-1, c))
    k = rois.shape[0]
    return {"out": out.permute(0, 2, 1).reshape(k, c, p, p), "argmax": None,
            "grads": [g.reshape(g.shape[0], f.shape[2], f.shape[3], c).permute(0, 3, 1, 2)
                      for g, f in zip(grads, feats)]}


def _exact_deform(case, st):
    feats, scales, c, s = st["feats"], st["scales"], case["channels"], case["sampling"]
    h = st["heads"][0]
    rois, p = h["rois"], h["out_size"][0]
    k = rois.shape[0]
    out = torch.zeros(k, c, p, p, dtype=torch.float64, device="cuda")
    g_off = torch.zeros(k, 2, p, p, dtype=torch.float64, device="cuda")
    g_mask = torch.zeros(k, p, p, dtype=torch.float64, device="cuda")
    grads = [torch.zeros(f.shape[0], f.shape[2] * f.shape[3], c, dtype=torch.float64,
                         device="cuda") for f in feats]
    gamma = torch.tensor(GAMMA, dtype=torch.float32, device="cuda")
    for l, b, idx in _groups(case, rois, 96):
        fm = feats[l][b]
        hh, ww = fm.shape[1:]
        f64 = fm.permute(1, 2, 0).double().reshape(hh * ww, c)
        r = rois[idx]
        x0, bx, gx, lx = _axis(r[:, 1], r[:, 3], scales[l], p, s)
        y0, by, gy, ly = _axis(r[:, 2], r[:, 4], scales[l], p, s)
        dx = (gamma * st["offset"][idx, 0]) * lx[:, None, None]
        dy = (gamma * st["offset"][idx, 1]) * ly[:, None, None]
        # [k, ph, pw, sample] along x, and along y with the bin axes exchanged back
        px, _ = _positions(x0, bx, gx, p, dx.transpose(1, 2))
        px = px.transpose(1, 2)
        py, _ = _positions(y0, by, gy, p, dy)
        vx, xl, xh, fx, cx = _taps(px, ww)
        vy, yl, yh, fy, cy = _taps(py, hh)
        m = st["mask"][idx].double()
        g = h["gout"][idx].double().permute(0, 2, 3, 1)             # [k, p, p, c]
        val = torch.zeros_like(g)
        sx, sy = torch.zeros_like(g), torch.zeros_like(g)
        for iy in range(s):
            for ix in range(s):
                v = (vy[..., iy] & vx[..., ix]).double()[..., None] / (s * s)
                ty, tx = fy[..., iy][..., None], fx[..., ix][..., None]
                corner = [(yl, xl, (1 - ty) * (1 - tx)), (yl, xh, (1 - ty) * tx),
                          (yh, xl, ty * (1 - tx)), (yh, xh, ty * tx)]
                f = []
                for yy, xx, w in corner:
                    pix = yy[..., iy] * ww + xx[..., ix]
                    f.append(f64[pix])
                    val += v * w * f[-1]
                    grads[l][b].index_add_(0, pix.reshape(-1),
                                           (g * m[..., None] * v * w).reshape(-1, c))
                free_x = (~cx[..., ix]).double()[..., None]
                free_y = (~cy[..., iy]).double()[..., None]
                sx += v * free_x * ((1 - ty) * (f[1] - f[0]) + ty * (f[3] - f[2]))
                sy += v * free_y * ((1 - tx) * (f[2] - f[0]) + tx * (f[3] - f[1]))
        out[idx] = (val * m[..., None]).permute(0, 3, 1, 2)
        g_mask[idx] = (g * val).sum(-1)
        scale = gamma.double() * m
        g_off[idx, 0] = (g * sx).sum(-1) * scale * lx.double()[:, None, None]
        g_off[idx, 1] = (g * sy).sum(-1) * scale * ly.double()[:, None, None]
    return {"out": out, "grad_offset": g_off, "grad_mask": g_mask,
            "grads": [t.reshape(t.shape[0], f.shape[2], f.shape[3], c).permute(0, 3, 1, 2)
                      for t, f in zip(grads, feats)]}


def _iou(a, b):
    """Binary32 IoU of boxes [n, 4] against [m, 4], one rounding per operation."""
    w = (torch.minimum(a[:, None, 2], b[None, :, 2]) -
         torch.maximum(a[:, None, 0], b[None, :, 0])).clamp(min=0)
    h = (torch.minimum(a[:, None, 3], b[None, :, 3]) -
         torch.maximum(a[:, None, 1], b[None, :, 1])).clamp(min=0)
    inter = w * h
    area_a = (a[:, 2] - a[:, 0]) * (a[:, 3] - a[:, 1])
    area_b = (b[:, 2] - b[:, 0]) * (b[:, 3] - b[:, 1])
    return inter / ((area_a[:, None] + area_b[None, :]) - inter)


def _exact_select(case, st):
    limit, method = case["max_keep"], case["method"]
    scores_out = torch.zeros(case["categories"], limit, dtype=torch.float64)
    per = case["per_category"]
    for cat in range(case["categories"]):
        s = st["scores"][cat * per:(cat + 1) * per]
        cand = torch.nonzero(s >= case["score_threshold"]).flatten()
        cand = cand[torch.argsort(s[cand], descending=True, stable=True)]
        box = st["boxes"][cat * per:(cat + 1) * per][cand]
        iou = _iou(box, box).cpu().numpy()
        cur = s[cand].cpu().numpy()
        alive = np.ones(len(cur), dtype=bool)
        for i in range(limit):
            if not alive.any():
                break
            j = int(np.argmax(np.where(alive, cur, -np.inf)))
            scores_out[cat, i] = float(cur[j])
            alive[j] = False
            row = iou[j]
            if method == "hard":
                alive &= ~(row > case["iou"])
                continue
            if method == "linear":
                w = np.where(row > np.float32(case["iou"]), np.float32(1) - row, np.float32(1))
            else:
                w = np.exp(-row.astype(np.float64) ** 2 / 0.5).astype(np.float32)
            w = np.where(np.isnan(row), np.float32(1), w)
            cur = np.where(alive, cur * w, cur)
            alive &= ~(cur < np.float32(case["score_threshold"]))
    return {"keep": None, "scores": scores_out, "num": None}


def exact(case, seed):
    if case["kind"] == "nms":
        return None                     # indices only
    st = prepare(case, seed)
    if case["kind"] == "select":
        return _exact_select(case, st)
    if case["kind"] == "pool":
        return _exact_pool(case, st)
    if case["kind"] == "deform":
        return _exact_deform(case, st)
    outs, grads = _exact_align(case, st)
    if case["kind"] == "heads":
        return {"outs": outs, "grads": grads}
    res = {"out": outs[0]}
    if case["kind"] == "align":
        res["levels"] = None
    if grads is not None:
        res["grads"] = grads
    return res
