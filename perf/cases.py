"""Performance cases of the library: what a program that fragments images has it do, each as one call
(or one round trip) through the public entry points, over the range of sizes that the tests, the
benchmark and the report's workloads use.

A case is a dict of plain values.  ``form`` names the entry points:

  image     frag_image then defrag_image (FP32, or the fp16 / bf16 precision form)
  batch     sf_frag_batch then sf_defrag_batch over a planned set of images in slabs
  pixel     pixel_frag_image then pixel_defrag_image (first or strong level, 11- or 8-bit fields)
  wavelet   dwt_frag_image then dwt_defrag_image
  cipher    encrypt_private over a buffer
  stats     security statistics of a protected image against its original
  step      one training step of the soft mask: public image, correlation loss, gradients
  tune      statistics pass and Adam loop of the soft-mask tuner

``keep`` says whether the program reuses its output buffers from call to call or lets every call
allocate them.  Images are smooth content (eight sinusoids per plane) with sensor-like noise, 8 bits
per sample, planar.
"""
from __future__ import annotations

import ctypes
import math
import random

import numpy as np
import torch

import paper_1512_02951_amd as sf
from paper_1512_02951_amd import batch as sf_batch
from paper_1512_02951_amd import dwt as sf_dwt
from paper_1512_02951_amd import pixel as sf_pixel
from paper_1512_02951_amd import softmask as sf_soft
from paper_1512_02951_amd import stats as sf_stats

DEVICE = "cuda:0"
PUBLIC_DTYPE = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
PER_TILE = sf.DEFAULT_PER_TILE


def prefix(k):
    """DC and the first k zigzag AC coefficients."""
    return (1 << (k + 1)) - 1


def listed():
    return [
        # The smallest call in use: one 512 x 512 gray image with DC + 2 AC private, each call
        # allocating its outputs.  Latency and launches count.
        {"name": "small gray image", "form": "image", "H": 512, "W": 512, "C": 1, "mask": prefix(2),
         "precision": "fp32", "keep": False},
        # The throughput workload: a 4096 x 4096 RGB image, DC + 5 AC, into kept buffers.
        {"name": "large RGB image", "form": "image", "H": 4096, "W": 4096, "C": 3, "mask": prefix(5),
         "precision": "fp32", "keep": True},
        # A video-sized RGB frame (rows not a multiple of the 64-block tile) with a selection as the
        # soft-mask tuner returns it: six low frequencies that are no zigzag prefix.
        {"name": "frame, tuned selection", "form": "image", "H": 1080, "W": 1920, "C": 3, "mask": 0x9F,
         "precision": "fp32", "keep": True},
        # The reduced-precision form on its own workload: one 8192 x 8192 gray image, DC + 9 AC.
        {"name": "fp16 large gray image", "form": "image", "H": 8192, "W": 8192, "C": 1, "mask": prefix(9),
         "precision": "fp16", "keep": True},
        # The same form in bf16 on an ordinary image whose last tile is partly filled.
        {"name": "bf16 ragged image", "form": "image", "H": 2056, "W": 3000, "C": 1, "mask": prefix(9),
         "precision": "bf16", "keep": True},
        # Many images of uneven sizes and selections in one call per direction.
        {"name": "batch of 128 images", "form": "batch", "images": 128, "lo": 256, "hi": 4096, "mix": 1},
        # The strong level in the report's storage format on the large RGB image.
        {"name": "strong level, RGB image", "form": "pixel", "H": 4096, "W": 4096, "C": 3, "mask": prefix(5),
         "strong": True, "bits": 11},
        # The wavelet variant on the large RGB image.
        {"name": "wavelet, RGB image", "form": "wavelet", "H": 4096, "W": 4096, "C": 3},
        # The cipher by itself, over a buffer that holds the private parts of many images.
        {"name": "cipher, 128 MiB", "form": "cipher", "bytes": 128 << 20, "first": 0},
        # Evaluation of a protected image (bytes that look like noise) against its original.
        {"name": "statistics, RGB image", "form": "stats", "H": 4096, "W": 4096, "C": 3, "protected": "noise"},
        # One training step of the soft mask on the tuning set.
        {"name": "soft-mask step", "form": "step", "B": 64, "H": 1024, "W": 1024},
        # The tuner on the same set: 200 Adam steps, six private coefficients.
        {"name": "soft-mask tuner", "form": "tune", "B": 64, "H": 1024, "W": 1024, "steps": 200, "private": 6},
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _side(v, lo, hi):
    return max(lo, min(hi, 8 * int(round(v / 8))))


def _image_shape(rng, lo, hi, channels=(1, 1, 3)):
    """(H, W, C) with lo .. hi samples in all, sides multiples of 8 and up to four to one."""
    n = _log(rng, lo, hi)
    C = rng.choice(channels)
    a = _log(rng, 0.5, 2.0)
    return _side(math.sqrt(n / C) * a, 64, 8192), _side(math.sqrt(n / C) / a, 64, 8192), C


def _mask(rng):
    if rng.random() < 0.75:
        return prefix(rng.choice((1, 2, 3, 5, 7, 9, 9, 14)))
    m = 1
    for z in rng.sample(range(1, 16), rng.randint(2, 9)):
        m |= 1 << z
    return m


def draw(rng):
    form = rng.choice(("image", "image", "image", "image", "batch", "pixel", "pixel", "wavelet", "cipher", "stats",
                       "step", "tune"))
    if form == "image":
        H, W, C = _image_shape(rng, 1 << 17, 1 << 25)
        return {"form": form, "H": H, "W": W, "C": C, "mask": _mask(rng),
                "precision": rng.choice(("fp32", "fp32", "fp16", "bf16")), "keep": rng.random() < 0.7}
    if form == "batch":
        return {"form": form, "images": rng.randint(4, 128), "lo": 256, "hi": rng.choice((1024, 2048, 4096)),
                "mix": rng.randrange(2, 1000)}
    if form == "pixel":
        H, W, C = _image_shape(rng, 1 << 17, 1 << 25)
        return {"form": form, "H": H, "W": W, "C": C, "mask": prefix(rng.choice((2, 3, 5, 9))),
                "strong": rng.random() < 0.5, "bits": rng.choice((11, 11, 8))}
    if form == "wavelet":
        H, W, C = _image_shape(rng, 1 << 17, 1 << 25)
        return {"form": form, "H": H, "W": W, "C": C}
    if form == "cipher":
        return {"form": form, "bytes": int(_log(rng, 1 << 12, 1 << 27)), "first": rng.randrange(1 << 34)}
    if form == "stats":
        H, W, C = _image_shape(rng, 1 << 17, 1 << 25)
        return {"form": form, "H": H, "W": W, "C": C, "protected": rng.choice(("noise", "residue"))}
    B = int(_log(rng, 1, 64.99))
    H, W = _side(_log(rng, 128, 1024), 128, 1024), _side(_log(rng, 128, 1024), 128, 1024)
    if form == "step":
        return {"form": form, "B": B, "H": H, "W": W}
    return {"form": form, "B": B, "H": H, "W": W, "steps": rng.randint(20, 200), "private": rng.randint(3, 12)}


# ------------------------------------------------------------------ inputs
def _plane(H, W, rng, gen):
    """One float32 plane (H, W): 128 + eight sinusoids + noise of variance 4, not yet rounded."""
    ys = torch.arange(H, dtype=torch.float32, device=DEVICE)
    xs = torch.arange(W, dtype=torch.float32, device=DEVICE)
    rows, cols = [], []
    for _ in range(8):
        A, T = rng.uniform(5, 30), rng.uniform(4, 128)
        th, ph = rng.uniform(0, 2 * math.pi), rng.uniform(0, 2 * math.pi)
        b = ys * (2 * math.pi * math.sin(th) / T) + ph
        a = xs * (2 * math.pi * math.cos(th) / T)
        rows += [A * torch.sin(b), A * torch.cos(b)]
        cols += [torch.cos(a), torch.sin(a)]
    v = torch.randn((H, W), dtype=torch.float32, device=DEVICE, generator=gen)
    return torch.addmm(v, torch.stack(rows, 1), torch.stack(cols, 0), beta=2.0).add_(128.0)


def _sources(seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return random.Random(seed), gen


def _image(H, W, C, rng, gen, out=None):
    """uint8 (C, H, W)."""
    out = torch.empty((C, H, W), dtype=torch.uint8, device=DEVICE) if out is None else out
    for c in range(C):
        out[c] = _plane(H, W, rng, gen).round_().clamp_(0, 255).to(torch.uint8)
    return out


def _keys(rng):
    return bytes(rng.randrange(256) for _ in range(16)), bytes(rng.randrange(256) for _ in range(8)) + bytes(8)


def _batch_specs(case):
    """(H, W, C, mask) per image: sides log-uniform, one or three channels, k from {1, 2, 5, 9}; ``mix``
    names one such set of shapes."""
    rng = random.Random(case["mix"])
    specs = []
    for _ in range(case["images"]):
        w, h = (_side(_log(rng, case["lo"], case["hi"]), 8, 1 << 14) for _ in range(2))
        specs.append((h, w, rng.choice((1, 3)), prefix(rng.choice((1, 2, 5, 9)))))
    return specs


def _slab_offsets(sizes):
    """Byte offsets of consecutive pieces, each on a 256-byte boundary, and the total."""
    offs, at = [], 0
    for n in sizes:
        offs.append(at)
        at += (n + 255) // 256 * 256
    return offs, max(at, 256)


def _batch_images(case, seed):
    rng, gen = _sources(seed)
    specs = _batch_specs(case)
    offs, total = _slab_offsets([h * w * c for h, w, c, _ in specs])
    slab = torch.zeros(total, dtype=torch.uint8, device=DEVICE)
    for (h, w, c, _), o in zip(specs, offs):
        _image(h, w, c, rng, gen, slab[o:o + h * w * c].view(c, h, w))
    return specs, offs, slab, rng


def _soft_inputs(case, seed):
    rng, gen = _sources(seed)
    x = torch.empty((case["B"], case["H"], case["W"]), dtype=torch.float32, device=DEVICE)
    for i in range(case["B"]):
        x[i] = _plane(case["H"], case["W"], rng, gen).round_().clamp_(0, 255).div_(255.0)
    return x, torch.randn(64, dtype=torch.float32, device=DEVICE, generator=gen)


def _stats_inputs(case, seed):
    rng, gen = _sources(seed)
    x = _image(case["H"], case["W"], case["C"], rng, gen)
    if case["protected"] == "noise":  # a strong-level public part
        y = torch.randint(0, 256, x.shape, dtype=torch.uint8, device=DEVICE, generator=gen)
    else:  # a first-level public part: the block means taken out, modulo 256
        C, H, W = x.shape
        b = x.view(C, H // 8, 8, W // 8, 8).to(torch.int32)
        y = ((b - b.sum(dim=(2, 4), keepdim=True) // 64) & 255).to(torch.uint8).view(C, H, W)
    return x, y


def prepare(case, seed):
    form = case["form"]
    s = {"case": case, "form": form}
    if form in ("image", "pixel", "wavelet"):
        rng, gen = _sources(seed)
        s["pixels"] = _image(case["H"], case["W"], case["C"], rng, gen)
        s["key"], s["ctr0"] = _keys(rng)
    if form == "image":
        s["out"] = s["restored"] = None
        if case["keep"]:
            shape = (case["C"], case["H"], case["W"])
            pb, qb, rb = sf.fragment_sizes(case["H"], case["W"], case["C"], case["mask"], case["precision"])
            pub = PUBLIC_DTYPE[case["precision"]]
            s["out"] = sf.Fragments(
                public=torch.zeros(pb // pub.itemsize, dtype=pub, device=DEVICE),
                private=torch.zeros(qb, dtype=torch.uint8, device=DEVICE),
                exceptions=sf.ExceptionList.empty(shape, case["mask"], device=DEVICE, precision=case["precision"]),
                residual=torch.zeros(rb, dtype=torch.uint8, device=DEVICE) if rb else None,
                shape=shape, mask=case["mask"], precision=case["precision"])
            s["restored"] = torch.zeros_like(s["pixels"])
    elif form == "pixel":
        pb, qb = sf_pixel.fragment_sizes(case["H"], case["W"], case["C"], case["mask"], case["strong"], case["bits"])
        s["out"] = sf_pixel.PixelFragments(
            torch.zeros_like(s["pixels"]), torch.zeros(qb, dtype=torch.uint8, device=DEVICE), case["mask"],
            case["strong"], tuple(s["pixels"].shape), case["bits"])
        s["restored"] = torch.zeros_like(s["pixels"])
    elif form == "wavelet":
        pb, qb = sf_dwt.fragment_sizes(case["H"], case["W"], case["C"])
        s["out"] = sf_dwt.DwtFragments(torch.zeros(pb // 2, dtype=torch.int16, device=DEVICE),
                                       torch.zeros(qb, dtype=torch.uint8, device=DEVICE), tuple(s["pixels"].shape))
        s["restored"] = torch.zeros_like(s["pixels"])
    elif form == "batch":
        specs, offs, s["pixels"], rng = _batch_images(case, seed)
        s["key"], _ = _keys(rng)
        sizes = [sf.fragment_sizes(h, w, c, m) for h, w, c, m in specs]
        exc = [sf.exception_bytes(h, w, c, m, PER_TILE) for h, w, c, m in specs]
        po, pt = _slab_offsets([z[0] for z in sizes])
        qo, qt = _slab_offsets([z[1] for z in sizes])
        eo, et = _slab_offsets([n if needed else 0 for n, needed in exc])
        s["public"] = torch.zeros(pt // 4, dtype=torch.float32, device=DEVICE)
        s["private"] = torch.zeros(qt, dtype=torch.uint8, device=DEVICE)
        s["exceptions"] = torch.zeros(et, dtype=torch.uint8, device=DEVICE)
        s["restored"] = torch.zeros_like(s["pixels"])
        items = (sf_batch.SfBatchItem * len(specs))()
        for i, (h, w, c, m) in enumerate(specs):
            it = items[i]
            it.height, it.width, it.channels, it.exc_per_tile, it.private_mask = h, w, c, PER_TILE, m
            it.d_pixels, it.d_restored = s["pixels"].data_ptr() + offs[i], s["restored"].data_ptr() + offs[i]
            it.d_public, it.d_private = s["public"].data_ptr() + po[i], s["private"].data_ptr() + qo[i]
            it.d_exc = s["exceptions"].data_ptr() + eo[i] if exc[i][1] else None
            it.ctr0[:] = list(_keys(rng)[1])
        n = sf_batch.lib().sf_batch_workspace_bytes(len(specs))
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEVICE)
        sf.check(sf_batch.lib().sf_batch_plan(items, len(specs), (ctypes.c_uint8 * 16)(*s["key"]),
                                              ctypes.c_void_p(s["workspace"].data_ptr()), n, sf._stream(None)))
    elif form == "cipher":
        rng, gen = _sources(seed)
        s["data"] = torch.randint(0, 256, (case["bytes"],), dtype=torch.uint8, device=DEVICE, generator=gen)
        s["key"], s["ctr0"] = _keys(rng)
        s["out"] = torch.zeros_like(s["data"])
    elif form == "stats":
        s["x"], s["y"] = _stats_inputs(case, seed)
        s["runner"] = sf_stats.StatsRunner(s["x"].device)
        s["blocks"] = torch.zeros(2 * s["x"].numel() // 64, dtype=torch.float32, device=DEVICE)
    else:
        s["x"], s["logits"] = _soft_inputs(case, seed)
        s["logits"].requires_grad_(form == "step")
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    form = s["form"]
    if form == "image":
        c = s["case"]
        f = sf.frag_image(s["pixels"], c["mask"], s["key"], s["ctr0"], precision=c["precision"], out=s["out"])
        y = sf.defrag_image(f, s["key"], s["ctr0"], out=s["restored"])
        return {"public": f.public, "private": f.private, "exceptions": f.exceptions.buf, "residual": f.residual,
                "restored": y}
    if form == "pixel":
        c = s["case"]
        f = sf_pixel.pixel_frag_image(s["pixels"], c["mask"], c["strong"], s["key"], s["ctr0"], out=s["out"],
                                      storage_bits=c["bits"])
        y = sf_pixel.pixel_defrag_image(f, s["key"], s["ctr0"], out=s["restored"])
        return {"public": f.public, "private": f.private, "restored": y}
    if form == "wavelet":
        f = sf_dwt.dwt_frag_image(s["pixels"], s["key"], s["ctr0"], out=s["out"])
        y = sf_dwt.dwt_defrag_image(f, s["key"], s["ctr0"], out=s["restored"])
        return {"public": f.public, "private": f.private, "restored": y}
    if form == "batch":
        ws = ctypes.c_void_p(s["workspace"].data_ptr())
        sf.check(sf_batch.lib().sf_frag_batch(ws, None, None, sf._stream(None)))
        sf.check(sf_batch.lib().sf_defrag_batch(ws, None, None, sf._stream(None)))
        return {k: s[k] for k in ("public", "private", "exceptions", "restored")}
    if form == "cipher":
        return sf.encrypt_private(s["key"], s["ctr0"], s["data"], out=s["out"], first_block=s["case"]["first"])
    if form == "stats":
        r = s["runner"]
        r.launch(s["x"], s["y"], s["blocks"])
        n = 8 * _STATS_INTS
        return {"counts": r.out[:n].view(torch.int64), "figures": r.out[n:].view(torch.float64),
                "joint": r.joint_histogram(), "block_entropy": s["blocks"]}
    if form == "step":
        x, logits = s["x"], s["logits"]
        logits.grad = None
        P = sf_soft.SoftMaskPublic.apply(x, logits)
        loss = sf_soft.CorrelationLoss.apply(x, P, logits)
        loss.backward()
        return {"public": P.detach(), "loss": loss.detach(), "grad": logits.grad}
    c = s["case"]
    logits, trace, mask = sf_soft.tune(s["x"], s["logits"], steps=c["steps"], n_private=c["private"])
    return {"logits": logits, "trace": trace, "mask": mask}


# samples, two histograms, two sets of 3 x 6 pair moments, six cross moments, differing bits
_STATS_INTS = 1 + 2 * 256 + 2 * 18 + 6 + 1


# ------------------------------------------------------------------ what a pass cannot do without
def _private(mask):
    return bin(mask).count("1")


def _image_bytes(n, mask, precision):
    P = _private(mask)
    elt = 4 if precision == "fp32" else 2
    extra = 0 if precision == "fp32" else n // 4  # 2-bit residual codes
    return 2 * (n + n // 64 * ((64 - P) * elt + 2 * P) + extra)


# additions and multiplications of an 8-point transform by even/odd parts, 16 of them to a block
_DCT_FLOPS = 16 * 36


def work(case):
    form = case["form"]
    if form == "batch":
        specs = _batch_specs(case)
        n = sum(h * w * c for h, w, c, _ in specs)
        return {"bytes": sum(_image_bytes(h * w * c, m, "fp32") for h, w, c, m in specs),
                "flops": 2 * n // 64 * _DCT_FLOPS}
    if form == "cipher":
        return {"bytes": 2 * case["bytes"], "flops": 0}
    if form in ("step", "tune"):
        n = case["B"] * case["H"] * case["W"]
        if form == "tune":  # the images once; the loop works on B x 65 sums
            return {"bytes": 4 * n, "flops": n // 64 * _DCT_FLOPS + case["steps"] * case["B"] * 64 * 10}
        # x in and P out; both in for the loss; both in and dL/dP out; x and dL/dP in for dL/dlogits
        return {"bytes": 4 * (2 + 2 + 3 + 2) * n, "flops": 4 * n // 64 * _DCT_FLOPS}
    n = case["H"] * case["W"] * case["C"]
    if form == "image":
        return {"bytes": _image_bytes(n, case["mask"], case["precision"]), "flops": 2 * n // 64 * _DCT_FLOPS}
    if form == "pixel":
        bits = sum((11 if z == 0 else case["bits"]) for z in range(64) if case["mask"] >> z & 1)
        return {"bytes": 2 * (2 * n + n // 64 * bits // 8), "flops": 2 * n // 64 * 64 * 2 * _private(case["mask"])}
    if form == "wavelet":
        return {"bytes": 2 * 3 * n, "flops": 0}
    return {"bytes": 2 * n + 2 * n // 64 * 4, "flops": 0}


# ------------------------------------------------------------------ in 64 bits
def _basis():
    """(64, 64) orthonormal 8x8 DCT-II basis, row 8u + v, column 8y + x, float64."""
    i = torch.arange(8, dtype=torch.float64, device=DEVICE)
    d = torch.cos((2 * i[None, :] + 1) * i[:, None] * math.pi / 16) * 0.5
    d[0] = math.sqrt(0.125)
    return torch.einsum("uy,vx->uvyx", d, d).reshape(64, 64)


def _zigzag():
    nat = []
    for d in range(15):
        us = [u for u in range(8) if 0 <= d - u < 8]
        nat += [8 * u + d - u for u in (us if d % 2 else us[::-1])]
    return nat


def _blocks(x):
    """(C, H, W) -> (blocks, 64) float64."""
    C, H, W = x.shape
    return x.view(C, H // 8, 8, W // 8, 8).permute(0, 1, 3, 2, 4).reshape(-1, 64).to(torch.float64)


def _public_exact(x, mask, halves):
    """The public fragment of (C, H, W) in the library's tile layout (halves: 32-block halves)."""
    nat = _zigzag()
    keep = [nat[z] for z in range(64) if not mask >> z & 1]
    c = _blocks(x) @ _basis()[keep].t().contiguous()
    nb, P = c.shape
    unit = 32 if halves else 64
    full = nb // 64 * 64
    parts = [c[:full].view(-1, unit, P).transpose(1, 2).reshape(-1)]
    parts += [c[i:min(i + unit, nb)].t().reshape(-1) for i in range(full, nb, unit)]
    return torch.cat(parts)


def _soft_exact(case, seed):
    x, logits = _soft_inputs(case, seed)
    return _blocks(x), logits.detach().to(torch.float64)


def _tune_exact(case, seed, lam=0.1, budget=6.0, lr=0.05):
    b, logits = _soft_exact(case, seed)
    B, N = case["B"], float(case["H"] * case["W"])
    E = ((b @ _basis().t()) ** 2).view(B, -1, 64).sum(1).cpu().numpy()
    sx = b.view(B, -1).sum(1).cpu().numpy()
    l = logits.cpu().numpy()
    xm, vx = sx / N, E.sum(1) / N - (sx / N) ** 2
    mom, vel, trace = np.zeros(64), np.zeros(64), []
    for t in range(case["steps"]):
        m = 1 / (1 + np.exp(-l))
        keep = 1 - m
        pm = keep[0] * xm
        cov, vp = E @ keep / N - xm * pm, E @ keep ** 2 / N - pm * pm
        rho = cov / np.sqrt(vx * vp)
        a, bb = 2 * rho / (B * N * np.sqrt(vx * vp)), -2 * rho ** 2 / (B * N * vp)
        dm = -(a @ E + (bb @ E) * keep)
        dm[0] += np.sum(a * N * xm * xm + bb * N * pm * xm)
        over = m.sum() - budget
        trace.append(np.mean(rho ** 2) + lam * over ** 2)
        g = m * keep * (dm + 2 * lam * over)
        mom, vel = 0.9 * mom + 0.1 * g, 0.999 * vel + 0.001 * g * g
        l = l - lr * (mom / (1 - 0.9 ** (t + 1))) / (np.sqrt(vel / (1 - 0.999 ** (t + 1))) + 1e-8)
    return {"logits": l, "trace": np.array(trace), "mask": None}


def _step_exact(case, seed, lam=0.1, budget=6.0):
    b, logits = _soft_exact(case, seed)
    B, H, W = case["B"], case["H"], case["W"]
    K = _basis()
    logits.requires_grad_(True)
    m = torch.sigmoid(logits)
    P = ((b @ K.t()) * (1 - m)) @ K
    x, p = b.view(B, -1), P.view(B, -1)
    dx, dp = x - x.mean(1, keepdim=True), p - p.mean(1, keepdim=True)
    rho2 = (dx * dp).mean(1) ** 2 / ((dx * dx).mean(1) * (dp * dp).mean(1))
    loss = rho2.mean() + lam * (m.sum() - budget) ** 2
    loss.backward()
    P = P.detach().view(B, H // 8, W // 8, 8, 8).permute(0, 1, 3, 2, 4).reshape(B, H, W)
    return {"public": P, "loss": loss.detach(), "grad": logits.grad}


def _entropy(counts):
    p = counts[counts > 0].to(torch.float64)
    p = p / p.sum()
    return float(-(p * torch.log2(p)).sum())


def _block_entropy(x):
    b = _blocks(x).to(torch.int64).sort(1).values
    # the length of the run that each sample lies in, from the places where runs begin
    first = torch.searchsorted(b, b, right=False)
    last = torch.searchsorted(b, b, right=True)
    return 6.0 - torch.log2((last - first).to(torch.float64)).sum(1) / 64.0


def _pearson(a, b):
    a, b = a.reshape(-1).to(torch.float64), b.reshape(-1).to(torch.float64)
    a, b = a - a.mean(), b - b.mean()
    return float((a * b).sum() / torch.sqrt((a * a).sum() * (b * b).sum()))


def _pairs(x):
    return [_pearson(x[:, :, :-1], x[:, :, 1:]), _pearson(x[:, :-1], x[:, 1:]), _pearson(x[:, :-1, :-1], x[:, 1:, 1:])]


def _stats_exact(case, seed):
    x, y = _stats_inputs(case, seed)
    n = x.numel()
    xi, yi = x.reshape(-1).to(torch.int64), y.reshape(-1).to(torch.int64)
    hx, hy = torch.bincount(xi, minlength=256), torch.bincount(yi, minlength=256)
    hxy = torch.bincount(256 * xi + yi, minlength=65536)
    Hx, Hy, Hxy = _entropy(hx), _entropy(hy), _entropy(hxy)
    e = n / 256.0
    chi2 = float(((hy.to(torch.float64) - e) ** 2 / e).sum())
    mi = Hx + Hy - Hxy
    table = torch.tensor([bin(i).count("1") for i in range(256)], device=DEVICE)
    bits = int(table[xi ^ yi].sum())
    sse = int(((xi - yi) ** 2).sum())
    bx, by = _block_entropy(x), _block_entropy(y)
    four = lambda h: [float(h.mean()), float(h.std(unbiased=False)), float(h.min()), float(h.max())]  # noqa: E731
    figures = [chi2, Hx, Hy, Hxy, mi, mi / math.sqrt(Hx * Hy)] + _pairs(x) + _pairs(y)
    figures += [_pearson(x, y), 100.0 * bits / (8.0 * n), 10 * math.log10(65025.0 * n / sse)] + four(bx) + four(by)
    return {"counts": None, "figures": torch.tensor(figures, dtype=torch.float64), "joint": None,
            "block_entropy": torch.cat([bx, by])}


def exact(case, seed):
    """What run() returns for these inputs in 64-bit arithmetic, from plain torch and numpy; None for
    bytes and integers, and for the forms that hold nothing else."""
    form = case["form"]
    if form == "image":
        rng, gen = _sources(seed)
        x = _image(case["H"], case["W"], case["C"], rng, gen)
        return {"public": _public_exact(x, case["mask"], case["precision"] != "fp32"), "private": None,
                "exceptions": None, "residual": None, "restored": None}
    if form == "batch":
        specs, offs, slab, _ = _batch_images(case, seed)
        po, pt = _slab_offsets([h * w * c // 64 * (64 - _private(m)) * 4 for h, w, c, m in specs])
        pub = torch.zeros(pt // 4, dtype=torch.float64, device=DEVICE)
        for (h, w, c, m), o, p in zip(specs, offs, po):
            v = _public_exact(slab[o:o + h * w * c].view(c, h, w), m, False)
            pub[p // 4:p // 4 + v.numel()] = v
        return {"public": pub, "private": None, "exceptions": None, "restored": None}
    if form == "stats":
        return _stats_exact(case, seed)
    if form == "step":
        return _step_exact(case, seed)
    if form == "tune":
        return _tune_exact(case, seed)
    return None
