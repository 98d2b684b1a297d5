"""Performance cases of the GSPN line scan: what a program that uses this package has it do.

The scan is called in three settings, and the cases cover each over its range:

* classification stages (feature maps of 7 to 72 pixels a side, hundreds to
  thousands of planes): training steps (forward and backward through autograd)
  and inference, plain weights and Eq. 6 logits, global and local (grouped)
  scans, square maps and ragged ones;
* diffusion latents (64 to 256 a side, square and with the aspect ratios of
  generated images) in inference and fine-tuning;
* high-resolution latents and single layers (512 to 2048 a side), where the
  plane no longer fits a compute unit: hundreds of planes for the latent of a
  16384 x 8192 image, a few dozen in training, one when a layer's speed is
  plotted over the image size.

`run` makes the calls such a program makes: `ops.gspn_scan_fwd` for inference,
`ops.gspn_scan` and autograd for a training step (which returns the output and
every gradient), and the module with its projections and learnable merger.
"""
from __future__ import annotations

import math

import torch

from paper_2501_12381_amd import ops
from paper_2501_12381_amd.module import GSPNModule

T2B, B2T, L2R, R2L = 1, 2, 4, 8
_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _scan(B, C, H, W, dtype, train=False, mask=15, logits=False, group_h=0, group_w=0, keep=False):
    return {"kind": "scan", "B": B, "C": C, "H": H, "W": W, "dtype": dtype, "train": train, "mask": mask,
            "logits": logits, "group_h": group_h, "group_w": group_w, "keep": keep}


def _module(B, dim, hidden, H, W):
    return {"kind": "module", "B": B, "C": hidden, "dim": dim, "H": H, "W": W, "dtype": "bf16", "train": True,
            "mask": 15, "logits": True, "group_h": 0, "group_w": 0, "keep": False}


def listed():
    return [
        # the smallest call: one direction over 8 planes of 16 x 16, where only latency counts
        {"name": "tiny16_f32_infer", **_scan(1, 8, 16, 16, "f32", mask=T2B)},
        # training step of a classifier's 14 x 14 stage (224-pixel input at stride 16), Eq. 6 logits
        {"name": "stage14_bf16_train", **_scan(32, 384, 14, 14, "bf16", train=True, logits=True)},
        # training step of the 28 x 28 stage, weights normalised by the caller
        {"name": "stage28_bf16_train", **_scan(32, 192, 28, 28, "bf16", train=True)},
        # fp32 training with local GSPN on a ragged map (an input whose sides are no multiple of the stride)
        {"name": "ragged45x77_f32_local_train",
         **_scan(4, 96, 45, 77, "f32", train=True, logits=True, group_h=23, group_w=39)},
        # latent of a 1024 x 1024 image: one denoising layer
        {"name": "lat128_bf16_infer", **_scan(2, 640, 128, 128, "bf16")},
        # the same latent in fine-tuning, Eq. 6 logits
        {"name": "lat128_bf16_train", **_scan(2, 640, 128, 128, "bf16", train=True, logits=True)},
        # latent of a wide 1344 x 768 image: one denoising layer
        {"name": "lat96x168_bf16_infer", **_scan(2, 640, 96, 168, "bf16")},
        # latent of a 1216 x 832 image in fine-tuning
        {"name": "lat104x152_bf16_train", **_scan(1, 640, 104, 152, "bf16", train=True)},
        # the whole module (projections, scan with unmerged outputs, merger) in training on a 64 x 64 map
        {"name": "module64_bf16_train", **_module(4, 320, 64, 64, 64)},
        # one channel on a large map: a single layer's latency over the image size
        {"name": "layer2048_bf16_infer", **_scan(1, 1, 2048, 2048, "bf16", logits=True)},
        # latent of a 16384 x 8192 image, all 320 channels
        {"name": "hires1024x2048_bf16_infer", **_scan(1, 320, 1024, 2048, "bf16")},
        # training step on large maps, the forward's states kept for the backward
        {"name": "hires1024_bf16_train", **_scan(1, 64, 1024, 1024, "bf16", train=True, logits=True, keep=True)},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: stages, latents, large maps, and now and then a module."""
    r = rng.random()
    dtype = "bf16" if rng.random() < 0.65 else "f32"
    train = rng.random() < 0.55
    logits = rng.random() < 0.5
    mask = 15 if rng.random() < 0.8 else rng.choice([T2B, L2R, T2B | B2T, L2R | R2L, T2B | L2R, 15 ^ R2L])
    if r < 0.08:  # module in training
        side = _log_uniform(rng, 14, 64)
        return _module(rng.randint(1, 4), 64 * rng.randint(1, 5), 16 * rng.randint(1, 4), side,
                       side if rng.random() < 0.6 else _log_uniform(rng, 14, 64))
    if r < 0.55:  # classification stage
        h = _log_uniform(rng, 7, 72)
        w = h if rng.random() < 0.6 else _log_uniform(rng, 7, 72)
        B, C = _log_uniform(rng, 1, 32), _log_uniform(rng, 32, 512)
        while B * C * h * w > 6_000_000:
            B, C = max(1, B // 2), max(16, C * 3 // 4)
        local = rng.random() < 0.3
        return _scan(B, C, h, w, dtype, train, mask, logits, rng.randint(2, h) if local else 0,
                     rng.randint(2, w) if local else 0)
    if r < 0.85:  # diffusion latent
        step = 8 if rng.random() < 0.75 else 1
        h, w = (step * max(1, _log_uniform(rng, 64, 256) // step) for _ in range(2))
        B, C = rng.randint(1, 2), _log_uniform(rng, 64, 640)
        while B * C * h * w > 20_000_000:
            B, C = 1, max(16, C * 3 // 4)
        return _scan(B, C, h, w, dtype, train, mask, logits)
    h, w = (8 * (_log_uniform(rng, 512, 2048) // 8) for _ in range(2))
    C = _log_uniform(rng, 1, 64)
    while C * h * w > 64_000_000:
        C = max(1, C * 3 // 4)
    return _scan(1, C, h, w, dtype, train, 15, logits, keep=train)


def _n(case):
    return bin(case["mask"]).count("1")


def _gen(seed, tid):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + tid * 7919 + 12345) & 0x7FFF_FFFF_FFFF)
    return g


def _randn(shape, seed, tid):
    return torch.randn(shape, generator=_gen(seed, tid), device="cuda")


def prepare(case, seed):
    dt = _DTYPES[case["dtype"]]
    B, C, H, W, n = case["B"], case["C"], case["H"], case["W"], _n(case)
    if case["kind"] == "module":
        with torch.random.fork_rng(devices=["cuda"]):
            torch.manual_seed(int(seed) & 0x7FFF_FFFF)
            m = GSPNModule(case["dim"], C, case["mask"]).to(device="cuda", dtype=dt)
        inp = _randn((B, case["dim"], H, W), seed, 0).to(dt).requires_grad_(True)
        return {"case": case, "module": m, "inp": inp, "dout": _randn((B, case["dim"], H, W), seed, 1).to(dt)}
    shape = (B, C, H, W)
    s = {"case": case, "x": _randn(shape, seed, 0).to(dt), "lam": torch.sigmoid(_randn(shape, seed, 1)).to(dt),
         "u": torch.sigmoid(_randn(shape, seed, 2)).to(dt)}
    w = torch.empty((n, 3) + shape, device="cuda", dtype=dt)
    for i in range(n):  # one direction at a time keeps the fp32 temporaries small
        lg = _randn((3,) + shape, seed, 4 + i)
        w[i].copy_(lg if case["logits"] else torch.softmax(lg, dim=0))
        del lg
    s["w"] = w
    if case["train"]:
        s["dy"] = _randn(shape, seed, 3).to(dt)
        for k in ("x", "w", "lam", "u"):
            s[k].requires_grad_(True)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "module":
        m = s["module"]
        out = m(s["inp"])
        names, params = zip(*m.named_parameters())
        grads = torch.autograd.grad(out, (s["inp"],) + params, s["dout"])
        return {"out": out, "inp": grads[0], **{"grad_" + k.replace(".", "_"): g for k, g in zip(names, grads[1:])}}
    opt = {"group_h": c["group_h"], "group_w": c["group_w"], "logits": c["logits"]}
    if not c["train"]:
        return ops.gspn_scan_fwd(s["x"], s["w"], s["lam"], s["u"], c["mask"], **opt)
    y = ops.gspn_scan(s["x"], s["w"], s["lam"], s["u"], c["mask"], save_state=c["keep"], **opt)
    dx, dw, dlam, du = torch.autograd.grad(y, (s["x"], s["w"], s["lam"], s["u"]), s["dy"])
    return {"y": y, "dx": dx, "dw": dw, "dlam": dlam, "du": du}


def work(case):
    n, es = _n(case), _DTYPES[case["dtype"]].itemsize
    pix = case["B"] * case["C"] * case["H"] * case["W"]
    # x, lam, u and three weights a direction in, y out; training: dy in and the gradients out as well
    maps = 4 + 3 * n + ((4 + 3 * n) if case["train"] else 0)
    # a direction's step: three multiply-adds and the merge; its adjoint: three products, their sum, three dw
    flops = pix * (7 * n + 2 + ((10 * n + 5) if case["train"] else 0))
    if case["kind"] == "module":
        hw, hid, dim = case["B"] * case["H"] * case["W"], case["C"], case["dim"]
        weights = dim * hid + hid * hid * (2 + 3 * n) + n * hid * dim
        # what cannot stay on chip: the module's input and output with their gradients, and the parameters with theirs
        return {"bytes": es * (4 * hw * dim + 2 * weights), "flops": flops + 6 * hw * weights}
    return {"bytes": es * pix * maps, "flops": flops}


def tolerance(case):
    # measured against `exact`: bf16 results carry the rounding of the stored value (relative 2-norm 1.7e-3,
    # at most half a unit in the last place); fp32 ones the rounding of the chain of line steps
    if case["kind"] == "module":
        return {"rel": 0.03, "max": 0.5}
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 0.03}
    return {"rel": 2e-6, "max": 1e-4}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _lines(t, vertical):
    """(..., N, H, W) -> (..., lines, N, positions)."""
    return t.movedim(-2, -3) if vertical else t.movedim(-1, -3)


def _starts(i, n, group, reverse):
    if not group or group >= n:
        return i == (n - 1 if reverse else 0)
    return (i == n - 1 or (i + 1) % group == 0) if reverse else i % group == 0


def _direction(lx, w3, vertical, reverse, group):
    """h of one direction.  lx: (N, H, W) float64; w3: (3, N, H, W), any float type."""
    b, w = _lines(lx, vertical), _lines(w3, vertical)
    L, N, P = b.shape
    h = torch.empty((L, N, P), device=lx.device, dtype=torch.float64)
    prev = torch.zeros((N, P + 2), device=lx.device, dtype=torch.float64)
    for i in (range(L - 1, -1, -1) if reverse else range(L)):
        if _starts(i, L, group, reverse):
            prev.zero_()
        wl = w[:, i].double()
        new = wl[0] * prev[:, :-2] + wl[1] * prev[:, 1:-1] + wl[2] * prev[:, 2:] + b[i]
        h[i] = new
        prev[:, 1:-1] = new
    return h.movedim(0, 1) if vertical else h.permute(1, 2, 0)


def _adjoint(src, w3, h, vertical, reverse, group):
    """g and dw of one direction; src = u dy, (N, H, W) float64."""
    b, w, hl = _lines(src, vertical), _lines(w3, vertical), _lines(h, vertical)
    L, N, P = b.shape
    dev = src.device
    g = torch.empty((L, N, P), device=dev, dtype=torch.float64)
    dw = torch.empty((3, L, N, P), device=dev, dtype=torch.float64)
    a = torch.zeros((3, N, P + 2), device=dev, dtype=torch.float64)
    pad = torch.zeros((N, P + 2), device=dev, dtype=torch.float64)
    for i in (range(L) if reverse else range(L - 1, -1, -1)):
        after, before = (i - 1, i + 1) if reverse else (i + 1, i - 1)
        new = b[i]
        if 0 <= after < L and not _starts(after, L, group, reverse):
            new = new + a[0][:, 2:] + a[1][:, 1:-1] + a[2][:, :-2]
        g[i] = new
        a[:, :, 1:-1] = w[:, i].double() * new
        if _starts(i, L, group, reverse):
            dw[:, i] = 0
        else:
            pad[:, 1:-1] = hl[before]
            for k in range(3):
                dw[k, i] = new * pad[:, k:k + P]
    if vertical:
        return g.movedim(0, 1), dw.movedim(1, 2)
    return g.permute(1, 2, 0), dw.permute(0, 2, 3, 1)


def _normalised(lg):
    s = torch.sigmoid(lg.double())
    return s / s.sum(dim=0, keepdim=True)


def _logit_grad(lg, dw):
    s = torch.sigmoid(lg.double())
    S = s.sum(dim=0, keepdim=True)
    inner = (s / S * dw).sum(dim=0, keepdim=True)
    return s * (1 - s) * (dw - inner) / S


def _exact_scan(x, w, lam, u, case, dys=None):
    """y_d of every direction, or with dys (the output gradients of the directions) the gradients too."""
    B, C, H, W = x.shape
    N = B * C
    flat = lambda t: t.reshape(t.shape[:-4] + (N, H, W))  # noqa: E731
    x, lam, u, w = (flat(t.detach()) for t in (x, lam, u, w))
    lx, ud = lam.double() * x.double(), u.double()
    ys, gsum, du, dws = [], torch.zeros_like(lx), torch.zeros_like(lx), []
    for i, d in enumerate([d for d in (T2B, B2T, L2R, R2L) if case["mask"] & d]):
        vertical, reverse = d in (T2B, B2T), d in (B2T, R2L)
        group = case["group_h"] if vertical else case["group_w"]
        w3 = _normalised(w[i]) if case["logits"] else w[i]
        h = _direction(lx, w3, vertical, reverse, group)
        ys.append(ud * h)
        if dys is not None:
            dy = flat(dys[i].detach()).double()
            g, dw = _adjoint(ud * dy, w3, h, vertical, reverse, group)
            gsum += g
            du += dy * h
            dws.append((_logit_grad(w[i], dw) if case["logits"] else dw).reshape(3, B, C, H, W))
        del h, w3
    back = lambda t: t.reshape(B, C, H, W)  # noqa: E731
    ys = [back(y) for y in ys]
    if dys is None:
        return ys
    return ys, back(lam.double() * gsum), torch.stack(dws), back(x.double() * gsum), back(du)


class _ExactModuleScan(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, w, lam, u, case):
        ctx.save_for_backward(x, w, lam, u)
        ctx.case = case
        return torch.stack(_exact_scan(x, w, lam, u, case))

    @staticmethod
    def backward(ctx, dys):
        _, dx, dw, dlam, du = _exact_scan(*ctx.saved_tensors, ctx.case, dys)
        return dx, dw, dlam, du, None


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "module":
        p = {k: v.detach().double().requires_grad_(True) for k, v in s["module"].named_parameters()}
        inp = s["inp"].detach().double().requires_grad_(True)
        B, dim, H, W = inp.shape
        n, C = _n(case), case["C"]

        def conv(t, name):
            y = p[name + ".weight"].flatten(1) @ t.flatten(2)
            return (y + p[name + ".bias"][:, None]).unflatten(2, (H, W))

        x = conv(inp, "reduce")
        w = conv(x, "proj_w").view(B, n, 3, C, H, W).permute(1, 2, 0, 3, 4, 5)
        ys = _ExactModuleScan.apply(x, w, conv(x, "proj_lam"), conv(x, "proj_u"), case)
        out = conv(ys.permute(1, 0, 2, 3, 4).reshape(B, n * C, H, W), "merge")
        grads = torch.autograd.grad(out, [inp] + list(p.values()), s["dout"].double())
        return {"out": out, "inp": grads[0],
                **{"grad_" + k.replace(".", "_"): g for k, g in zip(p, grads[1:])}}
    if not case["train"]:
        ys = _exact_scan(s["x"], s["w"], s["lam"], s["u"], case)
        total = ys[0]
        for y in ys[1:]:
            total = total + y
        return total
    ys, dx, dw, dlam, du = _exact_scan(s["x"], s["w"], s["lam"], s["u"], case, [s["dy"]] * _n(case))
    return {"y": sum(ys[1:], ys[0]), "dx": dx, "dw": dw, "dlam": dlam, "du": du}
