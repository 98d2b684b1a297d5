"""Generic resident kernels (any size that fits LDS, any alignment) against the
oracle at the sizes where their layout changes: rows narrower than a vector,
planes sharing a wave (lines of at most 15 and 31), lines of 64/65, 112/113
(half a line and its halo in one wave) and 128/129 positions, rows whose last
vector overlaps, plane counts that leave a wave partly empty, absent
directions, groups, and tensors that are only element-aligned."""
import pytest
import torch

import oracle as O
from paper_2501_12381_amd import ops, synth
from .parity_util import TOL, np64, normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (planes, H, W, mask, group_h, group_w, logits)
CASES = [(5, 3, 3, 15, 0, 0, False), (9, 7, 7, 15, 0, 0, True), (6, 7, 4, 15, 3, 2, False),
         (5, 14, 14, 15, 0, 0, True), (4, 15, 15, 11, 4, 6, False), (3, 16, 15, 15, 0, 0, False),
         (3, 31, 30, 13, 0, 0, True), (2, 32, 33, 15, 9, 7, False), (2, 64, 60, 15, 0, 0, True),
         (2, 65, 64, 15, 0, 0, False), (2, 45, 77, 15, 23, 39, True), (1, 96, 96, 7, 0, 0, False),
         (1, 112, 113, 15, 0, 0, True), (2, 113, 112, 14, 40, 0, False), (1, 128, 129, 15, 0, 0, False),
         (1, 129, 136, 15, 17, 50, True), (1, 40, 240, 15, 0, 0, True), (1, 241, 40, 5, 0, 0, False),
         (1, 20, 250, 15, 0, 0, True), (1, 250, 36, 10, 0, 0, False), (2, 150, 66, 3, 0, 0, True),
         (2, 66, 150, 12, 0, 0, True), (1, 8, 256, 15, 0, 0, False), (1, 256, 8, 15, 100, 3, True),
         # rows of more than two vectors: vectors in a group change at 16 rows and at 2560 pixels
         (3, 16, 64, 15, 0, 0, False), (2, 17, 60, 15, 5, 0, True), (2, 40, 64, 15, 0, 0, True),
         (2, 41, 63, 15, 0, 20, False),
         # one axis or one direction: arrays and registers of those alone
         (2, 16, 70, 1, 0, 0, True), (2, 100, 60, 2, 9, 0, False), (2, 70, 16, 4, 0, 0, False),
         (2, 60, 100, 8, 0, 30, True), (3, 30, 50, 8, 0, 0, False), (2, 14, 130, 5, 0, 0, True),
         (3, 12, 200, 15, 5, 0, False), (5, 9, 11, 4, 0, 0, False)]


def misalign(t):
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    v = buf[1:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("shifted", [False, True], ids=["aligned", "shifted"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_generic_resident(case, dtype, shifted):
    planes, H, W, mask, gh, gw, logits = case
    print(f"[generic] {case} {dtype} shifted={shifted}", flush=True)
    n = bin(mask).count("1")
    inp = synth.random_general((1, planes, H, W), n, device=DEV, seed=H * 300 + W, dtype=dtype)
    if shifted:
        inp = {k: misalign(v) for k, v in inp.items()}
    opt = dict(group_h=gh, group_w=gw, logits=logits)
    y = ops.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], mask, **opt)
    got = ops.gspn_scan_bwd(inp["dy"], inp["x"], inp["w"], inp["lam"], inp["u"], mask, **opt)
    torch.cuda.synchronize()
    a = {k: np64(v) for k, v in inp.items()}
    ref = (O.scan_fwd(a["x"], a["w"], a["lam"], a["u"], mask, **opt),) + tuple(
        O.scan_bwd(a["dy"], a["x"], a["w"], a["lam"], a["u"], mask, **opt))
    for name, g, r in zip(("y", "dx", "dw", "dlam", "du"), (y,) + tuple(got), ref):
        e = normwise(g, r)
        assert torch.isfinite(g).all() and e <= TOL[dtype], f"{name}: {e:.3e}"
    # the additions have a fixed order: a second run agrees bit for bit
    again = (ops.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], mask, **opt),) + tuple(
        ops.gspn_scan_bwd(inp["dy"], inp["x"], inp["w"], inp["lam"], inp["u"], mask, **opt))
    for g, h in zip((y,) + tuple(got), again):
        assert torch.equal(g, h)


@pytest.mark.parametrize("pd", [(True, False, False), (False, True, True), (True, True, True), (False, False, True)],
                         ids=lambda p: "".join("LUY"[i] if f else "-" for i, f in enumerate(p)))
@pytest.mark.parametrize("shape", [(7, 5), (13, 30), (16, 60), (17, 60), (40, 100), (70, 90)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_generic_resident_per_direction(shape, pd):
    """Per-direction maps on the generic kernels (three directions, both dtypes)."""
    H, W = shape
    mask, n = 0xD, 3
    for dtype in (torch.float32, torch.bfloat16):
        base = synth.random_general((1, 3, H, W), n, device=DEV, seed=7, dtype=dtype)
        many = synth.random_general((n, 3, H, W), n, device=DEV, seed=8, dtype=dtype)
        pick = lambda k, f: many[k].view(n, 1, 3, H, W) if f else base[k]
        x, w = base["x"], base["w"]
        lam, u, dy = pick("lam", pd[0]), pick("u", pd[1]), pick("dy", pd[2])
        opt = dict(lam_per_dir=pd[0], u_per_dir=pd[1], y_per_dir=pd[2])
        y = ops.gspn_scan_fwd(x, w, lam, u, mask, **opt)
        got = ops.gspn_scan_bwd(dy, x, w, lam, u, mask, **opt)
        torch.cuda.synchronize()
        a = [np64(t) for t in (dy, x, w, lam, u)]
        ref = (O.scan_fwd(*a[1:], mask, **opt),) + tuple(O.scan_bwd(*a, mask, **opt))
        for name, g, r in zip(("y", "dx", "dw", "dlam", "du"), (y,) + tuple(got), ref):
            e = normwise(g, r)
            assert e <= TOL[dtype], f"{name}: {e:.3e}"


# one sum in LDS (x and lam read once per axis): two arrays would fit but the
# planes are more than the compute units, only one fits, a side over 240 beside
# one over 112, and sums that leave no room for the exchange buffers (lines
# kept whole)
ONE_SUM = [(258, 104, 102, 15, 0, 0, False), (2, 160, 160, 15, 0, 0, True), (1, 200, 193, 13, 90, 50, False),
           (1, 250, 150, 15, 0, 0, False), (1, 130, 256, 7, 0, 0, True), (1, 209, 194, 15, 0, 0, False),
           (2, 193, 209, 11, 100, 60, True)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", ONE_SUM, ids=lambda c: "x".join(map(str, c)))
def test_generic_forward_one_sum(case, dtype):
    planes, H, W, mask, gh, gw, logits = case
    print(f"[one sum] {case} {dtype}", flush=True)
    n = bin(mask).count("1")
    inp = synth.random_general((1, planes, H, W), n, device=DEV, seed=H * 300 + W, dtype=dtype)
    lams = torch.stack([inp["lam"] * (0.5 + 0.25 * d) for d in range(n)])
    opt = dict(group_h=gh, group_w=gw, logits=logits)
    for lam, pd in ((inp["lam"], False), (lams, True)):
        if pd and planes > 2:
            continue
        for shift in (False, True):
            args = [inp["x"], inp["w"], lam, inp["u"]]
            if shift:
                args = [misalign(t) for t in args]
            y = ops.gspn_scan_fwd(*args, mask, lam_per_dir=pd, **opt)
            torch.cuda.synchronize()
            if not shift:
                first = y
                e = normwise(y, O.scan_fwd(*[np64(t) for t in args], mask, lam_per_dir=pd, **opt))
                assert torch.isfinite(y).all() and e <= TOL[dtype], f"{e:.3e}"
            assert torch.equal(y, first)


# more planes than compute units on lines of two waves with rings of four and
# eight rows (an odd and an even count of row blocks): workgroups start warm and
# at different times, which a single plane never shows
MANY = [((300, 104, 152, 15, 0, 0, False), torch.float32), ((300, 136, 144, 15, 0, 0, True), torch.float32),
        ((300, 64, 240, 15, 23, 0, False), torch.float32), ((300, 40, 240, 15, 0, 0, True), torch.bfloat16)]


@pytest.mark.parametrize("case,dtype", MANY, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v)[6:])
def test_generic_resident_many_planes(case, dtype):
    planes, H, W, mask, gh, gw, logits = case
    print(f"[many planes] {case} {dtype}", flush=True)
    inp = synth.random_general((1, planes, H, W), 4, device=DEV, seed=H * 300 + W, dtype=dtype)
    args = [inp[k] for k in ("x", "w", "lam", "u")]
    opt = dict(group_h=gh, group_w=gw, logits=logits)
    run = lambda: (ops.gspn_scan_fwd(*args, mask, **opt),) + tuple(ops.gspn_scan_bwd(inp["dy"], *args, mask, **opt))
    first = run()
    torch.cuda.synchronize()
    a = [np64(t) for t in args]
    ref = (O.scan_fwd(*a, mask, **opt),) + tuple(O.scan_bwd(np64(inp["dy"]), *a, mask, **opt))
    for name, g, r in zip(("y", "dx", "dw", "dlam", "du"), first, ref):
        e = normwise(g, r)
        assert torch.isfinite(g).all() and e <= TOL[dtype], f"{name}: {e:.3e}"
    for _ in range(5):
        for name, g, h in zip(("y", "dx", "dw", "dlam", "du"), first, run()):
            assert torch.equal(g, h), name


def test_generic_resident_more_planes_than_one_launch():
    """67.2 million planes of one pixel: more than one launch's threads (2^32) cover."""
    n = 67_200_000
    x, lam, u, dy = (torch.rand((1, n, 1, 1), device=DEV) for _ in range(4))
    w = torch.zeros((1, 3, 1, n, 1, 1), device=DEV)
    for got, ref in zip((ops.gspn_scan_fwd(x, w, lam, u, 1),) + tuple(ops.gspn_scan_bwd(dy, x, w, lam, u, 1)),
                        (u * (lam * x), lam * (u * dy), w, x * (u * dy), dy * (lam * x))):
        assert torch.equal(got, ref)  # one product of two at a time, each rounded once


# both sides of the line between the per-wave and the generic backward of 56 x 56 and 64 x 64 planes
@pytest.mark.parametrize("planes,S,mask,dtype", [(255, 56, 15, torch.float32), (256, 56, 15, torch.float32),
                                                 (341, 64, 7, torch.float32), (342, 64, 7, torch.float32),
                                                 (600, 56, 3, torch.float32), (1030, 64, 4, torch.float32),
                                                 (511, 64, 15, torch.bfloat16), (512, 64, 15, torch.bfloat16)],
                         ids=str)
def test_backward_of_56_and_64(planes, S, mask, dtype):
    n = bin(mask).count("1")
    print(f"[56 and 64] {planes} {S} {mask} {dtype}", flush=True)
    inp = synth.random_general((1, planes, S, S), n, device=DEV, seed=planes, dtype=dtype)
    args = [inp[k] for k in ("dy", "x", "w", "lam", "u")]
    got = ops.gspn_scan_bwd(*args, mask, logits=True)
    torch.cuda.synchronize()
    for first in (0, planes - 2):  # the oracle takes the first and the last planes
        cut = [t.narrow(-3, first, 2) for t in args]
        ref = O.scan_bwd(*[np64(t) for t in cut], mask, logits=True)
        for name, g, r in zip(("dx", "dw", "dlam", "du"), got, ref):
            e = normwise(g.narrow(-3, first, 2), r)
            assert e <= TOL[dtype], f"{name}: {e:.3e}"


# unmerged outputs on both sides of the line between the quad kernel and the two-pass family
@pytest.mark.parametrize("planes,H,W,dtype,mask", [(256, 136, 128, torch.float32, 15), (257, 136, 128, torch.float32, 15),
                                                   (257, 136, 124, torch.float32, 13), (257, 160, 208, torch.bfloat16, 15),
                                                   (300, 129, 256, torch.bfloat16, 3), (300, 128, 256, torch.float32, 12),
                                                   (97, 136, 248, torch.bfloat16, 12), (100, 136, 244, torch.float32, 7)],
                         ids=str)
def test_unmerged_outputs_many_planes(planes, H, W, dtype, mask):
    n = bin(mask).count("1")
    print(f"[unmerged] {planes} {H} {W} {dtype} {mask}", flush=True)
    inp = synth.random_general((1, planes, H, W), n, device=DEV, seed=H + W, dtype=dtype)
    args = [inp[k] for k in ("x", "w", "lam", "u")]
    for shift in (False, True):
        y = ops.gspn_scan_fwd(*([misalign(t) for t in args] if shift else args), mask, y_per_dir=True)
        torch.cuda.synchronize()
        for first in (0, planes - 2):  # the oracle takes the first and the last planes
            ref = O.scan_fwd(*[np64(t.narrow(-3, first, 2)) for t in args], mask, y_per_dir=True)
            e = normwise(y.narrow(-3, first, 2), ref)
            assert e <= TOL[dtype], f"shifted {shift}: {e:.3e}"
