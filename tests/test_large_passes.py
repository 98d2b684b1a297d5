"""Two-pass family at the sizes where its passes change shape, against the
oracle: rows at the edges of the vertical waves (64 lanes of 4 columns, 8-column
halos, 16 waves, then 8 columns a lane), column bands of the vertical scan
(few planes, wide rows) at the edges of their 128-row launches and in groups,
and the wide and narrow bands of the horizontal pass."""
import pytest
import torch

import oracle as O
from paper_2501_12381_amd import lib as L, ops, synth
from .parity_util import TOL, np64, normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (planes, H, W, mask, group_h, group_w, logits)
CASES = [(2, 9, 256, 15, 0, 0, False), (1, 8, 264, 15, 3, 0, True), (1, 7, 480, 3, 0, 0, False),
         (2, 17, 488, 6, 0, 0, True), (1, 33, 976, 15, 0, 0, False), (1, 16, 984, 15, 0, 100, True),
         # column bands: one row, all but one of a launch's rows, all of them, one more; several launches
         (1, 1, 1024, 15, 0, 0, False), (1, 127, 1024, 15, 0, 0, True), (2, 128, 1288, 15, 50, 0, False),
         (1, 129, 1288, 15, 128, 0, True), (1, 257, 1024, 13, 0, 0, False), (1, 136, 2048, 14, 129, 7, True),
         # many planes: one workgroup a plane and direction
         (44, 40, 1000, 15, 0, 0, False), (70, 9, 1024, 7, 4, 0, True),
         # horizontal bands: one, two and more narrow ones, and wide ones
         (1, 256, 64, 15, 0, 0, False), (2, 257, 72, 15, 0, 0, True), (1, 600, 64, 12, 0, 30, False),
         (100, 512, 64, 15, 0, 0, False)]
BF16 = [(1, 9, 2056, 15, 0, 0, True), (1, 20, 3840, 15, 0, 0, False), (2, 9, 3848, 15, 5, 0, False),
        (1, 140, 4096, 15, 0, 0, True), (30, 9, 3848, 7, 0, 0, False)]


@pytest.mark.parametrize("case,dtype", [(c, d) for c in CASES for d in (torch.float32, torch.bfloat16)]
                         + [(c, torch.bfloat16) for c in BF16],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v)[6:])
def test_two_pass_edges(case, dtype):
    planes, H, W, mask, gh, gw, logits = case
    print(f"[two-pass] {case} {dtype}", flush=True)
    n = bin(mask).count("1")
    inp = synth.random_general((1, planes, H, W), n, device=DEV, seed=H * 300 + W, dtype=dtype)
    opt = dict(group_h=gh, group_w=gw, logits=logits)
    args = [inp[k] for k in ("x", "w", "lam", "u")]
    a = [np64(t) for t in args]
    y = ops.gspn_scan_fwd(*args, mask, algo=L.GSPN_ALGO_TWO_PASS, **opt)
    torch.cuda.synchronize()
    e = normwise(y, O.scan_fwd(*a, mask, **opt))
    assert torch.isfinite(y).all() and e <= TOL[dtype], f"y: {e:.3e}"
    assert torch.equal(y, ops.gspn_scan_fwd(*args, mask, algo=L.GSPN_ALGO_TWO_PASS, **opt))
    if not mask & 12:
        return  # the two-pass backward needs a horizontal direction
    got = ops.gspn_scan_bwd(inp["dy"], *args, mask, algo=L.GSPN_ALGO_TWO_PASS, **opt)
    torch.cuda.synchronize()
    for name, g, r in zip(("dx", "dw", "dlam", "du"), got, O.scan_bwd(np64(inp["dy"]), *a, mask, **opt)):
        e = normwise(g, r)
        assert torch.isfinite(g).all() and e <= TOL[dtype], f"{name}: {e:.3e}"


def test_column_bands_equal_one_workgroup():
    """The bands form every sum in the order of the one-workgroup pass: a plane
    alone (bands) and among many (one workgroup each) gets the same bits."""
    for dtype in (torch.float32, torch.bfloat16):
        inp = synth.random_general((1, 70, 150, 1024), 4, device=DEV, seed=5, dtype=dtype)
        y = ops.gspn_scan_fwd(inp["x"], inp["w"], inp["lam"], inp["u"], 15, algo=L.GSPN_ALGO_TWO_PASS, logits=True)
        one = [inp[k][:, 3:4].contiguous() for k in ("x", "lam", "u")]
        w = inp["w"][:, :, :, 3:4].contiguous()
        y1 = ops.gspn_scan_fwd(one[0], w, one[1], one[2], 15, algo=L.GSPN_ALGO_TWO_PASS, logits=True)
        assert torch.equal(y[:, 3:4], y1)
