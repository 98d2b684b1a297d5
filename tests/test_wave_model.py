"""The generic resident kernels' own source, compiled for the host and run with
a workgroup's waves one after the other between two barriers, in several
orders (tests/wave_model).  What two waves leave unordered gives another result
in one of the orders; on the GPU the waves' timing can hide it.  Every order
has to give the same bits, and those the oracle's within the rounding of the
stored values."""
import ctypes
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle as O
from paper_2501_12381_amd import build as B, synth
from .parity_util import np64, normwise

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "wave_model")
F32, BF16 = torch.float32, torch.bfloat16
# fp32: the chain's rounding, as in the other parity tests; bf16: half a unit in
# the last place of the largest value on top of it
TOL = {F32: 1e-5, BF16: 2.0 ** -8 + 1e-5}
# waves in the order in which they run between barriers: either direction of a
# pair first, either half of a line first
ORDERS = [(0, 1, 2, 3), (3, 2, 1, 0), (2, 3, 0, 1), (1, 0, 3, 2)]


def clang():
    for c in ("/opt/rocm/llvm/bin/clang++", os.path.join(os.path.dirname(B.hipcc()), "amdclang++")):
        if os.path.exists(c):
            return c
    raise RuntimeError("no clang++ beside hipcc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    """{(dtype, logits): library}"""
    d = str(tmp_path_factory.mktemp("wave_model"))
    for f in os.listdir(B.CSRC):
        if f.endswith(".hpp"):
            text = open(os.path.join(B.CSRC, f)).read()
            text = text.replace("extern __shared__", "extern")
            text = text.replace('asm volatile("s_waitcnt lgkmcnt(0)\\n\\ts_barrier" ::: "memory");', "sim::barrier();")
            assert "s_barrier\"" not in text, f
            open(os.path.join(d, f), "w").write(text)

    def compile_one(key):
        out = os.path.join(d, f"model_{len(str(key[0]))}_{int(key[1])}.so")
        subprocess.run([clang(), "-x", "c++", "-std=c++17", "-O0", "-w", "-fPIC", "-shared",
                        f"-DMODEL_T={int(key[0] == BF16)}", f"-DMODEL_LG={'true' if key[1] else 'false'}",
                        "-I", HERE, "-I", d, os.path.join(HERE, "model.cpp"), "-o", out], check=True)
        return ctypes.CDLL(out)

    keys = [(t, lg) for t in (F32, BF16) for lg in (False, True)]
    with ThreadPoolExecutor(4) as ex:
        return dict(zip(keys, ex.map(compile_one, keys)))


def case_id(v):
    return "x".join(map(str, v)) if isinstance(v, tuple) else str(v)[6:]


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def inputs(case, dtype):
    planes, H, W, mask, gh, gw, logits = case
    n = bin(mask).count("1")
    inp = synth.random_general((1, planes, H, W), n, device="cpu", seed=H * 300 + W, dtype=dtype)
    return inp, {k: np64(v) for k, v in inp.items()}, dict(group_h=gh, group_w=gw, logits=logits)


def run_forward(model, case, dtype, inp, order):
    planes, H, W, mask, gh, gw, logits = case
    y = torch.full_like(inp["x"], float("nan"))
    st = model[dtype, logits].model_fwd(ptr(inp["x"]), ptr(inp["w"]), ptr(inp["lam"]), ptr(inp["u"]), ptr(y),
                                        ctypes.c_int64(planes), H, W, mask, gh, gw, 0, 0, (ctypes.c_int * 4)(*order))
    assert st == 0
    return y


def check_forward(model, case, dtype):
    inp, a, opt = inputs(case, dtype)
    ys = [run_forward(model, case, dtype, inp, o) for o in ORDERS]
    e = normwise(ys[0], O.scan_fwd(a["x"], a["w"], a["lam"], a["u"], case[3], **opt))
    assert torch.isfinite(ys[0]).all() and e <= TOL[dtype], f"{case}: {e:.3e}"
    for o, y in zip(ORDERS, ys):
        assert torch.equal(ys[0], y), f"{case}: the waves in the order {o} give another result"


# (planes, H, W, mask, group_h, group_w, logits): one, two and three blocks of
# eight rows, on lines that two waves share
@pytest.mark.parametrize("case,dtype", [((1, 8, 120, 15, 0, 0, False), F32), ((1, 16, 120, 15, 0, 0, True), F32),
                                        ((1, 24, 120, 3, 0, 0, False), F32), ((1, 19, 113, 15, 7, 40, True), F32),
                                        ((1, 24, 250, 15, 0, 0, False), F32), ((1, 24, 240, 15, 0, 0, True), BF16),
                                        ((1, 17, 200, 15, 0, 0, False), BF16), ((1, 24, 120, 14, 0, 0, False), F32)],
                         ids=case_id)
def test_merge_order(model, case, dtype):
    check_forward(model, case, dtype)


def check_backward(model, case, dtype, pair):
    planes, H, W, mask, gh, gw, logits = case
    inp, a, opt = inputs(case, dtype)
    runs = []
    for o in ORDERS:
        got = [torch.full_like(inp[k], float("nan")) for k in ("x", "w", "lam", "u")]
        sums = [torch.full(inp["x"].shape, float("nan")) for _ in range(2)]
        st = model[dtype, logits].model_bwd(*[ptr(inp[k]) for k in ("dy", "x", "w", "lam", "u")],
                                            *[ptr(t) for t in got + sums], ctypes.c_int64(planes), H, W, mask, gh,
                                            gw, int(pair), (ctypes.c_int * 4)(*o))
        assert st == 0
        runs.append(got)
    ref = O.scan_bwd(a["dy"], a["x"], a["w"], a["lam"], a["u"], mask, **opt)
    for i, name in enumerate(("dx", "dw", "dlam", "du")):
        e = normwise(runs[0][i], ref[i])
        assert torch.isfinite(runs[0][i]).all() and e <= TOL[dtype], f"{case}: {name}: {e:.3e}"
        for o, r in zip(ORDERS, runs):
            assert torch.equal(runs[0][i], r[i]), f"{case}: {name}: the waves in the order {o} give another result"


# rings of 4 to 16 rows on lines that two waves share; even and odd block counts
SHARED = [((1, 104, 152, 15, 0, 0, False), F32), ((1, 112, 144, 15, 0, 0, True), F32),
          ((1, 64, 240, 15, 17, 50, False), F32), ((1, 72, 66, 7, 0, 0, False), F32),
          ((1, 40, 240, 15, 0, 0, True), BF16), ((1, 48, 250, 13, 0, 0, False), BF16),
          ((1, 96, 168, 15, 0, 0, False), BF16), ((1, 130, 70, 15, 33, 0, True), BF16)]


@pytest.mark.parametrize("case,dtype", SHARED, ids=case_id)
def test_edge_exchange_forward(model, case, dtype):
    check_forward(model, case, dtype)


@pytest.mark.parametrize("case,dtype", SHARED, ids=case_id)
def test_edge_exchange_backward(model, case, dtype):
    check_backward(model, case, dtype, True)


@pytest.mark.parametrize("W,dtype", [(72, F32), (116, F32), (240, F32), (240, BF16)], ids=str)
def test_every_block_count(model, W, dtype):
    """1 to 20 blocks of rows at each ring depth (16, 8 and 4 rows; 8 for bf16)."""
    for nb in range(1, 21):
        H = 8 * nb - nb % 3
        if (H + 1) * (W + 2) * 4 <= 160 * 1024:
            check_forward(model, (1, H, W, 3, 0, 0, False), dtype)


@pytest.mark.parametrize("case,dtype", [((5, 14, 14, 15, 0, 0, True), BF16), ((3, 20, 31, 15, 6, 9, False), F32),
                                        ((2, 45, 33, 11, 0, 0, False), BF16), ((1, 64, 60, 15, 0, 0, True), F32),
                                        ((1, 41, 63, 15, 0, 0, False), F32), ((2, 16, 60, 8, 0, 9, True), BF16),
                                        ((2, 10, 60, 1, 4, 0, False), F32), ((3, 30, 50, 4, 0, 0, False), BF16)],
                         ids=case_id)
def test_one_wave_a_direction(model, case, dtype):
    """The quad kernels: the directions of an axis meet at the merge only."""
    check_forward(model, case, dtype)
    check_backward(model, case, dtype, False)


# (forward or backward, H, W, planes a workgroup, launches for 40 million planes)
@pytest.mark.parametrize("which,H,W,ppw,n", [(0, 1, 1, 4, 1), (0, 16, 2, 2, 2), (0, 33, 1, 1, 3), (0, 1, 66, 1, 3),
                                             (1, 3, 5, 4, 1), (1, 2, 20, 2, 2), (1, 40, 1, 1, 3)])
def test_more_planes_than_one_launch(model, which, H, W, ppw, n):
    """A launch's threads are counted in 32 bits; every plane gets a workgroup all the same."""
    planes, groups = 40_000_001, ctypes.c_int64()
    got = model[F32, False].model_launches(which, ctypes.c_int64(planes), H, W, ctypes.byref(groups))
    assert (got, groups.value) == (n, -(-planes // ppw))
