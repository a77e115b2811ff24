"""GPU parity: libhexconv (through its C ABI) against the fp64 oracle on the
same seeded inputs.

Tolerances: float32 rel-L2 <= 1e-5 per output tensor; bfloat16
|err| <= 1e-2 * (sum of |terms|) per element; max pooling and argmax taps
bit-exact; average pooling within one bf16 ulp of the rounded fp64 value.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1903_01814_amd import hexconv as hx
from paper_1903_01814_amd import inputs as gen

from gpu_helpers import (bf16_ulp, check, check_bf16, check_f32, empty,
                         from_dev, oracle_fwd_at, round_bf16_f64,
                         sample_indices, to_dev, torch_mod)

pytestmark = pytest.mark.gpu

CFG = gen.CONFIGS


def _sync():
    torch_mod().cuda.synchronize()


def _conv_inputs(cfg, N=None, seed=0):
    T = oracle.num_taps(cfg["k"])
    return gen.conv_inputs(cfg, T, oracle.out_shape(cfg["H"], cfg["W"],
                                                    cfg["stride"]),
                           seed=seed, N=N)


def run_fwd(x, w, b, k, s, dt, relu=False):
    torch = torch_mod()
    N, Ci, H, W = x.shape
    Ho, Wo = hx.hex_out_shape(H, W, k, s)
    xd, wd = to_dev(x, dt), to_dev(w, dt)
    bd = None if b is None else to_dev(b, dt)
    y = empty((N, w.shape[0], Ho, Wo), dt)
    hx.hexconv_fwd(xd, wd, bd, y, k, s, relu=relu)
    _sync()
    return from_dev(y)


def run_bwd_data(dy, w, k, s, H, W, dt):
    N = dy.shape[0]
    dx = empty((N, w.shape[1], H, W), dt)
    hx.hexconv_bwd_data(to_dev(dy, dt), to_dev(w, dt), dx, k, s)
    _sync()
    return from_dev(dx)


def run_bwd_weight(x, dy, k, s, dt, with_db=True):
    torch = torch_mod()
    N, Ci, H, W = x.shape
    Co = dy.shape[1]
    T = hx.hex_num_taps(k)
    dw = torch.full((Co, Ci, T), float("nan"), dtype=torch.float32, device="cuda:0")
    db = torch.full((Co,), float("nan"), dtype=torch.float32,
                    device="cuda:0") if with_db else None
    nbytes = hx.hexconv_bwd_weight_workspace(N, Ci, Co, H, W, k, s,
                                             hx.HEX_F32 if dt == "f32" else hx.HEX_BF16)
    ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda:0") if nbytes else None
    hx.hexconv_bwd_weight(to_dev(x, dt), to_dev(dy, dt), dw, db, ws, k, s)
    _sync()
    return from_dev(dw), (from_dev(db) if with_db else None)


def run_bwd(x, dy, w, k, s, dt, want_dx=True):
    """Both gradients through the combined entry point hexconv_bwd."""
    torch = torch_mod()
    N, Ci, H, W = x.shape
    Co = dy.shape[1]
    T = hx.hex_num_taps(k)
    dx = empty((N, Ci, H, W), dt) if want_dx else None
    if dx is not None:
        dx.fill_(float("nan"))
    dw = torch.full((Co, Ci, T), float("nan"), dtype=torch.float32, device="cuda:0")
    db = torch.full((Co,), float("nan"), dtype=torch.float32, device="cuda:0")
    nbytes = hx.hexconv_bwd_workspace(N, Ci, Co, H, W, k, s,
                                      hx.HEX_F32 if dt == "f32" else hx.HEX_BF16)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0") if nbytes else None
    wd = None if w is None else to_dev(w, dt)
    hx.hexconv_bwd(to_dev(x, dt), to_dev(dy, dt), wd, dx, dw, db, ws, k, s)
    _sync()
    return (from_dev(dx) if want_dx else None), from_dev(dw), from_dev(db)


def run_pool_fwd(x, k, s, mode, dt, want_argmax=True):
    torch = torch_mod()
    N, C, H, W = x.shape
    Ho, Wo = hx.hex_out_shape(H, W, k, s)
    y = empty((N, C, Ho, Wo), dt)
    am = torch.full((N, C, Ho, Wo), 255, dtype=torch.uint8,
                    device="cuda:0") if want_argmax else None
    hx.hexpool_fwd(to_dev(x, dt), y, am, k, s, mode)
    _sync()
    return from_dev(y), (am.cpu().numpy().astype(np.int32) if want_argmax else None)


def run_pool_bwd(dy, am, relu_y, k, s, mode, H, W, dt):
    torch = torch_mod()
    N, C = dy.shape[:2]
    dx = empty((N, C, H, W), dt)
    amd = None if am is None else torch.from_numpy(
        np.ascontiguousarray(am, np.uint8)).to("cuda:0")
    ry = None if relu_y is None else to_dev(relu_y, dt)
    hx.hexpool_bwd(to_dev(dy, dt), amd, ry, dx, k, s, mode)
    _sync()
    return from_dev(dx)


def check_fwd_full(x, w, b, k, s, dt, relu=False, what="fwd"):
    y = run_fwd(x, w, b, k, s, dt, relu)
    ref = oracle.conv_fwd(x, w, b, k, s)
    mag = oracle.conv_fwd(np.abs(x), np.abs(w), None if b is None else np.abs(b), k, s)
    if relu:
        ref = np.maximum(ref, 0.0)
    return check(dt, y, ref, mag, what)


def check_bwd_full(x, w, dy, k, s, dt, what="bwd"):
    N, Ci, H, W = x.shape
    dx = run_bwd_data(dy, w, k, s, H, W, dt)
    ref = oracle.conv_bwd_data(dy, w, k, s, H, W)
    mag = oracle.conv_bwd_data(np.abs(dy), np.abs(w), k, s, H, W)
    check(dt, dx, ref, mag, what + " dx")
    dw, db = run_bwd_weight(x, dy, k, s, dt)
    rw, rb = oracle.conv_bwd_weight(x, dy, k, s)
    mw, mb = oracle.conv_bwd_weight(np.abs(x), np.abs(dy), k, s)
    # dw / db are float32 outputs; bf16 operands -> magnitude metric
    check(dt, dw, rw, mw, what + " dw")
    check(dt, db, rb, mb, what + " db")
    # the combined entry point gives the same results (to the tolerance)
    dx2, dw2, db2 = run_bwd(x, dy, w, k, s, dt)
    check(dt, dx2, ref, mag, what + " bwd dx")
    check(dt, dw2, rw, mw, what + " bwd dw")
    check(dt, db2, rb, mb, what + " bwd db")


# ------------------------------------------------------------ workloads

def test_c1_tiny_fwd_fp32():
    cfg = CFG["c1"]
    d = _conv_inputs(cfg)
    check_fwd_full(d["x"], d["w"], d["b"], cfg["k"], cfg["stride"], "f32",
                   what="c1 fwd")


def test_c2_camera_fwd_bwd_fp32():
    cfg = CFG["c2"]
    d = _conv_inputs(cfg)
    check_fwd_full(d["x"], d["w"], d["b"], cfg["k"], 1, "f32", what="c2 fwd")
    check_bwd_full(d["x"], d["w"], d["dy"], cfg["k"], 1, "f32", what="c2")


@pytest.mark.parametrize("mode", [hx.HEX_POOL_MAX, hx.HEX_POOL_AVG])
def test_c3_pool_bf16(mode):
    cfg = CFG["c3"]
    x = gen.pool_inputs(cfg)["x"]
    y, am = run_pool_fwd(x, cfg["k"], cfg["stride"], mode, "bf16")
    ref, ram = oracle.pool_fwd(x, cfg["k"], cfg["stride"], mode)
    if mode == hx.HEX_POOL_MAX:
        np.testing.assert_array_equal(y, ref)           # bit-exact
        np.testing.assert_array_equal(am, ram)
    else:
        want = round_bf16_f64(ref)
        assert np.all(np.abs(y - want) <= bf16_ulp(want))


def test_c4_wide_fwd_bwd_bf16_full():
    """Config 4 at full size (64 images, 64 -> 64 channels, 128 x 128, bf16):
    every element of y, dx, dw and db against the oracle."""
    cfg = CFG["c4"]
    d = _conv_inputs(cfg)
    x, w, b, dy = d["x"], d["w"], d["b"], d["dy"]
    k, s = cfg["k"], cfg["stride"]
    H, W = x.shape[2:]
    y = run_fwd(x, w, b, k, s, "bf16")
    check_bf16(y, oracle.conv_fwd(x, w, b, k, s),
               oracle.conv_fwd(np.abs(x), np.abs(w), np.abs(b), k, s), "c4 fwd")
    del y
    dx = run_bwd_data(dy, w, k, s, H, W, "bf16")
    check_bf16(dx, oracle.conv_bwd_data(dy, w, k, s, H, W),
               oracle.conv_bwd_data(np.abs(dy), np.abs(w), k, s, H, W), "c4 dx")
    del dx
    dw, db = run_bwd_weight(x, dy, k, s, "bf16")
    rw, rb = oracle.conv_bwd_weight(x, dy, k, s)
    mw, mb = oracle.conv_bwd_weight(np.abs(x), np.abs(dy), k, s)
    check_bf16(dw, rw, mw, "c4 dw")
    check_bf16(db, rb, mb, "c4 db")
    # the fixed-order slot reduction gives the same bits on a second run
    dw2, db2 = run_bwd_weight(x, dy, k, s, "bf16")
    np.testing.assert_array_equal(dw, dw2)
    np.testing.assert_array_equal(db, db2)


def test_c5_stack_teacher_forced():
    """Config 5 layer by layer, every element: each GPU op gets the GPU's own
    bf16 inputs and the oracle recomputes that op from the same bits; max
    pooling and its argmax bit-exact."""
    torch = torch_mod()
    cfg = CFG["c5"]
    H, W = cfg["H"], cfg["W"]
    for layer in cfg["layers"]:
        k, s = (layer[3], layer[4]) if layer[0] == "conv" else (layer[2], layer[3])
        H, W = hx.hex_out_shape(H, W, k, s)
    d = gen.stack_inputs(cfg, oracle.num_taps, (H, W))
    acts = [d["x"]]                  # float64 copies of GPU activations
    argmaxes = []
    for li, layer in enumerate(cfg["layers"]):
        a = acts[-1]
        if layer[0] == "conv":
            _, ci, co, k, s, relu = layer
            p = d["params"][li]
            y = run_fwd(a, p["w"], p["b"], k, s, "bf16", relu=relu)
            ref = oracle.conv_fwd(a, p["w"], p["b"], k, s)
            if relu:
                ref = np.maximum(ref, 0.0)
            mag = oracle.conv_fwd(np.abs(a), np.abs(p["w"]), np.abs(p["b"]), k, s)
            check_bf16(y, ref, mag, "c5 L%d fwd" % li)
            acts.append(y)
            argmaxes.append(None)
        else:
            _, c, k, s = layer
            y, am = run_pool_fwd(a, k, s, hx.HEX_POOL_MAX, "bf16")
            ref, ram = oracle.pool_fwd(a, k, s, hx.HEX_POOL_MAX)
            np.testing.assert_array_equal(y, ref)
            np.testing.assert_array_equal(am, ram)
            acts.append(y)
            argmaxes.append(am)
    g = d["dy"]
    for li in range(len(cfg["layers"]) - 1, -1, -1):
        layer = cfg["layers"][li]
        a = acts[li]
        Hin, Win = a.shape[2:]
        if layer[0] == "conv":
            _, ci, co, k, s, relu = layer
            p = d["params"][li]
            dw, db = run_bwd_weight(a, g, k, s, "bf16")
            rw, rb = oracle.conv_bwd_weight(a, g, k, s)
            mw, mb = oracle.conv_bwd_weight(np.abs(a), np.abs(g), k, s)
            check_bf16(dw, rw, mw, "c5 L%d dw" % li)
            check_bf16(db, rb, mb, "c5 L%d db" % li)
            if li == 0:
                # the first layer as a network runs it: the combined entry
                # point without dx (fused small-channel kernel in bf16)
                _, dw2, db2 = run_bwd(a, g, p["w"], k, s, "bf16", want_dx=False)
                check_bf16(dw2, rw, mw, "c5 L0 combined dw")
                check_bf16(db2, rb, mb, "c5 L0 combined db")
                break                    # no gradient for the input image
            dx = run_bwd_data(g, p["w"], k, s, Hin, Win, "bf16")
            check_bf16(dx, oracle.conv_bwd_data(g, p["w"], k, s, Hin, Win),
                       oracle.conv_bwd_data(np.abs(g), np.abs(p["w"]), k, s, Hin, Win),
                       "c5 L%d dx" % li)
            g = dx
        else:
            _, c, k, s = layer
            am = argmaxes[li]
            # the ReLU sits right before the first pool
            relu_y = a if cfg["layers"][li - 1][0] == "conv" and cfg["layers"][li - 1][5] else None
            dx = run_pool_bwd(g, am, relu_y, k, s, hx.HEX_POOL_MAX, Hin, Win, "bf16")
            ref = oracle.pool_bwd(g, am, relu_y, k, s, hx.HEX_POOL_MAX, Hin, Win)
            mag = oracle.pool_bwd(np.abs(g), am, relu_y, k, s, hx.HEX_POOL_MAX, Hin, Win)
            check_bf16(dx, ref, mag, "c5 L%d pool dx" % li)
            # the tap-phase scatter is deterministic: same bits again
            dx2 = run_pool_bwd(g, am, relu_y, k, s, hx.HEX_POOL_MAX, Hin, Win, "bf16")
            np.testing.assert_array_equal(dx, dx2)
            g = dx


@pytest.mark.parametrize("ci,co,k", [(32, 32, 1), (64, 64, 1), (32, 32, 2)])
def test_wide_runs_across_images(ci, co, k):
    """bf16 matrix-core convolution with blocks that walk several row tiles:
    100 images of 48x16 in 3 tiles each (300 tiles), so runs of 2 consecutive
    tiles continue an image's window (only the new rows are staged) and some
    cross into the next image (whole window again); every output compared."""
    rng = np.random.default_rng(1000 * ci + 10 * co + k)
    N, H, W = 100, 48, 16
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, ci, H, W)), "bf16")
    w = gen.round_to(rng.normal(size=(co, ci, T)) / np.sqrt(ci * T), "bf16")
    b = gen.round_to(rng.normal(size=co) * 0.1, "bf16")
    check_fwd_full(x, w, b, k, 1, "bf16", what="fwd")
    dy = gen.round_to(rng.normal(size=(N, co, H, W)), "bf16")
    check_bwd_full(x, w, dy, k, 1, "bf16", what="bwd")


@pytest.mark.parametrize("N,ci,co,H,W,relu", [
    (3, 32, 48, 9, 96, True),     # 32 channels in, 48 out, rows of 96 pixels
    (300, 32, 32, 3, 72, False),  # more runs than blocks: blocks walk two runs
    (5, 64, 16, 130, 120, True),  # runs of 3 rows, the last run a single row
    (128, 64, 64, 4, 128, False), # runs of 2 rows
    (2, 64, 64, 37, 128, False),  # one image split into many runs
])
def test_wide_pipelined_rows(N, ci, co, H, W, relu):
    """bf16 matrix-core convolution with one-row tiles and split roles (k = 1,
    32 or 64 channels in, at most 64 out, rows of 64 < W <= 128 pixels):
    ring window of four rows, rows staged two tiles ahead, results stored
    one tile behind; runs of several rows per block, runs that end after one
    or two rows, blocks that take several runs; every output compared, and
    the data gradient where the output channels qualify as its input."""
    rng = np.random.default_rng(7 * N + ci + co + H + W)
    k = 1
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, ci, H, W)), "bf16")
    w = gen.round_to(rng.normal(size=(co, ci, T)) / np.sqrt(ci * T), "bf16")
    b = gen.round_to(rng.normal(size=co) * 0.1, "bf16")
    check_fwd_full(x, w, b, k, 1, "bf16", relu=relu, what="fwd")
    dy = gen.round_to(rng.normal(size=(N, co, H, W)), "bf16")
    check_bwd_full(x, w, dy, k, 1, "bf16", what="bwd")


@pytest.mark.parametrize("N,ci,co,H,k", [(10, 64, 64, 91, 1), (20, 32, 32, 57, 2)])
def test_wgrad32_regular_runs(N, ci, co, H, k):
    """bf16 matrix-core weight gradient with regular staging (rows of 128
    elements, as many input as output channels) over more tiles than blocks:
    block runs of several tiles, ragged last tiles (H not a multiple of the
    tile height) and runs crossing into the next image; dw and db compared
    in full."""
    rng = np.random.default_rng(N * 1000 + ci + H + k)
    W = 128
    x = gen.round_to(rng.normal(size=(N, ci, H, W)), "bf16")
    dy = gen.round_to(rng.normal(size=(N, co, H, W)), "bf16")
    dw, db = run_bwd_weight(x, dy, k, 1, "bf16")
    rw, rb = oracle.conv_bwd_weight(x, dy, k, 1)
    mw, mb = oracle.conv_bwd_weight(np.abs(x), np.abs(dy), k, 1)
    check("bf16", dw, rw, mw, "dw")
    check("bf16", db, rb, mb, "db")


# --------------------------------------------------------------- sweeps

SWEEP = [
    # N, Ci, Co, H, W, k, s
    (2, 1, 4, 16, 16, 1, 1), (1, 1, 16, 13, 11, 2, 1), (2, 3, 5, 9, 10, 1, 2),
    (1, 2, 3, 1, 7, 1, 1), (1, 2, 3, 7, 1, 2, 1), (2, 4, 2, 11, 12, 3, 1),
    (1, 3, 3, 12, 13, 2, 3), (1, 2, 2, 5, 5, 0, 1), (1, 5, 7, 17, 9, 1, 4),
    (2, 8, 8, 20, 21, 1, 1), (1, 16, 16, 18, 19, 2, 1), (1, 33, 17, 10, 14, 1, 1),
    (1, 64, 64, 12, 12, 1, 1), (1, 32, 64, 24, 24, 2, 1), (1, 1, 32, 48, 48, 2, 1),
    (2, 64, 16, 9, 70, 1, 1), (1, 7, 9, 6, 40, 2, 2), (1, 1, 1, 1, 1, 1, 1),
    (1, 2, 2, 2, 9, 4, 2), (3, 3, 24, 37, 8, 2, 1), (1, 2, 70, 5, 256, 1, 1),
    (2, 48, 40, 11, 32, 2, 1), (3, 2, 20, 13, 68, 2, 1), (2, 1, 24, 9, 8, 1, 1),
    (1, 2, 16, 5, 12, 2, 1),
    # small-channel forward with a 6-step contraction (3 x 7 taps), ragged rows
    (2, 3, 8, 10, 12, 1, 1), (1, 3, 16, 11, 40, 1, 1),
    # small-channel kernels at k = 3 (37 taps): forward, data and weight gradient
    # and the fused backward; 32 output channels; 3 input channels (fast data
    # gradient only)
    (2, 1, 16, 13, 20, 3, 1), (1, 1, 32, 9, 44, 3, 1), (3, 1, 8, 40, 40, 3, 1),
    (1, 3, 5, 10, 12, 3, 1),
    # dispatch boundaries of the few-channel gradients: the fused backward
    # with 20 output channels (a ragged second block of 16) at W = 44; 33
    # output channels (no fused kernel, W not a multiple of 8): the
    # small-channel weight gradient over three 16-channel blocks and the
    # small-channel data gradient over 33 channels, also in bf16
    (1, 1, 20, 9, 44, 2, 1), (2, 1, 33, 7, 44, 1, 1),
    # wide bf16 matrix-core path: registers (k=1: 32 and 64 channels, k=2: 32),
    # LDS-resident weights (long contractions), several channel chunks,
    # partial last tiles, narrow and wide rows
    (2, 32, 48, 10, 16, 1, 1), (1, 64, 128, 12, 12, 1, 1), (2, 64, 64, 37, 16, 1, 1),
    (1, 96, 32, 8, 24, 1, 1), (1, 32, 32, 6, 20, 2, 1), (1, 64, 64, 30, 12, 1, 1),
    (1, 32, 16, 6, 128, 2, 1), (1, 32, 32, 3, 256, 1, 1), (2, 128, 64, 5, 8, 2, 1),
    # matrix-core weight gradient in several output-channel passes (128 + 64
    # + 32, 64 + 64 at k=2, 64 + 32 with two input-channel blocks)
    (1, 32, 224, 6, 16, 1, 1), (2, 32, 128, 7, 12, 2, 1), (1, 64, 96, 5, 20, 1, 1),
    # four input-channel blocks per wave group at k = 1
    (1, 128, 32, 6, 16, 1, 1),
    # matrix-core weight gradient with regular staging (rows of whole 16-byte
    # chunks, as many input as output channels in the pass): 2 and 4 channel
    # blocks per row, ragged last tiles
    (2, 64, 64, 37, 128, 1, 1), (1, 32, 32, 19, 128, 2, 1), (3, 64, 64, 9, 64, 1, 1),
    (1, 32, 32, 10, 256, 2, 1),
    # k = 3 (37 taps)
    (2, 32, 32, 12, 16, 3, 1), (1, 64, 32, 9, 24, 3, 1), (1, 32, 64, 7, 40, 3, 1),
    # strided matrix-core weight gradient (W and W_out multiples of 8):
    # strides 2 and 3, k 1-3, ragged last tiles
    (2, 32, 32, 20, 32, 1, 2), (1, 64, 32, 17, 48, 2, 2), (1, 16, 24, 13, 48, 1, 3),
    (1, 32, 32, 14, 64, 3, 2), (3, 32, 64, 9, 16, 2, 2),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", SWEEP, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_conv_sweep(case, dt):
    N, Ci, Co, H, W, k, s = case
    rng = np.random.default_rng(abs(hash(case)) % (2 ** 31))
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, H, W)), dt)
    w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), dt)
    b = gen.round_to(rng.normal(size=Co) * 0.1, dt)
    Ho, Wo = oracle.out_shape(H, W, s)
    if Ho > 0:
        check_fwd_full(x, w, b, k, s, dt, what="fwd")
        check_fwd_full(x, w, None, k, s, dt, relu=True, what="fwd relu")
    dy = gen.round_to(rng.normal(size=(N, Co, Ho, Wo)), dt)
    if Ho > 0:
        check_bwd_full(x, w, dy, k, s, dt, what="bwd")


# Kernel sizes and strides up to the largest the ABI accepts (HEX_MAX_K = 8,
# HEX_MAX_STRIDE = 8): generic kernels for every op, including a block of
# 64 output channels at k = 5 and the k = 8 / stride 8 plan with 64 output
# channels (region plus staged weights within the block's LDS), and the
# bf16 matrix-core weight gradient at strides 4 and 8 (W and W_out
# multiples of 8).
LARGE_K_S = [
    # N, Ci, Co, H, W, k, s
    (1, 2, 3, 20, 22, 5, 1), (1, 3, 2, 25, 27, 8, 1), (1, 2, 2, 30, 33, 1, 5),
    (1, 2, 3, 41, 40, 2, 8), (1, 3, 3, 40, 41, 8, 8), (1, 4, 64, 40, 40, 8, 8),
    (1, 64, 64, 24, 24, 5, 1), (2, 5, 7, 37, 29, 5, 5), (1, 8, 40, 26, 26, 8, 5),
    (1, 32, 32, 30, 32, 2, 4), (2, 32, 32, 40, 64, 3, 8), (1, 32, 64, 24, 32, 1, 4),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", LARGE_K_S, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_conv_large_k_and_stride(case, dt):
    N, Ci, Co, H, W, k, s = case
    rng = np.random.default_rng(7000 + sum(case))
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, H, W)), dt)
    w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), dt)
    b = gen.round_to(rng.normal(size=Co) * 0.1, dt)
    Ho, Wo = oracle.out_shape(H, W, s)
    assert Ho > 0
    check_fwd_full(x, w, b, k, s, dt, what="fwd")
    dy = gen.round_to(rng.normal(size=(N, Co, Ho, Wo)), dt)
    check_bwd_full(x, w, dy, k, s, dt, what="bwd")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [hx.HEX_POOL_MAX, hx.HEX_POOL_AVG])
@pytest.mark.parametrize("case", [(1, 2, 20, 24, 5, 1), (1, 2, 25, 26, 8, 1),
                                  (2, 2, 30, 32, 1, 5), (1, 3, 40, 41, 2, 8),
                                  (1, 2, 33, 35, 8, 8), (1, 2, 30, 32, 5, 5)])
def test_pool_large_k_and_stride(case, mode, dt):
    N, C, H, W, k, s = case
    rng = np.random.default_rng(9000 + sum(case) + mode)
    x = gen.round_to(rng.normal(size=(N, C, H, W)), dt)
    x[0, 0, : H // 2, : W // 2] = 0.5            # plateaus: exercise ties
    y, am = run_pool_fwd(x, k, s, mode, dt)
    ref, ram = oracle.pool_fwd(x, k, s, mode)
    if mode == hx.HEX_POOL_MAX:
        np.testing.assert_array_equal(y, ref)
        np.testing.assert_array_equal(am, ram)
    elif dt == "bf16":
        want = round_bf16_f64(ref)
        assert np.all(np.abs(y - want) <= bf16_ulp(want))
    else:
        check_f32(y, ref, "avg pool")
    dy = gen.round_to(rng.normal(size=ref.shape), dt)
    for relu_y in (None, np.maximum(x, 0.0)):
        dx = run_pool_bwd(dy, ram if mode == 0 else None, relu_y, k, s, mode, H, W, dt)
        rdx = oracle.pool_bwd(dy, ram if mode == 0 else None, relu_y, k, s, mode, H, W)
        mag = oracle.pool_bwd(np.abs(dy), ram if mode == 0 else None, relu_y, k, s, mode, H, W)
        check(dt, dx, rdx, mag, "pool bwd")


# bf16 matrix-core convolution at any stride and k <= 3 (k_mfma_gen.hip):
# forward for C_in % 32 == 0, W % 8 == 0; data gradient (transposed lattice
# gather) for C_out % 32 == 0, W and W_out % 8 == 0, H a multiple of the
# stride.  Strides 1 (k = 3) to 8, several 32-channel chunks, 64-channel
# blocks cut short, ragged row tiles, output widths that are not a multiple
# of 8 (scalar stores), data-gradient tiles in several rounds of pixel
# groups (strides 3 and 4 over wide rows).  A call mostly goes to the kernels
# for any shape instead; test_any_gpu.py runs these cases with
# HEXCONV_PATH=rows, which puts k_mfma_gen.hip first.
GEN_CASES = [
    # N, Ci, Co, H, W, k, s
    (2, 32, 32, 12, 16, 3, 1), (1, 64, 96, 9, 24, 3, 1), (1, 96, 32, 8, 40, 3, 1),
    (2, 32, 64, 20, 32, 1, 2), (1, 64, 64, 34, 48, 2, 2), (1, 32, 32, 14, 64, 3, 2),
    (1, 32, 32, 30, 48, 1, 3), (2, 64, 32, 24, 96, 2, 3), (1, 32, 64, 24, 32, 1, 4),
    (1, 32, 32, 32, 128, 3, 4), (1, 32, 32, 40, 40, 2, 5), (2, 32, 32, 40, 64, 3, 8),
    (1, 32, 32, 21, 40, 1, 2), (1, 32, 48, 10, 24, 2, 1), (3, 64, 64, 16, 128, 1, 2),
    (1, 32, 32, 24, 256, 2, 3),
]


@pytest.mark.parametrize("case", GEN_CASES, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_conv_matrix_core_any_stride(case):
    N, Ci, Co, H, W, k, s = case
    rng = np.random.default_rng(5000 + sum(case))
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, H, W)), "bf16")
    w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), "bf16")
    b = gen.round_to(rng.normal(size=Co) * 0.1, "bf16")
    check_fwd_full(x, w, b, k, s, "bf16", what="fwd")
    check_fwd_full(x, w, None, k, s, "bf16", relu=True, what="fwd relu")
    Ho, Wo = oracle.out_shape(H, W, s)
    dy = gen.round_to(rng.normal(size=(N, Co, Ho, Wo)), "bf16")
    dx = run_bwd_data(dy, w, k, s, H, W, "bf16")
    check("bf16", dx, oracle.conv_bwd_data(dy, w, k, s, H, W),
          oracle.conv_bwd_data(np.abs(dy), np.abs(w), k, s, H, W), "dx")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [hx.HEX_POOL_MAX, hx.HEX_POOL_AVG])
@pytest.mark.parametrize("case", [(2, 3, 9, 10, 1, 2), (1, 4, 40, 40, 1, 2),
                                  (1, 2, 11, 12, 2, 1), (2, 2, 13, 7, 2, 3),
                                  (1, 3, 1, 9, 1, 1), (1, 5, 24, 24, 1, 2),
                                  (1, 2, 6, 6, 0, 1), (1, 1, 17, 18, 3, 4),
                                  # LDS-staged kernels: k 0..2, strides 1 and 2,
                                  # several planes per block with a partial last
                                  # block, 16 outputs per thread
                                  (2, 3, 16, 16, 2, 1), (1, 4, 48, 48, 1, 2),
                                  (3, 5, 7, 8, 0, 2), (1, 2, 8, 24, 2, 2),
                                  (1, 70, 24, 32, 1, 1), (2, 3, 5, 16, 1, 2),
                                  (1, 2, 64, 64, 1, 1),
                                  # k = 3 (37 taps) on the LDS-staged kernels
                                  (2, 3, 16, 16, 3, 1), (1, 4, 40, 40, 3, 2),
                                  (3, 2, 11, 24, 3, 2), (1, 70, 8, 16, 3, 1),
                                  # strides 3 and 4 on the LDS-staged kernels
                                  (1, 3, 20, 24, 1, 3), (2, 2, 17, 32, 2, 4),
                                  (1, 4, 30, 48, 3, 3), (2, 3, 9, 16, 0, 4),
                                  # k = 1, stride 2 in bf16 takes two outputs
                                  # per thread: odd H (the bottom border row
                                  # is read), 12 output pairs per row
                                  (2, 3, 13, 24, 1, 2), (1, 2, 9, 48, 1, 2)])
def test_pool_sweep(case, mode, dt):
    N, C, H, W, k, s = case
    rng = np.random.default_rng(sum(case) + mode)
    x = gen.round_to(rng.normal(size=(N, C, H, W)), dt)
    x[0, 0, : H // 2, : W // 2] = 0.5            # plateaus: exercise ties
    y, am = run_pool_fwd(x, k, s, mode, dt)
    ref, ram = oracle.pool_fwd(x, k, s, mode)
    if mode == hx.HEX_POOL_MAX:
        np.testing.assert_array_equal(y, ref)
        np.testing.assert_array_equal(am, ram)
    elif dt == "bf16":
        want = round_bf16_f64(ref)
        assert np.all(np.abs(y - want) <= bf16_ulp(want))
    else:
        check_f32(y, ref, "avg pool")
    dy = gen.round_to(rng.normal(size=ref.shape), dt)
    for relu_y in (None, np.maximum(x, 0.0)):
        dx = run_pool_bwd(dy, ram if mode == 0 else None, relu_y, k, s, mode, H, W, dt)
        rdx = oracle.pool_bwd(dy, ram if mode == 0 else None, relu_y, k, s, mode, H, W)
        mag = oracle.pool_bwd(np.abs(dy), ram if mode == 0 else None, relu_y, k, s, mode, H, W)
        check(dt, dx, rdx, mag, "pool bwd")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_bwd_without_dx(dt):
    """hexconv_bwd with dx = NULL (a first layer) still gives dw and db, with
    or without w (the header lets w be NULL then, and the fused kernel must
    not read it); hexconv_bwd_weight on the same shape takes the same kernel."""
    cfg = CFG["c2"]
    d = _conv_inputs(cfg, N=24)
    x, dy = gen.round_to(d["x"], dt), gen.round_to(d["dy"], dt)
    w = gen.round_to(d["w"], dt)
    rw, rb = oracle.conv_bwd_weight(x, dy, cfg["k"], 1)
    mw, mb = oracle.conv_bwd_weight(np.abs(x), np.abs(dy), cfg["k"], 1)
    for wv in (w, None):
        _, dw, db = run_bwd(x, dy, wv, cfg["k"], 1, dt, want_dx=False)
        check(dt, dw, rw, mw, "dw")
        check(dt, db, rb, mb, "db")
    dw, db = run_bwd_weight(x, dy, cfg["k"], 1, dt)
    check(dt, dw, rw, mw, "dw (hexconv_bwd_weight)")
    check(dt, db, rb, mb, "db (hexconv_bwd_weight)")


def test_debug_mode_golden():
    """All-ones kernel on a tensor of ones (tests/golden fixture)."""
    path = os.path.join(os.path.dirname(__file__), "golden", "debug_ones_3x4_k1.txt")
    rows = [[int(v) for v in l.split()] for l in open(path)
            if l.strip() and not l.startswith("#")]
    H, W, k = rows[0]
    y = run_fwd(np.ones((1, 1, H, W)), np.ones((1, 1, 7)), None, k, 1, "f32")
    np.testing.assert_array_equal(y[0, 0], np.array(rows[1:1 + H], np.float64))


# ----------------------------------------------------------- edge cases

def test_empty_batch_and_empty_output():
    torch = torch_mod()
    # N = 0: nothing to do, returns OK
    x = torch.empty((0, 1, 8, 8), dtype=torch.float32, device="cuda:0")
    w = to_dev(np.ones((2, 1, 7)), "f32")
    y = torch.empty((0, 2, 8, 8), dtype=torch.float32, device="cuda:0")
    hx.hexconv_fwd(x, w, None, y, 1, 1)
    # H too small for the odd output columns: empty output; gradients are 0
    H, W, k, s = 1, 5, 1, 2
    assert hx.hex_out_shape(H, W, k, s) == (0, 3)
    dy = np.zeros((1, 2, 0, 3))
    dx = run_bwd_data(dy, np.ones((2, 1, 7)), k, s, H, W, "f32")
    assert np.all(dx == 0)
    dw, db = run_bwd_weight(np.ones((1, 1, H, W)), dy, k, s, "f32")
    assert np.all(dw == 0) and np.all(db == 0)


def test_deterministic_repeat():
    """Same inputs, same bits: forward and both gradients."""
    cfg = CFG["c2"]
    d = _conv_inputs(cfg, N=32)
    a = run_bwd_weight(d["x"], d["dy"], cfg["k"], 1, "f32")
    b = run_bwd_weight(d["x"], d["dy"], cfg["k"], 1, "f32")
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])
    y1 = run_fwd(d["x"], d["w"], d["b"], cfg["k"], 1, "f32")
    y2 = run_fwd(d["x"], d["w"], d["b"], cfg["k"], 1, "f32")
    np.testing.assert_array_equal(y1, y2)
    # bf16 camera layer: the small-channel weight gradient (one block of 16
    # output channels) and data gradient called on their own
    xb = gen.round_to(d["x"], "bf16")
    dyb = gen.round_to(d["dy"], "bf16")
    wb = gen.round_to(d["w"], "bf16")
    a = run_bwd_weight(xb, dyb, cfg["k"], 1, "bf16")
    b = run_bwd_weight(xb, dyb, cfg["k"], 1, "bf16")
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])
    H, W = d["x"].shape[2:]
    dx1 = run_bwd_data(dyb, wb, cfg["k"], 1, H, W, "bf16")
    dx2 = run_bwd_data(dyb, wb, cfg["k"], 1, H, W, "bf16")
    np.testing.assert_array_equal(dx1, dx2)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_specialised_matches_generic(dt, monkeypatch):
    """The shape-specialised kernels and the generic kernels agree to the
    parity tolerance on the same inputs."""
    rng = np.random.default_rng(11)
    for (N, Ci, Co, H, W, k) in [(3, 1, 16, 40, 40, 2), (2, 16, 32, 24, 24, 2),
                                 (1, 64, 64, 32, 128, 1), (2, 1, 16, 40, 40, 3)]:
        T = oracle.num_taps(k)
        x = gen.round_to(rng.normal(size=(N, Ci, H, W)), dt)
        w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), dt)
        y_fast = run_fwd(x, w, None, k, 1, dt)
        monkeypatch.setenv("HEXCONV_PATH", "generic")
        y_gen = run_fwd(x, w, None, k, 1, dt)
        monkeypatch.delenv("HEXCONV_PATH")
        mag = oracle.conv_fwd(np.abs(x), np.abs(w), None, k, 1) if dt == "bf16" else None
        check(dt, y_fast, y_gen, mag, "fast vs generic")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_graph_replay_matches_eager(dt):
    """The library's launches captured into a HIP graph give, on every
    replay, the same bits as eager calls (outputs are poisoned and other
    eager work runs between replays)."""
    torch = torch_mod()
    rng = np.random.default_rng(21)
    cases = [(8, 1, 16, 40, 40, 2), (2, 32, 64, 24, 24, 2)]
    for (N, Ci, Co, H, W, k) in cases:
        T = hx.hex_num_taps(k)
        Ho, Wo = hx.hex_out_shape(H, W, k, 1)
        x = to_dev(gen.round_to(rng.normal(size=(N, Ci, H, W)), dt), dt)
        w = to_dev(gen.round_to(rng.normal(size=(Co, Ci, T)) * 0.1, dt), dt)
        b = to_dev(gen.round_to(rng.normal(size=Co) * 0.1, dt), dt)
        dy = to_dev(gen.round_to(rng.normal(size=(N, Co, Ho, Wo)), dt), dt)
        y = empty((N, Co, Ho, Wo), dt)
        dx = empty((N, Ci, H, W), dt)
        dw = torch.empty((Co, Ci, T), dtype=torch.float32, device="cuda:0")
        db = torch.empty((Co,), dtype=torch.float32, device="cuda:0")
        yp = empty((N, Co, *hx.hex_out_shape(Ho, Wo, 1, 2)), dt)
        am = torch.empty(yp.shape, dtype=torch.uint8, device="cuda:0")
        dxp = empty((N, Co, Ho, Wo), dt)
        nws = hx.hexconv_bwd_weight_workspace(N, Ci, Co, H, W, k, 1,
                                              hx.HEX_F32 if dt == "f32" else hx.HEX_BF16)
        ws = torch.empty(max(nws, 1), dtype=torch.uint8, device="cuda:0")

        def calls():
            hx.hexconv_fwd(x, w, b, y, k, 1)
            hx.hexconv_bwd_data(dy, w, dx, k, 1)
            hx.hexconv_bwd_weight(x, dy, dw, db, ws, k, 1)
            hx.hexpool_fwd(y, yp, am, 1, 2, hx.HEX_POOL_MAX)
            hx.hexpool_bwd(yp, am, y, dxp, 1, 2, hx.HEX_POOL_MAX)

        outs = (y, dx, dw, db, yp, am, dxp)
        calls()
        torch.cuda.synchronize()
        ref = [o.clone() for o in outs]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            calls()
        scratch = empty((N, Co, Ho, Wo), dt)
        for rep in range(3):
            for o in outs:
                o.fill_(7)
            hx.hexconv_fwd(x, w, None, scratch, k, 1)        # unrelated eager work
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            for o, r in zip(outs, ref):
                assert torch.equal(o, r), "replay %d differs" % rep


def test_kernel_timing_reports_launches():
    """hexconv_timing_* brackets each launch with events: one forward call of
    the camera shape reports its kernel once, with a positive duration, and
    the combined backward reports its main kernel and its reduction."""
    cfg = CFG["c2"]
    d = _conv_inputs(cfg, N=8)
    run_fwd(d["x"], d["w"], d["b"], cfg["k"], 1, "f32")  # warm (module load)
    hx.hexconv_timing_begin()
    run_fwd(d["x"], d["w"], d["b"], cfg["k"], 1, "f32")
    t = hx.hexconv_timing_end()
    assert list(t) == ["fwd_smallc_k"], t
    assert t["fwd_smallc_k"][0] == 1 and t["fwd_smallc_k"][1] > 0
    hx.hexconv_timing_begin()
    run_bwd(d["x"], d["dy"], d["w"], cfg["k"], 1, "f32")
    t = hx.hexconv_timing_end()
    assert list(t) == ["bwd_smallc_k", "reduce_chunked_k"], t
    assert all(c == 1 and ms > 0 for c, ms in t.values()), t
