"""Matrix-core kernels for planes of any size and channel count
(k_conv_any.hip, k_wgrad_any.hip) against the fp64 oracle, at the sizes where
they can go wrong: rows of odd length and of the shortest length taken (8),
one row, several tiles and a ragged last tile, channel counts just past a
chunk or a 32-channel tile, k = 1 .. 3, strides, both dtypes, 3-D.  Work this
little mostly goes to simpler kernels, so these cases run twice: as a call
does, and with HEXCONV_PATH putting the family under test first."""
import numpy as np
import pytest

import oracle
from gpu_helpers import check, rel_l2, torch_mod
from paper_1903_01814_amd import inputs as gen
from test_parity3d_gpu import run_bwd_data3, run_bwd_weight3, run_fwd3
from test_parity_gpu import (check_bwd_full, check_fwd_full, run_bwd_data, run_bwd_weight,
                             run_fwd, run_pool_bwd)
import test_parity_gpu as parity

pytestmark = pytest.mark.gpu

# N, C_in, C_out, H, W, k, stride
CASES = [
    (2, 5, 7, 9, 8, 1, 1),         # shortest rows
    (3, 24, 24, 1, 9, 1, 1),       # one row: every other window row is padding
    (2, 16, 17, 18, 19, 2, 1),     # one half chunk (bf16), 17 = half chunk + 1 back
    (2, 33, 65, 23, 43, 1, 1),     # one channel past a chunk and past two tiles
    (1, 70, 100, 12, 25, 2, 1),    # several chunks, streamed weights, 4 tiles out
    (1, 40, 36, 20, 250, 1, 1),    # one row per tile
    (1, 32, 40, 21, 51, 3, 1),     # k = 3
    (40, 12, 12, 20, 21, 1, 1),    # more tiles than a block's run
    (2, 48, 32, 29, 31, 1, 2),     # strides: split columns, odd centres
    (2, 40, 33, 31, 45, 2, 3),
    # data gradient at strides: classes cut at the border, streamed weights
    # (100 output channels at k = 2), one class row, strides up to 8
    (1, 5, 100, 33, 35, 2, 2), (1, 33, 16, 48, 47, 3, 2), (3, 16, 16, 16, 40, 1, 4),
    (1, 12, 8, 33, 64, 2, 8), (1, 3, 8, 2, 17, 1, 2), (1, 64, 64, 32, 32, 1, 2),
    # whole 16-byte rows that the tuned bf16 kernels leave to this one
    (2, 64, 96, 40, 48, 1, 1), (1, 96, 96, 33, 40, 1, 1), (2, 32, 32, 64, 64, 2, 1),
    # weight gradient: rows of 4 and of 8 pixels, more than 64 (channel, tap)
    # pairs, planes that end inside a step of 16 pixels
    (3, 12, 20, 9, 4, 1, 1), (2, 5, 33, 11, 4, 2, 1), (3, 12, 20, 9, 8, 1, 1),
    (2, 5, 33, 11, 8, 2, 1), (3, 16, 8, 13, 12, 1, 3),
    # weight gradient: fewer slots than tiles (k > 1), so that they fit the
    # scratch array of a call that may not allocate
    (30, 128, 128, 13, 17, 3, 1),
]


def conv_case(case, dt):
    N, Ci, Co, H, W, k, s = case
    rng = np.random.default_rng(300 + sum(case))
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, H, W)), dt)
    w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), dt)
    b = gen.round_to(rng.normal(size=Co) * 0.1, dt)
    check_fwd_full(x, w, b, k, s, dt, what="fwd")
    check_fwd_full(x, w, None, k, s, dt, relu=True, what="fwd relu")
    dy = gen.round_to(rng.normal(size=(N, Co) + oracle.out_shape(H, W, s)), dt)
    check_bwd_full(x, w, dy, k, s, dt, what="bwd")


@pytest.mark.parametrize("path", ["", "any"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_conv_any_shape(case, dt, path, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", path)
    conv_case(case, dt)


def conv3d_case(case, dt):
    N, Ci, Co, D, H, W, k, kz, s, sz = case
    rng = np.random.default_rng(400 + sum(case))
    Z, T = 2 * kz + 1, oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, D, H, W)), dt)
    w = gen.round_to(rng.normal(size=(Co, Ci, Z, T)) / np.sqrt(Ci * Z * T), dt)
    b = gen.round_to(rng.normal(size=Co) * 0.1, dt)
    a = np.abs
    check(dt, run_fwd3(x, w, b, k, kz, s, sz, dt), oracle.conv3d_fwd(x, w, b, k, kz, s, sz),
          oracle.conv3d_fwd(a(x), a(w), a(b), k, kz, s, sz), "fwd")
    Do, Ho, Wo = oracle.out_shape3d(D, H, W, s, sz)
    dy = gen.round_to(rng.normal(size=(N, Co, Do, Ho, Wo)), dt)
    check(dt, run_bwd_data3(dy, w, k, kz, s, sz, D, H, W, dt),
          oracle.conv3d_bwd_data(dy, w, k, kz, s, sz, D, H, W),
          oracle.conv3d_bwd_data(a(dy), a(w), k, kz, s, sz, D, H, W), "dx")
    dw, db = run_bwd_weight3(x, dy, k, kz, s, sz, dt)
    rw, rb = oracle.conv3d_bwd_weight(x, dy, k, kz, s, sz)
    mw, mb = oracle.conv3d_bwd_weight(a(x), a(dy), k, kz, s, sz)
    check(dt, dw, rw, mw, "dw")
    check(dt, db, rb, mb, "db")


@pytest.mark.parametrize("path", ["", "any"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    # N, C_in, C_out, D, H, W, k, kz, stride, stride_z
    (2, 6, 9, 3, 9, 11, 1, 1, 1, 1), (1, 17, 33, 4, 20, 19, 1, 1, 1, 1),
    (1, 8, 8, 2, 10, 13, 2, 2, 1, 1), (1, 40, 12, 5, 11, 17, 1, 1, 2, 2)])
def test_conv3d_any_shape(case, dt, path, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", path)
    conv3d_case(case, dt)


# Relative error of float32 sums whose terms are independent: a chain of n
# additions is off by about 2.5e-8 sqrt(n / 2) (half an ulp at most each, of a
# partial sum that grows as a random walk).  The weight gradients add chains of
# 16 pixels, of 8 of these and of the run's (20 at most here): 1.3e-7 with the
# slots' sums, and over the 40 and more values of db of all `runs` together a
# fifth to either side (24 values alone: 0.8e-7 to 1.9e-7).  One chain over a block's run of tiles has hundreds
# (1.8e-7 to 5.1e-7 in these cases).  A plane's part of the 3-D data gradient:
# 84 terms here, 1.7e-7 with the three planes' sum (3.0e-7 in one chain).
SUM_REL, PLANE_REL = 1.6e-7, 2.1e-7


@pytest.mark.parametrize("case", [
    # N, C_in, C_out, H, W, k, runs: the any-shape kernel, few channels, fused
    (227, 4, 8, 41, 39, 2, 5), (60, 12, 64, 37, 41, 1, 1), (119, 3, 24, 37, 30, 1, 2),
    (60, 2, 12, 37, 41, 2, 6)], ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_runs%d" % c)
def test_f32_weight_gradient_sums(case):
    N, Ci, Co, H, W, k, runs = case
    rng = np.random.default_rng(500 + sum(case[:6]))
    got, ref = [], []
    for _ in range(runs):
        x = gen.round_to(np.exp(rng.normal(size=(N, Ci, H, W))) *
                         (rng.uniform(size=(N, Ci, H, W)) < 0.1), "f32")
        dy = gen.round_to(rng.normal(size=(N, Co, H, W)), "f32")
        got.append(run_bwd_weight(x, dy, k, 1, "f32"))
        ref.append(oracle.conv_bwd_weight(x, dy, k, 1))
    err = [rel_l2(np.stack([g[i] for g in got]), np.stack([r[i] for r in ref])) for i in (0, 1)]
    assert max(err) <= SUM_REL, err


def test_f32_weight_gradient_sums_of_one_slot():
    """So many channels that the scratch array holds one slot of each type:
    one block adds all 3 600 steps of 16 pixels, as chains of 16, 60 and 60
    (2.5e-8 sqrt(136 / 2) = 2.1e-7, a fifth more allowed; chains of 8 and 450
    3.8e-7).  Eight output channels are checked."""
    N, C, H, W, k = 16, 512, 57, 57, 3
    rng = np.random.default_rng(550)
    x = rng.normal(size=(N, C, H, W)).astype(np.float32)
    dy = rng.normal(size=(N, C, H, W)).astype(np.float32)
    got = run_bwd_weight(x, dy, k, 1, "f32")
    ref = oracle.conv_bwd_weight(x, dy[:, 100:108], k, 1)
    err = rel_l2(got[0][100:108], ref[0])
    assert err <= 2.5e-7, err


def test_f32_volume_sums():
    rng = np.random.default_rng(600)
    got, ref = [], []
    for _ in range(5):
        x = gen.round_to(rng.normal(size=(6, 8, 10, 33, 35)), "f32")
        dy = gen.round_to(rng.normal(size=(6, 24, 10, 33, 35)), "f32")
        got.append(run_bwd_weight3(x, dy, 1, 1, 1, 1, "f32"))
        ref.append(oracle.conv3d_bwd_weight(x, dy, 1, 1, 1, 1))
    err = [rel_l2(np.stack([g[i] for g in got]), np.stack([r[i] for r in ref])) for i in (0, 1)]
    assert max(err) <= SUM_REL, err
    w = gen.round_to(rng.normal(size=(12, 1, 3, 7)), "f32")
    dx = run_bwd_data3(dy[:, :12], w, 1, 1, 1, 1, 10, 33, 35, "f32")
    rx = oracle.conv3d_bwd_data(dy[:, :12], w, 1, 1, 1, 1, 10, 33, 35)
    assert rel_l2(dx, rx) <= PLANE_REL, rel_l2(dx, rx)


# Little work, or channels that leave a matrix-core tile mostly empty: the
# simpler kernel that the estimates choose, and the sizes next to it that the
# kernels for any shape take.  The launch record names what ran.
ROUTES = [
    # op, N, C_in, C_out, H, W, k, stride, dtype, kernel
    ("fwd", 34, 2, 6, 73, 120, 3, 2, "bf16", "conv_fwd_generic_k"),
    ("fwd", 34, 16, 48, 33, 41, 1, 2, "bf16", "conv_any_k"),
    ("fwd", 125, 4, 6, 61, 128, 1, 2, "f32", "conv_fwd_generic_k"),
    ("fwd", 12, 16, 48, 33, 41, 1, 2, "f32", "conv_f32_k"),
    ("bwd_data", 170, 5, 2, 46, 18, 1, 1, "bf16", "conv_bwd_data_generic_k"),
    ("bwd_data", 2, 3, 3, 24, 32, 3, 1, "bf16", "bwd_data_f32_k"),
    ("bwd_data", 64, 4, 32, 41, 43, 1, 1, "bf16", "conv_any_k"),
    ("bwd_data", 6, 7, 3, 90, 72, 1, 2, "f32", "conv_bwd_data_generic_k"),
    ("bwd_data", 10, 6, 5, 46, 98, 1, 3, "bf16", "conv_bwd_data_generic_k"),
    ("bwd_data", 8, 48, 64, 46, 47, 1, 2, "bf16", "conv_any_dgs_k"),
    # one walk over dy for all classes of pixels; too wide a row for the
    # any-shape window, which the other bf16 kernel still holds
    ("bwd_data", 2, 3, 192, 112, 96, 1, 2, "bf16", "conv_gen_dgrad_k"),
    ("fwd", 2, 32, 32, 72, 128, 3, 4, "bf16", "conv_gen_fwd_k"),
    ("bwd_weight", 112, 3, 5, 63, 77, 1, 2, "f32", "wgrad_partial_generic_k"),
    ("bwd_weight", 1, 7, 2, 29, 57, 1, 1, "f32", "wgrad_partial_generic_k"),
    ("bwd_weight", 20, 16, 24, 33, 41, 1, 2, "f32", "wgrad_any_k"),
    ("bwd_weight", 1, 1, 85, 18, 88, 3, 1, "bf16", "wgrad_bf16_k"),
    ("bwd_weight", 6, 5, 40, 24, 32, 1, 1, "bf16", "wgrad_bf16_k"),
    ("bwd_weight", 55, 7, 40, 24, 24, 1, 3, "bf16", "wgrad_bf16_k"),
    ("bwd_weight", 40, 48, 64, 24, 32, 2, 1, "bf16", "wgrad_any_k"),
    # rows of 4 pixels, 32 channels and more: several passes over x
    ("bwd_weight", 40, 32, 160, 9, 4, 1, 1, "bf16", "wgrad32_k"),
    ("bwd_weight", 4, 7, 5, 60, 71, 1, 4, "bf16", "wgrad_partial_generic_k"),
]


@pytest.mark.parametrize("case", ROUTES, ids=lambda c: "%s_N%d_ci%d_co%d_%dx%d_k%d_s%d_%s" % c[:9])
def test_route(case):
    from paper_1903_01814_amd import hexconv as hx
    op, N, Ci, Co, H, W, k, s, dt, kernel = case
    rng = np.random.default_rng(700 + N + Ci + H)
    T = oracle.num_taps(k)
    x = gen.round_to(rng.normal(size=(N, Ci, H, W)), dt)
    w = gen.round_to(rng.normal(size=(Co, Ci, T)) / np.sqrt(Ci * T), dt)
    dy = gen.round_to(rng.normal(size=(N, Co) + oracle.out_shape(H, W, s)), dt)
    a = np.abs
    hx.hexconv_timing_begin()
    try:
        if op == "fwd":
            got = [run_fwd(x, w, None, k, s, dt)]
        elif op == "bwd_data":
            got = [run_bwd_data(dy, w, k, s, H, W, dt)]
        else:
            got = run_bwd_weight(x, dy, k, s, dt)
    finally:
        ran = hx.hexconv_timing_end()
    assert kernel in ran, ran
    if op == "fwd":
        ref, mag = [oracle.conv_fwd(x, w, None, k, s)], [oracle.conv_fwd(a(x), a(w), None, k, s)]
    elif op == "bwd_data":
        ref = [oracle.conv_bwd_data(dy, w, k, s, H, W)]
        mag = [oracle.conv_bwd_data(a(dy), a(w), k, s, H, W)]
    else:
        ref, mag = oracle.conv_bwd_weight(x, dy, k, s), oracle.conv_bwd_weight(a(x), a(dy), k, s)
    for g, r, m in zip(got, ref, mag):
        check(dt, g, r, m, kernel)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    # N, C, H, W, kernel: 1024 and 2048 pixels a plane, 3 << 20 in all
    (2, 3, 32, 32, "pool_bwd_k"), (2, 3, 26, 40, "pool_any_bwd_k"),
    (4, 400, 50, 40, "pool_bwd_k"), (4, 400, 52, 40, "pool_any_bwd_k")])
def test_mean_gradient_route(case, dt):
    from paper_1903_01814_amd import hexconv as hx
    N, C, H, W, kernel = case
    rng = np.random.default_rng(H + W)
    dy = gen.round_to(rng.normal(size=(N, C, H, W)), dt)
    hx.hexconv_timing_begin()
    try:
        got = run_pool_bwd(dy, None, None, 1, 1, 1, H, W, dt)
    finally:
        ran = hx.hexconv_timing_end()
    assert list(ran) == [kernel]
    ref = oracle.pool_bwd(dy, None, None, 1, 1, 1, H, W)
    mag = oracle.pool_bwd(np.abs(dy), None, None, 1, 1, 1, H, W)
    check(dt, got, ref, mag, kernel)


# Few input channels on rows that are no multiple of 4 (the last group of four
# columns is moved back to end with the row): each remainder, the shortest and
# the longest row that a tile holds whole, a row past it, one input row.
SMALL = [
    # N, C_in, C_out, H, W, k
    (2, 1, 4, 9, 5, 1), (2, 1, 16, 21, 43, 2), (3, 2, 16, 25, 45, 1), (2, 2, 20, 17, 46, 2),
    (1, 1, 32, 33, 127, 2), (2, 3, 16, 20, 21, 1), (2, 1, 17, 13, 6, 3), (2, 3, 33, 15, 49, 2),
    (1, 1, 8, 20, 131, 1), (1, 2, 16, 7, 255, 1), (100, 1, 16, 24, 37, 1), (2, 2, 5, 1, 11, 1)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", SMALL, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d" % c)
def test_few_channels_any_width(case, dt, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", "few")
    conv_case(case + (1,), dt)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    (2, 1, 8, 5, 20, 25, 1, 1, 1, 1), (1, 2, 16, 4, 13, 43, 1, 1, 1, 1),
    (1, 1, 16, 3, 9, 130, 1, 1, 1, 1), (1, 2, 40, 4, 15, 19, 1, 1, 1, 1),
    (1, 1, 8, 3, 10, 7, 2, 2, 1, 1), (1, 1, 12, 6, 17, 46, 1, 1, 1, 2)])
def test_few_channels_any_width_3d(case, dt, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", "few")
    conv3d_case(case, dt)


# The general sweeps' shapes, whose work is as little: through the families
# that a larger tensor of the same shape is given to.
@pytest.mark.parametrize("dt,path", [("f32", "few"), ("bf16", "few"), ("bf16", "rows")])
@pytest.mark.parametrize("case", parity.SWEEP, ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_sweep_families(case, dt, path, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", path)
    parity.test_conv_sweep(case, dt)


@pytest.mark.parametrize("case", parity.GEN_CASES + [c for c in parity.LARGE_K_S if c[1] >= 32],
                         ids=lambda c: "N%d_ci%d_co%d_%dx%d_k%d_s%d" % c)
def test_rows_any_stride(case, monkeypatch):
    monkeypatch.setenv("HEXCONV_PATH", "rows")
    conv_case(case, "bf16")


# Pools on planes that are no whole 16-byte rows, and 3-D pools: single rows and
# columns, every stride's cells cut at the right and bottom border, planes
# beside the volume; one-tap mean (the ReLU mask) with a tail past 16 bytes.
POOL = [
    # N, C, H, W, k, stride
    (2, 3, 9, 11, 1, 2), (1, 2, 45, 51, 1, 2), (2, 5, 1, 7, 1, 1), (1, 3, 7, 1, 1, 2),
    (2, 3, 13, 10, 2, 2), (1, 9, 22, 23, 2, 3), (1, 2, 17, 9, 3, 1), (3, 3, 8, 13, 3, 3),
    (1, 3, 16, 16, 1, 1), (1, 2, 16, 24, 2, 1)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", POOL, ids=lambda c: "N%d_c%d_%dx%d_k%d_s%d" % c)
def test_pool_any_shape(case, mode, dt):
    parity.test_pool_sweep(case, mode, dt)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 3, 5, 7), (2, 4, 16, 16), (1, 1, 1, 3)])
def test_relu_mask_any_shape(shape, dt):
    rng = np.random.default_rng(sum(shape))
    dy = gen.round_to(rng.normal(size=shape), dt)
    y = np.maximum(gen.round_to(rng.normal(size=shape), dt), 0.0)
    H, W = shape[2:]
    np.testing.assert_array_equal(run_pool_bwd(dy, None, y, 0, 1, 1, H, W, dt), dy * (y > 0))
    np.testing.assert_array_equal(run_pool_bwd(dy, None, None, 0, 1, 1, H, W, dt), dy)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", [
    (1, 2, 5, 9, 11, 1, 1, 2, 1), (2, 2, 7, 12, 10, 1, 1, 2, 2), (1, 3, 4, 8, 9, 2, 2, 1, 3),
    (1, 2, 1, 5, 6, 1, 1, 3, 1), (1, 2, 10, 7, 8, 1, 4, 2, 5)])
def test_pool3d_any_shape(case, mode, dt):
    """Against the generic kernels, bit for bit: the same terms in the same order."""
    import os
    from paper_1903_01814_amd import hexconv as hx
    torch = torch_mod()
    N, C, D, H, W, k, kz, s, sz = case
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(sum(case))
    x = (torch.randn((N, C, D, H, W), generator=g) * 2).round().div(2).to(tdt).cuda()
    shape = (N, C) + tuple(hx.hex_out_shape3d(D, H, W, k, kz, s, sz))
    dy = torch.randn(shape, generator=g).to(tdt).cuda()
    got = []
    try:
        for path in ("", "generic"):
            os.environ["HEXCONV_PATH"] = path
            y = torch.full(shape, float("nan"), dtype=tdt, device="cuda")
            am = torch.zeros(shape, dtype=torch.int16, device="cuda") if mode == 0 else None
            hx.hexpool3d_fwd(x, y, am, k, kz, s, sz, mode)
            res = [y]
            for relu in (None, x):
                dx = torch.full(x.shape, float("nan"), dtype=tdt, device="cuda")
                hx.hexpool3d_bwd(dy, am, relu, dx, k, kz, s, sz, mode)
                res.append(dx)
            got.append(res + ([am] if mode == 0 else []))
    finally:
        os.environ.pop("HEXCONV_PATH", None)
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("case", [
    # N, C_in, C_out, D (None: 2-D), H, W, k, kz, stride, stride_z
    (2, 33, 70, None, 17, 29, 1, 0, 2, 1), (1, 40, 20, None, 12, 13, 2, 0, 1, 1),
    (1, 24, 24, None, 1, 9, 1, 0, 1, 1), (1, 16, 7, None, 9, 250, 1, 0, 1, 1),
    (2, 16, 33, None, 9, 8, 3, 0, 1, 1), (1, 1, 16, None, 20, 21, 2, 0, 1, 1),
    (1, 130, 40, None, 11, 24, 1, 0, 3, 1), (30, 16, 24, None, 20, 21, 1, 0, 1, 1),
    (2, 9, 32, 4, 12, 13, 1, 1, 1, 1), (1, 8, 12, 5, 9, 11, 1, 2, 1, 2),
    (1, 5, 40, 3, 12, 13, 2, 1, 2, 1)])
def test_f32_forward_order(case):
    """The float32 forward of rows that the generic kernel used to take equals
    that kernel bit for bit: the same products in the same order from the
    bias on, so what a ReLU or a maximum decides does not change."""
    import os
    from paper_1903_01814_amd import hexconv as hx
    torch = torch_mod()
    N, Ci, Co, D, H, W, k, kz, s, sz = case
    g = torch.Generator().manual_seed(N + Ci + H)
    T = hx.hex_num_taps(k)
    vol = D is not None
    x = torch.randn((N, Ci) + ((D,) if vol else ()) + (H, W), generator=g).cuda()
    w = torch.randn((Co, Ci) + ((2 * kz + 1,) if vol else ()) + (T,), generator=g).cuda()
    b = torch.randn(Co, generator=g).cuda()
    o = hx.hex_out_shape3d(D, H, W, k, kz, s, sz) if vol else hx.hex_out_shape(H, W, k, s)
    got = []
    try:
        for path in ("any", "generic"):
            os.environ["HEXCONV_PATH"] = path
            y = torch.full((N, Co) + tuple(o), float("nan"), device="cuda")
            if vol:
                hx.hexconv3d_fwd(x, w, b, y, k, kz, s, sz)
            else:
                hx.hexconv_fwd(x, w, b, y, k, s)
            got.append(y)
    finally:
        os.environ.pop("HEXCONV_PATH", None)
    assert torch.equal(*got)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_weight_gradient_keeps_infinities(dt):
    """An infinity in x next to a tile's end reaches the sums of its own taps
    as an infinity, and no other sum: 19 x 27 pixels end inside a step (the
    generic kernel here; the families with tiles in the test below)."""
    torch = torch_mod()
    from paper_1903_01814_amd import hexconv as hx
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(0)
    x = torch.rand((1, 8, 19, 27), generator=g).to(tdt)
    dy = (torch.rand((1, 8, 19, 27), generator=g) + 0.5).to(tdt)
    x[0, 3, 18, 26] = float("inf")
    dw = torch.empty((8, 8, 7), device="cuda")
    nws = hx.hexconv_bwd_weight_workspace(1, 8, 8, 19, 27, 1, 1, 0 if dt == "f32" else 1)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    hx.hexconv_bwd_weight(x.cuda(), dy.cuda(), dw, None, ws, 1, 1)
    dw = dw.cpu()
    hit = torch.isinf(dw)
    assert not torch.isnan(dw).any()
    # corner (18, 26), an even column: the window centres that reach it inside
    # the tensor are itself and its neighbours (17, 26), (18, 25), (17, 25)
    assert hit[:, 3].sum(1).eq(4).all() and not hit[:, [0, 1, 2, 4, 5, 6, 7]].any()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    # N, C_in, C_out, H, W, kernel: planes that end inside a step of 16 pixels
    # (few tiles a block and many), a row of tiles cut at the bottom
    (20, 16, 24, 33, 41, "wgrad_any_k"), (60, 48, 40, 25, 45, "wgrad_any_k"),
    (9, 8, 16, 19, 27, "wgrad_f32_k"), (9, 2, 12, 37, 41, "bwd_smallc_k"),
    (9, 1, 20, 18, 40, "bwd_smallc_k")], ids=lambda c: "%d_%d_%d_%dx%d_%s" % c)
def test_infinity_stays_with_its_taps(case, dt):
    """An infinity in the last pixel of an image reaches the sums of the taps
    that read it from a centre inside the tensor, as an infinity, and no other
    sum: neither rows and pixels past a tile's end nor borders multiply it."""
    torch = torch_mod()
    from paper_1903_01814_amd import hexconv as hx
    N, Ci, Co, H, W, kernel = case
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(1)
    x = torch.rand((N, Ci, H, W), generator=g).to(tdt)
    dy = (torch.rand((N, Co, H, W), generator=g) + 0.5).to(tdt)
    c = Ci // 2
    for n in (0, N - 1):
        x[n, c, H - 1, W - 1] = float("inf")
    dw, db = torch.empty((Co, Ci, 7), device="cuda"), torch.empty(Co, device="cuda")
    nws = hx.hexconv_bwd_weight_workspace(N, Ci, Co, H, W, 1, 1, 0 if dt == "f32" else 1)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    hx.hexconv_timing_begin()
    try:
        hx.hexconv_bwd_weight(x.cuda(), dy.cuda(), dw, db, ws, 1, 1)
    finally:
        ran = hx.hexconv_timing_end()
    assert kernel in ran, ran
    dw = dw.cpu()
    nan = torch.isnan(dw).sum().item()
    assert nan == 0 and torch.isfinite(db).all().item()
    # centres that reach the corner from inside: itself, the pixel above, and
    # the left column's one (odd corner column) or two
    hit, want = torch.isinf(dw), 4 if W % 2 else 3
    assert hit[:, c].sum(1).unique().tolist() == [want]
    hit[:, c] = False
    assert hit.sum().item() == 0


@pytest.mark.parametrize("path", ["", "generic", "any", "few", "rows"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    # N, C_in, C_out, H, W, k: any width, few channels, whole 16-byte rows
    (2, 6, 9, 19, 27, 1), (2, 2, 9, 14, 24, 2), (2, 32, 32, 12, 16, 1),
    (2, 32, 32, 12, 16, 3)], ids=lambda c: "%d_%d_%d_%dx%d_k%d" % c)
def test_infinite_weight(case, dt, path, monkeypatch):
    """An infinite weight makes the outputs of its channel infinite where its
    tap lies inside the tensor; where the tap is padding, they are NaN or the
    sum of the other taps; other channels keep their sums.  Both directions."""
    monkeypatch.setenv("HEXCONV_PATH", path)
    N, Ci, Co, H, W, k = case
    rng = np.random.default_rng(800 + sum(case))
    T = oracle.num_taps(k)
    x = gen.round_to(rng.uniform(0.5, 1.0, size=(N, Ci, H, W)), dt)
    dy = gen.round_to(rng.uniform(0.5, 1.0, size=(N, Co, H, W)), dt)
    w = gen.round_to(rng.uniform(0.5, 1.0, size=(Co, Ci, T)), dt)
    co, ci, t = Co - 1, Ci // 2, 0
    one = np.zeros((1, 1, T))
    one[0, 0, t] = 1.0
    ones = np.ones((1, 1, H, W))
    wi, w0 = w.copy(), w.copy()
    wi[co, ci, t], w0[co, ci, t] = np.inf, 0.0
    for got, ref, inside, c in (
            (run_fwd(x, wi, None, k, 1, dt), oracle.conv_fwd(x, w0, None, k, 1),
             oracle.conv_fwd(ones, one, None, k, 1)[0, 0] > 0, co),
            (run_bwd_data(dy, wi, k, 1, H, W, dt), oracle.conv_bwd_data(dy, w0, k, 1, H, W),
             oracle.conv_bwd_data(ones, one, k, 1, H, W)[0, 0] > 0, ci)):
        assert 0 < inside.sum() < H * W
        hit = got[:, c]
        assert np.isposinf(hit[:, inside]).all()
        got[:, c][:, inside] = ref[:, c][:, inside]
        edge = np.isnan(got)
        assert not edge[:, np.arange(got.shape[1]) != c].any()
        check(dt, np.where(edge, ref, got), ref, ref, "finite sums")
