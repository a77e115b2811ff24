"""The work that a user of this library has it do, as cases to be timed.

Every case is one pass through the public entry points: the C ABI's binding
(``paper_1903_01814_amd.hexconv``) with buffers that the caller owns, as a
serving or training loop holds them, or the autograd layers
(``paper_1903_01814_amd.nn``).  ``listed()`` gives fixed cases, ``draw`` more
of the same ranges.  ``exact`` evaluates the definitions (HexagDLy,
arXiv:1903.01814, Sec. 2) in 64 bits with plain torch indexing and matrix
products.
"""
from __future__ import annotations

import math

import torch

from paper_1903_01814_amd import hexconv as hx
from paper_1903_01814_amd import nn as hnn

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
CODES = {"f32": hx.HEX_F32, "bf16": hx.HEX_BF16}


# ------------------------------------------------------------------- cases

def conv(name, N, Ci, Co, H, W, k, s, dtype, data, bwd=True):
    return dict(name=name, kind="conv", N=N, Ci=Ci, Co=Co, H=H, W=W, k=k, s=s, dtype=dtype,
                data=data, bwd=bwd)


def pool(name, N, C, H, W, k, s, dtype, mode, bwd):
    return dict(name=name, kind="pool", N=N, C=C, H=H, W=W, k=k, s=s, dtype=dtype, mode=mode,
                bwd=bwd)


def volume(name, N, Ci, Co, D, H, W, k, kz, dtype):
    return dict(name=name, kind="volume", N=N, Ci=Ci, Co=Co, D=D, H=H, W=W, k=k, kz=kz,
                dtype=dtype)


def listed():
    return [
        # a handful of small images through one layer: a serving call, whose
        # time is its launch
        conv("tiny_fwd_f32", 4, 1, 4, 16, 16, 1, 1, "f32", "uniform", bwd=False),
        # the first layer of a camera network in training, images on the
        # camera's square tensor
        conv("camera_f32", 256, 1, 16, 40, 40, 2, 1, "f32", "camera"),
        # the same for a camera whose tensor has odd sizes, with two values a
        # pixel (amplitude and time)
        conv("camera_odd_f32", 192, 2, 16, 45, 43, 1, 1, "f32", "camera"),
        # downsampling between layers in inference: max pool, then mean pool
        pool("pools_bf16", 256, 64, 40, 40, 1, 2, "bf16", "both", False),
        # a max pool in training on an odd grid
        pool("pool_odd_f32", 96, 48, 45, 51, 1, 2, "f32", "max", True),
        # a wide layer in training on large images: the largest case
        conv("wide_bf16", 64, 64, 64, 128, 128, 1, 1, "bf16", "normal"),
        # a wide layer of a camera network on an odd grid, widening
        conv("wide_odd_bf16", 96, 64, 96, 45, 51, 1, 1, "bf16", "normal"),
        # a wide layer that downsamples by its stride
        conv("wide_strided_bf16", 64, 64, 64, 128, 128, 1, 2, "bf16", "normal"),
        # a wide layer in torch's default dtype
        conv("wide_f32", 128, 32, 64, 40, 40, 1, 1, "f32", "normal"),
        # a whole camera network in training through the autograd layers
        dict(name="stack_bf16", kind="stack", N=512, H=48, W=48, dtype="bf16"),
        # the first 3-D layer over time-resolved camera events, in training
        volume("volume_f32", 64, 1, 16, 32, 40, 40, 1, 1, "f32"),
        # the next block of that network through the autograd layers: 3-D max
        # pool of stride 2 in the plane and along time, then a wider layer
        dict(name="volume_block_f32", kind="volume_block", N=32, Ci=16, Co=32, D=16, H=40, W=40,
             k=1, kz=1, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["serve", "camera", "pool", "wide", "wide", "stack", "volume",
                       "volume_block"])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "serve":
        c = conv("", _log(rng, 1, 8), rng.randint(1, 4), rng.randint(4, 16), rng.randint(12, 48),
                 rng.randint(12, 48), rng.choice([1, 1, 2]), rng.choice([1, 1, 2]), dtype,
                 "uniform", bwd=False)
    elif kind == "camera":
        c = conv("", _log(rng, 24, 320), rng.randint(1, 4), rng.choice([8, 12, 16, 24, 32]),
                 rng.randint(24, 56), rng.randint(24, 56), rng.choice([1, 2]), 1, dtype, "camera")
    elif kind == "pool":
        c = pool("", _log(rng, 16, 200), rng.choice([8, 16, 24, 32, 48, 64]), rng.randint(20, 56),
                 rng.randint(20, 56), rng.choice([1, 1, 2]), rng.choice([2, 2, 3]), dtype,
                 rng.choice(["max", "max", "both"]), rng.random() < 0.6)
    elif kind == "wide":
        s = rng.choice([1, 1, 2])
        size = rng.randint(24, 96) if dtype == "bf16" else rng.randint(20, 48)
        c = conv("", _log(rng, 8, 64), rng.choice([16, 32, 48, 64, 96]),
                 rng.choice([16, 32, 48, 64, 96]), size, max(16, size + rng.randint(-6, 6)),
                 rng.choice([1, 1, 2]), s, dtype, "normal")
    elif kind == "stack":
        c = dict(kind="stack", N=_log(rng, 32, 384), H=rng.randint(32, 56), W=rng.randint(32, 56),
                 dtype=dtype)
    elif kind == "volume":
        c = volume("", _log(rng, 4, 48), rng.choice([1, 1, 2]), rng.choice([8, 12, 16]),
                   rng.randint(8, 32), rng.randint(24, 44), rng.randint(24, 44), 1, 1, dtype)
    else:
        c = dict(kind="volume_block", N=_log(rng, 4, 24), Ci=rng.choice([8, 12, 16]),
                 Co=rng.choice([16, 24, 32]), D=rng.randint(8, 20), H=rng.randint(24, 44),
                 W=rng.randint(24, 44), k=1, kz=1, dtype=dtype)
    c.pop("name", None)
    most = 18e9 if dtype == "f32" else 60e9  # operations: within the largest listed case's cost
    while c["N"] > 1 and work(c)["flops"] > most:
        c["N"] = (c["N"] + 1) // 2
    return c


# ------------------------------------------------------------------ inputs

class _Gen:
    """Inputs drawn on the device from the seed alone, rounded to the dtype."""

    def __init__(self, case, seed):
        self.dev = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
        self.g = torch.Generator(device=self.dev).manual_seed(seed)
        self.dt = DTYPES[case["dtype"]]

    def normal(self, shape, std=1.0):
        t = torch.randn(shape, generator=self.g, device=self.dev)
        return (t * std).to(self.dt)

    def data(self, shape, dist):
        if dist == "normal":
            return self.normal(shape)
        u = torch.rand(shape, generator=self.g, device=self.dev)
        if dist == "uniform":
            return u.to(self.dt)
        # sparse positive camera images: log-normal amplitudes in a tenth of
        # the pixels
        amp = torch.randn(shape, generator=self.g, device=self.dev).exp_()
        return (amp * (u < 0.1)).to(self.dt)

    def weight(self, *shape):
        return self.normal(shape, math.sqrt(2.0 / math.prod(shape[1:])))  # He, hexagonal fan-in


def _taps(k):
    return 1 + 3 * k * (k + 1)


def _out(H, W, s):
    Wo = (W - 1) // s + 1
    Ho = (H - 1 - (s // 2 if Wo > 1 else 0)) // s + 1
    return Ho, Wo


STACK = [("conv", 1, 32, 2, True), ("pool",), ("conv", 32, 64, 2, False), ("pool",),
         ("conv", 64, 128, 1, False)]


def _stack_sizes(c):
    h, w = c["H"], c["W"]
    sizes = []
    for layer in STACK:
        o = _out(h, w, 2) if layer[0] == "pool" else (h, w)
        sizes.append(((h, w), o))
        h, w = o
    return sizes


def _inputs(c, seed):
    """Every input of a case, in the order they are drawn."""
    g = _Gen(c, seed)
    kind = c["kind"]
    if kind == "conv":
        Ho, Wo = _out(c["H"], c["W"], c["s"])
        d = dict(x=g.data((c["N"], c["Ci"], c["H"], c["W"]), c["data"]),
                 w=g.weight(c["Co"], c["Ci"], _taps(c["k"])), b=g.normal((c["Co"],), 0.1))
        if c["bwd"]:
            d["dy"] = g.normal((c["N"], c["Co"], Ho, Wo))
        return d
    if kind == "pool":
        Ho, Wo = _out(c["H"], c["W"], c["s"])
        d = dict(x=g.data((c["N"], c["C"], c["H"], c["W"]), "normal"))
        if c["bwd"]:
            d["dy"] = g.normal((c["N"], c["C"], Ho, Wo))
        return d
    if kind == "stack":
        d = dict(x=g.data((c["N"], 1, c["H"], c["W"]), "camera"), w=[], b=[])
        for layer in STACK:
            if layer[0] == "conv":
                d["w"].append(g.weight(layer[2], layer[1], _taps(layer[3])))
                d["b"].append(g.normal((layer[2],), 0.1))
        d["dy"] = g.normal((c["N"], 128) + _stack_sizes(c)[-1][1])
        return d
    Z, T = 2 * c["kz"] + 1, _taps(c["k"])
    D, (Ho, Wo) = c["D"], (c["H"], c["W"])
    if kind == "volume_block":
        D, (Ho, Wo) = (D - 1) // 2 + 1, _out(c["H"], c["W"], 2)
    dist = "camera" if kind == "volume" else "normal"
    return dict(x=g.data((c["N"], c["Ci"], c["D"], c["H"], c["W"]), dist),
                w=g.weight(c["Co"], c["Ci"], Z, T), b=g.normal((c["Co"],), 0.1),
                dy=g.normal((c["N"], c["Co"], D, Ho, Wo)))


def _ws(nbytes, dev):
    return torch.empty((nbytes,), dtype=torch.uint8, device=dev) if nbytes else None


def prepare(case, seed):
    c = case
    st = dict(_inputs(c, seed), case=c)
    x = st["x"]
    dev, code, kind = x.device, CODES[c["dtype"]], c["kind"]
    f32 = dict(dtype=torch.float32, device=dev)
    if kind == "conv":
        st["y"] = x.new_empty((c["N"], c["Co"]) + _out(c["H"], c["W"], c["s"]))
        if c["bwd"]:
            st.update(dx=torch.empty_like(x), dw=torch.empty(st["w"].shape, **f32),
                      db=torch.empty((c["Co"],), **f32),
                      ws=_ws(hx.hexconv_bwd_workspace(c["N"], c["Ci"], c["Co"], c["H"], c["W"],
                                                      c["k"], c["s"], code), dev))
    elif kind == "pool":
        shape = (c["N"], c["C"]) + _out(c["H"], c["W"], c["s"])
        st.update(ymax=x.new_empty(shape), am=torch.empty(shape, dtype=torch.uint8, device=dev))
        if c["mode"] == "both":
            st["yavg"] = x.new_empty(shape)
        if c["bwd"]:
            st.update(dxmax=torch.empty_like(x))
            if c["mode"] == "both":
                st.update(dxavg=torch.empty_like(x))
    elif kind == "volume":
        st.update(y=x.new_empty((c["N"], c["Co"], c["D"], c["H"], c["W"])),
                  dx=torch.empty_like(x), dw=torch.empty(st["w"].shape, **f32),
                  db=torch.empty((c["Co"],), **f32),
                  ws=_ws(hx.hexconv3d_bwd_weight_workspace(
                      c["N"], c["Ci"], c["Co"], c["D"], c["H"], c["W"], c["k"], c["kz"], 1, 1,
                      code), dev))
    elif kind == "stack":
        layers, i = [], 0
        for layer in STACK:
            if layer[0] == "pool":
                layers.append(hnn.HexMaxPool2d(1, 2))
                continue
            m = hnn.HexConv2d(layer[1], layer[2], layer[3], relu=layer[4], device=dev,
                              dtype=x.dtype)
            m.weight.data.copy_(st["w"][i])
            m.bias.data.copy_(st["b"][i])
            layers.append(m)
            i += 1
        st["net"] = torch.nn.Sequential(*layers)
        st["params"] = list(st["net"].parameters())
    else:
        m = hnn.HexConv3d(c["Ci"], c["Co"], (c["k"], c["kz"]), device=dev, dtype=x.dtype,
                          relu=True)
        m.weight.data.copy_(st["w"])
        m.bias.data.copy_(st["b"])
        st["net"] = torch.nn.Sequential(hnn.HexMaxPool3d((1, 1), (2, 2)), m)
        st["params"] = list(st["net"].parameters())
        st["x"] = x.requires_grad_(True)
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "conv":
        k, s = c["k"], c["s"]
        hx.hexconv_fwd(st["x"], st["w"], st["b"], st["y"], k, s)
        if not c["bwd"]:
            return st["y"]
        hx.hexconv_bwd(st["x"], st["dy"], st["w"], st["dx"], st["dw"], st["db"], st["ws"], k, s)
        return st["y"], st["dx"], st["dw"], st["db"]
    if kind == "pool":
        k, s = c["k"], c["s"]
        out = []
        if c["bwd"]:
            hx.hexpool_fwd(st["x"], st["ymax"], st["am"], k, s, hx.HEX_POOL_MAX)
            hx.hexpool_bwd(st["dy"], st["am"], None, st["dxmax"], k, s, hx.HEX_POOL_MAX)
            out += [st["ymax"], st["am"], st["dxmax"]]
        else:
            hx.hexpool_fwd(st["x"], st["ymax"], None, k, s, hx.HEX_POOL_MAX)
            out += [st["ymax"]]
        if c["mode"] == "both":
            hx.hexpool_fwd(st["x"], st["yavg"], None, k, s, hx.HEX_POOL_AVG)
            out += [st["yavg"]]
            if c["bwd"]:
                hx.hexpool_bwd(st["dy"], None, None, st["dxavg"], k, s, hx.HEX_POOL_AVG)
                out += [st["dxavg"]]
        return out
    if kind == "volume":
        k, kz = c["k"], c["kz"]
        hx.hexconv3d_fwd(st["x"], st["w"], st["b"], st["y"], k, kz, 1, 1)
        hx.hexconv3d_bwd_data(st["dy"], st["w"], st["dx"], k, kz, 1, 1)
        hx.hexconv3d_bwd_weight(st["x"], st["dy"], st["dw"], st["db"], st["ws"], k, kz, 1, 1)
        return st["y"], st["dx"], st["dw"], st["db"]
    y = st["net"](st["x"])
    wanted = st["params"] + ([st["x"]] if kind == "volume_block" else [])
    return [y.detach()] + list(torch.autograd.grad(y, wanted, st["dy"]))


# -------------------------------------------------------------------- work

def _conv_work(c, e, N, Ci, Co, P, Po, taps, grads):
    """Bytes and operations of a layer: forward, and with `grads` ("w" or
    "xw") its gradients; P and Po input and output elements per channel."""
    x, y, w = N * Ci * P, N * Co * Po, Co * Ci * taps
    byts = (x + w + Co + y) * e
    flops = 2 * N * Po * Co * Ci * taps
    if grads:
        byts += (x + y) * e + (w + Co) * 4
        flops *= 2
        if "x" in grads:
            byts += (w + x) * e
            flops += flops // 2
    return byts, flops


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    kind = c["kind"]
    if kind == "conv":
        Ho, Wo = _out(c["H"], c["W"], c["s"])
        b, f = _conv_work(c, e, c["N"], c["Ci"], c["Co"], c["H"] * c["W"], Ho * Wo,
                          _taps(c["k"]), "xw" if c["bwd"] else "")
        return {"bytes": b, "flops": f}
    if kind == "pool":
        Ho, Wo = _out(c["H"], c["W"], c["s"])
        x, y = c["N"] * c["C"] * c["H"] * c["W"], c["N"] * c["C"] * Ho * Wo
        passes = 2 if c["mode"] == "both" else 1
        b = passes * (x + y) * e
        if c["bwd"]:
            b += 2 * y + passes * (x + y) * e  # argmax written and read; dy read, dx written
        return {"bytes": b, "flops": passes * y * _taps(c["k"])}
    if kind == "volume":
        P = c["D"] * c["H"] * c["W"]
        b, f = _conv_work(c, e, c["N"], c["Ci"], c["Co"], P, P, (2 * c["kz"] + 1) * _taps(c["k"]),
                          "xw")
        return {"bytes": b, "flops": f}
    if kind == "stack":
        b = f = 0
        C = 1
        first = True
        for layer, ((h, w), (ho, wo)) in zip(STACK, _stack_sizes(c)):
            if layer[0] == "conv":
                bb, ff = _conv_work(c, e, c["N"], layer[1], layer[2], h * w, ho * wo,
                                    _taps(layer[3]), "w" if first else "xw")
                if layer[4]:
                    bb += c["N"] * layer[2] * ho * wo * e  # the output's signs, for the gradient
                C, first = layer[2], False
            else:
                n = c["N"] * C
                bb = 2 * n * (h * w + ho * wo) * e + 2 * n * ho * wo
                ff = n * ho * wo * 7
            b, f = b + bb, f + ff
        return {"bytes": b, "flops": f}
    D, (Ho, Wo) = (c["D"] - 1) // 2 + 1, _out(c["H"], c["W"], 2)
    P, Po = c["D"] * c["H"] * c["W"], D * Ho * Wo
    n = c["N"] * c["Ci"]
    b, f = _conv_work(c, e, c["N"], c["Ci"], c["Co"], Po, Po, (2 * c["kz"] + 1) * _taps(c["k"]),
                      "xw")
    b += c["N"] * c["Co"] * Po * e + 2 * n * (P + Po) * e + 4 * n * Po
    return {"bytes": b, "flops": f + n * Po * 21}


def tolerance(case):
    c = case
    kind = c["kind"]
    if kind == "pool":
        # maxima and their taps are exact; the gradient adds up to seven
        # terms, the mean 7 or 19
        if c["dtype"] == "f32":
            return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
        return {"rel": 2e-3, "max": 2e-2, "differ": 0.0}
    if kind == "stack":
        # a 1-ulp change in one layer moves some maxima of the pools after it
        if c["dtype"] == "f32":
            return {"rel": 1e-3, "max": 0.9}
        return {"rel": 1e-2, "max": 0.9}
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 5e-3, "max": 5e-2}


# ------------------------------------------------------------------- exact

def _index(D, H, W, k, kz, s, sz):
    """Flat input index of every (dz, tap) of every output element, D*H*W
    where the tap lies outside: [Z * T][Do * Ho * Wo]."""
    Ho, Wo = _out(H, W, s)
    Do = (D - 1) // sz + 1
    l = torch.arange(Do).view(-1, 1, 1)
    i = torch.arange(Ho).view(1, -1, 1)
    j = torch.arange(Wo).view(1, 1, -1)
    c0 = s * j
    s0 = s * i + (j % 2) * (s // 2) - c0 // 2  # axial (q, s) = (c, r - floor(c / 2))
    rows = []
    for dz in range(-kz, kz + 1):
        for dq in range(-k, k + 1):
            for ds in range(-k, k + 1):
                if max(abs(dq), abs(ds), abs(dq + ds)) > k:
                    continue
                z, col = sz * l + dz, c0 + dq
                r = s0 + ds + torch.div(col, 2, rounding_mode="floor")
                ok = (z >= 0) & (z < D) & (col >= 0) & (col < W) & (r >= 0) & (r < H)
                rows.append(torch.where(ok, (z * H + r) * W + col, D * H * W).reshape(-1))
    return rows


def _rows(x):
    """[N][C][...] -> [C][N][P + 1] float64 with a zero behind every image."""
    n, ch = x.shape[:2]
    flat = x.double().reshape(n, ch, -1).transpose(0, 1)
    return torch.nn.functional.pad(flat, (0, 1))


def _conv64(x, w, b, idx, shape):
    xr = _rows(x)
    ci, n, _ = xr.shape
    w = w.double().reshape(w.shape[0], ci, -1)
    y = b.double().view(-1, 1).expand(-1, n * idx[0].numel()).clone()
    for t, ix in enumerate(idx):
        y += w[:, :, t].contiguous() @ xr[:, :, ix.to(x.device)].reshape(ci, -1)
    return y.view(w.shape[0], n, -1).transpose(0, 1).reshape((n, w.shape[0]) + tuple(shape))


def _conv64_bwd(x, w, dy, idx):
    xr = _rows(x)
    ci, n, p1 = xr.shape
    co = w.shape[0]
    w3 = w.double().reshape(co, ci, -1)
    g = dy.double().reshape(n, co, -1).transpose(0, 1).reshape(co, -1)
    dx = torch.zeros_like(xr)
    dw = torch.empty_like(w3)
    for t, ix in enumerate(idx):
        ix = ix.to(x.device)
        dw[:, :, t] = g @ xr[:, :, ix].reshape(ci, -1).T.contiguous()
        dx.index_add_(2, ix, (w3[:, :, t].T.contiguous() @ g).view(ci, n, -1))
    dx = dx[:, :, :p1 - 1].transpose(0, 1).reshape(x.shape)
    return dx, dw.view(w.shape), g.sum(1)


def _max64(x, idx, shape):
    xr = _rows(x)
    best = arg = None
    for t, ix in enumerate(idx):
        v = xr[:, :, ix.to(x.device)]
        if best is None:
            best, arg = v, torch.zeros(v.shape, dtype=torch.int64, device=x.device)
        else:
            m = v > best
            best = torch.where(m, v, best)
            arg = torch.where(m, t, arg)
    full = (x.shape[0], x.shape[1]) + tuple(shape)
    return best.transpose(0, 1).reshape(full), arg.transpose(0, 1).reshape(full)


def _max64_bwd(x, arg, dy, idx):
    n, ch = x.shape[:2]
    at = torch.stack([ix.to(x.device) for ix in idx])  # [T][P]
    a = arg.reshape(n * ch, -1)
    to = at.gather(0, a)
    dx = torch.zeros((n * ch, x[0, 0].numel() + 1), dtype=torch.float64, device=x.device)
    dx.scatter_add_(1, to, dy.double().reshape(n * ch, -1))
    return dx[:, :-1].reshape(x.shape)


def exact(case, seed):
    c = case
    d = _inputs(c, seed)
    kind = c["kind"]
    if kind == "conv":
        idx = _index(1, c["H"], c["W"], c["k"], 0, c["s"], 1)
        y = _conv64(d["x"], d["w"], d["b"], idx, _out(c["H"], c["W"], c["s"]))
        return (y,) + _conv64_bwd(d["x"], d["w"], d["dy"], idx) if c["bwd"] else y
    if kind == "pool":
        shape = _out(c["H"], c["W"], c["s"])
        idx = _index(1, c["H"], c["W"], c["k"], 0, c["s"], 1)
        y, arg = _max64(d["x"], idx, shape)
        out = [y]
        if c["bwd"]:
            out += [arg, _max64_bwd(d["x"], arg, d["dy"], idx)]
        if c["mode"] == "both":
            n, ch = c["N"], c["C"]
            w = torch.full((1, 1, len(idx)), 1.0 / len(idx), dtype=torch.float64,
                           device=d["x"].device)
            zero = torch.zeros(1, device=w.device)
            flat = d["x"].reshape(n * ch, 1, c["H"], c["W"])
            out.append(_conv64(flat, w, zero, idx, shape).reshape((n, ch) + shape))
            if c["bwd"]:
                g = d["dy"].reshape((n * ch, 1) + shape)
                out.append(_conv64_bwd(flat, w, g, idx)[0].reshape(d["x"].shape))
        return out
    if kind == "volume":
        idx = _index(c["D"], c["H"], c["W"], c["k"], c["kz"], 1, 1)
        y = _conv64(d["x"], d["w"], d["b"], idx, (c["D"], c["H"], c["W"]))
        return (y,) + _conv64_bwd(d["x"], d["w"], d["dy"], idx)
    # the networks: what passes between two layers is rounded to the case's
    # dtype, which is what the layers hand on
    dt = d["x"].dtype
    if kind == "volume_block":
        D1, hw1 = (c["D"] - 1) // 2 + 1, _out(c["H"], c["W"], 2)
        idx0 = _index(c["D"], c["H"], c["W"], 1, 1, 2, 2)
        idx1 = _index(D1, hw1[0], hw1[1], c["k"], c["kz"], 1, 1)
        p, arg = _max64(d["x"], idx0, (D1,) + hw1)
        y = _conv64(p, d["w"], d["b"], idx1, (D1,) + hw1).clamp_min(0.0)
        g = d["dy"] * (y.to(dt) > 0)
        dp, dw, db = _conv64_bwd(p, d["w"], g, idx1)
        return [y, dw, db, _max64_bwd(d["x"], arg, dp.to(dt), idx0)]
    x, acts, i = d["x"], [], 0
    for layer, ((h, w), o) in zip(STACK, _stack_sizes(c)):
        idx = _index(1, h, w, 1 if layer[0] == "pool" else layer[3], 0,
                     2 if layer[0] == "pool" else 1, 1)
        if layer[0] == "pool":
            y, arg = _max64(x, idx, o)
            acts.append((x, arg, idx, None))
        else:
            y = _conv64(x, d["w"][i], d["b"][i], idx, o)
            y = y.clamp_min(0.0) if layer[4] else y
            acts.append((x, i, idx, y.to(dt) if layer[4] else None))
            i += 1
        x = y.to(dt)
    grads, g = {}, d["dy"]
    for n, (layer, (a, b, idx, relu)) in reversed(list(enumerate(zip(STACK, acts)))):
        if layer[0] == "pool":
            g = _max64_bwd(a, b, g, idx).to(dt)
            continue
        if relu is not None:
            g = g * (relu > 0)
        dx, dw, db = _conv64_bwd(a, d["w"][b], g, idx)
        grads[b] = [dw, db]
        g = dx.to(dt)
    return [y] + [t for b in sorted(grads) for t in grads[b]]
