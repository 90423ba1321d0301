"""What users of this library have it do, as cases that can be timed.

A case is one call sequence of a program built on the package: a layer's forward pass ("infer") or its forward and
backward pass ("train"), on tensors that are already on the GPU and with the grid handle (and the parameters) made
once beforehand.  Calls are the plain ones of the binding: outputs and scratch are left to the default, torch's
caching allocator.

`listed()` holds the shapes of the library's own workloads, the two layers around them and a few general ones;
`draw()` gives further cases of the same ranges: any latitude and longitude count (odd ones too), the head widths 16,
32 and 64, float32 and bf16 tensors, equal grids, 2:1 downsampling and 1:2 upsampling, cutoffs of two to seven grid
spacings, few and many (batch, head) slices.
"""
import math

import numpy as np
import torch

import paper_2505_11157_amd as S

EQUIANGULAR, GAUSS = S.S2_GRID_EQUIANGULAR, S.S2_GRID_LEGENDRE_GAUSS


def _case(layer, op, grid, sizes, theta, batch, dtype, **more):
    lat_in, lon_in, lat_out, lon_out = sizes
    return dict(layer=layer, op=op, grid=grid, nlat_in=lat_in, nlon_in=lon_in, nlat_out=lat_out, nlon_out=lon_out,
                theta=theta, batch=batch, dtype=dtype, **more)


def _nattn(op, grid, sizes, theta, batch, heads, d, dtype, **more):
    return _case("nattn", op, grid, sizes, theta, batch, dtype, heads=heads, d=d, **more)


def _global(op, grid, nlat, nlon, batch, heads, **more):
    # the cutoff of the handle plays no part in the global variant; bf16 and d = 64 are what it takes
    return _case("global", op, grid, (nlat, nlon) * 2, math.pi, batch, "bf16", heads=heads, d=64, **more)


def _mha(op, grid, nlat, nlon, theta, batch, channels, heads, **more):
    return _case("mha", op, grid, (nlat, nlon) * 2, theta, batch, "f32", channels=channels, heads=heads, **more)


def _disco(op, grid, sizes, theta, batch, cin, cout, nbasis, **more):
    return _case("disco", op, grid, sizes, theta, batch, "f32", cin=cin, cout=cout, nbasis=nbasis, **more)


def listed():
    pi, swe, down, up = math.pi, (129, 256) * 2, (257, 512, 129, 256), (129, 256, 257, 512)
    return [
        # a toy model or a unit test (workload 1): nothing but launches and the host path
        _nattn("train", EQUIANGULAR, (17, 32) * 2, pi / 8, 1, 1, 8, "f32", name="tiny_train"),
        # inference of a medium layer on the Gaussian grid (workload 2): a launch that barely fills the chip
        _nattn("infer", GAUSS, (64, 128) * 2, 7 * pi / 64, 2, 4, 32, "f32", name="gauss64_infer"),
        # training step of the shallow-water-sized layer (workload 3, the headline of the benchmark)
        _nattn("train", EQUIANGULAR, swe, 4 * pi / 128, 4, 8, 32, "f32", name="swe129_train"),
        # the same layer on bf16 tensors (workload 7)
        _nattn("train", EQUIANGULAR, swe, 4 * pi / 128, 4, 8, 32, "bf16", name="swe129_bf16_train"),
        # the same layer with wide heads (workload 9)
        _nattn("train", EQUIANGULAR, swe, 4 * pi / 128, 4, 8, 64, "f32", name="swe129_d64_train"),
        # an encoder's downsampling layer (workload 4)
        _nattn("train", EQUIANGULAR, down, 2 * pi / 128, 2, 4, 32, "f32", name="down257_train"),
        # a decoder's upsampling layer (workload 6)
        _nattn("train", EQUIANGULAR, up, 2 * pi / 128, 2, 4, 32, "f32", name="up257_train"),
        # inference on a two-degree grid (91 x 180: no power of two anywhere), bf16, narrow heads
        _nattn("infer", EQUIANGULAR, (91, 180) * 2, 4 * pi / 90, 2, 8, 16, "bf16", name="twodeg_bf16_infer"),
        # training step of the global layer (workload 5): the largest product
        _global("train", EQUIANGULAR, 65, 128, 4, 8, name="global65_train"),
        # inference of a small global layer, one sample, a token count that is no multiple of any tile
        _global("infer", EQUIANGULAR, 46, 90, 1, 4, name="global46_infer"),
        # training step of the attention sub-block with the head width of the paper's segmentation models
        _mha("train", EQUIANGULAR, 129, 256, 4 * pi / 128, 4, 128, 8, name="mha129_train"),
        # training step of the DISCO convolution
        _disco("train", EQUIANGULAR, swe, 4 * pi / 128, 4, 64, 64, 9, name="disco129_train"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_sizes(rng, lo, hi, multiple=1):
    """A latitude count spread over its logarithm and about twice as many longitudes (a multiple of `multiple`)."""
    gt = rng.choice((EQUIANGULAR, EQUIANGULAR, GAUSS))
    nlat = _log_int(rng, lo, hi)
    nlon = 2 * (nlat - 1) if gt == EQUIANGULAR else 2 * nlat
    if multiple == 1 and rng.random() < 0.25:
        nlon = max(8, nlon + rng.choice((-3, -1, 1, 3)))
    return gt, nlat, max(multiple, nlon // multiple * multiple)


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = {}                                              # no drawn case is larger than the layer's largest listed one
    for c in listed():
        most[c["layer"]] = max(most.get(c["layer"], 0.0), _cost(c))
    while True:
        op = rng.choice(("infer", "train"))
        kind = rng.choices(("equal", "resample", "global", "mha", "disco"), (10, 4, 3, 2, 2))[0]
        batch, heads = rng.choice((1, 2, 3, 4)), rng.choice((1, 2, 4, 6, 8))
        d, dtype = rng.choice((16, 32, 32, 64)), rng.choice(("f32", "bf16"))
        nlat_most = {"equal": 181, "global": 65}.get(kind, 129)
        grid, nlat, nlon = _grid_sizes(rng, 16, nlat_most, 16 if kind in ("mha", "disco") else 1)
        fine = (2 * nlat - 1 if grid == EQUIANGULAR else 2 * nlat, 2 * nlon)
        # cutoffs in latitude spacings: of the grid itself, or of the coarse one of two
        near, coarse = rng.uniform(2.0, 7.0) * math.pi / nlat, rng.uniform(1.5, 3.0) * math.pi / nlat
        if kind == "equal":
            c = _nattn(op, grid, (nlat, nlon) * 2, near, batch, heads, d, dtype)
        elif kind == "resample":
            sizes = rng.choice((fine + (nlat, nlon), (nlat, nlon) + fine))
            c = _nattn(op, grid, sizes, coarse, batch, heads, d, dtype)
        elif kind == "global":
            c = _global(op, grid, nlat, nlon, batch, heads)
        elif kind == "mha":
            width, heads = rng.choice((16, 32)), rng.choice((4, 6, 8))
            c = _mha(op, grid, nlat, nlon, near, batch, width * heads, heads)
        else:
            sizes, theta = rng.choice((((nlat, nlon) * 2, near), (fine + (nlat, nlon), coarse)))
            c = _disco(op, grid, sizes, theta, batch, rng.choice((16, 32, 48, 64)), rng.choice((32, 64, 96)),
                       rng.choice((4, 7, 9)))
        if _cost(c) <= most[c["layer"]]:
            return c


def _theta_nodes(gt, n):
    if gt == GAUSS:
        return np.arccos(np.polynomial.legendre.leggauss(n)[0])[::-1]
    return math.pi * np.arange(n) / (n - 1)


def _pairs(c):
    """(output, input) pairs of one (batch, head) slice: the points of every disk, latitude by latitude."""
    a, b = (_theta_nodes(c["grid"], c[k])[s] for k, s in (("nlat_out", np.s_[:, None]), ("nlat_in", np.s_[None, :])))
    x = math.cos(c["theta"] + 1e-9) - np.cos(a) * np.cos(b)
    s = np.sin(a) * np.sin(b)
    half = np.where(x <= -s, math.pi, np.where(x > s, -1.0, np.arccos(np.clip(x / np.maximum(s, 1e-300), -1, 1))))
    step = 2 * math.pi / c["nlon_in"]
    n = np.where(half < 0, 0, np.minimum(c["nlon_in"], 2 * np.floor(half / step) + 1))
    return float(n.sum()) * c["nlon_out"]


def work(case):
    """Operations of the contractions and bytes of the inputs and outputs, each once."""
    c, train = case, case["op"] == "train"
    n_in, n_out = c["nlat_in"] * c["nlon_in"], c["nlat_out"] * c["nlon_out"]
    if c["layer"] in ("nattn", "global"):
        bh, d, size = c["batch"] * c["heads"], c["d"], 2 if c["dtype"] == "bf16" else 4
        pairs = n_in * n_out if c["layer"] == "global" else _pairs(c)
        # q, k, v -> out, lse; and dout -> dq, dk, dv
        elements = 2 * n_out + 2 * n_in + (2 * n_out + 2 * n_in if train else 0)
        return {"flops": (14.0 if train else 4.0) * d * pairs * bh, "bytes": bh * (size * d * elements + 4.0 * n_out)}
    B = c["batch"]
    if c["layer"] == "mha":
        C = c["channels"]
        flops = B * (8.0 * C * C * n_in * (3 if train else 1) + (14.0 if train else 4.0) * C * _pairs(c))
        planes = (2 * B + 1 + (2 * B + 1 if train else 0)) * C * n_in        # x, y, pos; dy, dx, dpos
        return {"flops": flops, "bytes": 4.0 * (planes + (8 if train else 4) * C * C)}
    cin, cout, K = c["cin"], c["cout"], c["nbasis"]
    gather, mix = 2.0 * cin * K * _pairs(c), 2.0 * cin * K * cout * n_out
    x, y, w = cin * n_in, cout * n_out, cin * cout * K
    return {"flops": B * ((2 * gather + 3 * mix) if train else (gather + mix)),
            "bytes": 4.0 * (B * (x + y) + w) * (2 if train else 1)}


def tolerance(case):
    # bf16 tensors carry 8 bits; float32 sums of up to some thousand terms, chained three to five deep in the layers
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 2e-5 if case["layer"] == "mha" else 1e-5, "max": 5e-4}


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    grid = S.s2_grid_init(c["grid"], c["nlat_in"], c["nlon_in"], c["nlat_out"], c["nlon_out"], c["theta"])
    st = {"layer": c["layer"], "train": c["op"] == "train", "grid": grid}
    B, n_in, n_out = c["batch"], (c["nlat_in"], c["nlon_in"]), (c["nlat_out"], c["nlon_out"])
    if c["layer"] in ("nattn", "global"):
        H, d = c["heads"], c["d"]
        if c["layer"] == "global":
            s_in = s_out = (B, H, n_in[0] * n_in[1], d)
        else:
            s_in, s_out = (B, H, d) + n_in, (B, H, d) + n_out
        cast = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        st.update(scale=1 / math.sqrt(d), q=rnd(*s_out).to(cast), k=rnd(*s_in).to(cast), v=rnd(*s_in).to(cast))
        if st["train"]:
            st["dout"] = rnd(*s_out).to(cast)
    elif c["layer"] == "mha":
        C = c["channels"]
        # no key bias: it shifts all logits of a query alike, so its gradient is zero
        p = {"gamma": 1 + 0.3 * rnd(C), "beta": 0.3 * rnd(C), "pos": 0.5 * rnd(C, *n_in)}
        for n in "qkvo":
            p["W" + n] = rnd(C, C) / math.sqrt(C)
        for n in "qvo":
            p["b" + n] = 0.3 * rnd(C)
        st.update(heads=c["heads"], params=p, x=rnd(B, C, *n_in))
        if st["train"]:
            st["dy"] = rnd(B, C, *n_in)
    else:
        cin, cout, K = c["cin"], c["cout"], c["nbasis"]
        st.update(disco=S.s2_disco_init(grid, K), x=rnd(B, cin, *n_in), weight=rnd(cout, cin, K) / math.sqrt(cin * K),
                  bias=rnd(cout))
        if st["train"]:
            st["dy"] = rnd(B, cout, *n_out)
    return st


def run(st):
    if st["layer"] == "nattn":
        g, q, k, v, scale = st["grid"], st["q"], st["k"], st["v"], st["scale"]
        out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
        return (out, lse) + (S.s2_nattn_bwd(g, q, k, v, out, lse, st["dout"], scale) if st["train"] else ())
    if st["layer"] == "global":
        g, q, k, v, scale = st["grid"], st["q"], st["k"], st["v"], st["scale"]
        out, lse = S.s2_attn_global_fwd(g, q, k, v, scale)
        return (out, lse) + (S.s2_attn_global_bwd(g, q, k, v, out, lse, st["dout"], scale) if st["train"] else ())
    if st["layer"] == "mha":
        y, ws = S.s2_mha_fwd(st["grid"], st["x"], st["params"], st["heads"])
        return (y,) + (S.s2_mha_bwd(st["grid"], st["x"], st["params"], st["heads"], st["dy"], ws) if st["train"] else ())
    y, ws = S.s2_disco_fwd(st["disco"], st["x"], st["weight"], st["bias"])
    return (y,) + (S.s2_disco_bwd(st["disco"], st["x"], st["weight"], st["dy"], ws) if st["train"] else ())
