"""Performance cases: the work that programs built on this package have it do,
each through its public entry points.

``listed()`` names the fixed cases, ``draw(rng)`` gives further ones of the
same ranges, ``prepare`` builds what a program holds before the call (inputs
from the seed, the solver handle or the network with its buffers), ``run`` is
one pass, ``work`` the bytes and operations no implementation can do without,
and ``exact`` the same outputs in 64-bit arithmetic, written with plain torch.

Kinds of case
  smooth    red-black sweeps on the finest level (a program's own cycle)
  residual  residual field and norms (judging an iterate or a prediction)
  vcycle    one V(2,2) cycle from a zero guess (a preconditioner's call)
  solve     adaptive solve to a tolerance from a zero guess
  step      one time step of a moving body: new faces, then the FP64
            refinement solve around FP32 cycles
  batch     many uneven problems refined together
  conv      one forward convolution of the network (with bias and ReLU)
  conv_bwd  one layer's backward: ReLU gate, weight, bias and data gradients
  infer     the network's warm start of one problem
  train     forward and backward of the network on one batch
"""
import math

import torch

from paper_2607_07687_amd import gmg as G
from paper_2607_07687_amd import unet as UN
from paper_2607_07687_amd import unet_net as NET

DEV = "cuda"
STORE = {"f32": G.GMG_F32, "f64": G.GMG_F64, "bf16": G.GMG_BF16}
LAYERS = [(8, 16), (16, 16), (32, 16), (16, 32), (32, 32), (64, 32), (32, 64), (64, 64),
          (128, 64), (64, 128), (128, 128)]


def listed():
    return [
        # two sweeps on a mid-sized uneven grid: the smoother alone
        dict(name="smooth_200x120x88_f32", kind="smooth", nx=200, ny=120, nz=88, prec="f32",
             store="f32", per="", sweeps=2),
        # the 512 x 192 x 192 channel's residual with both norms: the largest
        # single pass over memory
        dict(name="residual_channel_512x192x192_f32", kind="residual", nx=512, ny=192, nz=192,
             prec="f32", store="f32", per=""),
        # a cycle on a smaller uneven grid, periodic in z: many short launches
        dict(name="vcycle_120x88x72_f32", kind="vcycle", nx=120, ny=88, nz=72, prec="f32",
             store="f32", per="z"),
        # the benchmark problem: 256^3, a sphere in a box, to 1e-6
        dict(name="solve_sphere_256_f32", kind="solve", nx=256, ny=256, nz=256, prec="f32",
             store="f32", per="", rtol=1e-6),
        # the smallest solve: 32^3 periodic Taylor-Green box in FP64, to 1e-10
        dict(name="solve_tgv_32_f64", kind="solve", nx=32, ny=32, nz=32, prec="f64",
             store="f64", per="xyz", rtol=1e-10),
        # one step of the moving-sphere sequence
        dict(name="step_moving_256x64x64", kind="step", nx=256, ny=64, nz=64, store="f32",
             rtol=1e-6),
        # the batch of 64 uneven problems, refined to 1e-10
        dict(name="batch_64", kind="batch", count=64, store="f32", rtol=1e-10),
        # the widest full-resolution layer of a 128^3 training batch
        dict(name="conv_128_32to16", kind="conv", n=2, d=128, h=128, w=128, cin=32, cout=16),
        # the bottleneck layer: few voxels, many channels
        dict(name="conv_16_128to128", kind="conv", n=2, d=16, h=16, w=16, cin=128, cout=128),
        # backward of a half-resolution layer
        dict(name="conv_bwd_64_32to32", kind="conv_bwd", n=2, d=64, h=64, w=64, cin=32, cout=32),
        # the warm start of one problem of the uneven batch's sizes
        dict(name="infer_104x56x48", kind="infer", nx=104, ny=56, nz=48),
        # one training step's forward and backward at the training size
        dict(name="train_128", kind="train", n=2, nx=128, ny=128, nz=128),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi, step, cells):
    """Three sizes, multiples of `step` (1: odd ones too), at most `cells`."""
    while True:
        n = [max(lo, step * (_logint(rng, lo, hi) // step)) for _ in range(3)]
        if n[0] * n[1] * n[2] <= cells:
            return n


def draw(rng):
    kind = rng.choice(["smooth", "residual", "vcycle", "solve", "step", "batch", "conv", "conv",
                       "conv_bwd", "conv_bwd", "infer", "train"])
    if kind in ("smooth", "residual"):
        n = _grid(rng, 24, 400, 1, 16 << 20)
        per = rng.choice(["", "", "z", "xy"])
        n = [v + v % 2 if d in per else v for v, d in zip(n, "xyz")]
        prec = rng.choice(["f32", "f32", "f32", "f64"])
        store = "f64" if prec == "f64" else rng.choice(["f32", "f32", "bf16"])
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], prec=prec, store=store, per=per)
        if kind == "smooth":
            c["sweeps"] = rng.choice([1, 2, 2, 3, 4])
        return c
    if kind in ("vcycle", "solve"):
        n = _grid(rng, 32, 160, 8, 2 << 20) if rng.random() < 0.7 else _grid(rng, 64, 256, 32,
                                                                            16 << 20)
        prec = rng.choice(["f32", "f32", "f64"])
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], prec=prec,
                 store="f64" if prec == "f64" else rng.choice(["f32", "f32", "bf16"]),
                 per=rng.choice(["", "", "z"]))
        if kind == "solve":
            c["rtol"] = 1e-5 if prec == "f32" else 1e-9
        return c
    if kind == "step":
        n = _grid(rng, 32, 256, 16, 2 << 20)
        return dict(kind="step", nx=max(n[0], 64), ny=n[1], nz=n[2],
                    store=rng.choice(["f32", "bf16"]), rtol=rng.choice([1e-6, 1e-8]))
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(3, 48), store=rng.choice(["f32", "bf16"]),
                    rtol=rng.choice([1e-8, 1e-10]))
    if kind in ("conv", "conv_bwd"):
        cin, cout = rng.choice(LAYERS if kind == "conv" else LAYERS[1:])
        n = rng.choice([1, 1, 2])
        while True:
            s = [_logint(rng, 6, 144) for _ in range(3)]
            if rng.random() < 0.5:  # the network's own sizes: multiples of 8
                s = [max(8, 8 * (v // 8)) for v in s]
            if n * s[0] * s[1] * s[2] * cin * cout <= (1 << 21) * 512:
                return dict(kind=kind, n=n, d=s[0], h=s[1], w=s[2], cin=cin, cout=cout)
    if kind == "infer":
        n = _grid(rng, 32, 160, 8, 1 << 21)
        return dict(kind="infer", nx=n[0], ny=n[1], nz=n[2])
    n = _grid(rng, 32, 128, 8, 1 << 20)
    return dict(kind="train", n=rng.choice([1, 2]), nx=n[0], ny=n[1], nz=n[2])


# ---------------------------------------------------------------------------
# Inputs (FP64 on the GPU; a run rounds them to its own precision)
# ---------------------------------------------------------------------------

AX = (2, 1, 0)  # tensor axis of direction d


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _sel(d, i):
    s = [slice(None)] * 3
    s[AX[d]] = i
    return tuple(s)


def _per(case):
    return tuple(d in case.get("per", "") for d in "xyz")


def _coords(n, d):
    o = [0.0 if e == d else 0.5 for e in range(3)]
    t = [torch.arange(n[e], dtype=torch.float64, device=DEV) + o[e] for e in range(3)]
    return t[0][None, None, :], t[1][None, :, None], t[2][:, None, None]


def _sphere(n, per, centre, radius):
    """Faces mu0(|f - C| - R) of a sphere smoothed over a 2-cell band, with
    zero faces on the walls."""
    L = torch.empty((3, n[2], n[1], n[0]), dtype=torch.float64, device=DEV)
    for d in range(3):
        X, Y, Z = _coords(n, d)
        r = torch.sqrt((X - centre[0]) ** 2 + (Y - centre[1]) ** 2 + (Z - centre[2]) ** 2) - radius
        b = r.clamp(-1.0, 1.0)
        L[d] = 0.5 * (1.0 + b) + torch.sin(math.pi * b) / (2.0 * math.pi)
        L[d][r <= -1.0] = 0.0
        L[d][r >= 1.0] = 1.0
        if not per[d]:
            L[d][_sel(d, 0)] = 0.0
    return L


def _touched(L, per):
    t = torch.zeros(L.shape[1:], dtype=torch.bool, device=DEV)
    for d in range(3):
        hi = torch.roll(L[d], -1, AX[d])
        if not per[d]:
            hi[_sel(d, -1)] = 0.0
        t |= (L[d] != 0) | (hi != 0)
    return t


def _rhs(L, u, per):
    """Flux divergence of the face velocity, its mean over the open cells removed."""
    s = torch.zeros(L.shape[1:], dtype=torch.float64, device=DEV)
    for d in range(3):
        f = L[d] * u[d]
        fh = torch.roll(f, -1, AX[d])
        if not per[d]:
            fh[_sel(d, -1)] = 0.0
        s += fh - f
    t = _touched(L, per)
    s[t] -= s[t].mean()
    s[~t] = 0.0
    return s


def _problem(n, per, seed, tgv=False):
    """(faces, right-hand side) of a sphere in a box with a random velocity,
    or (tgv) of an empty box with a noisy Taylor-Green velocity."""
    g = _gen(seed)
    u = torch.rand((3, n[2], n[1], n[0]), dtype=torch.float64, device=DEV, generator=g) * 2 - 1
    if tgv:
        L = torch.ones((3, n[2], n[1], n[0]), dtype=torch.float64, device=DEV)
        for d in range(3):
            if not per[d]:
                L[d][_sel(d, 0)] = 0.0
        u *= 0.02
        for d in range(2):
            X, Y, Z = (2 * math.pi * c / m for c, m in zip(_coords(n, d), n))
            u[d] += (torch.sin(X) * torch.cos(Y) if d == 0 else -torch.cos(X) * torch.sin(Y)) * \
                torch.cos(Z)
    else:
        q = torch.rand(3, dtype=torch.float64, device=DEV, generator=g).tolist()
        c = [m * (0.4 + 0.2 * v) for m, v in zip(n, q)]
        L = _sphere(n, per, c, min(n) / 8.0)
    return L, _rhs(L, u, per)


def _moving(n, seed):
    """A sphere in a box at a time drawn from the seed, and the right-hand side
    of its accelerating motion along x with a travelling Taylor-Green wave."""
    per = (False, False, False)
    t = (seed * 7919 % 97) / 97.0 * 0.3
    xc = n[0] * (0.25 + t)
    L = _sphere(n, per, (xc, n[1] / 2.0, n[2] / 2.0), min(n) / 8.0)
    U = 1.0 + 0.05 * xc
    u = torch.zeros_like(L)
    k = 2.0 * math.pi / n[1]
    for d in range(2):
        X, Y, Z = (k * c for c in _coords(n, d))
        X = X - k * xc
        w = torch.sin(X) * torch.cos(Y) if d == 0 else -torch.cos(X) * torch.sin(Y)
        u[d] = 0.1 * U * w * torch.cos(Z)
    u[0] += U
    return L, _rhs(L, u, per)


def _batch(case, seed):
    size, g = torch.Generator(), torch.Generator()
    size.manual_seed(3)  # the sizes are the case's, whatever the seed
    g.manual_seed(int(seed) + 17)
    out = []
    for i in range(case["count"]):
        m = torch.rand(3, generator=size).tolist()
        n = (8 * (4 + int(m[0] * 13)), 8 * (4 + int(m[1] * 5)), 8 * (4 + int(m[2] * 5)))
        r = [0.0] * 3 + torch.rand(4, generator=g).tolist()
        rad = 0.5 * (8.0 + 16.0 * r[3])
        c = [rad + 3.0 + v * (m - 2.0 * rad - 6.0) for v, m in zip(r[4:], n)]
        L = _sphere(n, (False,) * 3, c, rad)
        u = torch.rand(L.shape, dtype=torch.float64, device=DEV, generator=_gen(seed * 97 + i))
        out.append((n, L, _rhs(L, 2 * u - 1, (False,) * 3)))
    return out


def _real(case):
    return torch.float64 if case.get("prec", "f64") == "f64" else torch.float32


def _gmg_inputs(case, seed):
    n = (case["nx"], case["ny"], case["nz"])
    if case["kind"] == "step":
        return n, (False,) * 3, _moving(n, seed)
    per = _per(case)
    L, s = _problem(n, per, seed, tgv=all(per))
    dt = _real(case)
    return n, per, (L.to(dt), s.to(dt))


def _guess(case, seed):
    """A smooth iterate with some noise, of order one."""
    n = (case["nx"], case["ny"], case["nz"])
    X, Y, Z = _coords(n, 0)
    x = torch.cos(math.pi * X / n[0]) * torch.cos(2 * math.pi * Y / n[1]) + 0.3 * Z / n[2]
    x = x + 0.05 * torch.randn(x.shape, dtype=torch.float64, device=DEV, generator=_gen(seed + 5))
    return x.to(_real(case)).contiguous()


def _bf16(shape, seed, scale=1.0, relu=False):
    t = torch.randn(shape, dtype=torch.float32, device=DEV, generator=_gen(seed)) * scale
    return (t.clamp_min(0.0) if relu else t).to(torch.bfloat16)


def _conv_inputs(case, seed):
    """Activations after a ReLU, He-sized weights, small biases; for the
    backward a gradient and the layer's own (ReLU) output."""
    vol = (case["n"], case["d"], case["h"], case["w"])
    ci, co = case["cin"], case["cout"]
    x = _bf16(vol + (ci,), seed, 1.0, relu=True)
    w = _bf16((co, 27, ci), seed + 1, math.sqrt(2.0 / (27 * ci)))
    b = torch.randn(co, dtype=torch.float32, device=DEV, generator=_gen(seed + 2)) * 0.1
    if case["kind"] == "conv":
        return x, w, b
    return x, w, _bf16(vol + (co,), seed + 3, 0.01), _bf16(vol + (co,), seed + 4, 1.0, relu=True)


def _net_inputs(case, seed):
    n, b = (case["nx"], case["ny"], case["nz"]), case.get("n", 1)
    vol = (n[2], n[1], n[0])
    sig, faces, mask, scale = [], [], [], []
    for k in range(b):
        g = _gen(seed * 31 + k)
        q = torch.rand(7, dtype=torch.float64, device=DEV, generator=g).tolist()
        rad = min(4.0 + 8.0 * q[0], min(n) / 2.0 - 4.0)
        c = [rad + 3.0 + v * (m - 2.0 * rad - 6.0) for v, m in zip(q[1:4], n)]
        L = _sphere(n, (False,) * 3, c, rad)
        u = torch.zeros_like(L)
        for d in range(2):
            X, Y, Z = (2 * math.pi * (1 + int(3 * p)) * e / m
                       for e, m, p in zip(_coords(n, d), n, q[4:]))
            u[d] = (torch.sin(X) * torch.cos(Y) if d == 0 else -torch.cos(X) * torch.sin(Y)) * \
                torch.cos(Z)
        s = _rhs(L, u, (False,) * 3)
        t = _touched(L, (False,) * 3)
        scale.append(float(s[t].pow(2).mean().sqrt()))
        sig.append(s.float())
        faces.append(L.float())
        mask.append(t)
    g = _gen(seed + 9)
    target = 3.0 * torch.randn((b,) + vol, dtype=torch.float32, device=DEV, generator=g)
    net = [torch.randn(co * taps * ci, generator=g, device=DEV) *
           math.sqrt(2.0 / ((4 if k == 0 else ci) * taps)) for k, (_, ci, co, taps)
           in enumerate(NET.layers())]
    net[0].view(16, 27, 8)[:, :, 4:] = 0.0
    flat = torch.cat([torch.cat([w, 0.05 * torch.randn(co, generator=g, device=DEV)])
                      for w, (_, _, co, _) in zip(net, NET.layers())])
    return (torch.stack(sig).contiguous(), torch.stack(faces).contiguous(),
            torch.stack(mask).to(torch.uint8).contiguous(), scale, target, flat)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    k = case["kind"]
    st = dict(case=case)
    if k in ("smooth", "residual", "vcycle", "solve", "step"):
        n, per, (L, s) = _gmg_inputs(case, seed)
        code = G.GMG_F64 if L.dtype == torch.float64 else G.GMG_F32
        kw = dict(l_storage=STORE[case["store"]])
        if k == "step":
            kw["cycle_dtype"] = G.GMG_F32
            first = _moving(n, seed + 1)[0].contiguous()  # the previous step's faces
        else:
            first = L.contiguous()
        st["h"] = G.gmg_setup(G.gmg_default_params(n, per, code, **kw), first)
        st["L"], st["s"] = L.contiguous(), s.contiguous()
        st["x"] = _guess(case, seed) if k == "residual" else torch.zeros_like(st["s"])
        st["r"] = torch.zeros_like(st["s"]) if k == "residual" else None
    elif k == "batch":
        pb = _batch(case, seed)
        prm = [G.gmg_default_params(n, (False,) * 3, G.GMG_F64, cycle_dtype=G.GMG_F32,
                                    l_storage=STORE[case["store"]]) for n, _, _ in pb]
        st["b"] = G.gmg_batch_setup(prm, [L.contiguous() for _, L, _ in pb])
        st["s"] = [s.contiguous() for _, _, s in pb]
        # one allocation for all the problems' iterates
        st["all"] = torch.zeros(sum(s.numel() for s in st["s"]), dtype=torch.float64, device=DEV)
        st["x"], o = [], 0
        for s in st["s"]:
            st["x"].append(st["all"][o:o + s.numel()].view(s.shape))
            o += s.numel()
    elif k in ("conv", "conv_bwd"):
        vol = (case["n"], case["d"], case["h"], case["w"])
        ci, co = case["cin"], case["cout"]
        st["sh"] = UN.shape(*vol)
        if k == "conv":
            st["x"], st["w"], st["b"] = _conv_inputs(case, seed)
            st["y"] = torch.zeros(vol + (co,), dtype=torch.bfloat16, device=DEV)
        else:
            st["x"], st["w"], st["dy"], st["y"] = _conv_inputs(case, seed)
            st["g"] = torch.zeros_like(st["dy"])
            st["dx"] = torch.zeros_like(st["x"])
            st["dw"] = torch.zeros((co, 27, ci), dtype=torch.float32, device=DEV)
            st["db"] = torch.zeros(co, dtype=torch.float32, device=DEV)
            st["flip"] = torch.empty(co * 27 * ci, dtype=torch.bfloat16, device=DEV)
            st["ws"] = torch.empty(UN.unet_wgrad_workspace(st["sh"], ci, co, 27) // 4 + 1,
                                   dtype=torch.float32, device=DEV)
    else:
        st["sig"], st["L"], mask, st["scale"], target, flat = _net_inputs(case, seed)
        st["net"] = NET.UNet()
        st["net"].set_flat(flat.cpu().numpy())
        b, vol = case.get("n", 1), (case["nz"], case["ny"], case["nx"])
        st["sh"] = UN.shape(b, *vol)
        st["in"] = torch.zeros((b,) + vol + (NET.IN_CH,), dtype=torch.int16, device=DEV)
        if k == "train":
            st["mask"], st["target"] = mask, target
        else:
            st["p"] = torch.zeros(vol, dtype=torch.float64, device=DEV)
    return st


def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "smooth":
        state["x"].zero_()
        G.gmg_smooth(state["h"], 0, state["x"], state["s"], case["sweeps"])
        return state["x"]
    if k == "residual":
        rn, sn = G.gmg_residual(state["h"], state["x"], state["s"], state["r"])
        return [state["r"], rn, sn]
    if k == "vcycle":
        state["x"].zero_()
        G.gmg_vcycle(state["h"], state["x"], state["s"])
        return state["x"]
    if k == "solve":
        state["x"].zero_()
        info = G.gmg_solve(state["h"], state["x"], state["s"], case["rtol"], 12)
        return [state["x"], info["cycles"], info["rnorm"]]
    if k == "step":
        state["x"].zero_()
        G.gmg_update_faces(state["h"], state["L"])
        info = G.gmg_solve_ir(state["h"], state["x"], state["s"], case["rtol"])
        return [state["x"], info["outer"], info["inner_total"]]
    if k == "batch":
        state["all"].zero_()
        infos = G.gmg_batch_solve_ir(state["b"], state["x"], state["s"], case["rtol"])
        return [state["all"], torch.tensor([[i["outer"], i["inner_total"]] for i in infos])]
    if k == "conv":
        ci, co = case["cin"], case["cout"]
        UN.unet_conv_fwd(state["sh"], UN.act(state["x"], ci, 0, ci), state["w"], state["b"], 27,
                         UN.act(state["y"], co, 0, co), None, 1)
        return state["y"]
    if k == "conv_bwd":
        ci, co = case["cin"], case["cout"]
        sh, g = state["sh"], UN.act(state["g"], co, 0, co)
        UN.unet_relu_bwd(sh, UN.act(state["y"], co, 0, co), UN.act(state["dy"], co, 0, co), g)
        UN.unet_conv_wgrad(sh, UN.act(state["x"], ci, 0, ci), g, 27, state["dw"], state["db"],
                           state["ws"])
        UN.unet_conv_dgrad(sh, g, state["w"], 27, UN.act(state["dx"], ci, 0, ci), state["flip"])
        return [state["dx"], state["dw"], state["db"]]
    UN.unet_pack_input(state["sh"], state["sig"], state["L"], state["scale"], state["in"])
    vol = (case["nz"], case["ny"], case["nx"])
    out = state["net"].forward(state["in"], case.get("n", 1), *vol)
    if k == "infer":
        UN.unet_scale_f64(out, state["scale"][0], state["p"])
        return state["p"]
    state["net"].backward(state["in"], state["target"], state["mask"], want_loss=False)
    return [out, state["net"].grad]


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------

def _net_flops(case, backward):
    vox = case.get("n", 1) * case["nx"] * case["ny"] * case["nz"]
    f = 0.0
    for name, ci, co, taps in NET.layers():
        lvl = 0 if name == "head" else int("".join(c for c in name if c.isdigit()))
        one = 2.0 * (vox >> (3 * lvl)) * taps * ci * co
        f += one * ((2 if name == "enc0a" else 3) if backward else 1)
    return f


def work(case):
    """Each input read once and each output written once; operations of the
    method (a sweep 20 per cell, a residual 19)."""
    k = case["kind"]
    if k in ("smooth", "residual", "vcycle", "solve", "step"):
        cells = case["nx"] * case["ny"] * case["nz"]
        e = 8 if k == "step" or case["prec"] == "f64" else 4
        face = {"f32": 4, "f64": 8, "bf16": 2}[case["store"]]
        if k == "smooth":
            return dict(bytes=cells * (2 * e + 3 * face), flops=20.0 * cells * case["sweeps"])
        if k == "residual":
            return dict(bytes=cells * (3 * e + 3 * face), flops=19.0 * cells)
        cycle = cells * 8.0 / 7.0 * (4 * 20 + 19)
        if k == "vcycle":
            return dict(bytes=cells * (2 * e + 3 * face), flops=cycle)
        if k == "solve":
            return dict(bytes=cells * (2 * e + 3 * face), flops=cycle * (4 if e == 4 else 8))
        return dict(bytes=cells * (2 * e + 3 * 8), flops=cycle * 10)
    if k == "batch":
        cells = case["count"] * 96 * 48 * 48 * 0.8
        return dict(bytes=cells * (2 * 8 + 3 * 8), flops=cells * 8.0 / 7.0 * 99 * 11)
    if k in ("conv", "conv_bwd"):
        vox, ci, co = case["n"] * case["d"] * case["h"] * case["w"], case["cin"], case["cout"]
        one = 2.0 * vox * 27 * ci * co
        if k == "conv":
            return dict(bytes=vox * 2 * (ci + co) + 54 * ci * co, flops=one)
        return dict(bytes=vox * 2 * (2 * ci + 2 * co) + 27 * ci * co * 6, flops=2 * one)
    vox = case.get("n", 1) * case["nx"] * case["ny"] * case["nz"]
    par = sum(t * ci * co + co for _, ci, co, t in NET.layers())
    if k == "infer":
        return dict(bytes=vox * (16 + 8) + 2 * par, flops=_net_flops(case, False))
    return dict(bytes=vox * (16 + 4 + 4 + 1) + 6 * par, flops=_net_flops(case, True))


# ---------------------------------------------------------------------------
# The same outputs in 64-bit arithmetic
# ---------------------------------------------------------------------------

def _ax(L, x, per):
    """(A x, D): flux form, D = -(sum of a cell's six faces)."""
    y, D = torch.zeros_like(x), torch.zeros_like(x)
    for d in range(3):
        lo = L[d]
        hi = torch.roll(lo, -1, AX[d])
        if not per[d]:
            hi[_sel(d, -1)] = 0.0
        y += hi * (torch.roll(x, -1, AX[d]) - x) + lo * (torch.roll(x, 1, AX[d]) - x)
        D -= lo + hi
    return y, D


def _residual(L, x, s, per):
    y, D = _ax(L, x, per)
    return torch.where(D != 0, s - y, torch.zeros_like(s)), D


def _sweeps(L, x, s, per, count, omega=1.0):
    nz, ny, nx = x.shape
    par = (torch.arange(nx, device=DEV)[None, None, :] + torch.arange(ny, device=DEV)[:, None] +
           torch.arange(nz, device=DEV)[:, None, None]) % 2
    for _ in range(count):
        for colour in (0, 1):
            r, D = _residual(L, x, s, per)
            x = torch.where((par == colour) & (D != 0), x + omega * r / D, x)
    return x


def _blocksum(a, c):
    z, y, x = a.shape
    return a.reshape(z // c[2], c[2], y // c[1], c[1], x // c[0], c[0]).sum((1, 3, 5))


def _levels(L, per):
    out = []
    while True:
        n = (L.shape[3], L.shape[2], L.shape[1])
        c = [2 if m % 2 == 0 and m // 2 >= 4 and not (p and (m // 2) % 2) else 1
             for m, p in zip(n, per)]
        last = c == [1, 1, 1]
        out.append((L, None if last else c))
        if last:
            return out
        nxt = []
        for d in range(3):
            cut = [slice(None)] * 3
            cut[AX[d]] = slice(None, None, c[d])
            e = [1 if i == d else c[i] for i in range(3)]
            nxt.append(_blocksum(L[d][tuple(cut)], e) / c[d])
        L = torch.stack(nxt)


def _coarsest(L, x, s, per, omega):
    r, D = _residual(L, x, s, per)
    s = torch.where(D != 0, s - s[D != 0].mean(), s)
    lim = 0.1 * _residual(L, x, s, per)[0].norm()
    for _ in range(16):
        x = _sweeps(L, x, s, per, 4, omega)
        if _residual(L, x, s, per)[0].norm() <= lim:
            break
    return x


def _cycle(levels, x, s, per, l=0, omega=1.0):
    L, c = levels[l]
    if c is None:
        return _coarsest(L, x, s, per, omega) if l else _sweeps(L, x, s, per, 4, omega)
    x = _sweeps(L, x, s, per, 2, omega)
    r, D = _residual(L, x, s, per)
    sc = _blocksum(r, c)
    e = _cycle(levels, torch.zeros_like(sc), sc, per, l + 1, omega)
    for d in range(3):
        e = e.repeat_interleave(c[d], AX[d])
    x = torch.where(D != 0, x + e, x)
    return _sweeps(L, x, s, per, 2, omega)


def _solve(levels, s, per, rtol, most):
    L = levels[0][0]
    x, omega = torch.zeros_like(s), 1.0
    snorm = s[_residual(L, x, s, per)[1] != 0].norm()
    rho, cycles = _residual(L, x, s, per)[0].norm(), 0
    while cycles < most and not rho <= rtol * snorm:
        y = _cycle(levels, x, s, per, 0, omega)
        rn = _residual(L, y, s, per)[0].norm()
        cycles += 1
        if rn > rho:
            omega = max(0.1, 0.5 * omega)
        else:
            x, rho, omega = y, rn, min(1.0, 1.2 * omega)
    return x, cycles, float(rho)


class _Conv(torch.autograd.Function):
    """3x3x3 cross-correlation with zero padding in FP64, channels last:
    one matrix product per tap.  w: [taps][cin][cout]."""

    @staticmethod
    def _taps(x):
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        d, h, w = x.shape[1:4]
        for t in range(27):
            a, b, c = t // 9, t // 3 % 3, t % 3
            yield t, (slice(None), slice(a, a + d), slice(b, b + h), slice(c, c + w)), p

    @staticmethod
    def forward(ctx, x, w):
        ctx.save_for_backward(x, w)
        y = torch.zeros(x.shape[:-1] + (w.shape[2],), dtype=x.dtype, device=x.device)
        for t, cut, p in _Conv._taps(x):
            y += (p[cut].reshape(-1, p.shape[-1]) @ w[t]).reshape(y.shape)
        return y

    @staticmethod
    def backward(ctx, dy):
        x, w = ctx.saved_tensors
        dw, dp = torch.zeros_like(w), None
        f = dy.reshape(-1, dy.shape[-1])
        for t, cut, p in _Conv._taps(x):
            dp = torch.zeros_like(p) if dp is None else dp
            dw[t] = p[cut].reshape(-1, p.shape[-1]).t() @ f
            dp[cut] += (f @ w[t].t().contiguous()).reshape(p[cut].shape)
        return dp[:, 1:-1, 1:-1, 1:-1], dw


def _taps64(w):  # [cout][27][cin] -> FP64 [27][cin][cout]
    return w.double().permute(1, 2, 0).contiguous()


def _net64(case, x, flat):
    """The network in FP64 (weights as the convolutions read them: BF16, the
    head's and the biases FP32); returns the output and its parameters in
    layer order."""
    par, off = {}, 0
    for name, ci, co, taps in NET.layers():
        w = flat[off:off + co * taps * ci].view(co, taps, ci)
        w = w if name == "head" else w.to(torch.bfloat16)
        b = flat[off + co * taps * ci:off + co * taps * ci + co]
        par[name] = (w.double().requires_grad_(True), b.double().requires_grad_(True))
        off += co * taps * ci + co

    def conv(a, name):
        w, b = par[name]
        return torch.relu(_Conv.apply(a, w.permute(1, 2, 0).contiguous()) + b)

    def pool(a):
        n, d, h, w, c = a.shape
        return a.reshape(n, d // 2, 2, h // 2, 2, w // 2, 2, c).mean((2, 4, 6))

    def up(a):
        n, d, h, w, c = a.shape
        return a[:, :, None, :, None, :, None].expand(n, d, 2, h, 2, w, 2, c).reshape(
            n, 2 * d, 2 * h, 2 * w, c)

    skip = []
    for i in range(4):
        x = conv(conv(x, f"enc{i}a"), f"enc{i}b")
        if i < 3:
            skip.append(x)
            x = pool(x)
    for i in (2, 1, 0):
        x = torch.cat([conv(up(x), f"up{i}"), skip[i]], -1)
        x = conv(conv(x, f"dec{i}a"), f"dec{i}b")
    w, b = par["head"]
    return (x @ w.reshape(-1, 1)).squeeze(-1) + b, [t for p in par.values() for t in p]


def exact(case, seed):
    k = case["kind"]
    if k in ("step", "batch"):
        # the iterate at which a refinement stops depends on FP32 inner
        # cycles; there is no 64-bit value of it
        return None
    if k in ("smooth", "residual", "vcycle", "solve"):
        n, per, (L, s) = _gmg_inputs(case, seed)
        if case["store"] == "bf16":
            L = L.to(torch.bfloat16)
        L, s = L.double(), s.double()
        z = torch.zeros_like(s)
        if k == "smooth":
            return _sweeps(L, z, s, per, case["sweeps"])
        if k == "residual":
            r, D = _residual(L, _guess(case, seed).double(), s, per)
            return [r, float(r.norm()), float(s[D != 0].norm())]
        if k == "vcycle":
            return _cycle(_levels(L, per), z, s, per)
        x, cycles, rn = _solve(_levels(L, per), s, per, case["rtol"], 12)
        return [x, None, rn]
    if k == "conv":
        x, w, b = _conv_inputs(case, seed)
        return torch.relu(_Conv.apply(x.double(), _taps64(w)) + b.double())
    if k == "conv_bwd":
        x, w, dy, y = _conv_inputs(case, seed)
        g = torch.where(y > 0, dy, torch.zeros_like(dy)).double()
        xr, wr = x.double().requires_grad_(True), _taps64(w).requires_grad_(True)
        _Conv.apply(xr, wr).backward(g)
        return [xr.grad, wr.grad.permute(2, 0, 1).contiguous(), g.sum((0, 1, 2, 3))]
    sig, L, mask, scale, target, flat = _net_inputs(case, seed)
    sc = torch.tensor(scale, dtype=torch.float64, device=DEV)[:, None, None, None]
    x = torch.stack([sig.double() / sc] + [L[:, d].double() for d in range(3)] +
                    [torch.zeros_like(sig, dtype=torch.float64)] * 4, -1)
    if k == "infer":
        with torch.no_grad():
            return _net64(case, x, flat)[0][0] * scale[0]
    out, par = _net64(case, x, flat)
    m = mask.double()
    loss = (m * (out - target.double()) ** 2).sum() / m.sum()
    grads = torch.autograd.grad(loss, par)
    return [out.detach(), torch.cat([g.reshape(-1) for g in grads])]
