"""The work that a program has this library do, as timed cases.

A case is one call pattern of the spectral-convolution layer (or of the whole
FNO block around it) on one GPU:

  "fwd"    inference: one forward call, no spectral cache
  "step"   training: the forward (keeping the input spectrum) and the combined
           backward (data and weight gradients)
  "split"  training with bwd_data and bwd_weight as two calls (both spectra
           kept between them)
  "block"  training of one FNO block: the layer, then skip + bias + GELU +
           residual, and the backward through both

on a 1-, 2- or 3-D grid, in fp16+tanh or fp32 storage, with dense, Tucker or
CP weights.  "graph": the calls are captured once and each pass replays them,
as the benchmark and latency-bound training loops do; otherwise each pass
makes the calls.

`listed()` are the fixed cases, `draw()` gives others of the same ranges.
"""
from __future__ import annotations

import math

import torch

from paper_2307_15034_amd import binding as B
from paper_2307_15034_amd.layer import BlockEpilogue, SpectralConv


def _case(name, do, n, modes, batch, c_in, c_out, prec="fp16", weight="dense", rank="",
          policy="min_result", graph=False):
    """Shapes are written as text ("128x128") so that a case is plain values."""
    c = {"do": do, "n": n, "modes": modes, "batch": batch, "c_in": c_in, "c_out": c_out,
         "prec": prec, "weight": weight, "rank": rank, "policy": policy, "graph": graph}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A small training step, bound by latency and launches: the smallest
        # workload of the benchmark, captured in a graph as the benchmark does.
        _case("step-2d-64", "step", "64x64", "8x8", 2, 16, 16, graph=True),
        # One sample through one layer, called from Python: the smallest call
        # a serving loop makes.
        _case("fwd-2d-64", "fwd", "64x64", "12x12", 1, 32, 32),
        # The Navier-Stokes-shaped training step (benchmark workload 2).
        _case("step-2d-128", "step", "128x128", "32x32", 32, 64, 64),
        # The largest training step, the default benchmark workload.
        _case("step-2d-1024", "step", "1024x1024", "64x64", 8, 64, 64),
        # Zero-shot super-resolution inference: one 1024^2 sample.
        _case("fwd-2d-1024", "fwd", "1024x1024", "64x64", 1, 64, 64),
        # The 3-D latent grid of a geometry-informed operator (workload 4).
        _case("step-3d-64", "step", "64x64x64", "16x16x16", 4, 32, 32),
        # The Tucker-factorised operator in the layer's default greedy order
        # (workload 5).
        _case("step-tucker-256", "step", "256x256", "32x32", 16, 128, 128, weight="tucker",
              rank="13,13,6,3"),
        # The CP-factorised Navier-Stokes step (workload 6).
        _case("step-cp-128", "step", "128x128", "32x32", 32, 64, 64, weight="cp", rank="16"),
        # The full-precision baseline of the Navier-Stokes step.
        _case("step-fp32-128", "step", "128x128", "32x32", 32, 64, 64, prec="fp32"),
        # An odd grid, as finite-element data sets on node grids have.
        _case("step-2d-odd", "step", "241x241", "20x20", 16, 32, 32),
        # A 1-D operator on long signals.
        _case("step-1d-8192", "step", "8192", "32", 32, 64, 64),
        # One whole FNO block, forward and backward.
        _case("block-2d-256", "block", "256x256", "32x32", 8, 64, 64),
    ]


# ---------------------------------------------------------------------------
# Other cases of the same ranges
# ---------------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extent(rng, lo, hi):
    """A grid extent: a power of two, a multiple of eight, or any number."""
    v = _log(rng, lo, hi)
    how = rng.random()
    if how < 0.4:
        return max(lo, 1 << max(1, round(math.log2(v))))
    return max(lo, v // 8 * 8) if how < 0.7 else v


def draw(rng):
    kind = rng.choice(["2d", "2d", "2d-odd", "3d", "1d", "tucker", "cp", "fp32", "block", "fwd"])
    do = rng.choice(["step", "step", "split"])
    policy = rng.choice(["min_result", "min_net"])
    prec, weight, rank = "fp16", "dense", ""
    if kind == "3d":
        n = [_extent(rng, 16, 96) for _ in range(3)]
    elif kind == "1d":
        n = [_extent(rng, 256, 16384)]
    elif kind == "2d-odd":
        n = [_log(rng, 40, 500) | 1 for _ in range(2)]
    else:
        a = _extent(rng, 32, 1024)
        n = [a, a if rng.random() < 0.6 else _extent(rng, 32, 1024)]
    d = len(n)
    cap = {1: 64, 2: 64, 3: 16}[d]
    modes = []
    for j, v in enumerate(n):
        top = min(v // 2, cap)
        modes.append(max(2, min(top, _log(rng, 4, cap))))
    c_in = rng.choice([16, 20, 32, 48, 64, 64, 128])
    c_out = c_in if kind == "block" or rng.random() < 0.7 else rng.choice([16, 24, 32, 64])
    if kind == "tucker":
        weight = "tucker"
        rank = ",".join(str(rng.randint(4, 16)) for _ in range(2)) + "," + ",".join(
            str(rng.randint(2, 8)) for _ in range(d))
    if kind == "cp":
        weight, rank = "cp", str(_log(rng, 4, 32))
    if kind == "fp32":
        prec = "fp32"
    if kind == "fwd":
        do = "fwd"
        prec = rng.choice(["fp16", "fp16", "fp32"])
    if kind == "block":
        do = "block"
    # as many samples as the kind's share of the largest listed case allows
    points = math.prod(n)
    room = {"2d": 1 << 26, "fwd": 1 << 25, "block": 1 << 25}.get(kind, 1 << 24)
    most = max(1, min(32, room // (points * max(c_in, c_out))))
    batch = _log(rng, 1, most)
    return _case(None, do, "x".join(map(str, n)), "x".join(map(str, modes)), batch, c_in, c_out,
                 prec, weight, rank, policy)


# ---------------------------------------------------------------------------
# Shapes
# ---------------------------------------------------------------------------
def _shape(case):
    n = tuple(int(v) for v in case["n"].split("x"))
    modes = tuple(int(v) for v in case["modes"].split("x"))
    rank = tuple(int(v) for v in case["rank"].split(",")) if case["rank"] else None
    kd = tuple(2 * m if j < len(n) - 1 else m for j, m in enumerate(modes))
    return n, modes, kd, rank


def _params(case, seed, dtype, dev):
    """Inputs of the case from the seed: {"x", "gy", "w", and for a block
    "skip", "bias"} on `dev` in the storage type.  x: smooth random fields of
    unit variance (periodic, power falling off as the benchmark's Gaussian
    fields do); gy: white noise; weights with the variance the layer is
    initialised with."""
    n, _, kd, rank = _shape(case)
    g = torch.Generator(device=dev).manual_seed(int(seed))
    f32 = dict(device=dev, dtype=torch.float32, generator=g)
    bt, ci, co = case["batch"], case["c_in"], case["c_out"]

    def basis(length):
        """[length, 2 m] cosines and sines of the wavenumbers 0..m-1, and the
        wavenumbers of the columns."""
        m = max(1, min(24, length // 2))
        k = torch.arange(m, device=dev, dtype=torch.float64)
        ph = 2 * math.pi / length * torch.arange(length, device=dev, dtype=torch.float64)[:, None]
        f = torch.cat([torch.cos(ph * k), torch.sin(ph * k)], 1).float()
        return f, torch.cat([k, k]).float()

    bases = [basis(v) for v in n]
    k2 = torch.zeros((), device=dev)
    for j, (_, k) in enumerate(bases):
        k2 = k2 + (k * k).reshape([-1 if q == j else 1 for q in range(len(n))])
    amp = (k2 + 49.0) ** -1.25
    # mean variance of a field: each axis' columns have mean square 1/2
    # (the sine of wavenumber zero vanishes)
    pw = amp * amp
    for f, _ in bases:
        pw = torch.tensordot((f * f).mean(0), pw, dims=([0], [0]))
    amp = amp / pw.sqrt()

    def fields(c):
        out = torch.empty((bt, c) + n, device=dev, dtype=dtype)
        for b in range(bt):
            z = torch.randn((c,) + amp.shape, **f32) * amp
            for f, _ in bases:  # the first grid axis each time; it moves to the back
                z = torch.tensordot(z, f, dims=([1], [1]))
            out[b] = z.to(dtype)
        return out

    def noise(shape):
        out = torch.empty(shape, device=dev, dtype=dtype)
        for b in range(shape[0]):
            out[b] = torch.randn(shape[1:], **f32).to(dtype)
        return out

    def cplx(shape, std):
        return (torch.randn(tuple(shape) + (2,), **f32) * std).to(dtype)

    p = {"x": fields(ci)}
    if case["do"] != "fwd":
        p["gy"] = noise((bt, co) + n)
    if case["weight"] == "tucker":
        p["w"] = {"core": cplx(rank, 1 / math.sqrt(ci * co)),
                  "u_in": cplx((ci, rank[0]), 1 / math.sqrt(2 * rank[0])),
                  "u_out": cplx((co, rank[1]), 1 / math.sqrt(2 * rank[1])),
                  "u_mode": [cplx((k, r), 1 / math.sqrt(2 * r)) for k, r in zip(kd, rank[2:])]}
    elif case["weight"] == "cp":
        r = rank[0]
        p["w"] = {"core": cplx((r,), 1 / math.sqrt(ci * co * r)),
                  "u_in": cplx((ci, r), math.sqrt(0.5)), "u_out": cplx((co, r), math.sqrt(0.5)),
                  "u_mode": [cplx((k, r), math.sqrt(0.5)) for k in kd]}
    else:
        p["w"] = cplx((ci, co) + kd, 1 / math.sqrt(ci * co))
    if case["do"] == "block":
        p["skip"] = (torch.randn((co, ci), **f32) / math.sqrt(ci)).to(dtype)
        p["bias"] = (torch.randn((co,), **f32) * 0.1).to(dtype)
    return p


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    n, modes, _, rank = _shape(case)
    prec = B.FNO_PREC_FP16_TANH if case["prec"] == "fp16" else B.FNO_PREC_FP32
    kind = {"dense": B.FNO_WEIGHT_DENSE, "tucker": B.FNO_WEIGHT_TUCKER,
            "cp": B.FNO_WEIGHT_CP}[case["weight"]]
    pol = B.FNO_PATH_MIN_RESULT if case["policy"] == "min_result" else B.FNO_PATH_MIN_NET
    layer = SpectralConv(n, modes, case["batch"], case["c_in"], case["c_out"], precision=prec,
                         weight_kind=kind, rank=rank, path_policy=pol)
    s = {"do": case["do"], "layer": layer}
    s.update(_params(case, seed, layer.dtype, "cuda"))
    if case["do"] != "fwd":
        s["x_hat"] = layer.spectrum_buffer(0)  # kept from the forward to the backward
    if case["do"] == "split":
        s["gy_hat"] = layer.spectrum_buffer(1)
    if case["do"] == "block":
        s["epi"] = BlockEpilogue(n, case["batch"], case["c_in"], case["c_out"], precision=prec,
                                 residual=case["c_in"] == case["c_out"])
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _calls(s)  # builds the plan, as the library asks before a capture
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["out"] = _calls(s)
    return s


def _calls(s):
    layer, x, w = s["layer"], s["x"], s["w"]
    if s["do"] == "fwd":
        return {"y": layer.fwd(x, w)}
    y = layer.fwd(x, w, x_hat=s["x_hat"])
    if s["do"] == "step":
        gx, gw = layer.bwd(x, w, s["gy"], x_hat=s["x_hat"])
        return {"y": y, "gx": gx, "gw": gw}
    if s["do"] == "split":
        gx = layer.bwd_data(x, w, s["gy"], gy_hat=s["gy_hat"])
        gw = layer.bwd_weight(None, None, w, x_hat=s["x_hat"], gy_hat=s["gy_hat"])
        return {"y": y, "gx": gx, "gw": gw}
    epi = s["epi"]
    out, z = epi.fwd(x, y, s["skip"], s["bias"])
    gz, g_skip, g_bias = epi.bwd_weight(x, z, s["gy"])
    gx, gw = layer.bwd(x, w, gz, x_hat=s["x_hat"])
    gx = epi.bwd_data(gz, s["skip"], gx, g_out=s["gy"] if epi.residual else None, gx=gx)
    return {"out": out, "gx": gx, "gw": gw, "g_skip": g_skip, "g_bias": g_bias}


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return _calls(state)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: the inputs of each call read once and its outputs written once
    (x is an input of the forward and, through the derivative of tanh, of the
    backward; the kept spectra are written once and read once).  Operations:
    real FFTs of every plane and the channel contractions of each direction
    (of a factorised weight: through the ranks)."""
    n, _, kd, rank = _shape(case)
    es = 2 if case["prec"] == "fp16" else 4
    bt, ci, co = case["batch"], case["c_in"], case["c_out"]
    pts, modes = math.prod(n), math.prod(kd)
    xin, yout = bt * ci * pts * es, bt * co * pts * es
    xhat, ghat = bt * ci * modes * 2 * es, bt * co * modes * 2 * es
    fft = 2.5 * pts * math.log2(max(2, pts))
    if case["weight"] == "dense":
        wn = ci * co * modes
        mix = 8.0 * bt * ci * co * modes
    elif case["weight"] == "tucker":
        wn = math.prod(rank) + ci * rank[0] + co * rank[1] + sum(
            k * r for k, r in zip(kd, rank[2:]))
        mix = 8.0 * bt * modes * (ci * rank[0] + co * rank[1] + rank[0] * rank[1])
    else:
        wn = rank[0] * (1 + ci + co + sum(kd))
        mix = 8.0 * bt * modes * rank[0] * (ci + co + 1)
    wb = wn * 2 * es
    nbytes = xin + wb + yout
    flops = bt * (ci + co) * fft + mix
    if case["do"] != "fwd":
        nbytes += 2 * xhat + yout + wb + xin + wn * 8
        nbytes += xin if case["prec"] == "fp16" else 0  # tanh'(x)
        nbytes += 2 * ghat if case["do"] == "split" else 0
        flops += bt * (ci + co) * fft + 2 * mix
    if case["do"] == "block":
        # forward: x, y -> out, z; backward: x, z, g_out -> g_z; then g_z,
        # the layer's gx (and g_out) -> gx
        nbytes += xin + 3 * yout + xin + 3 * yout + yout + 2 * xin
        nbytes += yout if ci == co else 0
        flops += 3 * 2.0 * bt * ci * co * pts
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what was measured against `exact` over the listed and
    24 drawn cases.  fp16 storage (spectra and outputs rounded to 11 bits
    between the steps): relative error at most 7.5e-4, largest difference over
    the root mean square 2.7e-2 (the weight gradient of the 1024^2 step, whose
    modes differ much in size).  fp32 storage (32-bit sums and twiddles):
    5.5e-7 and 1.1e-5."""
    if case["prec"] == "fp32":
        return {"rel": 2.4e-6, "max": 8e-5}
    return {"rel": 3e-3, "max": 8e-2}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
def exact(case, seed):
    """The pass in float64 by the definitions (dense DFT matrices of the
    retained modes, full weights, autograd for the gradients), one sample at
    a time."""
    n, modes, kd, _ = _shape(case)
    fp16 = case["prec"] == "fp16"
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    p = _params(case, seed, torch.float16 if fp16 else torch.float32, dev)
    d, points = len(n), math.prod(n)

    def dft(j):
        """cos and sin of 2 pi k n / N, [K_j, N_j], the phase reduced in integers."""
        t = torch.arange(kd[j], device=dev)
        k = t if j == d - 1 else torch.where(t < modes[j], t, n[j] - 2 * modes[j] + t)
        ph = (k[:, None] * torch.arange(n[j], device=dev)) % n[j]
        ph = ph.double() * (2 * math.pi / n[j])
        return torch.cos(ph), torch.sin(ph)

    tw = [dft(j) for j in range(d)]
    t = torch.arange(kd[-1], device=dev)
    cm = torch.where((t == 0) | (2 * t == n[-1]), 1.0, 2.0).double()

    def along(re, im, axis, c, s, sign):
        """sum over `axis` of (re + i im)(c + i sign s), c and s [out, in]."""
        re = re.movedim(axis, -1)
        im = None if im is None else im.movedim(axis, -1)
        a, b = re @ c.t(), re @ s.t() * sign
        if im is not None:
            a, b = a - im @ s.t() * sign, b + im @ c.t()
        return a.movedim(-1, axis), b.movedim(-1, axis)

    def layer(x, w):
        re, im = (torch.tanh(x) if fp16 else x) / points, None
        for j in reversed(range(d)):
            re, im = along(re, im, 1 + j, tw[j][0], tw[j][1], -1.0)
        k = math.prod(kd)
        xs = torch.complex(re, im).reshape(-1, k).t().unsqueeze(1)          # [K, 1, ci]
        ws = w.reshape(case["c_in"], case["c_out"], k).permute(2, 0, 1)     # [K, ci, co]
        ys = torch.bmm(xs, ws.contiguous()).squeeze(1).t().reshape((case["c_out"],) + kd)
        re, im = ys.real * cm, ys.imag * cm
        for j in range(d - 1):
            re, im = along(re, im, 1 + j, tw[j][0].t(), tw[j][1].t(), 1.0)
        return re @ tw[-1][0] - im @ tw[-1][1]

    def leaf(v):
        return v.double().requires_grad_(case["do"] != "fwd")

    def full(w):
        """Dense complex weights [ci, co, K..] of the stored parameters."""
        c = torch.view_as_complex
        if case["weight"] == "dense":
            return c(w)
        core, u_in, u_out = c(w["core"]), c(w["u_in"]), c(w["u_out"])
        um = [c(u) for u in w["u_mode"]]
        if case["weight"] == "tucker":
            t = torch.tensordot(u_in, core, dims=([1], [0]))   # [ci, e, r..]
            t = torch.tensordot(t, u_out, dims=([1], [1]))     # [ci, r.., co]
            for u in um:                                       # the next rank is axis 1
                t = torch.tensordot(t, u, dims=([1], [1]))     # [ci, .., co, K..]
            return t
        left = u_in * core
        for u in [u_out] + um:                                 # [.., R] x [k, R]
            left = left.unsqueeze(-2) * u
        return left.sum(-1)

    dense = case["weight"] == "dense"
    w = leaf(p["w"]) if dense else {
        k: [leaf(u) for u in v] if isinstance(v, list) else leaf(v) for k, v in p["w"].items()}
    grads = case["do"] != "fwd"
    wf = full(w)
    # the gradient of the dense weights is summed over the samples first
    wl = wf.detach().requires_grad_(grads)
    block = case["do"] == "block"
    skip, bias = (leaf(p["skip"]), leaf(p["bias"])) if block else (None, None)
    ys, gxs = [], []
    for b in range(case["batch"]):
        x = leaf(p["x"][b])
        y = layer(x, wl)
        if block:
            z = (skip @ x.reshape(case["c_in"], -1)).reshape(y.shape) + y
            z = z + bias.reshape((-1,) + (1,) * d)
            y = torch.nn.functional.gelu(z)
            if case["c_in"] == case["c_out"]:
                y = y + x
        if grads:
            y.backward(p["gy"][b].double())
            gxs.append(x.grad.float())
        ys.append(y.detach().float())
    res = {"out" if block else "y": torch.stack(ys)}
    if not grads:
        return res
    res["gx"] = torch.stack(gxs)
    if dense:
        res["gw"] = torch.view_as_real(wl.grad.resolve_conj()).contiguous()
    else:
        wf.backward(wl.grad)
        res["gw"] = {k: [u.grad for u in v] if isinstance(v, list) else v.grad
                     for k, v in w.items()}
    if block:
        res["g_skip"], res["g_bias"] = skip.grad, bias.grad
    return res
