"""Performance cases of the library's public entry points (gemm, conv1d, dwsep_conv, gru_forward).

``listed()`` holds the fixed cases, ``draw(rng)`` gives more of the same ranges.  ``prepare``
makes what a program holds before the call (inputs, weights, output buffers and the workspace
the size query asks for, on the GPU); ``run`` is one call; ``work`` the bytes and operations the
call cannot do without; ``exact`` the same result from plain torch in 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_1810_09958_amd as isam

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_ES = {"bf16": 2, "f32": 4}


def listed():
    return [
        # A layer of a very small network (and the smallest call): launch latency.
        dict(name="gemm_f32_128", op="gemm", M=128, N=128, K=128, dt="f32", ct="f32", ta=False, tb=False, acc=False),
        # The largest product: matrix-core rate of the whole chip.
        dict(name="gemm_bf16_8192", op="gemm", M=8192, N=8192, K=8192, dt="bf16", ct="bf16", ta=False, tb=False,
             acc=False),
        # Weight gradient of a GRU input projection (3 x 1024 gate rows, 1024 inputs, 64 steps x 32
        # sequences): dW += dG^T X, both operands with the sum over rows.
        dict(name="gemm_bf16_gradient", op="gemm", M=3072, N=1024, K=2048, dt="bf16", ct="f32", ta=True, tb=False,
             acc=True),
        # A linear layer (weights [N][K]) whose sizes are nobody's multiple.
        dict(name="gemm_bf16_ragged", op="gemm", M=1000, N=1537, K=1023, dt="bf16", ct="bf16", ta=False, tb=True,
             acc=False),
        # The same kind of layer in fp32 at ordinary sizes.
        dict(name="gemm_f32_layer", op="gemm", M=2048, N=1024, K=1024, dt="f32", ct="f32", ta=False, tb=True,
             acc=False),
        # One RNN step at batch 32: weights times a narrow block of activations.
        dict(name="skinny_bf16_n32", op="gemm", M=4096, N=32, K=4096, dt="bf16", ct="f32", ta=False, tb=False,
             acc=False),
        # A speech-model convolution over time: 32 sequences of 1024 positions, 5 taps.
        dict(name="conv1d_bf16", op="conv1d", batch=32, L=1028, Ki=512, D=5, Ko=512, dt="bf16", ct="f32"),
        # GRU layer of the benchmark: 64 steps, batch 32.
        dict(name="gru_bf16_b32", op="gru", T=64, batch=32, I=1024, H=1024, dt="bf16", extra=False),
        # A smaller fp32 GRU with an initial state and the inner bias.
        dict(name="gru_f32_b12", op="gru", T=50, batch=12, I=200, H=400, dt="f32", extra=True),
        # MobileNet-style separable layers: an early one ...
        dict(name="dwsep_bf16_56", op="dwsep", batch=32, hw=56, C=128, cm=1, k=3, stride=1, Co=256, dt="bf16", ct="bf16"),
        # ... the deep one such networks repeat most ...
        dict(name="dwsep_bf16_14", op="dwsep", batch=32, hw=14, C=512, cm=1, k=3, stride=1, Co=512, dt="bf16", ct="bf16"),
        # ... and a down-sampling one, in fp32.
        dict(name="dwsep_f32_down", op="dwsep", batch=16, hw=112, C=64, cm=1, k=3, stride=2, Co=128, dt="f32", ct="f32"),
    ]


# ---------------------------------------------------------------------------------------
# Drawn cases
# ---------------------------------------------------------------------------------------
def _log(rng, lo, hi, step=1):
    """An integer in [lo, hi], even over its logarithm, a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v) // step * step))


def _draw_gemm(rng):
    dt = "bf16" if rng.random() < 0.7 else "f32"
    layout = rng.choices(("nn", "nt", "tn"), (4, 3, 3))[0]
    odd = rng.random() < 0.35
    step = 1 if odd else rng.choice((8, 64))
    cap = 1e10 if odd else 3e10 if dt == "f32" else 1.4e11
    m, n, k = (_log(rng, 64, 2400 if odd else 8192, step) for _ in range(3))
    n = max(n, 40)
    while 2.0 * m * n * k > cap:
        if k >= max(m, n):
            k = max(64, k // 2 // step * step)
        elif m >= n:
            m = max(64, m // 2 // step * step)
        else:
            n = max(64, n // 2 // step * step)
    return dict(op="gemm", M=m, N=n, K=k, dt=dt, ct=rng.choice(("bf16", "f32")) if dt == "bf16" else "f32",
                ta=layout == "tn", tb=layout == "nt", acc=layout == "tn" and rng.random() < 0.5)


def _draw_skinny(rng):
    dt = "bf16" if rng.random() < 0.7 else "f32"
    return dict(op="gemm", M=_log(rng, 256, 16384, 8), N=rng.choice((1, rng.randint(2, 32), 8 * rng.randint(1, 4))),
                K=_log(rng, 256, 8192, 8), dt=dt, ct="f32", ta=False, tb=False, acc=False)


def _draw_conv1d(rng):
    dt = "bf16" if rng.random() < 0.8 else "f32"
    step = 1 if rng.random() < 0.2 else 8
    c = dict(op="conv1d", batch=_log(rng, 1, 32), L=_log(rng, 50, 2048), Ki=_log(rng, 16, 512, step),
             D=rng.randint(1, 11), Ko=_log(rng, 16, 512, step), dt=dt,
             ct=rng.choice(("bf16", "f32")) if dt == "bf16" else "f32")
    while 2.0 * c["batch"] * c["L"] * c["Ki"] * c["D"] * c["Ko"] > (9e10 if dt == "bf16" and step == 8 else 8e9):
        key = "batch" if c["batch"] > 1 else "L"
        c[key] = c[key] // 2
    return c


def _draw_gru(rng):
    dt = "bf16" if rng.random() < 0.6 else "f32"
    H = rng.choice((256, 512, 768, 1024)) if rng.random() < 0.5 else _log(rng, 64, 1024, 8)
    return dict(op="gru", T=_log(rng, 1, 128 if dt == "bf16" and H % 256 == 0 else 50), batch=_log(rng, 1, 64 if dt == "bf16" else 32),
                I=_log(rng, 40, 1024, 8), H=H, dt=dt, extra=rng.random() < 0.5)


def _draw_dwsep(rng):
    dt = "bf16" if rng.random() < 0.65 else "f32"
    hw = rng.choice((7, 14, 28, 56, 112)) if rng.random() < 0.7 else _log(rng, 7, 113)
    c = dict(op="dwsep", batch=_log(rng, 1, 32), hw=hw, C=_log(rng, 16, 1024, 8), cm=2 if rng.random() < 0.1 else 1,
             k=5 if rng.random() < 0.2 else 3, stride=2 if rng.random() < 0.35 else 1, Co=_log(rng, 16, 1024, 8), dt=dt,
             ct=rng.choice(("bf16", "f32")) if dt == "bf16" else "f32")
    if rng.random() < 0.1:
        c["C"], c["Co"] = c["C"] + 3, c["Co"] + 1
    while c["batch"] > 1 and (c["batch"] * hw * hw * c["C"] * c["cm"] > 13e6
                              or 2.0 * c["batch"] * hw * hw * c["C"] * c["cm"] * c["Co"] > 1.4e10 * c["stride"] ** 2):
        c["batch"] //= 2
    while c["batch"] == 1 and (hw * hw * c["C"] * c["cm"] > 13e6 or 2.0 * hw * hw * c["C"] * c["cm"] * c["Co"] > 1.4e10):
        c["C"], c["Co"] = max(16, c["C"] // 2), max(16, c["Co"] // 2)
    return c


def draw(rng):
    f = rng.choices((_draw_gemm, _draw_skinny, _draw_conv1d, _draw_gru, _draw_dwsep), (40, 15, 10, 15, 20))[0]
    return f(rng)


# ---------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------
class _Source:
    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(int(seed))

    def normal(self, shape, dt, scale=1.0):
        return torch.randn(shape, generator=self.g, device=self.dev).mul_(scale).to(_DT[dt])

    def uniform(self, shape, dt, r):
        return torch.rand(shape, generator=self.g, device=self.dev).mul_(2 * r).sub_(r).to(_DT[dt])


def _out_hw(c):
    pad = c["k"] // 2
    return pad, (c["hw"] + 2 * pad - c["k"]) // c["stride"] + 1


def _inputs(c, seed):
    s, dt = _Source(seed), c["dt"]
    if c["op"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        x = dict(A=s.normal((K, M) if c["ta"] else (M, K), dt, 1 / math.sqrt(K)),
                 B=s.normal((N, K) if c["tb"] else (K, N), dt))
        if c["acc"]:
            x["C"] = s.normal((M, N), c["ct"])
        return x
    if c["op"] == "conv1d":
        return dict(A=s.normal((c["batch"], c["L"], c["Ki"]), dt),
                    B=s.uniform((c["D"], c["Ki"], c["Ko"]), dt, 1 / math.sqrt(c["D"] * c["Ki"])))
    if c["op"] == "gru":
        T, b, I, H = c["T"], c["batch"], c["I"], c["H"]
        r = 1 / math.sqrt(H)
        x = dict(x=s.normal((T, b, I), dt), W=s.uniform((3 * H, I), dt, r), U=s.uniform((3 * H, H), dt, r),
                 bias=s.normal((3 * H,), "f32", 0.01))
        if c["extra"]:
            x["bias_hn"] = s.normal((H,), "f32", 0.01)
            x["h0"] = s.uniform((b, H), "f32", 1.0)
        return x
    b, hw, C, cm, k, Co = (c[n] for n in ("batch", "hw", "C", "cm", "k", "Co"))
    return dict(x=s.normal((b, hw, hw, C), dt), D=s.uniform((k, k, C, cm), dt, 1 / k),
                P=s.uniform((C * cm, Co), dt, 1 / math.sqrt(C * cm)))


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    dev = torch.device("cuda")
    code = {"f32": isam.ISAM_F32, "bf16": isam.ISAM_BF16}

    def room(nbytes):
        return torch.empty(max(nbytes, 1), device=dev, dtype=torch.uint8)

    if c["op"] == "gemm":
        out = x["C"] if c["acc"] else torch.empty((c["M"], c["N"]), device=dev, dtype=_DT[c["ct"]])
        ws = room(isam.gemm_workspace_size(c["M"], c["N"], c["K"], code[c["dt"]], code[c["ct"]], int(c["ta"]),
                                           int(c["tb"])))
        return dict(op="gemm", A=x["A"], B=x["B"], kw=dict(out=out, trans_a=c["ta"], trans_b=c["tb"],
                                                           accumulate=c["acc"], workspace=ws))
    if c["op"] == "conv1d":
        out = torch.empty((c["batch"], c["L"] - c["D"] + 1, c["Ko"]), device=dev, dtype=_DT[c["ct"]])
        return dict(op="conv1d", A=x["A"], B=x["B"], kw=dict(out=out))
    if c["op"] == "gru":
        T, b, H = c["T"], c["batch"], c["H"]
        ws = room(isam.gru_forward_workspace_size(T, b, c["I"], H, code[c["dt"]]))
        return dict(op="gru", x=x["x"], W=x["W"], U=x["U"],
                    kw=dict(bias=x["bias"], bias_hn=x.get("bias_hn"), h0=x.get("h0"),
                            h_seq=torch.empty((T, b, H), device=dev), h_T=torch.empty((b, H), device=dev),
                            workspace=ws))
    pad, o = _out_hw(c)
    ws = room(isam.dwsep_conv_workspace_size(c["batch"], c["hw"], c["hw"], c["C"], c["cm"], c["k"], c["k"], c["stride"],
                                             pad, c["Co"], code[c["dt"]], code[c["ct"]]))
    out = torch.empty((c["batch"], o, o, c["Co"]), device=dev, dtype=_DT[c["ct"]])
    return dict(op="dwsep", x=x["x"], D=x["D"], P=x["P"], kw=dict(stride=c["stride"], pad=pad, out=out, workspace=ws))


def run(state):
    op = state["op"]
    if op == "gemm":
        return isam.gemm(state["A"], state["B"], **state["kw"])
    if op == "conv1d":
        return isam.conv1d(state["A"], state["B"], **state["kw"])
    if op == "gru":
        return isam.gru_forward(state["x"], state["W"], state["U"], **state["kw"])
    return isam.dwsep_conv(state["x"], state["D"], state["P"], **state["kw"])


# ---------------------------------------------------------------------------------------
# Work, tolerance, 64-bit results
# ---------------------------------------------------------------------------------------
def work(case):
    c, e = case, _ES[case["dt"]]
    if c["op"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        return dict(bytes=e * (M * K + K * N) + _ES[c["ct"]] * M * N * (2 if c["acc"] else 1), flops=2.0 * M * N * K)
    if c["op"] == "conv1d":
        b, X = c["batch"], c["L"] - c["D"] + 1
        return dict(bytes=e * (b * c["L"] * c["Ki"] + c["D"] * c["Ki"] * c["Ko"]) + _ES[c["ct"]] * b * X * c["Ko"],
                    flops=2.0 * b * X * c["D"] * c["Ki"] * c["Ko"])
    if c["op"] == "gru":
        T, b, I, H = c["T"], c["batch"], c["I"], c["H"]
        return dict(bytes=e * (T * b * I + 3 * H * (I + H)) + 4 * (3 * H + T * b * H + b * H),
                    flops=2.0 * T * b * 3 * H * (I + H))
    o = _out_hw(c)[1]
    px, Cm = c["batch"] * o * o, c["C"] * c["cm"]
    return dict(bytes=e * (c["batch"] * c["hw"] ** 2 * c["C"] + c["k"] ** 2 * Cm + Cm * c["Co"]) + _ES[c["ct"]] * px * c["Co"],
                flops=2.0 * px * Cm * (c["k"] ** 2 + c["Co"]))


def tolerance(case):
    """About four times the distance seen between the results and exact()."""
    c = case
    if c["op"] == "gru":
        # bf16: h is rounded to bf16 as each step's operand, so one rounding that falls the other
        # way travels on (seen 3.3e-4); fp32: 32-bit sums over up to 50 steps (seen 2.7e-7).
        return {"rel": 1.5e-3, "max": 2e-2} if c["dt"] == "bf16" else {"rel": 5e-6, "max": 5e-5}
    if c["ct"] == "bf16" or (c["op"] == "dwsep" and c["dt"] == "bf16"):
        # one rounding of the result to bf16 (seen 1.7e-3); bf16 separable convolutions round the
        # depthwise result before the product (with the result's rounding: seen 2.3e-3)
        return {"rel": 7e-3, "max": 3e-2}
    return {"rel": 5e-6, "max": 5e-5}   # 32-bit sums (of exact products where the inputs are bf16; seen 1e-7 to 7e-7)


def exact(case, seed):
    c = case
    x = {k: v.double() for k, v in _inputs(case, seed).items()}
    if c["op"] == "gemm":
        r = (x["A"].t().contiguous() if c["ta"] else x["A"]) @ (x["B"].t().contiguous() if c["tb"] else x["B"])
        return r + x["C"] if c["acc"] else r
    if c["op"] == "conv1d":
        X = c["L"] - c["D"] + 1
        r = torch.zeros((c["batch"] * X, c["Ko"]), device=x["A"].device, dtype=torch.float64)
        for d in range(c["D"]):
            r += x["A"][:, d:d + X].reshape(-1, c["Ki"]).contiguous() @ x["B"][d]
        return r.view(c["batch"], X, c["Ko"])
    if c["op"] == "gru":
        T, b, H = c["T"], c["batch"], c["H"]
        gx = (x["x"].reshape(T * b, -1) @ x["W"].t().contiguous() + x["bias"]).view(T, b, 3 * H)
        Ut = x["U"].t().contiguous()
        h = x["h0"] if c["extra"] else torch.zeros((b, H), device=gx.device, dtype=torch.float64)
        hs = torch.empty((T, b, H), device=gx.device, dtype=torch.float64)
        for t in range(T):
            gh = h @ Ut
            r = torch.sigmoid(gx[t, :, :H] + gh[:, :H])
            z = torch.sigmoid(gx[t, :, H:2 * H] + gh[:, H:2 * H])
            hn = gh[:, 2 * H:] + x["bias_hn"] if c["extra"] else gh[:, 2 * H:]
            n = torch.tanh(gx[t, :, 2 * H:] + r * hn)
            h = (1 - z) * n + z * h
            hs[t] = h
        return hs, h
    pad, o = _out_hw(c)
    s, k = c["stride"], c["k"]
    xp = torch.nn.functional.pad(x["x"], (0, 0, pad, pad, pad, pad))
    Y = torch.zeros((c["batch"], o, o, c["C"], c["cm"]), device=xp.device, dtype=torch.float64)
    for i in range(k):
        for j in range(k):
            Y += xp[:, i:i + s * (o - 1) + 1:s, j:j + s * (o - 1) + 1:s, :, None] * x["D"][i, j]
    return (Y.view(-1, c["C"] * c["cm"]) @ x["P"]).view(c["batch"], o, o, c["Co"])
