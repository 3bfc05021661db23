"""The work that users of this framework have it do, as timed cases.

A case is one pass of orthogonalization (batched or grouped call) or of the
optimizer over the matrices that its ``shapes`` text lists ("16x64x576" is 16
matrices of 64 x 576, several shapes separated by spaces).  Every call works in
place on a buffer that the program owns, so a pass first puts this step's
gradients into it, as the momentum part of an optimizer does.
"""
import math

import torch

from paper_2512_04632_amd import _lib as tm
from paper_2512_04632_amd.optim import TurboMuon

TRIPLE = (3.4445, -4.7750, 2.0315)     # the library's default coefficients


def schedule():
    """A five-row coefficient table that falls towards the convergent quintic."""
    return [(a, 2.5 - 2.0 * a, a - 1.5) for a in (3.0, 2.6, 2.2, 1.875, 1.6)]


def listed():
    def case(name, shapes, **more):
        base = {"name": name, "kind": "batched", "dtype": "bf16", "precond": "aol", "iters": 4,
                "schedule": False, "alpha": 0.8, "shapes": shapes}
        return {**base, **more}

    return [
        # the smallest calls, where latency counts: the first stage of a ResNet (3 x 3
        # kernels as 64 x 576 matrices), and one small matrix in fp32
        case("conv_stage1", "16x64x576", alpha=1.0),
        case("f32_256", "1x256x256", dtype="f32", alpha=1.0),
        # one MLP matrix of a 768-wide transformer, as a program that treats its parameters one
        # by one sends it; and its transpose with plain Muon (Frobenius scale, 5 iterations)
        case("mlp_768", "1x768x3072"),
        case("mlp_768_tall_muon", "1x3072x768", precond="frobenius", iters=5),
        # every matrix of a 12-layer 768-wide transformer in one grouped call
        case("gpt2_12layer", "48x768x768 12x768x3072 12x3072x768", kind="grouped"),
        # the 3 x 3 convolutions of a ResNet, four stages in one grouped call
        case("conv_64", "16x64x576 16x128x1152 16x256x2304 16x512x4608", kind="grouped", alpha=1.0),
        # odd and ragged sizes in one grouped call (heads, embeddings, adapters), Schatten-4
        # scale, a five-row schedule
        case("ragged", "1x1000x2731 3x515x515 1x3001x777 2x129x1153 1x50x4001 2x333x90",
             kind="grouped", precond="schatten4", iters=5, schedule=True),
        # an 8B-class transformer: its attention and MLP matrices, eight layers a call
        case("attn_8b", "8x4096x4096", alpha=0.5),
        case("mlp_8b", "8x4096x14336", alpha=0.5),
        # fp32 storage: one layer of the 768-wide transformer, and one 4096-wide matrix
        case("f32_layer", "4x768x768 1x768x3072 1x3072x768", kind="grouped", dtype="f32"),
        case("f32_4096", "1x4096x4096", dtype="f32", alpha=0.5),
        # the optimizer's step (momentum, orthogonalization, update) over the 12 layers
        case("optimizer_12layer", "48x768x768 12x768x3072 12x3072x768", kind="optimizer"),
    ]


# Drawn cases cost at most this many operations (fp32 products are about ten times slower).
CAP = {"bf16": 1.2e13, "f32": 6e11}


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case: sides 32 .. 4096 on the short side, aspect ratios 1 .. 9, either
    orientation, every scale and 3 .. 5 iterations, odd sizes in half of the cases."""
    kind = rng.choice(["batched", "batched", "batched", "grouped", "grouped", "optimizer"])
    dtype = "f32" if kind != "optimizer" and rng.random() < 0.25 else "bf16"
    precond, iters = rng.choice([("aol", 4), ("aol", 4), ("aol", 3), ("aol", 5),
                                 ("frobenius", 5), ("schatten4", 4)])
    even = rng.random() < 0.5
    cap = 0.5 * CAP[dtype] * rng.random()
    parts, total = [], 0.0
    for _ in range(1 if kind == "batched" else rng.randint(2, 6)):
        k = _log_uniform(rng, 32, 4096 if kind == "batched" else 2048)
        n = min(k * _log_uniform(rng, 1.0, 9.0), 16384)
        count = int(_log_uniform(rng, 1, 40))
        k, n = (max(64, 64 * round(k / 64)), max(64, 64 * round(n / 64))) if even else (round(k), round(n))
        k, n = min(k, n), max(k, n)
        each = 4 * iters * (3.0 * k * k * n + k ** 3)
        count = max(1, min(count, int((CAP[dtype] - cap - total) / each)))
        if parts and total + count * each > CAP[dtype]:
            break
        total += count * each
        parts.append("%dx%dx%d" % ((count, k, n) if rng.random() < 0.6 else (count, n, k)))
    return {"kind": kind, "dtype": dtype, "precond": precond, "iters": iters,
            "schedule": rng.random() < 0.2, "alpha": round(rng.uniform(0.5, 1.0), 2),
            "shapes": " ".join(parts)}


def _shapes(case):
    return [tuple(int(v) for v in part.split("x")) for part in case["shapes"].split()]


def _coeffs(case):
    return tm.schedule_tail(schedule(), case["iters"]) if case["schedule"] else None


def _gradients(case, seed, dtype):
    """Gradient-like matrices: a power-law part plus 1% Gaussian noise, a (count, m, n)
    tensor for each shape, all views of one flat buffer."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    shapes = _shapes(case)
    flat = torch.empty(sum(c * m * n for c, m, n in shapes), device="cuda", dtype=dtype)
    for x in _views(flat, shapes):
        count, m, n = x.shape
        k = min(m, n)
        sigma = torch.arange(1, k + 1, device="cuda", dtype=torch.float32) ** -case["alpha"]
        for i in range(count):
            u = torch.randn((m, k), generator=g, device="cuda") * (sigma / math.sqrt(m * n))
            v = torch.randn((k, n), generator=g, device="cuda")
            x[i] = u @ v + 0.01 * torch.randn((m, n), generator=g, device="cuda")
    return flat


def _views(flat, shapes):
    out, at = [], 0
    for count, m, n in shapes:
        out.append(flat[at:at + count * m * n].view(count, m, n))
        at += count * m * n
    return out


def prepare(case, seed):
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    state = {"case": case, "coeffs": _coeffs(case)}
    if case["kind"] == "optimizer":
        start = _optimizer_start(case, seed)
        state["start"] = start
        state["w"], state["m"] = start["w"].clone(), start["m"].clone()
        params, shapes = [], _shapes(case)
        for w, grad in zip(_views(state["w"], shapes), _views(start["g"], shapes)):
            for i in range(w.shape[0]):
                p = torch.nn.Parameter(w[i])
                p.grad = grad[i]
                params.append(p)
        opt = TurboMuon(params, lr=0.02, momentum=0.95, weight_decay=0.01, iters=case["iters"],
                        precond=case["precond"], coeffs=state["coeffs"])
        bufs = [m[i] for m in _views(state["m"], shapes) for i in range(m.shape[0])]
        for p, m in zip(params, bufs):       # a step in the middle of training
            opt.state[p]["momentum_buffer"] = m
        state["opt"] = opt
    else:
        state["grads"] = _gradients(case, seed, dtype)
        state["buffer"] = torch.empty_like(state["grads"])
        state["views"] = _views(state["buffer"], _shapes(case))
    return state


def _optimizer_start(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 7)
    grads = _gradients(case, seed, torch.float32)
    w = 0.02 * torch.randn(grads.shape, generator=g, device="cuda")
    m = 4.0 * grads + 0.02 * torch.randn(grads.shape, generator=g, device="cuda")
    return {"w": w, "m": m, "g": grads}


def run(state):
    case = state["case"]
    if case["kind"] == "optimizer":
        # every pass is the same step: weights and momentum as they were before it
        state["w"].copy_(state["start"]["w"])
        state["m"].copy_(state["start"]["m"])
        state["opt"].step()
        return {"w": state["w"], "m": state["m"]}
    state["buffer"].copy_(state["grads"])
    if case["kind"] == "batched":
        tm.orthogonalize(state["views"][0], case["iters"], state["coeffs"], case["precond"])
    else:
        tm.orthogonalize_grouped([x[i] for x in state["views"] for i in range(x.shape[0])],
                                 case["iters"], state["coeffs"], case["precond"])
    return {"o": state["buffer"]}


def work(case):
    """Symmetric products counted once per pair.  With k = min, N = max: the iterations as
    printed take (3 N + k) k^2 each; in bf16 two of them taken together through the k x k
    side take (3 N + 5 k) k^2, and the smaller of the two counts."""
    flops, elements, t = 0.0, 0, case["iters"]
    for count, m, n in _shapes(case):
        k, N = float(min(m, n)), float(max(m, n))
        one = (3 * N + k) * k * k
        two = min(2 * one, (3 * N + 5 * k) * k * k) if case["dtype"] == "bf16" else 2 * one
        flops += count * ((t // 2) * two + (t % 2) * one)
        elements += count * m * n
    size = 20 if case["kind"] == "optimizer" else (4 if case["dtype"] == "bf16" else 8)
    return {"bytes": size * elements, "flops": flops}


def tolerance(case):
    if case["kind"] == "optimizer":
        return {"rel": 2e-3}      # the weights move by a fortieth of themselves, in bf16
    # four times the error against 64 bits that is seen: 4e-3 to 1.1e-2 in bf16, and in fp32
    # 1e-6 to 6e-6 (the iteration amplifies what rounding leaves in the small directions)
    return {"rel": 0.03} if case["dtype"] == "bf16" else {"rel": 2.5e-5}


def _polar(x, case):
    """One matrix in 64 bits, straight from the definition."""
    tall = x.shape[0] > x.shape[1]
    y = x.double()
    y = y.t().contiguous() if tall else y
    a0 = y @ y.t()
    if case["precond"] == "aol":
        s = a0.abs().sum(1).rsqrt()
    elif case["precond"] == "frobenius":
        s = torch.ones_like(a0[0]) / y.norm()
    else:
        s = torch.ones_like(a0[0]) / a0.norm().sqrt()
    y = s[:, None] * y
    for a, b, c in _coeffs(case) or [TRIPLE] * case["iters"]:
        g = y @ y.t()
        p = b * g + c * (g @ g)
        y = a * y + p @ y
    return y.t() if tall else y


def exact(case, seed):
    shapes = _shapes(case)
    if case["kind"] != "optimizer":
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        grads = _gradients(case, seed, dtype)
        out = torch.empty(grads.shape, device="cuda", dtype=torch.float64)
        for x, o in zip(_views(grads, shapes), _views(out, shapes)):
            for i in range(x.shape[0]):
                o[i] = _polar(x[i], case)
        return {"o": out}
    start = _optimizer_start(case, seed)
    mom = 0.95 * start["m"].double() + start["g"].double()
    u = start["g"].double() + 0.95 * mom
    w = start["w"].double() * (1.0 - 0.02 * 0.01)
    for x, o in zip(_views(u, shapes), _views(w, shapes)):
        scale = 0.02 * math.sqrt(max(1.0, x.shape[1] / x.shape[2]))
        for i in range(x.shape[0]):
            o[i] -= scale * _polar(x[i], case)
    return {"w": w, "m": mom}
