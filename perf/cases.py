"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values.  Its "kind" says which public calls of ``paper_2511_04063_amd.binding`` one pass makes:

* ``step``    one calibration step (QR of the latent, rotation, Eq. 4 and its gradient, derivative through the QR, update)
  with the update rule ``update``: "sgd" or "adam"; ``b`` problems in one call.
* ``staged``  the same step made of the stage calls, with heavy-ball momentum: a program that keeps R, G and dZ.
* ``qr``      the factorisation alone: reading the calibrated rotation off a latent.
* ``cayley``  one step of the comparison optimiser, which moves the rotation itself.
* ``pass``    loss and gradient of one objective on a rotated block that is already there.

All cases of a process share one context and one workspace, as a program does that calibrates one layer after another on
one stream.
"""

import math

import torch

from paper_2511_04063_amd import binding as B

_DTYPE = {"bf16": (torch.bfloat16, B.DQ_BF16), "f32": (torch.float32, B.DQ_F32)}
_OBJECTIVE = {"whip": B.DQ_OBJ_WHIP, "variance": B.DQ_OBJ_VARIANCE, "kurtosis": B.DQ_OBJ_KURTOSIS, "quant": B.DQ_OBJ_QUANT}
_QUANT_BITS = 4
_LR = {"sgd": 1e-3, "adam": 2e-5}


def listed():
    def case(name, kind, n, T, x="bf16", b=1, latent="moved", **more):
        return {"name": name, "kind": kind, "n": n, "T": T, "x": x, "b": b, "latent": latent, **more}

    return [
        # the smallest whole step: one small rotation in fp32, all launches and latency
        case("step_tiny", "step", 256, 2048, "f32", latent="gauss", update="sgd", lr=1e-2),
        # a small residual width with Adam on the latent
        case("step_1k_adam", "step", 1024, 4096, update="adam", lr=2e-5),
        # a width and a token count that are multiples of nothing: what token sampling and pruned models leave
        case("step_ragged", "step", 2890, 3001, update="sgd", lr=1e-3),
        # the residual rotations of the three model sizes that the benchmark is quoted on
        case("step_7b", "step", 4096, 8192, latent="gauss", update="sgd", lr=1e-2),
        case("step_13b", "step", 5120, 8192, latent="gauss", update="sgd", lr=1e-2),
        case("step_70b", "step", 8192, 16384, latent="gauss", update="sgd", lr=1e-3),
        # per-head rotations, every head of a layer in one call: the usual head size, and a smaller one on a ragged block
        case("step_heads_128", "step", 128, 16384, b=64, latent="gauss", update="sgd", lr=1e-3),
        case("step_heads_80", "step", 80, 3000, b=32, update="sgd", lr=1e-3),
        # the rotation of a finished latent
        case("qr_2k", "qr", 2048, 1, "f32"),
        # a program with its own optimiser, fp32 activations, ragged tokens
        case("staged_1536", "staged", 1536, 4099, "f32", lr=1e-3, mu=0.9),
        # the optimiser that the method is compared with
        case("cayley_4k", "cayley", 4096, 8192, lr=1e-3, beta=0.9),
        # per-token quantisation error of a rotated block and its gradient
        case("pass_quant", "pass", 4096, 8192, objective="quant"),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, round_to):
    """A size between lo and hi, even over its logarithm; half of them multiples of round_to, as configured widths are."""
    v = _spread(rng, lo, hi)
    if rng.random() < 0.5:
        v = max(round_to, (v + round_to // 2) // round_to * round_to)
    return min(max(v, lo), hi)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "heads", "heads", "staged", "qr", "cayley", "pass"])
    if kind == "heads":
        update = rng.choice(["sgd", "sgd", "adam"])
        # a pass over all heads of a layer; per-head blocks are no larger than the listed ones
        return {"kind": "step", "n": rng.choice([64, 80, 96, 112, 128, 128, 128]), "T": _size(rng, 1024, 16384, 256), "x": "bf16",
                "b": rng.randint(8, 64), "latent": "moved", "update": update, "lr": _LR[update]}
    if kind == "qr":
        return {"kind": "qr", "n": _size(rng, 64, 7168, 256), "T": 1, "x": "f32", "b": 1, "latent": "moved"}
    if kind == "pass":
        n = _size(rng, 256, 8192, 256)
        return {"kind": "pass", "n": n, "T": _size(rng, 512, 16384, 256), "x": rng.choice(["bf16", "bf16", "f32"]), "b": 1, "latent": "moved",
                "objective": rng.choice(["whip", "variance", "kurtosis", "quant"])}
    if kind == "cayley":
        return {"kind": "cayley", "n": _size(rng, 256, 5120, 256), "T": _size(rng, 2048, 8192, 256), "x": "bf16", "b": 1, "latent": "moved",
                "lr": 1e-3, "beta": 0.9}
    if kind == "staged":
        x = rng.choice(["bf16", "f32"])
        return {"kind": "staged", "n": _size(rng, 128, 3072, 256), "T": _size(rng, 4096, 8192, 256), "x": x, "b": 1, "latent": "moved",
                "lr": 1e-3, "mu": 0.9}
    x, update = rng.choice(["bf16", "bf16", "bf16", "f32"]), rng.choice(["sgd", "sgd", "adam"])
    n = _size(rng, 96, 7168 if x == "bf16" else 2048, 256)
    return {"kind": "step", "n": n, "T": _size(rng, 512 if update == "sgd" else 4096, 12288, 256), "x": x, "b": 1, "latent": "moved",
            "update": update, "lr": _LR[update]}


def _round_up(v, m):
    return (v + m - 1) // m * m


def _matrix(b, rows, cols, dtype, fill=None):
    """b row-major matrices whose rows start at 16-byte multiples, as the library asks for."""
    ld = _round_up(cols, 8)
    shape = (b, rows, ld) if b > 1 else (rows, ld)
    m = torch.empty(shape, dtype=dtype, device="cuda") if fill is None else torch.full(shape, fill, dtype=dtype, device="cuda")
    return m[..., :cols]


def _activations(case, g):
    """Activations of zero mean and unit variance with a few channels that stand out (2 % of them 6 times the rest, two of
    a per-head block 40 times) and a log-normal scale per token: kurtosis 40 to 200, as reported for hidden states."""
    b, T, n = case["b"], case["T"], case["n"]
    X = _matrix(b, T, n, _DTYPE[case["x"]][0])
    scale, count = (40.0, 2) if b > 1 else (6.0, max(1, n // 50))
    rms = math.sqrt(math.exp(2 * 0.3 ** 2) * (1.0 + count / n * (scale ** 2 - 1.0)))
    for i in range(b):
        x = torch.randn(T, n, generator=g, device="cuda")
        x[:, torch.randperm(n, generator=g, device="cuda")[:count]] *= scale
        x *= torch.exp(0.3 * torch.randn(T, 1, generator=g, device="cuda")) / rms
        (X[i] if b > 1 else X).copy_(x)
    return X


def _rotation(b, n, g):
    """Randomised orthogonal matrices: a cosine transform with permuted columns and random signs of the rows (the initial
    latent of the method is a randomised Hadamard matrix, which exists for few n)."""
    k = torch.arange(n, device="cuda", dtype=torch.float64)
    C = torch.cos((math.pi / (2 * n)) * k[:, None] * (2 * k + 1)[None, :]) * math.sqrt(2.0 / n)
    C[0] *= math.sqrt(0.5)
    Q = _matrix(b, n, n, torch.float32)
    for i in range(b):
        sign = torch.randint(0, 2, (n, 1), generator=g, device="cuda", dtype=torch.float64) * 2 - 1
        (Q[i] if b > 1 else Q).copy_(sign * C[:, torch.randperm(n, generator=g, device="cuda")])
    return Q


def _latent(case, g):
    """"gauss": a Gaussian start, as the benchmark has it.  "moved": a rotation as the start, moved by the steps since."""
    b, n = case["b"], case["n"]
    noise = torch.randn((b, n, n) if b > 1 else (n, n), generator=g, device="cuda")
    if case["latent"] == "gauss":
        Z = _matrix(b, n, n, torch.float32)
        Z.copy_(noise)
        return Z
    Z = _rotation(b, n, g)
    Z += noise * (0.3 / math.sqrt(n))
    return Z


_context = None


def _ctx(b, n, T, xdt):
    global _context
    if _context is None:
        _context = B.Context()
    _context.ensure_workspace(b, n, T, xdt)
    return _context


def prepare(case, seed):
    b, n, T, kind = case["b"], case["n"], case["T"], case["kind"]
    dtype, xdt = _DTYPE[case["x"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    st = {"case": case, "ctx": _ctx(b, n, T, xdt), "xdt": xdt, "loss": torch.zeros(b, device="cuda")}
    if kind == "pass":
        # the channels of a rotated block are close to normal with a scale per token
        Y = torch.randn(T, n, generator=g, device="cuda") * torch.exp(0.5 * torch.randn(T, 1, generator=g, device="cuda"))
        st["Y"] = _matrix(1, T, n, torch.float32)
        st["Y"].copy_(Y)
        st["dY"] = _matrix(1, T, n, dtype, 0.0)
        return st
    if kind != "cayley":
        st["Z"] = _latent(case, g)
    if kind == "qr":
        st["R"], st["U"] = _matrix(b, n, n, torch.float32, 0.0), _matrix(b, n, n, torch.float32, 0.0)
        return st
    st["X"] = _activations(case, g)
    if kind == "step" and case["update"] == "adam":
        st["m"], st["v"], st["t"] = _matrix(b, n, n, torch.float32, 0.0), _matrix(b, n, n, torch.float32, 0.0), 0
    if kind == "staged":
        for k in ("R", "U", "G", "dZ", "buf"):
            st[k] = _matrix(b, n, n, torch.float32, 0.0)
    if kind == "cayley":
        # this optimiser starts from a rotation
        st["R"], st["M"] = _rotation(b, n, g), _matrix(b, n, n, torch.float32, 0.0)
    return st


def run(st):
    case, ctx, xdt, loss = st["case"], st["ctx"], st["xdt"], st["loss"]
    kind, red = case["kind"], B.DQ_REDUCE_TOKEN_MEAN
    if kind == "step" and case["update"] == "sgd":
        ctx.dq_calib_step(st["X"], xdt, st["Z"], case["lr"], red, loss)
        return loss, st["Z"]
    if kind == "step":
        st["t"] += 1
        ctx.dq_calib_step_adam(st["X"], xdt, st["Z"], st["m"], st["v"], st["t"], case["lr"], red, loss)
        return loss, st["Z"], st["m"], st["v"]
    if kind == "staged":
        ctx.dq_qr_orth(st["Z"], st["R"], st["U"])
        ctx.dq_rotate_loss_grad(st["X"], xdt, st["R"], red, loss, st["G"])
        ctx.dq_qr_backward(st["R"], st["U"], st["G"], st["dZ"])
        ctx.dq_sgd_momentum_update(st["Z"], st["dZ"], st["buf"], case["lr"], case["mu"])
        return loss, st["R"], st["U"], st["G"], st["dZ"], st["Z"], st["buf"]
    if kind == "qr":
        ctx.dq_qr_orth(st["Z"], st["R"], st["U"])
        return st["R"], st["U"]
    if kind == "cayley":
        ctx.dq_cayley_step(st["X"], xdt, st["R"], st["M"], case["lr"], red, loss, beta=case["beta"])
        return loss, st["R"], st["M"]
    ctx.dq_objective_loss_grad(_OBJECTIVE[case["objective"]], _QUANT_BITS, st["Y"], red, loss, st["dY"], xdt)
    return loss, st["dY"]


def work(case):
    """Dense operation counts (QR 4/3 n^3, forming R 4/3 n^3, derivative 4 n^3, 2 T n^2 a product with the block, 2 n^3 a
    product of the comparison optimiser) and each input read once, each output written once."""
    b, n, T, kind = case["b"], float(case["n"]), float(case["T"]), case["kind"]
    e = 2.0 if case["x"] == "bf16" else 4.0
    nn = 4.0 * n * n
    if kind == "pass":
        return {"bytes": T * n * (4.0 + e), "flops": 5.0 * T * n}
    if kind == "qr":
        return {"bytes": 3.0 * nn, "flops": 8.0 / 3.0 * n ** 3}
    if kind == "cayley":
        return {"bytes": e * T * n + 4.0 * nn, "flops": 4.0 * T * n * n + 12.0 * n ** 3}
    flops = b * (4.0 * T * n * n + 20.0 / 3.0 * n ** 3)
    if kind == "staged":
        return {"bytes": b * (e * T * n + 8.0 * nn), "flops": flops}
    return {"bytes": b * (e * T * n + (6.0 if case["update"] == "adam" else 2.0) * nn), "flops": flops}


def tolerance(case):
    """About four times what two routes of the library differ by after two passes (Householder panels against CholeskyQR,
    fp32 products against split ones, staged against fused), over three seeds of every listed and two dozen drawn cases.

    dY jumps at y = 0: an entry of Y within rounding of zero takes either sign, and each such entry moves its column of the
    gradient by 2 x_t / T.  With Y good to 1e-6 that is 4 sqrt(0.8e-6) = 4e-3 of the gradient's norm, most of a single
    entry where it happens; the rotation and the latent do not feel it."""
    kind = case["kind"]
    if kind == "pass":
        # the codes of the quantiser are decided in fp32; bf16 gradients agree but for their last bit
        return {"rel": 1e-3, "max": 0.02} if case["x"] == "bf16" else {"rel": 1e-5, "max": 1e-3}
    if kind == "qr":
        return {"rel": 4e-6, "max": 1e-4}
    if kind == "cayley":
        return {"rel": 4e-3, "max": 0.9}
    if kind == "step" and case["update"] == "sgd":
        return {"rel": 2e-5, "max": 6e-3}
    return {"rel": 2.5e-2, "max": 0.99}
