"""The work a user of the framework has it do, as cases that can be timed and compared.

A case names a kind of model, its sizes, a solver and a batch.  Networks are random ones of that shape (weights
N(0, 1/fan_in), hidden degrees drawn uniformly), made once per shape and kept, as a program that samples keeps its
model; what changes from call to call -- the noise, or for the recurrent network everything it is given -- is drawn
from the seed.  One pass is one whole call (for the recurrent network one training step: forward pass, loss
gradient, backward pass, parameter gradients).
"""
import functools
import math
import weakref

import numpy as np
import torch

from paper_2002_03629_amd import binding as B

DEV = "cuda"


def listed():
    return [
        # the smallest call: 64 binary positions, one hidden layer, single precision, a handful of samples; launches
        # and latencies only
        {"name": "tiny_f32_b16", "kind": "mlp", "solver": "jacobi", "D": 64, "H": 256, "L": 1, "dtype": "f32", "N": 16},
        # about a hundred 28 x 28 binary images drawn in parallel: the ordinary sampling call
        {"name": "made_b128", "kind": "mlp", "solver": "jacobi", "D": 784, "H": 2000, "L": 2, "dtype": "bf16", "N": 128},
        # a server's or an evaluation's batch, not a multiple of any tile
        {"name": "made_b1000", "kind": "mlp", "solver": "jacobi", "D": 784, "H": 2000, "L": 2, "dtype": "bf16", "N": 1000},
        # a data set's worth of samples in one call: throughput
        {"name": "made_b32768", "kind": "mlp", "solver": "jacobi", "D": 784, "H": 2000, "L": 2, "dtype": "bf16", "N": 32768},
        # the hybrid solver with short blocks: many small passes, one after the other
        {"name": "made_gs16_b128", "kind": "mlp", "solver": "gs", "block": 16, "D": 784, "H": 2000, "L": 2, "dtype": "bf16", "N": 128},
        # the sequential sampler, one position at a time: what the parallel solvers are compared with
        {"name": "made_seq_b128", "kind": "mlp", "solver": "sequential", "D": 784, "H": 2000, "L": 2, "dtype": "bf16", "N": 128},
        # 32 x 32 grey images of 256 levels: an output layer of 2 GiB, read once per iteration
        {"name": "cat256_b64", "kind": "cat", "onehot": False, "D": 1024, "C": 256, "H": 4096, "L": 2, "dtype": "bf16", "N": 64},
        # one-hot symbols of another class count, a batch that fills no tile
        {"name": "onehot64_b100", "kind": "cat", "onehot": True, "D": 512, "C": 64, "H": 1024, "L": 2, "dtype": "bf16", "N": 100},
        # real-valued pixels with logistic conditionals, 100 images, solved to the fixed point
        {"name": "logistic_b100", "kind": "real", "eps": 0.0, "D": 784, "H": 512, "L": 2, "dtype": "bf16", "N": 100},
        # 32 x 32 colour images from a masked convolutional network, 8 layers of 5 x 5
        {"name": "conv_b32", "kind": "conv", "rows": 32, "F": 128, "k": 5, "layers": 8, "dtype": "bf16", "N": 32},
        # a training step of the recurrent network on one sequence, backward pass by ten Jacobi iterations
        {"name": "rnn_b1", "kind": "rnn", "n": 10, "T": 100, "H": 128, "I": 1, "B": 1},
        # the same step on a batch with a sequence for every compute unit
        {"name": "rnn_b256", "kind": "rnn", "n": 10, "T": 100, "H": 128, "I": 1, "B": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mlp", "mlp", "mlp", "mlp", "cat", "real", "conv", "rnn"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "mlp":
        solver = rng.choice(["jacobi", "jacobi", "jacobi", "gs", "sequential"])
        c = {"kind": kind, "solver": solver, "D": _log_int(rng, 40, 1024), "H": _log_int(rng, 100, 2048), "L": rng.randint(1, 2),
             "dtype": dtype, "N": _log_int(rng, 1, 32768)}
        if solver != "jacobi":
            c["N"] = _log_int(rng, 1, 1024 if solver == "gs" else 256)
        elif dtype == "f32":          # single precision has a sixteenth of the matrix rate
            c["N"] = _log_int(rng, 1, 2048)
        if solver == "gs":
            c["block"] = _log_int(rng, 4, max(8, c["D"] // 4))
        return c
    if kind == "cat":
        onehot = rng.random() < 0.5
        return {"kind": kind, "onehot": onehot, "D": _log_int(rng, 24, 512), "C": rng.choice([256, 256, rng.randint(5, 255)]),
                "H": _log_int(rng, 96, 2048), "L": rng.randint(1, 2), "dtype": dtype, "N": _log_int(rng, 1, 128)}
    if kind == "real":
        return {"kind": kind, "eps": rng.choice([0.0, 0.01, 0.1]), "D": _log_int(rng, 50, 1024), "H": _log_int(rng, 64, 1024),
                "L": rng.randint(1, 2), "dtype": dtype, "N": _log_int(rng, 1, 512)}
    if kind == "conv":
        return {"kind": kind, "rows": rng.randint(3, 32), "F": rng.choice([64, 128]), "k": rng.choice([3, 5, 7]),
                "layers": rng.randint(2, 8), "dtype": dtype if rng.random() < 0.5 else "bf16", "N": _log_int(rng, 1, 32)}
    H = rng.randint(17, 128)
    T = rng.randint(20, min(200, B.rnn_jacobi_max_steps(H)))
    # n = 0: the standard backward pass, one step after the other
    return {"kind": kind, "n": rng.choice([0, 5, 10, 20]), "T": T, "H": H, "I": rng.randint(1, 4), "B": _log_int(rng, 1, 512)}


# ------------------------------------------------------------------------------------------------
# models: one per shape, kept by the program
# ------------------------------------------------------------------------------------------------
class _Model:
    def __init__(self, handle):
        self.handle = handle
        weakref.finalize(self, B.made_free, handle)


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weights(shape, fan_in, gen, gain=1.0):
    """A host matrix of the given shape, drawn on the GPU in slices (the largest has 2^30 entries)."""
    out = np.empty(shape, np.float32)
    flat = torch.from_numpy(out).view(-1)
    step = 1 << 27
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n].copy_(torch.randn(n, generator=gen, device=DEV).mul_(gain / math.sqrt(fan_in)))
    return out


def _degrees(D, H, L):
    r = np.random.Generator(np.random.Philox(1000003 * D + 1009 * H + L))
    return [r.integers(1, D, size=H).astype(np.int32) for _ in range(L)]


@functools.lru_cache(maxsize=2)
def _mlp(D, C, H, L, dtype, real, onehot):
    gen = _generator(D + 7 * C + 13 * H + L)
    dims = [D * C if onehot else D] + [H] * L + [D * C]
    W = []
    for l in range(L + 1):
        fan_in = D if l == 0 else dims[l]
        W.append(_weights((dims[l + 1], dims[l]), fan_in, gen))
    handle = B.made_init(D, C, [H] * L, B.MADE_BF16 if dtype == "bf16" else B.MADE_F32, _degrees(D, H, L), W, None, real, onehot)
    return _Model(handle)


@functools.lru_cache(maxsize=2)
def _conv(rows, F, k, layers, dtype):
    gen = _generator(rows + 7 * F + 13 * k + layers)
    shapes = [(F, k, k, 3)] + [(F, k, k, F)] * (layers - 1) + [(3 * 256, 1, 1, F)]
    # about half of the taps are visible and ReLU halves the variance: this gain keeps the logits' scale over the depth
    W = [_weights(s, s[1] * s[2] * s[3], gen, 2.3) for s in shapes]
    return _Model(B.made_conv_init(rows, 32, 256, F, k, layers, B.MADE_BF16 if dtype == "bf16" else B.MADE_F32, W))


def _gumbel(shape, gen):
    u = torch.rand(shape, generator=gen, device=DEV).clamp_(2.0 ** -24, 1.0 - 2.0 ** -24)
    return u.log_().neg_().log_().neg_()


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind == "rnn":
        b, T, H, I = case["B"], case["T"], case["H"], case["I"]
        f = functools.partial(torch.empty, device=DEV)
        s = {"W": torch.randn(H, H, generator=gen, device=DEV) * 0.1, "U": torch.randn(H, I, generator=gen, device=DEV) * 0.1,
             "b": torch.zeros(H, device=DEV), "x": torch.rand(b, T, I, generator=gen, device=DEV),
             "y": torch.rand(b, T, H, generator=gen, device=DEV) * 0.9 + 0.3,
             "z": f(b, T, H), "h": f(b, T, H), "g": f(b, T, H), "d": f(b, T, H), "dW": f(H, H), "dU": f(H, I), "db": f(H)}
        return {"case": case, **s}
    N = case["N"]
    if kind == "conv":
        D = case["rows"] * 96
        model = _conv(case["rows"], case["F"], case["k"], case["layers"], case["dtype"])
        return {"case": case, "model": model, "noise": _gumbel((N, D, 256), gen), "x": torch.empty(N, D, dtype=torch.uint8, device=DEV)}
    D, H, L = case["D"], case["H"], case["L"]
    if kind == "mlp":
        noise = torch.rand(N, D, generator=gen, device=DEV)
        model = _mlp(D, 1, H, L, case["dtype"], False, False)
    elif kind == "cat":
        noise = _gumbel((N, D, case["C"]), gen)
        model = _mlp(D, case["C"], H, L, case["dtype"], False, case["onehot"])
    else:
        noise = torch.rand(N, D, generator=gen, device=DEV).clamp_(2.0 ** -24, 1.0 - 2.0 ** -24).logit_()
        model = _mlp(D, 2, H, L, case["dtype"], True, False)
    x = torch.empty(N, D, dtype=torch.float32 if kind == "real" else torch.uint8, device=DEV)
    return {"case": case, "model": model, "noise": noise, "x": x}


def run(s):
    c = s["case"]
    if c["kind"] == "rnn":
        b, T, H, I = c["B"], c["T"], c["H"], c["I"]
        B.rnn_forward(s["W"], s["U"], s["b"], s["x"], None, b, T, H, I, s["z"], s["h"])
        torch.sub(s["h"], s["y"], out=s["g"])
        if c["n"]:
            B.rnn_backward_jacobi(s["W"], s["z"], s["g"], None, b, T, H, c["n"], 0.0, s["d"])
        else:
            B.rnn_backward_sequential(s["W"], s["z"], s["g"], b, T, H, s["d"])
        B.rnn_param_grads(s["z"], s["h"], s["x"], s["d"], None, b, T, H, I, s["dW"], s["dU"], s["db"])
        return {k: s[k] for k in ("h", "d", "dW", "dU", "db")}
    m, noise, x = s["model"].handle, s["noise"], s["x"]
    if c["kind"] == "real":
        B.jacobi_sample_real(m, noise, c["N"], None, c["eps"], 0, x)
    elif c.get("solver") == "gs":
        B.gs_jacobi_sample(m, noise, c["N"], None, c["block"], x)
    elif c.get("solver") == "sequential":
        B.sequential_sample(m, noise, c["N"], 1, x)
    else:
        B.jacobi_sample(m, noise, c["N"], None, 0, x)
    return x


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct results may be apart
# ------------------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "rnn":
        b, T, H, I, n = case["B"], case["T"], case["H"], case["I"], case["n"] or 1
        step = 2.0 * b * T * H
        # inputs x and y, outputs z, h, d and the gradients; products: forward, n passes (the first one has a zero
        # iterate), parameter gradients
        return {"bytes": 4.0 * (b * T * (I + 4 * H) + 2 * H * (H + I + 1)), "flops": step * ((H + I) + max(1, n - 1) * H + (H + I))}
    N = case["N"]
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "conv":
        F, k, rows, layers = case["F"], case["k"], case["rows"], case["layers"]
        D, mid = rows * 96, k // 2
        taps = mid * k + mid + 1
        macs = taps * F * (3 + (layers - 1) * F) + 3 * 256 * F * 2 // 3
        # two evaluations: one that reaches the fixed point and one that confirms it
        return {"bytes": float(N * D * (256 * 4 + 1) + es * macs), "flops": 2.0 * 2 * N * rows * 32 * macs}
    D, H, L = case["D"], case["H"], case["L"]
    C = {"mlp": 1, "cat": case.get("C"), "real": 2}[kind]
    degs = _degrees(D, H, L)
    first = float(degs[0].sum())
    hidden = sum(float(np.searchsorted(np.sort(degs[l - 1]), degs[l], side="right").sum()) for l in range(1, L))
    output = C * float(np.searchsorted(np.sort(degs[-1]), np.arange(1, D + 1), side="left").sum())
    nnz = first + hidden + output
    weights = nnz - first + min(C, N) * first if case.get("onehot") else nnz
    noise = 4 * (C if kind == "cat" else 1)
    evaluations = 1 if case.get("solver") == "sequential" else 2
    return {"bytes": float(weights * es + N * D * (noise + (4 if kind == "real" else 1))), "flops": 2.0 * evaluations * nnz * N}


def tolerance(case):
    kind = case["kind"]
    if kind == "rnn":       # against float64: 4e-6 (iterate), 2e-6 (gradients); largest 2e-5 of rms
        return {"rel": 2e-5, "max": 1e-4}
    if kind == "real":      # against float64 sums with the same roundings to bf16: 6e-8; a rounding that falls the other
        return {"rel": 1e-4 if case["dtype"] == "bf16" else 1e-6}     # way moves an activation by 2^-9 of itself
    if kind == "conv":      # sums taken in another order: up to 6e-2 of the symbols, the errors of 8 rounded layers
        return {"differ": 1e-2}                                       # feeding back through up to 3072 states
    # symbols: a logit within rounding of the draw's threshold falls either way and the positions behind it may follow;
    # no difference seen in 25 M symbols between three orders of the sums, and one flip may take a few with it
    return {"differ": 2e-4}
