"""GPU parity of the recurrent-network entry points (include/jacobi_rnn.h) against oracle/rnn_oracle.py on the
same seeded inputs.  Tolerances, relative to the largest entry of the compared tensor: 1e-5 where the GPU
computes in fp32 (forward pass, standard backward pass), 1e-4 where a matrix product takes its operands as two
bf16 parts each (Jacobi passes: ~2^-16 per product) or sums tens of thousands of fp32 terms (parameter gradients)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import rnn_oracle as R
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

from gpu_util import dev, progress

pytestmark = pytest.mark.gpu

F32_TOL, SPLIT_TOL = 1e-5, 1e-4


def rel_err(a, ref):
    return float(np.abs(np.asarray(a, np.float64) - ref).max() / max(np.abs(ref).max(), 1e-30))


class Case:
    """Parameters and inputs of one workload; the backward pass gets the oracle's forward results rounded to fp32,
    and the oracle continues from those same fp32 values."""

    def __init__(self, w, rep=0):
        self.w = w
        W, U, b = S.make_rnn_params(w)
        b = (b + 0.05 * np.arange(w.H, dtype=np.float32) / w.H).astype(np.float32)
        x, y = S.make_rnn_inputs(w, rep)
        self.W, self.U, self.b, self.x, self.y = W, U, b, x, y
        z, h = R.rnn_forward(W.astype(np.float64), U.astype(np.float64), b.astype(np.float64), x)
        self.z_ref, self.h_ref = z, h
        self.z32, self.h32 = z.astype(np.float32), h.astype(np.float32)
        self.g32 = (h - y).astype(np.float32)
        self.W64 = W.astype(np.float64)

    def oracle_jacobi(self, n=0, eps=0.0, init=None):
        return R.jacobi_reference(self.W64, self.z32.astype(np.float64), self.g32.astype(np.float64), n, eps, init)

    def oracle_backprop(self):
        return R.backprop_sequential(self.W64, self.z32.astype(np.float64), self.g32.astype(np.float64))

    def gpu_jacobi(self, n=0, eps=0.0, init=None):
        w = self.w
        d = torch.empty((w.B, w.T, w.H), dtype=torch.float32, device="cuda")
        it = torch.full((w.B,), -1, dtype=torch.int32, device="cuda")
        cv = torch.full((w.B,), -1, dtype=torch.int32, device="cuda")
        B.rnn_backward_jacobi(dev(self.W), dev(self.z32), dev(self.g32), None if init is None else dev(init), w.B, w.T, w.H, n,
                              eps, d, it, cv)
        torch.cuda.synchronize()
        return d.cpu().numpy(), it.cpu().numpy(), cv.cpu().numpy()


@pytest.mark.parametrize("name", ["rnn_small", "rnn_wide", "rnn_paper"])
def test_rnn_parity(name):
    w = S.rnn_workload(name)
    c = Case(w)
    progress(f"rnn parity {name}: forward")
    z = torch.empty((w.B, w.T, w.H), dtype=torch.float32, device="cuda")
    h = torch.empty_like(z)
    B.rnn_forward(dev(c.W), dev(c.U), dev(c.b), dev(c.x), None, w.B, w.T, w.H, w.I, z, h)
    torch.cuda.synchronize()
    assert rel_err(z.cpu().numpy(), c.z_ref) <= F32_TOL and rel_err(h.cpu().numpy(), c.h_ref) <= F32_TOL
    h0 = np.random.default_rng(5).uniform(0, 1, (w.B, w.H)).astype(np.float32)
    B.rnn_forward(dev(c.W), dev(c.U), dev(c.b), dev(c.x), dev(h0), w.B, w.T, w.H, w.I, z, h)
    torch.cuda.synchronize()
    z0, h0_ref = R.rnn_forward(c.W64, c.U.astype(np.float64), c.b.astype(np.float64), c.x, h0)
    assert rel_err(z.cpu().numpy(), z0) <= F32_TOL and rel_err(h.cpu().numpy(), h0_ref) <= F32_TOL

    progress(f"rnn parity {name}: standard backward pass")
    d_ref = c.oracle_backprop()
    d = torch.empty((w.B, w.T, w.H), dtype=torch.float32, device="cuda")
    B.rnn_backward_sequential(dev(c.W), dev(c.z32), dev(c.g32), w.B, w.T, w.H, d)
    torch.cuda.synchronize()
    assert rel_err(d.cpu().numpy(), d_ref) <= F32_TOL

    progress(f"rnn parity {name}: Jacobi_n")
    for n in (1, 2, 7, w.T // 2, w.T, 0):
        dj, it, cv = c.gpu_jacobi(n)
        ref, it_ref, cv_ref, _ = c.oracle_jacobi(n)
        assert rel_err(dj, ref) <= SPLIT_TOL, (n, rel_err(dj, ref))
        assert (it == it_ref).all() and (it == (w.T if n in (0, w.T) else n)).all()
        assert (cv == 0).all() or n in (0, w.T)      # eps = 0 is only met if a pass changes nothing at all
    # T passes reproduce the standard backward pass (Proposition 1), and truncation approaches it (Section 5.1)
    dj, _, _ = c.gpu_jacobi(0)
    assert rel_err(dj, d_ref) <= SPLIT_TOL
    errs = [rel_err(c.gpu_jacobi(n)[0], d_ref) for n in (1, 4, 16)]
    assert errs[0] > errs[1] > errs[2]

    progress(f"rnn parity {name}: forward-difference stop, initial iterate")
    scale = np.abs(d_ref).max()
    for eps in (1e-2 * scale, 1e-4 * scale):
        dj, it, cv = c.gpu_jacobi(0, float(eps))
        ref, it_ref, cv_ref, diffs = c.oracle_jacobi(0, float(eps))
        # a sequence whose forward differences all stay clear of eps must stop at the oracle's pass
        clear = np.ones(w.B, dtype=bool)
        for dk in diffs:
            clear &= ~(np.abs(dk - eps) <= 0.05 * eps)
        assert clear.any()
        assert (it[clear] == it_ref[clear]).all() and (cv[clear] == cv_ref[clear]).all(), (eps, it, it_ref)
        assert np.abs(it - it_ref).max() <= 1
        for bi in np.nonzero(clear)[0]:
            assert rel_err(dj[bi], ref[bi]) <= SPLIT_TOL
    init = np.random.default_rng(6).standard_normal((w.B, w.T, w.H)).astype(np.float32)
    for n in (1, 3, 0):
        dj, it, cv = c.gpu_jacobi(n, 0.0, init)
        ref, it_ref, _, _ = c.oracle_jacobi(n, 0.0, init.astype(np.float64))
        assert rel_err(dj, ref) <= SPLIT_TOL * max(1.0, np.abs(init).max() / np.abs(ref).max()) and (it == it_ref).all()

    progress(f"rnn parity {name}: parameter gradients")
    dW = torch.empty((w.H, w.H), dtype=torch.float32, device="cuda")
    dU = torch.empty((w.H, w.I), dtype=torch.float32, device="cuda")
    db = torch.empty((w.H,), dtype=torch.float32, device="cuda")
    d32 = d_ref.astype(np.float32)
    B.rnn_param_grads(dev(c.z32), dev(c.h32), dev(c.x), dev(d32), None, w.B, w.T, w.H, w.I, dW, dU, db)
    torch.cuda.synchronize()
    rW, rU, rb = R.param_grads(c.z32.astype(np.float64), c.h32.astype(np.float64), c.x, d32.astype(np.float64))
    assert rel_err(dW.cpu().numpy(), rW) <= SPLIT_TOL and rel_err(dU.cpu().numpy(), rU) <= SPLIT_TOL
    assert rel_err(db.cpu().numpy(), rb) <= SPLIT_TOL
    B.rnn_param_grads(dev(c.z32), dev(c.h32), dev(c.x), dev(d32), dev(h0), w.B, w.T, w.H, w.I, dW, dU, db)
    torch.cuda.synchronize()
    rW0, _, _ = R.param_grads(c.z32.astype(np.float64), c.h32.astype(np.float64), c.x, d32.astype(np.float64), h0)
    assert rel_err(dW.cpu().numpy(), rW0) <= SPLIT_TOL


def test_rnn_edge_cases():
    # largest shape of the Jacobi call at H = 128, a single step, an empty batch, and the argument errors
    for (Bn, T, H, I) in ((2, 128, 128, 1), (3, 1, 40, 2), (2, 256, 64, 1), (1, 33, 1, 1), (2, 97, 65, 1)):
        progress(f"rnn edge case B={Bn} T={T} H={H}")
        w = dataclasses.replace(S.rnn_workload("rnn_small"), B=Bn, T=T, H=H, I=I, w_std=min(0.2, 1.2 / np.sqrt(H)))
        c = Case(w)
        for n in (0, 3):
            dj, it, cv = c.gpu_jacobi(n)
            ref, it_ref, _, _ = c.oracle_jacobi(n)
            assert rel_err(dj, ref) <= SPLIT_TOL
            # with eps = 0 a sequence ends before the pass limit only if a pass changed nothing at all, and when
            # that happens depends on the arithmetic (fp64 there, fp32 with split products here)
            assert ((it == it_ref) | ((cv == 1) & (it <= it_ref))).all(), (it, it_ref, cv)
        d = torch.empty((Bn, T, H), dtype=torch.float32, device="cuda")
        B.rnn_backward_sequential(dev(c.W), dev(c.z32), dev(c.g32), Bn, T, H, d)
        torch.cuda.synchronize()
        assert rel_err(d.cpu().numpy(), c.oracle_backprop()) <= F32_TOL
    w = S.rnn_workload("rnn_small")
    c = Case(w)
    empty = torch.empty((0, w.T, w.H), dtype=torch.float32, device="cuda")
    B.rnn_backward_jacobi(dev(c.W), empty, empty, None, 0, w.T, w.H, 0, 0.0, empty)
    B.rnn_backward_sequential(dev(c.W), empty, empty, 0, w.T, w.H, empty)
    d = torch.empty((w.B, w.T, w.H), dtype=torch.float32, device="cuda")
    for call in (lambda: B.rnn_backward_jacobi(dev(c.W), dev(c.z32), dev(c.g32), None, w.B, 200, 100, 0, 0.0, d),
                 lambda: B.rnn_backward_jacobi(dev(c.W), dev(c.z32), dev(c.g32), None, w.B, w.T, w.H, 0, -1.0, d),
                 lambda: B.rnn_backward_jacobi(dev(c.W), dev(c.z32), dev(c.g32), None, w.B, w.T, 129, 0, 0.0, d),
                 lambda: B.rnn_backward_sequential(dev(c.W), None, dev(c.g32), w.B, w.T, w.H, d)):
        with pytest.raises(B.MadeError) as e:
            call()
        assert e.value.code == B.MADE_ERR_ARG


def test_rnn_full_batch():
    """256 sequences of the paper's shape in one call (the launch bench.py times); the oracle checks a sample of them."""
    w = S.rnn_workload("rnn_batch")
    c = Case(w)
    progress("rnn full batch: Jacobi_10, Jacobi_T, standard backward pass")
    d_ref = c.oracle_backprop()
    for n in (10, 0):
        dj, it, cv = c.gpu_jacobi(n)
        ref, it_ref, _, _ = c.oracle_jacobi(n)
        assert rel_err(dj, ref) <= SPLIT_TOL and (it == it_ref).all()
    d = torch.empty((w.B, w.T, w.H), dtype=torch.float32, device="cuda")
    B.rnn_backward_sequential(dev(c.W), dev(c.z32), dev(c.g32), w.B, w.T, w.H, d)
    torch.cuda.synchronize()
    assert rel_err(d.cpu().numpy(), d_ref) <= F32_TOL


@pytest.mark.parametrize("B_,T,H,I", [(1, 1, 1, 1), (1, 63, 31, 7), (2, 32, 32, 8), (13, 5, 33, 6), (1, 512, 64, 1), (27, 19, 65, 2),
                                      (3, 171, 96, 16), (4, 200, 97, 1), (180, 100, 128, 3)])
def test_param_grads_slices_and_strips(B_, T, H, I):
    """Edges of the gradient kernel: chunks of 64 rows, one slice (up to 512 rows) and several, strips of 32 units, the
    eight [1, x] columns per block.  fp32 sums of R rows: about sqrt(R) ulp each way, 2e-6 of the largest entry at most."""
    progress(f"rnn gradients B={B_} T={T} H={H} I={I}")
    r = np.random.default_rng(17)
    z, h, d = (r.standard_normal((B_, T, H)).astype(np.float32) for _ in range(3))
    x, h0 = r.standard_normal((B_, T, I)).astype(np.float32), r.standard_normal((B_, H)).astype(np.float32)
    for init in (None, h0):
        dW, dU, db = (torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((H, H), (H, I), (H,)))
        B.rnn_param_grads(dev(z), dev(h), dev(x), dev(d), None if init is None else dev(init), B_, T, H, I, dW, dU, db)
        torch.cuda.synchronize()
        ref = R.param_grads(*(a.astype(np.float64) for a in (z, h, x, d)), None if init is None else init.astype(np.float64))
        for got, want in zip((dW, dU, db), ref):
            assert rel_err(got.cpu().numpy(), want) <= 2e-6 * max(1.0, np.sqrt(B_ * T) / 20)


@pytest.mark.parametrize("B_,T,H,I", [(1, 1, 1, 1), (2, 3, 31, 5), (1, 4, 32, 1), (3, 5, 33, 2), (1, 7, 64, 1), (2, 9, 95, 3), (1, 8, 96, 1),
                                      (1, 2, 97, 1), (2, 131, 127, 1), (1, 65, 128, 6)])
def test_recurrences_at_tile_edges(B_, T, H, I):
    """The step kernels at the edges of their 32-unit widths and of the groups of four steps.  F32_TOL as elsewhere."""
    progress(f"rnn recurrences B={B_} T={T} H={H} I={I}")
    w = dataclasses.replace(S.rnn_workload("rnn_small"), B=B_, T=T, H=H, I=I, w_std=min(0.2, 1.2 / np.sqrt(H)))
    c = Case(w)
    z, h, d = (torch.empty((B_, T, H), dtype=torch.float32, device="cuda") for _ in range(3))
    h0 = np.random.default_rng(5).uniform(0, 1, (B_, H)).astype(np.float32)
    for init in (None, h0):
        B.rnn_forward(dev(c.W), dev(c.U), dev(c.b), dev(c.x), None if init is None else dev(init), B_, T, H, I, z, h)
        torch.cuda.synchronize()
        z_ref, h_ref = R.rnn_forward(c.W64, c.U.astype(np.float64), c.b.astype(np.float64), c.x, init)
        assert rel_err(z.cpu().numpy(), z_ref) <= F32_TOL and rel_err(h.cpu().numpy(), h_ref) <= F32_TOL
    B.rnn_backward_sequential(dev(c.W), dev(c.z32), dev(c.g32), B_, T, H, d)
    torch.cuda.synchronize()
    assert rel_err(d.cpu().numpy(), c.oracle_backprop()) <= F32_TOL


def _activations(v, what):
    """softplus (forward pass, one unit and one step, z = x) or sigmoid (backward pass, W = 1: d_0[j] = sigmoid(z_1[j])) of a
    float32 array whose length is a multiple of 128."""
    n = v.size // 128
    if what == "softplus":
        z, h = (torch.empty((v.size, 1, 1), dtype=torch.float32, device="cuda") for _ in range(2))
        W, U, b = np.zeros((1, 1), np.float32), np.ones((1, 1), np.float32), np.zeros(1, np.float32)
        B.rnn_forward(dev(W), dev(U), dev(b), dev(v.reshape(-1, 1, 1)), None, v.size, 1, 1, 1, z, h)
        return h.cpu().numpy().reshape(-1)
    n = v.size // 128
    zz, g = np.zeros((n, 2, 128), np.float32), np.zeros((n, 2, 128), np.float32)
    zz[:, 1], g[:, 1] = v.reshape(n, 128), 1.0
    d = torch.empty((n, 2, 128), dtype=torch.float32, device="cuda")
    B.rnn_backward_sequential(dev(np.eye(128, dtype=np.float32)), dev(zz), dev(g), n, 2, 128, d)
    return d.cpu().numpy()[:, 0].reshape(-1)


@pytest.mark.parametrize("lo,hi,largest,mean", [(-110, -87.4, 2.0, 0.53), (-87.3, -20, 2.0, 0.40), (-20, -5, 2.25, 0.472), (-5, -1, 2.15, 0.485),
                                                (-1, 0, 1.87, 0.45), (0, 1, 1.6, 0.43), (1, 5, 1.35, 0.382), (5, 100, 1.1, 0.259)])
def test_activations_over_their_range(lo, hi, largest, mean):
    """softplus and sigmoid of single values against extended precision, in units of 2^-24 of the value (of the smallest
    normal number below it).  The bounds are what log1pf(expf(z)) of the device library shows on these ranges (its
    sigmoid, 1 / (1 + expf(-z)), is worse by a third); a last rounding alone has a largest error of 1 and a mean of 0.35."""
    progress(f"rnn activations {lo}..{hi}")
    v = np.linspace(lo, hi, 1 << 17, dtype=np.float32)
    x = v.astype(np.longdouble)
    for what, want in (("softplus", np.maximum(x, 0) + np.log1p(np.exp(-np.abs(x)))), ("sigmoid", 1 / (1 + np.exp(-x)))):
        err = np.abs(_activations(v, what) - want) / (np.maximum(want, 2.0 ** -126) * 2.0 ** -24)
        assert err.max() <= largest and err.mean() <= mean, (what, float(err.max()), float(err.mean()))


def test_activations_of_special_values():
    v = np.resize(np.array([0.0, -0.0, 1e-40, -1e-40, 104.0, -104.0, 1e30, -1e30, np.inf, -np.inf, np.nan], np.float32), 128)
    x = v.astype(np.float64)
    with np.errstate(over="ignore", invalid="ignore"):
        for what, want in (("softplus", np.maximum(x, 0) + np.log1p(np.exp(-np.abs(x)))), ("sigmoid", 1 / (1 + np.exp(-x)))):
            got = _activations(v, what) if what == "softplus" else _activations(np.where(np.isnan(v), 0, v), what)
            want = np.where(np.isnan(v) & (what == "sigmoid"), 0.5, want)
            assert np.array_equal(got, want.astype(np.float32), equal_nan=True), (what, got, want)


@pytest.mark.parametrize("B_,T,H,I", [(180, 100, 128, 3), (40, 64, 33, 2), (70, 100, 20, 1), (30, 100, 96, 9)])
def test_param_grads_repeat_bit_for_bit(B_, T, H, I):
    """Gradients of many rows are summed in slices: the same bits from call to call, from eight streams at once (more
    calls than there are places for partial sums), and from replays of a recorded call with other calls in between."""
    progress(f"rnn gradients repeat B={B_} T={T} H={H} I={I}")
    gen = torch.Generator(device="cuda").manual_seed(3)
    z, h, d = (torch.randn(B_, T, H, generator=gen, device="cuda") for _ in range(3))
    x, h0 = torch.randn(B_, T, I, generator=gen, device="cuda"), torch.randn(B_, H, generator=gen, device="cuda")
    outputs = lambda: [torch.full(s, 7.0, device="cuda") for s in ((H, H), (H, I), (H,))]
    call = lambda out: B.rnn_param_grads(z, h, x, d, h0, B_, T, H, I, *out)
    first = outputs()
    call(first)
    torch.cuda.synchronize()
    same = lambda out: all(torch.equal(a, b) for a, b in zip(out, first))
    streams = [torch.cuda.Stream() for _ in range(8)]
    outs = [[outputs() for _ in range(6)] for _ in streams]
    torch.cuda.synchronize()
    for i in range(6):
        for s, o in zip(streams, outs):
            with torch.cuda.stream(s):
                call(o[i])
    torch.cuda.synchronize()
    assert all(same(o) for stream in outs for o in stream)
    recorded, eager = outputs(), outputs()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(recorded)
    for _ in range(4):
        for o in recorded + eager:
            o.fill_(3.0)
        graph.replay()
        call(eager)
        torch.cuda.synchronize()
        assert same(recorded) and same(eager)


@pytest.mark.parametrize("T", [1, 2, 5])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_last_state_does_not_read_the_weights(T, bad):
    """d_T = g_T in the standard backward pass, also with weights that are infinite or no numbers."""
    B_, H = 2, 33
    r = np.random.default_rng(2)
    z, g = (r.standard_normal((B_, T, H)).astype(np.float32) for _ in range(2))
    W = np.full((H, H), bad, np.float32)
    d = torch.empty((B_, T, H), dtype=torch.float32, device="cuda")
    B.rnn_backward_sequential(dev(W), dev(z), dev(g), B_, T, H, d)
    assert np.array_equal(d.cpu().numpy()[:, -1], g[:, -1])


@pytest.mark.parametrize("H,T", [(20, 480), (20, 481), (32, 512), (1, 500), (33, 256)])
def test_jacobi_with_one_and_two_copies_of_the_product_s_input(H, T):
    """A pass reads one copy of X in LDS and writes the other where two fit: up to 480 steps of up to 32 units, and every
    longer shape of more units; beyond, one copy is updated in place.  Two samples, from zeros and from a start of one's own."""
    progress(f"rnn jacobi H={H} T={T}")
    w = dataclasses.replace(S.rnn_workload("rnn_small"), B=2, T=T, H=H, I=2, w_std=min(0.2, 1.2 / np.sqrt(H)))
    c = Case(w)
    init = np.random.default_rng(2).standard_normal((w.B, T, H)).astype(np.float32)
    for start in (None, init):
        for n in (1, 2, 3, 10):
            d, it, cv = c.gpu_jacobi(n, 0.0, start)
            ref, it_ref, _, _ = c.oracle_jacobi(n, 0.0, start)
            # (one unit of weight 0.0116: a pass moves its iterate by 0.006 of what the one before did, so that fp32 stands still
            # after six)
            assert n > 3 or ((it == n).all() and (it_ref == n).all() and (cv == 0).all())
            assert rel_err(d, ref) <= SPLIT_TOL, (start is None, n)
        d, it, cv = c.gpu_jacobi(0, 1e-3, start)
        assert (cv == 1).all() and (it < T).all()
        d, it, cv = c.gpu_jacobi(0, 0.0, start)
        assert rel_err(d, c.oracle_backprop()) <= SPLIT_TOL
