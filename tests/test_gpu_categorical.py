"""Categorical output layer with the draw fused in, at the class counts and sizes where its tiling changes: classes
per 32-row tile below and above one, runs of positions that straddle tiles, a position over nine tiles, batches around
the pair of sample tiles.  Judged by the oracle's fixed-point certificate (positions whose decision margin is below
1e-3 exempt) and against the sampler that draws from logits in memory."""
import numpy as np
import pytest
import torch

from oracle import made_oracle as O
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,D,N,dtype", [(2, 75, 65, "bf16"), (5, 40, 1, "f32"), (31, 17, 33, "bf16"), (32, 24, 64, "f32"),
                                         (33, 19, 70, "bf16"), (64, 21, 129, "bf16"), (100, 9, 32, "f32"),
                                         (225, 6, 66, "bf16"), (226, 7, 31, "bf16"), (255, 11, 96, "f32")])
def test_fused_draw_of_any_class_count(C, D, N, dtype):
    w = S.Workload(f"any{C}", D, C, [90, 70], dtype, N, "random", "fan_in", S.SEED_BASE + 900 + C, gain=2.0)
    net = S.make_network(w, with_bias=True)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16" if dtype == "bf16" else None)
    u = torch.from_numpy(noise).cuda()
    h = B.model_from_network(net)
    try:
        out = {}
        for fused in (1, 0):
            B.made_set_option(h, B.MADE_OPT_FUSED_CATEGORICAL, fused)
            for call in ("jacobi", "gs", "sequential"):
                x = torch.full((N, D), 255, dtype=torch.uint8, device="cuda")
                it = torch.zeros((N,), dtype=torch.int32, device="cuda")
                if call == "jacobi":
                    B.jacobi_sample(h, u, N, None, 0, x, it)
                elif call == "gs":
                    B.gs_jacobi_sample(h, u, N, None, 4, x, it)
                else:
                    B.sequential_sample(h, u, N, 1, x)
                torch.cuda.synchronize()
                out[call, fused] = (x.cpu().numpy(), it.cpu().numpy(), B.made_last_stats(h)["kernels"])
        for call in ("jacobi", "gs", "sequential"):
            x = out[call, 1][0]
            ok, margin = O.fixed_point_check(ref, x, noise)
            assert (ok | (margin < 1e-3)).all(), call
            clear = margin.min(axis=1) >= 1e-3       # (at a fixed point both forms reached: the same one)
            assert (x[clear] == out[call, 0][0][clear]).all(), call
        assert (out["jacobi", 1][0][clear] == out["sequential", 1][0][clear]).all()
        # (a launch less per position where the draw is fused)
        assert out["sequential", 1][2] == out["sequential", 0][2] - D
    finally:
        B.made_free(h)


@pytest.mark.parametrize("C,D,N,dtype,onehot,hidden", [(2, 75, 65, "bf16", False, [200, 1000]), (5, 40, 1, "f32", True, [90, 333]),
                                                       (64, 40, 100, "bf16", True, [700, 900]), (33, 19, 70, "bf16", False, [500]),
                                                       (7, 100, 16, "f32", False, [150, 520]), (226, 7, 31, "bf16", False, [640]),
                                                       (100, 9, 32, "f32", False, [300]), (128, 12, 64, "bf16", False, [1024])])
def test_logits_have_the_same_bits_in_every_sampler(C, D, N, dtype, onehot, hidden):
    """Noise that is exactly minus the logits of the all-zero state: every class then scores exactly 0 and class 0 is drawn
    everywhere -- if and only if a sampler's logits have the bits of made_forward_logits, whatever run of positions and
    batch a workgroup takes them for."""
    w = S.Workload(f"bits{C}", D, C, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 950 + C, gain=2.0, onehot=onehot)
    net = S.make_network(w, with_bias=True)
    h = B.model_from_network(net)
    try:
        z = torch.empty((N, D, C), device="cuda")
        B.made_forward_logits(h, torch.zeros((N, D), dtype=torch.uint8, device="cuda"), N, z)
        noise = -z
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        it = torch.zeros((N,), dtype=torch.int32, device="cuda")
        for what, call in (("jacobi", lambda: B.jacobi_sample(h, noise, N, None, 0, x, it)),
                           ("gs 1", lambda: B.gs_jacobi_sample(h, noise, N, None, 1, x)),
                           ("gs 3", lambda: B.gs_jacobi_sample(h, noise, N, None, 3, x)),
                           ("seq 0", lambda: B.sequential_sample(h, noise, N, 0, x)), ("seq 1", lambda: B.sequential_sample(h, noise, N, 1, x))):
            x.fill_(255)
            call()
            torch.cuda.synchronize()
            assert (x == 0).all(), (what, int((x != 0).sum()))
        B.jacobi_sample(h, noise, N, None, 0, x, it)
        assert (it == 1).all()
    finally:
        B.made_free(h)
