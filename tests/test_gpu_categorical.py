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
                out[call, fused] = (x.cpu().numpy(), it.cpu().numpy())
        for call in ("jacobi", "gs", "sequential"):
            x, it = out[call, 1]
            ok, margin = O.fixed_point_check(ref, x, noise)
            assert (ok | (margin < 1e-3)).all(), call
            clear = margin.min(axis=1) >= 1e-3       # (at a fixed point both forms reached: the same one)
            assert (x[clear] == out[call, 0][0][clear]).all(), call
        assert (out["jacobi", 1][0][clear] == out["sequential", 1][0][clear]).all()
    finally:
        B.made_free(h)
