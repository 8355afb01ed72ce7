"""256 classes, workgroups of four waves and of eight: at positions and chunks on both sides of the line between them and with a
second pair of sample tiles (whose workgroups pass it), against the oracle's decisions and the on-GPU sequential sampler.  Both
forms give the same bits and nothing a call returns names the one that ran: the sizes are taken from the rule itself
(257 .. 512 workgroups, positions times pairs of sample tiles, and 16 chunks: eight waves)."""
import numpy as np
import pytest
import torch

from oracle import made_oracle as O
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,N", [(256, 520, 33), (257, 520, 1), (257, 470, 33), (257, 520, 64), (257, 520, 65)])
def test_both_shapes(D, H, N):
    w = S.Workload(f"cw{D}", D, 256, [H], "f32", N, "random", "fan_in", S.SEED_BASE + 2400 + H, gain=1.5)
    net = S.make_network(w, with_bias=True)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, None)
    h = B.model_from_network(net)
    try:
        g = torch.from_numpy(noise).cuda()
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        B.jacobi_sample(h, g, N, None, 0, x)
        torch.cuda.synchronize()
        xj = x.cpu().numpy()
        ok, margin = O.fixed_point_check(ref, xj[:8], noise[:8])
        assert (ok | (margin < 1e-3)).all()
        x.fill_(9)
        B.sequential_sample(h, g, N, 1, x)
        torch.cuda.synchronize()
        assert (x.cpu().numpy() == xj).all()           # (one order of sums: the same bits)
    finally:
        B.made_free(h)
