"""Real states, Jacobi on up to 256 samples: the stop test without a tail against the one with it (the same kernels but
for where a pass's list of active samples is made: same states bit for bit, same pass counts), at the sizes where the
list fills or passes a word, a tile or the limit, with pass limits and a tolerance."""
import numpy as np
import pytest
import torch

from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hidden,dtype", [(50, [70], "f32"), (131, [96, 160], "bf16")])
@pytest.mark.parametrize("N", [1, 31, 33, 64, 100, 256, 257])
def test_with_and_without_tail(D, hidden, dtype, N):
    w = S.Workload(f"stop{D}", D, 2, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 1500 + D, gain=1.5, real=True)
    net = S.make_network(w, with_bias=True)
    gen = np.random.default_rng(D + N)
    noise = torch.from_numpy(gen.logistic(size=(N, D)).astype(np.float32)).cuda()
    x0 = torch.from_numpy(gen.normal(size=(N, D)).astype(np.float32)).cuda()
    h = B.model_from_network(net)
    B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)   # (the call in one launch makes no list)
    try:
        for init, eps, cap in ((None, 0.0, 0), (x0, 0.0, 0), (x0, 0.05, 0), (None, 0.0, 1), (None, 0.0, 3)):
            out = []
            for lazy in (1, 0):
                B.made_set_option(h, B.MADE_OPT_LAZY_STOP_TEST, lazy)
                x = torch.full((N, D), 7.0, device="cuda")
                it = torch.full((N,), -1, dtype=torch.int32, device="cuda")
                try:
                    B.jacobi_sample_real(h, noise, N, init, eps, cap, x, it)
                    stopped = True
                except B.MadeError as e:             # the pass limit was reached
                    stopped = False
                    assert cap
                out.append((x.cpu().numpy(), it.cpu().numpy(), stopped, B.made_last_stats(h)))
            (xa, ia, sa, ta), (xb, ib, sb, tb) = out
            assert (xa == xb).all() and (ia == ib).all() and sa == sb, (N, eps, cap)
            assert ta["sample_passes"] == tb["sample_passes"] == ia.sum()
            # (every pass but the last allowed one goes without a tail, on up to 256 samples)
            assert (ta["tail_less_passes"] > 0) == (N <= 256 and cap != 1) and tb["tail_less_passes"] == 0
            assert ia.min() >= 1 and (not cap or ia.max() <= cap)
    finally:
        B.made_free(h)
