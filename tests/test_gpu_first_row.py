"""Large batches started from zeros: the first pass evaluates its layers for one row and draws every sample from it.  Against
the pass with every row evaluated (MADE_OPT_ZERO_START = 0): symbols after one pass, at the fixed point, pass counts and verdicts
-- at batches around the line and ragged ones, with positions that end inside a piece, a chunk or a line, buffers at odd
addresses, and a network whose first draw leaves most samples at zero (they stop after that pass)."""
import numpy as np
import pytest
import torch

from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hidden,dtype,shift", [
    (5, [9], "bf16", -4.0), (64, [100], "bf16", 0.0), (131, [96, 160], "f32", 0.0), (130, [70, 40], "bf16", -5.0),
    (784, [300, 200], "bf16", 0.0), (100, [50], "f32", -4.0)])
@pytest.mark.parametrize("N", [511, 512, 545, 2100])
def test_against_every_row_evaluated(D, hidden, dtype, shift, N):
    w = S.Workload(f"first{D}", D, 1, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 2300 + D, gain=2.0)
    net = S.make_network(w, with_bias=True)
    net.b[-1] = net.b[-1] + np.float32(shift)
    noise_h = np.random.default_rng(D).random((N, D)).astype(np.float32)
    h = B.model_from_network(net)
    try:
        for offset in (0, 1):
            noise = torch.empty(N * D + 1, device="cuda")[offset:offset + N * D].view(N, D)
            noise.copy_(torch.from_numpy(noise_h))
            for cap in (0, 1, 2):
                out = []
                for zero in (1, 0):
                    B.made_set_option(h, B.MADE_OPT_ZERO_START, zero)
                    B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
                    x = torch.full((N * D + 40,), 9, dtype=torch.uint8, device="cuda")
                    it = torch.full((N,), -1, dtype=torch.int32, device="cuda")
                    code = 0
                    try:
                        B.jacobi_sample(h, noise, N, None, cap, x[3 * offset:3 * offset + N * D].view(N, D), it)
                    except B.MadeError as e:
                        code = e.code
                        assert cap and code == B.MADE_ERR_NOT_CONVERGED
                    torch.cuda.synchronize()
                    out.append((x.cpu().numpy(), it.cpu().numpy(), code, B.made_last_stats(h)))
                a, b = out
                # (at these batches both sides sum a logit in the same order: see tile_edge)
                assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and a[2] == b[2], (offset, cap)
                assert a[3]["passes"] == b[3]["passes"] and a[3]["sample_passes"] == b[3]["sample_passes"] == a[1].sum()
                assert shift == 0.0 or (a[1] == 1).any()
    finally:
        B.made_free(h)


@pytest.mark.parametrize("N", [20199, 32761])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_batches_on_which_a_wave_draws_several_chunks(dtype, N):
    """20192 samples and more of 784 positions: a wave takes 2 or 3 of 13 chunks (fp32: 3 or 6 of 25), the last one what is
    left.  On 32 x 32 tiles for both sides, so that a logit's sum has one order."""
    D = 784
    w = S.Workload("firstw", D, 1, [40], dtype, N, "random", "fan_in", S.SEED_BASE + 2390, gain=2.0)
    net = S.make_network(w, with_bias=True)
    h = B.model_from_network(net)
    try:
        B.made_set_option(h, B.MADE_OPT_MID_TILE_BATCH, 1 << 30)
        B.made_set_option(h, B.MADE_OPT_BIG_TILE_BATCH, 1 << 30)
        noise = torch.rand(N * D + 1, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
        for offset in (0, 1):
            u = noise[offset:offset + N * D].view(N, D)
            for cap in (0, 1):
                out = []
                for zero in (1, 0):
                    B.made_set_option(h, B.MADE_OPT_ZERO_START, zero)
                    x = torch.full((N * D + 40,), 9, dtype=torch.uint8, device="cuda")
                    it = torch.full((N,), -1, dtype=torch.int32, device="cuda")
                    code = 0
                    try:
                        B.jacobi_sample(h, u, N, None, cap, x[3 * offset:3 * offset + N * D].view(N, D), it)
                    except B.MadeError as e:
                        code = e.code
                        assert cap and code == B.MADE_ERR_NOT_CONVERGED
                    torch.cuda.synchronize()
                    out.append((x, it, code, B.made_last_stats(h)))
                a, b = out
                assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2], (offset, cap)
                assert a[3]["passes"] == b[3]["passes"] and a[3]["sample_passes"] == b[3]["sample_passes"] == int(a[1].sum())
                assert int((a[1] == 1).sum()) < N or cap
    finally:
        B.made_free(h)
