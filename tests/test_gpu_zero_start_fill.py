"""Calls started from zeros clear the caller's states 16 bytes at a time between ragged ends: buffers at any address,
shorter than a piece and longer, neighbours untouched, and the result that a start from given zeros reaches."""
import numpy as np
import pytest
import torch

from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("D,N", [(2, 1), (5, 3), (33, 31), (50, 65), (131, 300)])
def test_any_address(D, N, real):
    w = S.Workload(f"zero{D}", D, 2 if real else 1, [40], "bf16", N, "random", "fan_in", S.SEED_BASE + 1700 + D, gain=1.5, real=real)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    gen = np.random.default_rng(D)
    noise = torch.from_numpy((gen.logistic(size=(N, D)) if real else gen.random((N, D))).astype(np.float32)).cuda()
    dtype = torch.float32 if real else torch.uint8
    try:
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)

        def call(out, init):
            if real:
                B.jacobi_sample_real(h, noise, N, init, 0.0, 0, out, None)
            else:
                B.jacobi_sample(h, noise, N, init, 0, out, None)

        want = torch.empty(N, D, dtype=dtype, device="cuda")
        call(want, torch.zeros(N, D, dtype=dtype, device="cuda"))
        for offset in (0, 1, 3) if real else (0, 1, 7, 15):
            buf = torch.full((N * D + 48,), 9, dtype=dtype, device="cuda")
            call(buf[offset:offset + N * D].view(N, D), None)
            torch.cuda.synchronize()
            assert (buf[:offset] == 9).all() and (buf[offset + N * D:] == 9).all()
            assert torch.equal(buf[offset:offset + N * D].view(N, D), want)
    finally:
        B.made_free(h)
