"""Masked layers on 64 x 64 tiles, where their tiles come out ragged: odd numbers of unit tiles, rows that fill no
tile, rows of noise and symbols that no 16-byte load may take, windows of positions that start and end inside a run of
four, several hidden layers (activations by sample and by list position).  Judged by the oracle: hidden activations
within bf16 rounding, symbols by the fixed-point certificate (positions whose decision margin is below 1e-3 exempt)."""
import numpy as np
import pytest
import torch

from gpu_util import GpuModel, dev, oracle_models
from oracle import made_oracle as O
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


def make(D, hidden, N):
    w = S.Workload(f"quad{D}", D, 1, hidden, "bf16", N, "random", "fan_in", S.SEED_BASE + 1100 + D + N, gain=2.5)
    net = S.make_network(w, with_bias=True)
    return net, oracle_models(net)[1], S.make_noise(w)


def certify(ref, x, noise, what):
    ok, margin = O.fixed_point_check(ref, x, noise)
    assert (ok | (margin < 1e-3)).all(), what


@pytest.mark.parametrize("D,hidden,N", [(1050, [1100], 641), (1056, [1100, 1057], 704), (999, [1250, 1100], 1027),
                                        (322, [330], 4033), (330, [600, 340], 2300)])
def test_jacobi(D, hidden, N):
    net, ref, noise = make(D, hidden, N)
    x0 = np.random.default_rng(D).integers(0, 2, size=(N, D)).astype(np.uint8)
    with GpuModel(net) as g:
        for init, chains in ((None, 1), (x0, 1), (x0, 2)):
            B.made_set_option(g.h, B.MADE_OPT_CHAINS, chains)
            x, it = g.jacobi(noise, init)
            certify(ref, x, noise, (D, init is None, chains))
            assert it.min() >= 1 and it.max() <= D
        B.made_set_option(g.h, B.MADE_OPT_CHAINS, 1)
        # the same rows at addresses that are multiples of 4 only
        pad = torch.empty(N * D + 1, device="cuda")
        pad[1:] = dev(noise).flatten()
        xs = torch.empty(N * D + 1, dtype=torch.uint8, device="cuda")
        B.jacobi_sample(g.h, pad[1:].view(N, D), N, dev(x0), 0, xs[1:].view(N, D), None)
        certify(ref, xs[1:].view(N, D).cpu().numpy(), noise, (D, "unaligned"))
        # a hidden unit is a bf16 of an fp32 sum: half an ulp of it, 2^-9, where both round the same way, one ulp else
        for l in range(len(hidden)):
            act = g.activations(x, l)
            want = O.encode(x, net.C, False) if l == 0 else g.activations(x, l - 1)
            want = np.maximum(want.astype(np.float64) @ ref.WM[l].T + ref.b[l], 0)
            assert np.abs(act - want).max() <= 2.0 ** -8 * np.abs(want).max()


@pytest.mark.parametrize("D,hidden,N", [(300, [1100, 1057], 900), (322, [330], 3700), (784, [2000, 2000], 257)])
def test_same_bits_as_the_32_x_32_tiles(D, hidden, N):
    """Hidden activations, symbols and pass counts against a model that MADE_OPT_MID_TILE_BATCH keeps on the 32 x 32 tiles."""
    net, _, noise = make(D, hidden, N)
    x0 = np.random.default_rng(D).integers(0, 2, size=(N, D)).astype(np.uint8)
    with GpuModel(net) as g, GpuModel(net, mid_tile_batch=1 << 30) as small:
        for h in (g.h, small.h):
            B.made_set_option(h, B.MADE_OPT_CHAINS, 1)
        for l in range(len(hidden)):
            assert (g.activations(x0, l) == small.activations(x0, l)).all(), l
        for init in (None, x0):
            (x, it), (xs, its) = g.jacobi(noise, init), small.jacobi(noise, init)
            assert (x == xs).all() and (it == its).all()


@pytest.mark.parametrize("D,hidden,N,block", [(330, [1100], 2300, 299), (650, [700, 650], 2051, 301)])
def test_windows_of_positions(D, hidden, N, block):
    net, ref, noise = make(D, hidden, N)
    with GpuModel(net) as g:
        B.made_set_option(g.h, B.MADE_OPT_CHAINS, 1)
        for cache in (0, 1):
            B.made_set_option(g.h, B.MADE_OPT_PREFIX_CACHE, cache)
            x, _ = g.gs_jacobi(noise, block)
            certify(ref, x, noise, (D, block, cache))


@pytest.mark.parametrize("D,hidden,N", [(60, [1100, 1057], 900), (41, [1900], 1100), (30, [700, 2100], 641)])
def test_real_states_equal_the_sequential_ones_bit_for_bit(D, hidden, N):
    """Passes of one call run on 64 x 64 or 32 x 32 tiles, by the number of samples still active; with tolerance 0 the
    states are those of the sequential samplers (whose narrow launches take 32 x 32 tiles) to the last bit, every time."""
    w = S.Workload(f"quadreal{D}", D, 2, hidden, "bf16", N, "random", "fan_in", S.SEED_BASE + 1400 + D, gain=1.5, real=True)
    net = S.make_network(w, with_bias=True)
    noise = dev(np.random.default_rng(D).logistic(size=(N, D)).astype(np.float32))
    h = B.model_from_network(net)
    try:
        want = torch.empty((N, D), device="cuda")
        B.sequential_sample_real(h, noise, N, 0, want)
        got = torch.empty((N, D), device="cuda")
        B.sequential_sample_real(h, noise, N, 1, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        for init in (None, torch.randn(N, D, device="cuda", generator=torch.Generator("cuda").manual_seed(1))):
            for _ in range(4):
                B.jacobi_sample_real(h, noise, N, init, 0.0, 0, got)
                torch.cuda.synchronize()
                assert torch.equal(got, want), int((got != want).sum())
        B.gs_jacobi_sample_real(h, noise, N, None, 7, 0.0, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    finally:
        B.made_free(h)


@pytest.mark.parametrize("dtype,N", [("bf16", 5300), ("f32", 8300)])
def test_real_states_of_large_batches_bit_for_bit(dtype, N):
    """Whole-layer and narrow launches of the sequential samplers, and passes over any number of samples, sum in the same
    order also where whole layers take the 128 x 128 tiles: the same states to the last bit."""
    D = 24
    w = S.Workload(f"seqreal{dtype}", D, 2, [1100, 1100], dtype, N, "random", "fan_in", S.SEED_BASE + 1450, gain=1.5, real=True)
    net = S.make_network(w, with_bias=True)
    noise = dev(np.random.default_rng(D).logistic(size=(N, D)).astype(np.float32))
    h = B.model_from_network(net)
    try:
        out = [torch.empty((N, D), device="cuda") for _ in range(2)]
        for mode in (0, 1):
            B.sequential_sample_real(h, noise, N, mode, out[mode])
        torch.cuda.synchronize()
        assert torch.equal(*out), int((out[0] != out[1]).sum())
        for chains in (1, 3):                # (the line is the call's, not a chain's or a pass's)
            B.made_set_option(h, B.MADE_OPT_CHAINS, chains)
            for _ in range(3):
                B.jacobi_sample_real(h, noise, N, None, 0.0, 0, out[1])
                torch.cuda.synchronize()
                assert torch.equal(*out), (chains, int((out[0] != out[1]).sum()))
    finally:
        B.made_free(h)


@pytest.mark.parametrize("D,hidden,dtype,sizes", [(160, [700], "bf16", (960, 961, 6016, 6017)), (160, [700], "f32", (9472, 9473)),
                                                  (64, [120], "bf16", (6143, 6144)), (64, [120], "f32", (12287, 12288)),
                                                  (40, [2000], "bf16", (16383, 16384))])
def test_batches_around_the_lines_between_the_tiles(D, hidden, dtype, sizes):
    """The last batch on one tile and the first on the next: 32 and 64 (176 workgroups), 64 and 128 (144 paired ones, fp32
    224), networks of one column (6144 rows, fp32 12288), 128 and 256 (256 paired ones at 16384)."""
    for N in sizes:
        w = S.Workload(f"line{D}", D, 1, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 1600 + D, gain=2.5)
        net = S.make_network(w, with_bias=True)
        ref, noise = oracle_models(net)[1], S.make_noise(w)
        with GpuModel(net) as g:
            B.made_set_option(g.h, B.MADE_OPT_CHAINS, 1)
            certify(ref, g.jacobi(noise)[0], noise, (D, dtype, N))
            certify(ref, g.gs_jacobi(noise, 30)[0], noise, (D, dtype, N, "gs"))
