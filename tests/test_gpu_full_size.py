"""Parity at the benchmark's full sizes, in the launch configuration bench.py times.

A full sequential oracle run of the whole batch would take minutes, so the whole batch is graded
with the one-pass fixed-point certificate (the triangular system has a unique solution) and a
sub-batch is compared with the oracle's own sequential run symbol by symbol."""
import numpy as np
import pytest

from oracle import made_oracle as O
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

from gpu_util import (LOGIT_TOL, MARGIN, GpuModel, assert_logits_close, assert_sample_parity, mlp_layer_certificate,
                      oracle_models, progress)


def assert_counts_close(it, it_ref, min_margin, x, x_ref, same_floor):
    """Iteration counts at full size.  Nearly every sample of a large network meets SOME decision within 1e-3 of a
    tie in one of its passes (cfg2: 784 positions x 3-4 passes), so the strict comparison -- equal counts where
    every margin is clear -- covers only a few samples.  Therefore, for EVERY sample: the count is within one pass
    of the oracle's (a near-tie that falls the other way in an intermediate pass costs or saves one pass), and
    the count is equal wherever the final symbols are the oracle's; and the share of samples whose symbols are
    identical to the oracle's own Jacobi run has a floor."""
    clear = min_margin >= MARGIN
    assert (it[clear] == it_ref[clear]).all()
    assert (np.abs(it - it_ref) <= 1).all(), (it, it_ref)
    same = (x == x_ref).all(axis=1)
    assert same.mean() >= same_floor, f"only {same.mean():.3f} of the samples equal the oracle's Jacobi result"
    assert (it[same] != it_ref[same]).mean() <= 0.05
    return float(clear.mean()), float(same.mean()), float((it == it_ref).mean())

pytestmark = pytest.mark.gpu


@pytest.fixture
def library_defaults():
    """The models of a test run with the options the library itself defaults to (what bench.py times): one chain, the
    tail-less stop test, the one-launch kernels where the library chooses them."""
    import gpu_util
    old = (gpu_util.CHAINS, gpu_util.RESIDENT, gpu_util.XCD, gpu_util.LAZY, gpu_util.RETIRE_SPLIT)
    gpu_util.CHAINS, gpu_util.RESIDENT, gpu_util.XCD, gpu_util.LAZY, gpu_util.RETIRE_SPLIT = 1, 2, None, None, None
    yield
    gpu_util.CHAINS, gpu_util.RESIDENT, gpu_util.XCD, gpu_util.LAZY, gpu_util.RETIRE_SPLIT = old


def test_cfg2_full_batch_as_benchmarked(library_defaults):
    """cfg2 in the launch configuration bench.py times (library defaults): Jacobi and GS-Jacobi in one-launch kernels; and Jacobi on
    the per-layer launches with the tail-less stop test, with the same result."""
    test_cfg2_jacobi_and_gs_jacobi_full_batch(False, expect_default_paths=True)


@pytest.mark.parametrize("persistent", [True, False])
def test_cfg2_jacobi_and_gs_jacobi_full_batch(persistent, expect_default_paths=False):
    w = S.workload("cfg2")
    net = S.make_network(w)
    exact, same = oracle_models(net)
    noise = S.make_noise(w)
    sub = 6
    xs, mg = O.sequential_sample(same, noise[:sub])
    xr, it_ref, _, _, mm = O.jacobi_reference(same, noise)
    with GpuModel(net, persistent) as g:
        x, it = g.jacobi(noise)
        if expect_default_paths:
            assert g.stats()["kernels"] == 1, g.stats()
            one = (x, it)
            B.made_set_option(g.h, B.MADE_OPT_XCD_RESIDENT, 0)
            x, it = g.jacobi(noise)
            st = g.stats()
            B.made_set_option(g.h, B.MADE_OPT_XCD_RESIDENT, 1)
            assert (x == one[0]).all() and (it == one[1]).all()
            assert st["tail_less_passes"] >= st["passes"] > 0 and st["kernels"] > 3, st
        exempt, _ = assert_sample_parity(same, noise, x)
        assert_sample_parity(same, noise[:sub], x[:sub], xs, mg)
        clear, same_frac, equal_counts = assert_counts_close(it, it_ref, mm, x, xr, same_floor=0.85)
        print(f"cfg2 jacobi: passes mean {it.mean():.2f} max {it.max()}, exempt positions {exempt}, samples with all "
              f"margins clear {clear:.3f}, identical to oracle jacobi {same_frac:.3f}, equal pass counts {equal_counts:.3f}")
        z = g.logits(x[:16])
        assert_logits_close(z, O.logits_all(exact, x[:16]), LOGIT_TOL["bf16"])
        worst = mlp_layer_certificate(g, same, x, noise)
        print(f"cfg2 layer certificate at the Jacobi result: worst logit accumulation error {worst:.2f} x 2^-24 sum|a w|")
        for block in w.block_sizes:
            xb, itb = g.gs_jacobi(noise, block)
            if expect_default_paths:
                assert g.stats()["kernels"] == 1, g.stats()      # (the whole call in one launch)
            assert_sample_parity(same, noise, xb)
            assert_sample_parity(same, noise[:sub], xb[:sub], xs, mg)
            ref = O.gs_jacobi_reference(same, noise[:sub], block)
            clear = ref[3] >= MARGIN
            assert (itb[:sub][clear] == ref[1][clear]).all()
            # every sample of the sub-batch: a block's inner loop may take one pass more or less per near-tie
            assert (np.abs(itb[:sub] - ref[1]) <= 2).all(), (block, itb[:sub], ref[1])
        for mode in (0, 1):
            xq = g.sequential(noise, mode)
            assert_sample_parity(same, noise, xq)
            assert_sample_parity(same, noise[:sub], xq[:sub], xs, mg)


@pytest.mark.timeout(900)
def test_cfg4_categorical_full_size(library_defaults):
    """D = 1024 positions x 256 classes, 2 x 4096 hidden, 2 GiB output layer, batch 64.  The whole batch is
    certified with one oracle pass per sample; a sub-batch is compared with the oracle's sequential run."""
    w = S.workload("cfg4")
    progress("cfg4: drawing the network")
    net = S.make_network(w)
    progress("cfg4: building the oracle models")
    exact, same = oracle_models(net)
    noise = S.make_noise(w)
    sub = 2
    progress("cfg4: oracle sequential run of 2 samples")
    xs, mg = O.sequential_sample(same, noise[:sub])
    progress("cfg4: made_init")
    with GpuModel(net) as g:
        progress("cfg4: jacobi on the GPU, then the oracle certificate")
        x, it = g.jacobi(noise)
        exempt, _ = assert_sample_parity(same, noise, x)
        assert_sample_parity(same, noise[:sub], x[:sub], xs, mg)
        st = g.stats()
        print(f"cfg4 jacobi: passes mean {it.mean():.2f} max {it.max()}, exempt positions {exempt}, stats {st}")
        progress("cfg4: oracle jacobi of 8 samples")
        ref = O.jacobi_reference(same, noise[:8])
        clear = ref[4] >= MARGIN
        assert (it[:8][clear] == ref[1][clear]).all()
        assert (np.abs(it[:8] - ref[1]) <= 1).all(), (it[:8], ref[1])
        print(f"cfg4 jacobi vs oracle jacobi on 8 samples: clear {clear.mean():.2f}, equal counts {(it[:8] == ref[1]).mean():.2f}, "
              f"identical symbols {(x[:8] == ref[0]).all(axis=1).mean():.2f}")
        z = g.logits(x[:2])
        assert_logits_close(z, O.logits_all(exact, x[:2]), LOGIT_TOL["bf16"])
        progress("cfg4: gs-jacobi, sequential")
        xb, itb = g.gs_jacobi(noise, 128)
        assert_sample_parity(same, noise, xb)
        assert_sample_parity(same, noise[:sub], xb[:sub], xs, mg)
        xq = g.sequential(noise[:8], 1)
        assert_sample_parity(same, noise[:8], xq)
        assert_sample_parity(same, noise[:sub], xq[:sub], xs, mg)


@pytest.mark.timeout(900)
def test_cfg4_onehot_full_size_certificate(library_defaults):
    """cfg4 with one-hot input at full size (first layer = gather over a 4096 x 262144 weight matrix): the Jacobi
    result of all 64 samples is certified as the fixed point of the oracle's network (one oracle evaluation of
    every position from the GPU's output; exact except where the oracle's margin is below 1e-3), the logits of
    two samples are compared, and GS-Jacobi and the lean sequential mode must reach the same certificate."""
    w = S.workload("cfg4_onehot")
    progress("cfg4_onehot: weights")
    net = S.make_network(w)
    progress("cfg4_onehot: building the oracle models")
    exact, same = oracle_models(net)
    noise = S.make_noise(w)
    progress("cfg4_onehot: made_init")
    with GpuModel(net) as g:
        progress("cfg4_onehot: jacobi on the GPU, then the oracle certificate")
        x, it = g.jacobi(noise)
        exempt, _ = assert_sample_parity(same, noise, x)
        assert (it >= 2).all() and (it <= w.D).all()
        print(f"cfg4_onehot jacobi: passes mean {it.mean():.2f} max {it.max()}, exempt positions {exempt}, stats {g.stats()}")
        z = g.logits(x[:2])
        assert_logits_close(z, O.logits_all(exact, x[:2]), LOGIT_TOL["bf16"])
        progress("cfg4_onehot: gs-jacobi, sequential")
        xb, _ = g.gs_jacobi(noise, 128)
        assert_sample_parity(same, noise, xb)
        xq = g.sequential(noise[:8], 1)
        assert_sample_parity(same, noise[:8], xq)
        # the three solvers agree with each other wherever the oracle's margins are clear
        ok, margin = O.fixed_point_check(same, x, noise)
        clear = (margin >= MARGIN).all(axis=1)
        assert (xb[clear] == x[clear]).all() and (xq[clear[:8]] == x[:8][clear[:8]]).all()


@pytest.mark.timeout(600)
def test_cfg2_jacobi_gs_full_batch():
    """Algorithm 2 on cfg2 at full batch: the result is certified for all 128 samples (one oracle pass), and a
    sub-batch is compared with the oracle's Algorithm 2 run (iteration counts) and with its sequential run.
    The virtual batch (13 blocks x 128 samples) goes through the hidden layers on the 32 x 32 tile kernels for
    block 64 and on the 256 x 256 tile kernels for block 16 (49 x 128 = 6272 rows)."""
    w = S.workload("cfg2")
    net = S.make_network(w)
    _, same = oracle_models(net)
    noise = S.make_noise(w)
    sub = 4
    xs, mg = O.sequential_sample(same, noise[:sub])
    with GpuModel(net) as g:
        for block in (64, 16):
            progress(f"cfg2 jacobi_gs block {block}")
            x, it = g.jacobi_gs(noise, block)
            st = g.stats()
            assert_sample_parity(same, noise, x)
            assert_sample_parity(same, noise[:sub], x[:sub], xs, mg)
            ref = O.jacobi_gs_reference(same, noise[:sub], block)
            clear = ref[3] >= MARGIN
            assert (it[:sub][clear] == ref[1][clear]).all()
            print(f"cfg2 jacobi_gs block {block}: iterations mean {it.mean():.2f} max {it.max()}, stats {st}")


@pytest.mark.parametrize("tile", [256, 128])
def test_cfg2_large_batch_vector_epilogue(tile):
    """cfg2's network at batch 300: the 256 x 256 / 128 x 128 tile kernels with the 16-byte epilogue I/O (D % 16 == 0)."""
    import dataclasses
    w = dataclasses.replace(S.workload("cfg2"), N=300)
    net = S.make_network(w)
    exact, same = oracle_models(net)
    noise = S.make_noise(w)
    sub = 4
    xs, mg = O.sequential_sample(same, noise[:sub])
    ref = O.jacobi_reference(same, noise)
    with GpuModel(net, big_tile_batch=256 if tile == 256 else 1 << 30, mid_tile_batch=128 if tile == 128 else None) as g:
        x, it = g.jacobi(noise)
        assert_sample_parity(same, noise, x)
        assert_sample_parity(same, noise[:sub], x[:sub], xs, mg)
        assert_counts_close(it, ref[1], ref[4], x, ref[0], same_floor=0.85)
        z = g.logits(x[:300])
        assert_logits_close(z, O.logits_all(exact, x), LOGIT_TOL["bf16"])
        xb, _ = g.gs_jacobi(noise, 196)
        assert_sample_parity(same, noise, xb)
        # a block size that is no multiple of four: windows cut the epilogue's runs of four positions
        xc, _ = g.gs_jacobi(noise, 50)
        assert_sample_parity(same, noise, xc)
        assert_sample_parity(same, noise[:sub], xc[:sub], xs, mg)


def test_cfg2_batch_8192_stop_test_as_its_own_kernel():
    """cfg2's network at batch 8192, one chain, library defaults: lists this long are retired by a kernel of their own
    (MADE_OPT_RETIRE_SPLIT).  Whole batch by the fixed-point certificate, a sub-batch against the oracle's sequential
    run, and symbols and pass counts as in the run that keeps the stop test inside the output kernel."""
    import dataclasses
    import gpu_util
    w = dataclasses.replace(S.workload("cfg2"), N=8192)
    net = S.make_network(w)
    _, same = oracle_models(net)
    noise = S.make_noise(w)
    sub = 4
    xs, mg = O.sequential_sample(same, noise[:sub])
    ref = O.jacobi_reference(same, noise[:64])
    results = []
    old = gpu_util.CHAINS, gpu_util.RETIRE_SPLIT
    try:
        for split in (None, 1 << 30):
            gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = 1, split
            progress(f"cfg2 batch 8192, retire split {split}")
            with GpuModel(net) as g:
                x, it = g.jacobi(noise)
                xb, itb = g.gs_jacobi(noise, 196)
            results.append((x, it, xb, itb))
    finally:
        gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = old
    x, it, xb, itb = results[0]
    assert_sample_parity(same, noise, x)
    assert_sample_parity(same, noise[:sub], x[:sub], xs, mg)
    assert_sample_parity(same, noise, xb)
    assert_counts_close(it[:64], ref[1], ref[4], x[:64], ref[0], same_floor=0.85)
    # the other run: same symbols and pass counts, except where a draw lies within rounding of its threshold (which
    # tile shape a late pass runs on depends on the active count the host had seen when it enqueued the pass, and
    # the shapes sum in different orders)
    x2, it2, xb2, itb2 = results[1]
    assert_sample_parity(same, noise, x2)
    assert_sample_parity(same, noise, xb2)
    for xa, ia, xo, io in ((x, it, x2, it2), (xb, itb, xb2, itb2)):
        rows_equal = (xa == xo).all(axis=1)
        assert rows_equal.mean() > 0.999
        assert (ia[rows_equal] != io[rows_equal]).mean() < 1e-3     # (a near-tie in an intermediate pass costs a pass)


@pytest.mark.parametrize("N", [1535, 1536, 1537, 2047, 2048, 2049, 2600])
def test_batches_around_the_tile_and_stop_test_thresholds(N):
    """Batches just below, at and above the sizes where the layers are told to move to the LDS-staged 128 x 128 tiles
    (1536, by option) and the stop test becomes a kernel of its own (2048, the default); late passes of the same call
    fall back below both.  Whole batch by the fixed-point certificate; pass counts against a run that stays on the
    32 x 32 tiles with the fused stop test."""
    import dataclasses
    import gpu_util
    w = dataclasses.replace(S.workload("mid_bf16"), N=N)
    net = S.make_network(w, with_bias=True)
    _, same = oracle_models(net)
    noise = S.make_noise(w)
    old = gpu_util.CHAINS, gpu_util.RETIRE_SPLIT
    try:
        gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = 1, None
        with GpuModel(net, mid_tile_batch=1536) as g:
            x, it = g.jacobi(noise)
            xb, _ = g.gs_jacobi(noise, 50)
        gpu_util.RETIRE_SPLIT = 1 << 30
        with GpuModel(net, mid_tile_batch=1 << 30) as g:
            x_small, it_small = g.jacobi(noise)
    finally:
        gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = old
    assert_sample_parity(same, noise, x)
    assert_sample_parity(same, noise, xb)
    assert_sample_parity(same, noise, x_small)
    rows_equal = (x == x_small).all(axis=1)
    assert rows_equal.mean() > 0.99                      # (the two tile shapes sum in different orders: near-ties may flip)
    assert (it[rows_equal] != it_small[rows_equal]).mean() < 1e-3     # (a near-tie in an intermediate pass costs a pass)


def test_four_chains_of_large_sub_batches():
    """8200 samples cut into four chains on their own streams: each chain runs the 128 x 128 tiles (from 1536 samples on, by
    option) and its own stand-alone stop test concurrently with the others.  Whole batch by the fixed-point certificate, pass counts
    against the single-chain run."""
    import dataclasses
    import gpu_util
    w = dataclasses.replace(S.workload("mid_bf16"), N=8200)
    net = S.make_network(w, with_bias=True)
    _, same = oracle_models(net)
    noise = S.make_noise(w)
    old = gpu_util.CHAINS, gpu_util.RETIRE_SPLIT
    try:
        out = []
        for chains in (4, 1):
            gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = chains, None
            with GpuModel(net, mid_tile_batch=1536) as g:
                out.append(g.jacobi(noise))
    finally:
        gpu_util.CHAINS, gpu_util.RETIRE_SPLIT = old
    (x4, it4), (x1, it1) = out
    assert_sample_parity(same, noise, x4)
    assert_sample_parity(same, noise, x1)
    # (which tile shape a late pass runs on depends on the active count the host had seen when it enqueued the pass;
    # the shapes sum in different orders, so a draw within rounding of its threshold may come out differently)
    rows_equal = (x4 == x1).all(axis=1)
    assert rows_equal.mean() > 0.999
    assert (it4[rows_equal] != it1[rows_equal]).mean() < 1e-3     # (a near-tie in an intermediate pass costs a pass)
