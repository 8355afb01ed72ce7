"""GS-Jacobi and the lean sequential sampler in the one-launch kernel that walks the positions block by block, at the
sizes where its blocks change shape: one sample to several workgroups, one to three hidden layers, sparse and crowded
degrees (blocks cut short by the units of a degree), positions that are no multiple of a block.  Judged by the
oracle's fixed-point certificate and its sequential run, pass counts by the oracle's GS-Jacobi, and against the
per-layer launches."""
import numpy as np
import pytest
import torch

from oracle import made_oracle as O
from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hidden,N,dtype,blocks", [
    (64, [256], 16, "f32", (4, 16)), (50, [77, 45], 1, "f32", (1, 7, 32)), (100, [203, 150], 37, "bf16", (3, 32)),
    (33, [500], 5, "bf16", (2,)), (130, [96, 160, 64], 6, "bf16", (8, 31)), (20, [700, 30], 4, "f32", (1,)),
    (40, [3, 2], 9, "bf16", (5, 32)), (300, [1000, 900], 130, "bf16", (16,)), (2, [5], 3, "f32", (1, 2))])
def test_block_substitution(D, hidden, N, dtype, blocks):
    w = S.Workload(f"col{D}", D, 1, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 700 + D, gain=2.5)
    net = S.make_network(w, with_bias=True)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16" if dtype == "bf16" else None)
    xs, margin = O.sequential_sample(ref, noise)
    clear = margin.min(axis=1) >= 1e-3
    u = torch.from_numpy(noise).cuda()
    x0 = np.random.default_rng(D).integers(0, 2, size=(N, D)).astype(np.uint8)
    h = B.model_from_network(net)
    try:
        def call(block, init=None):
            x = torch.full((N, D), 9, dtype=torch.uint8, device="cuda")
            it = torch.full((N,), -1, dtype=torch.int32, device="cuda")
            if block:
                B.gs_jacobi_sample(h, u, N, None if init is None else torch.from_numpy(init).cuda(), block, x, it)
            else:
                B.sequential_sample(h, u, N, 1, x)
            torch.cuda.synchronize()
            x = x.cpu().numpy()
            ok, at = O.fixed_point_check(ref, x, noise)
            assert (ok | (at < 1e-3)).all(), block
            assert (x[clear] == xs[clear]).all(), block
            return x, it.cpu().numpy(), B.made_last_stats(h)

        compared = 0
        for block in (0,) + blocks:
            x, it, st = call(block)
            assert st["kernels"] == 1, (block, st)
            if block:
                r = O.gs_jacobi_reference(ref, noise, block)
                calm = r[3] >= 1e-3
                assert (it[calm] == r[1][calm]).all(), block
                assert st["sample_passes"] == it.sum()
                xi, iti, sti = call(block, x0)
                B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
                B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
                xl, itl, stl = call(block, x0)
                assert stl["kernels"] > 1 and stl["passes"] >= 1
                # (a draw within rounding of its threshold may cost a sample a pass on one side; with none of them apart the
                # blocks' passes are the per-layer launches')
                ri = O.gs_jacobi_reference(ref, noise, block, x0)
                calm = ri[3] >= 1e-3
                assert (iti[calm] == ri[1][calm]).all(), block
                assert sti["sample_passes"] == iti.sum()
                fits = all(((d >= a) & (d < a + block)).sum() <= 64 for d in net.degrees for a in range(0, D, block))
                if fits and (iti == itl).all() and (xi == xl).all():
                    assert sti["passes"] == stl["passes"], block
                    compared += 1
                B.made_set_option(h, B.MADE_OPT_RESIDENT, 2)
                B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 1)
                assert (xi[clear] == xl[clear]).all()
        assert compared >= 1 or not fits
    finally:
        B.made_free(h)


def test_too_many_units_of_one_degree_take_the_other_paths():
    """70 units of one degree are more than the kernel's lanes: same results, more launches."""
    D, N = 12, 5
    w = S.Workload("crowded", D, 1, [90], "f32", N, "random", "fan_in", S.SEED_BASE + 799, gain=2.0)
    net = S.make_network(w, with_bias=True)
    net.degrees[0][:70] = 4
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, None)
    xs, margin = O.sequential_sample(ref, noise)
    clear = margin.min(axis=1) >= 1e-3
    h = B.model_from_network(net)
    try:
        u = torch.from_numpy(noise).cuda()
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        B.sequential_sample(h, u, N, 1, x)
        torch.cuda.synchronize()
        assert B.made_last_stats(h)["kernels"] > 1
        assert (x.cpu().numpy()[clear] == xs[clear]).all()
        B.gs_jacobi_sample(h, u, N, None, 4, x)
        torch.cuda.synchronize()
        assert (x.cpu().numpy()[clear] == xs[clear]).all()
    finally:
        B.made_free(h)


@pytest.mark.parametrize("crowd,at,before,dtype", [(64, 5, 31, "bf16"), (64, 5, 32, "bf16"), (61, 3, 7, "bf16"), (63, 9, 1, "f32"), (60, 5, 2, "bf16")])
def test_a_position_with_as_many_units_as_a_wave_has_lanes(crowd, at, before, dtype):
    """`crowd` units of degree `at` in both layers behind `before` units of lower degree (the block's weights then begin at an
    odd or an even input): the widest blocks the kernel takes, alone and among others."""
    D, N = 14, 5
    w = S.Workload(f"crowd{crowd}", D, 1, [crowd + before + 20] * 2, dtype, N, "random", "fan_in", S.SEED_BASE + 760 + before, gain=2.5)
    net = S.make_network(w, with_bias=True)
    for d in net.degrees:
        d[:] = D - 1 - np.arange(d.size) % 3
        d[:crowd] = at
        d[crowd:crowd + before] = 1 + np.arange(before) % (at - 1)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16" if dtype == "bf16" else None)
    xs, margin = O.sequential_sample(ref, noise)
    clear = margin.min(axis=1) >= 1e-3
    h = B.model_from_network(net)
    try:
        u = torch.from_numpy(noise).cuda()
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        for call in (lambda: B.sequential_sample(h, u, N, 1, x), lambda: B.gs_jacobi_sample(h, u, N, None, 1, x)):
            x.fill_(9)
            call()
            torch.cuda.synchronize()
            assert B.made_last_stats(h)["kernels"] == 1
            ok, at_ = O.fixed_point_check(ref, x.cpu().numpy(), noise)
            assert (ok | (at_ < 1e-3)).all()
            assert (x.cpu().numpy()[clear] == xs[clear]).all()
    finally:
        B.made_free(h)


@pytest.mark.parametrize("D,hidden,dtype", [(100, [2500, 2200], "f32"), (90, [2300, 2100, 1900], "bf16"), (60, [1200, 900, 700], "f32")])
def test_models_that_leave_room_for_one_buffer_of_staged_weights(D, hidden, dtype):
    """Inputs of 60 to 100 KB per workgroup: a block's own weights are written between two blocks."""
    N = 6
    w = S.Workload(f"one{D}", D, 1, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 740 + D, gain=2.5)
    net = S.make_network(w, with_bias=True)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16" if dtype == "bf16" else None)
    h = B.model_from_network(net)
    try:
        u = torch.from_numpy(noise).cuda()
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        for call in (lambda: B.sequential_sample(h, u, N, 1, x), lambda: B.gs_jacobi_sample(h, u, N, None, 1, x)):
            x.fill_(9)
            call()
            torch.cuda.synchronize()
            assert B.made_last_stats(h)["kernels"] == 1
            ok, margin = O.fixed_point_check(ref, x.cpu().numpy(), noise)
            assert (ok | (margin < 1e-3)).all()
    finally:
        B.made_free(h)


@pytest.mark.parametrize("kernel", ["column", "resident"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_noise_and_logits_at_the_ends(dtype, kernel):
    """Logits of any size against noise at and outside the ends of [0, 1): the symbols are those of the kernels that compute the
    probability.  Every pair of them; none is within 1e-6 of a tie."""
    logits = np.array([-1e30, -1e4, -200, -89, -86, -20, 0.5, 20, 86, 89, 200, 1e4, 1e30], np.float32)
    us = np.array([0.0, -1.0, -0.0, 2.0 ** -24, 1e-30, 0.25, 0.75, 1 - 2.0 ** -24, 1.0, 2.0, np.nan, -np.inf, np.inf], np.float32)
    D, N = logits.size, us.size * 2
    w = S.Workload("ends", D, 1, [40], dtype, N, "random", "fan_in", S.SEED_BASE + 770, gain=0.0)
    net = S.make_network(w, with_bias=True)
    net.W[-1][:] = 0.0
    net.b[-1] = logits.reshape(np.asarray(net.b[-1]).shape)
    noise = torch.from_numpy(np.repeat(np.tile(us, 2)[:, None], D, axis=1).copy()).cuda()
    h = B.model_from_network(net)
    try:
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
        want = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        B.jacobi_sample(h, noise, N, None, 0, want)
        if kernel == "column":
            B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 1)
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 2 if kernel == "column" else 1)
        p = 1 / (1 + np.exp(-np.clip(logits.astype(np.float64), -700, 700)))
        assert (want.cpu().numpy()[3:8] == (us[3:8, None] < p)).all()          # (the ordinary values, against 64 bits)
        calls = [lambda x: B.gs_jacobi_sample(h, noise, N, None, 5, x)]
        calls.append((lambda x: B.sequential_sample(h, noise, N, 1, x)) if kernel == "column" else
                     (lambda x: B.jacobi_sample(h, noise, N, None, 0, x)))
        for call in calls:
            x = torch.full((N, D), 9, dtype=torch.uint8, device="cuda")
            call(x)
            torch.cuda.synchronize()
            assert B.made_last_stats(h)["kernels"] == 1
            bad = (x != want).cpu().numpy()
            assert not bad.any(), [(float(np.tile(us, 2)[i]), float(logits[j])) for i, j in np.argwhere(bad)]
    finally:
        B.made_free(h)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_weights_that_are_no_numbers_stay_where_they_are(dtype):
    """The kernel multiplies what is staged past a block's last unit, an earlier block's weights, with 0.  A NaN among them must not
    reach the units of another block: ReLU ends it in its own unit."""
    D, N = 90, 24
    w = S.Workload("nonum", D, 1, [150, 130], dtype, N, "random", "fan_in", S.SEED_BASE + 760, gain=2.5)
    net = S.make_network(w, with_bias=True)
    deg = [np.arange(1, D + 1)] + [np.asarray(d) for d in net.degrees]
    for l, unit_deg, limit in ((0, 9, 9), (0, 12, 10), (1, 13, 12), (1, 17, 15)):          # unit of a degree, input up to one
        i = int(np.argmin(np.abs(deg[l + 1] - unit_deg)))
        j = int(np.argmin(np.where(deg[l] <= deg[l + 1][i], np.abs(deg[l] - limit), 10 ** 6)))
        net.W[l][i, j] = np.nan
    noise = S.make_noise(w)
    h = B.model_from_network(net)
    try:
        u = torch.from_numpy(noise).cuda()
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
        want = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        B.sequential_sample(h, u, N, 0, want)
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 2)
        for block in (0, 8, 13, 32):
            x = torch.full((N, D), 9, dtype=torch.uint8, device="cuda")
            if block:
                B.gs_jacobi_sample(h, u, N, None, block, x)
            else:
                B.sequential_sample(h, u, N, 1, x)
            torch.cuda.synchronize()
            assert torch.equal(x, want), (block, int((x != want).sum()), B.made_last_stats(h)["kernels"])
    finally:
        B.made_free(h)


def test_a_smaller_model_made_later_leaves_the_larger_one_its_lds():
    """Two models of one depth and type alive, the larger (about 130 KB of LDS) called after the smaller was made."""
    models = []
    try:
        for D, H in ((784, 2000), (20, 30)):
            w = S.Workload(f"lds{D}", D, 1, [H, H], "bf16", 6, "random", "fan_in", S.SEED_BASE + 780 + D, gain=2.5)
            net = S.make_network(w, with_bias=True)
            models.append((w, S.make_noise(w), O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16"), B.model_from_network(net)))
        for w, noise, ref, h in models:
            x = torch.empty((w.N, w.D), dtype=torch.uint8, device="cuda")
            for call in (lambda: B.gs_jacobi_sample(h, torch.from_numpy(noise).cuda(), w.N, None, 8, x),
                         lambda: B.sequential_sample(h, torch.from_numpy(noise).cuda(), w.N, 1, x)):
                call()
                torch.cuda.synchronize()
                assert B.made_last_stats(h)["kernels"] == 1
                ok, margin = O.fixed_point_check(ref, x.cpu().numpy(), noise)
                assert (ok | (margin < 1e-3)).all()
    finally:
        for m in models:
            B.made_free(m[-1])


@pytest.mark.parametrize("D,hidden,N,dtype", [(64, [100], 2048, "bf16"), (64, [100], 2049, "bf16"), (16, [40], 32768, "f32"), (16, [40], 32769, "f32")])
def test_batches_around_the_lines_to_the_other_paths(D, hidden, N, dtype):
    """GS-Jacobi up to and beyond 2048 samples on a model the sample-resident kernel holds, the sequential sampler of a narrow
    network up to and beyond 32768."""
    w = S.Workload(f"line{D}", D, 1, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 790 + D, gain=2.5)
    net = S.make_network(w, with_bias=True)
    noise = S.make_noise(w)
    ref = O.build_model(net.D, net.C, net.degrees, net.W, net.b, "bf16" if dtype == "bf16" else None)
    h = B.model_from_network(net)
    try:
        u = torch.from_numpy(noise).cuda()
        x = torch.empty((N, D), dtype=torch.uint8, device="cuda")
        for call in (lambda: B.gs_jacobi_sample(h, u, N, None, 4, x), lambda: B.sequential_sample(h, u, N, 1, x)):
            x.fill_(9)
            call()
            torch.cuda.synchronize()
            ok, margin = O.fixed_point_check(ref, x.cpu().numpy(), noise)
            assert (ok | (margin < 1e-3)).all()
        assert (B.made_last_stats(h)["kernels"] == 1) == (N <= 32768)
    finally:
        B.made_free(h)
