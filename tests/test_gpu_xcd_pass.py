"""A Jacobi call in one launch, every XCD on its own eighth of the batch, against the per-layer launches: the same sums in the
same order, so the same symbols or states bit for bit, the same pass counts and the same verdict -- where the rows of an XCD, the
unit tiles of its workgroups (none, one, two) or the K chunks of a wave (none, those requested ahead, more) run out, with a
start of one's own, pass limits and a tolerance."""
import numpy as np
import pytest
import torch

from paper_2002_03629_amd import binding as B
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu

SHAPES = [  # D, hidden, dtype
    (64, [256], "f32"), (2, [3], "bf16"), (33, [31, 65], "bf16"), (131, [96, 160, 40], "f32"), (200, [1024, 1025], "bf16"),
    (100, [2048], "bf16"), (60, [1500, 300], "f32"), (784, [512, 512], "bf16")]


def _call(h, real, noise, N, init, eps, cap, D):
    x = torch.full((N, D), 7, dtype=torch.float32 if real else torch.uint8, device="cuda")
    it = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    code = 0
    try:
        if real:
            B.jacobi_sample_real(h, noise, N, init, eps, cap, x, it)
        else:
            B.jacobi_sample(h, noise, N, init, cap, x, it)
    except B.MadeError as e:
        code = e.code
        assert code == B.MADE_ERR_NOT_CONVERGED
    torch.cuda.synchronize()
    return x.cpu().numpy(), it.cpu().numpy(), code, B.made_last_stats(h)


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("D,hidden,dtype", SHAPES)
def test_against_launches(D, hidden, dtype, real):
    w = S.Workload(f"xp{D}", D, 2 if real else 1, hidden, dtype, 256, "random", "fan_in", S.SEED_BASE + 2100 + D, gain=2.0, real=real)
    net = S.make_network(w, with_bias=True)
    gen = np.random.default_rng(D)
    h = B.model_from_network(net)
    try:
        for N in (1, 8, 9, 100, 255, 256):
            noise = (gen.logistic(size=(N, D)) if real else gen.random((N, D))).astype(np.float32)
            start = gen.normal(size=(N, D)).astype(np.float32) if real else gen.integers(0, 2, size=(N, D)).astype(np.uint8)
            noise, start = torch.from_numpy(noise).cuda(), torch.from_numpy(start).cuda()
            for init, eps, cap, zero in ((None, 0.0, 0, 1), (start, 0.0, 0, 1), (None, 0.05, 3, 1), (None, 0.0, 2, 0)):
                if not real and eps:
                    continue
                B.made_set_option(h, B.MADE_OPT_ZERO_START, zero)
                out = []
                for xcd in (2, 0):
                    B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, xcd)
                    out.append(_call(h, real, noise, N, init, eps, cap, D))
                (xa, ia, ca, sa), (xb, ib, cb, sb) = out
                assert sa["kernels"] == 1 and sb["kernels"] > 1, B.made_last_error()
                assert (xa == xb).all() and (ia == ib).all() and ca == cb, (N, init is not None, eps, cap)
                assert sa["sample_passes"] == sb["sample_passes"] == ia.sum() and sa["passes"] == sb["passes"]
    finally:
        B.made_free(h)


@pytest.mark.parametrize("real", [False, True])
def test_one_launch_whatever_the_stop_test_of_the_launches(real):
    """MADE_OPT_LAZY_STOP_TEST belongs to the per-layer launches: with either value, and with a single allowed pass, the call is
    one launch, and no pass of it counts as one whose list the next pass derived."""
    D, N = 50, 33
    w = S.Workload(f"xps{real}", D, 2 if real else 1, [70], "bf16", N, "random", "fan_in", S.SEED_BASE + 2180, gain=2.0, real=real)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    try:
        gen = np.random.default_rng(5)
        noise = torch.from_numpy((gen.logistic(size=(N, D)) if real else gen.random((N, D))).astype(np.float32)).cuda()
        for lazy in (1, 0):
            B.made_set_option(h, B.MADE_OPT_LAZY_STOP_TEST, lazy)
            for cap in (0, 1, 2):
                out = []
                for xcd in (1, 0):
                    B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, xcd)
                    out.append(_call(h, real, noise, N, None, 0.0, cap, D))
                (xa, ia, ca, sa), (xb, ib, cb, sb) = out
                assert sa["kernels"] == 1 and sa["tail_less_passes"] == 0, (lazy, cap, sa)
                assert (xa == xb).all() and (ia == ib).all() and ca == cb and sa["passes"] == sb["passes"], (lazy, cap)
                assert (sb["tail_less_passes"] > 0) == (lazy == 1 and cap != 1), (lazy, cap, sb)
    finally:
        B.made_free(h)


@pytest.mark.parametrize("gs", [False, True])
def test_a_wait_that_runs_out_switches_the_kernels_off_for_a_while(gs):
    """MADE_OPT_WAIT_LIMIT = 0: whichever workgroup arrives first backs out.  The call's result is that of the launches, the next
    16 calls take them, twice as many after another call that backs out, and then the kernel serves the model again."""
    D, N = 90, 40
    w = S.Workload("xpw", D, 1, [70, 60], "bf16", N, "random", "fan_in", S.SEED_BASE + 2185, gain=2.0)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    noise = torch.from_numpy(np.random.default_rng(6).random((N, D)).astype(np.float32)).cuda()

    def call():
        if not gs:
            return _call(h, False, noise, N, None, 0.0, 0, D)
        x, it = torch.empty((N, D), dtype=torch.uint8, device="cuda"), torch.empty((N,), dtype=torch.int32, device="cuda")
        B.gs_jacobi_sample(h, noise, N, None, 40, x, it)
        torch.cuda.synchronize()
        return x.cpu().numpy(), it.cpu().numpy(), 0, B.made_last_stats(h)

    try:
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
        want = call()
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 2)
        kernels = []
        for calls, limit in ((2, 1 << 20), (1, 0), (16, 1 << 20), (2, 1 << 20), (1, 0), (16, 0), (1, 0), (32, 0), (1, 1 << 20)):
            B.made_set_option(h, B.MADE_OPT_WAIT_LIMIT, limit)
            for _ in range(calls):
                got = call()
                assert (got[0] == want[0]).all() and (got[1] == want[1]).all()
                kernels.append(got[3]["kernels"] == 1)
        assert kernels == [True] * 2 + [False] * 17 + [True] * 2 + [False] * 50 + [True], kernels
        B.made_set_option(h, B.MADE_OPT_WAIT_LIMIT, 0)
        assert call()[3]["kernels"] > 1
        B.made_set_option(h, B.MADE_OPT_WAIT_LIMIT, 1 << 20)
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 2)
        assert call()[3]["kernels"] == 1
    finally:
        B.made_free(h)


@pytest.mark.parametrize("real", [False, True])
def test_a_wait_that_runs_out_at_the_last_barrier(real):
    """A workgroup may give up on a barrier that the others then see complete.  Where it is the call's last one the call is served:
    the result has to be whole.  Waits of a few polls, one pass, so that the barriers are few and the last one is met often (whether
    a workgroup gives up there and the call is served all the same is a matter of microseconds that nothing here can force)."""
    D, N = 90, 256
    w = S.Workload("xpl", D, 2 if real else 1, [70], "bf16", N, "random", "fan_in", S.SEED_BASE + 2186, gain=2.0, real=real)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    gen = np.random.default_rng(11)
    noise = torch.from_numpy((gen.logistic(size=(N, D)) if real else gen.random((N, D))).astype(np.float32)).cuda()
    x = torch.empty((N, D), dtype=torch.float32 if real else torch.uint8, device="cuda")

    def call():
        x.fill_(9)
        try:
            B.jacobi_sample_real(h, noise, N, None, 0.0, 1, x) if real else B.jacobi_sample(h, noise, N, None, 1, x)
        except B.MadeError as e:
            assert e.code == B.MADE_ERR_NOT_CONVERGED
        return B.made_last_stats(h)["kernels"] == 1

    try:
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
        call()
        want = x.clone()
        wrong, one = [], 0
        for limit in [n for n in range(24) for _ in range(100)]:
            B.made_set_option(h, B.MADE_OPT_WAIT_LIMIT, limit)
            B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 2)
            served = call()
            one += served
            if not torch.equal(x, want):
                wrong.append((limit, served, int((x != want).sum())))
        print(real, "served in one launch:", one, "of 2400")
        assert not wrong, (len(wrong), wrong[:5])
        assert 0 < one < 2400, one
    finally:
        B.made_free(h)


def test_one_launch_after_a_batch_that_needs_buffers_past_2_gib():
    D, H, big, N = 4, 2048, (1 << 19) + 70, 100
    w = S.Workload("xpb", D, 1, [H], "bf16", N, "random", "fan_in", S.SEED_BASE + 2188, gain=2.0)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    try:
        noise = torch.rand(big, D, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        before = _call(h, False, noise[:N], N, None, 0.0, 0, D)
        many = _call(h, False, noise, big, None, 0.0, 0, D)
        after = _call(h, False, noise[:N], N, None, 0.0, 0, D)
        assert before[3]["kernels"] == after[3]["kernels"] == 1, (before[3], after[3])
        assert (before[0] == after[0]).all() and (before[1] == after[1]).all()
        assert (many[0][:N] == before[0]).mean() > 0.99      # (other tiles, another order of sums)
    finally:
        B.made_free(h)


@pytest.mark.parametrize("hidden,dtype,few", [([2048] * 3, "bf16", False), ([2000, 1500], "bf16", True), ([1024] * 6, "f32", True)])
def test_where_the_library_takes_one_launch(hidden, dtype, few):
    """By default: 12 MB of visible weights from 64 samples on, 6 MB and layers of at most 1024 units (13 MB) always."""
    D = 784
    w = S.Workload("xpv", D, 1, hidden, dtype, 64, "random", "fan_in", S.SEED_BASE + 2189, gain=1.5)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    try:
        noise = torch.from_numpy(np.random.default_rng(4).random((64, D)).astype(np.float32)).cuda()
        for N in (63, 64):
            B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 1)
            a = _call(h, False, noise[:N], N, None, 0.0, 0, D)
            B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
            b = _call(h, False, noise[:N], N, None, 0.0, 0, D)
            assert (a[3]["kernels"] == 1) == (few or N == 64), a[3]
            assert (a[0] == b[0]).all() and (a[1] == b[1]).all()
    finally:
        B.made_free(h)


@pytest.mark.parametrize("kind", ["bernoulli", "real", "gs"])
def test_a_start_that_the_result_overwrites(kind):
    """x_out is x_init: in one launch, and where the kernel backs out with some XCDs' results written (waits of a few polls run out
    on some XCDs and not on others), the call's iterate, pass counts and verdict are those of its own start."""
    real = kind == "real"
    D, N = 90, 200
    w = S.Workload("xpa", D, 2 if real else 1, [70, 60], "bf16", N, "random", "fan_in", S.SEED_BASE + 2187, gain=2.0, real=real)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    gen = np.random.default_rng(9)
    noise = torch.from_numpy((gen.logistic(size=(N, D)) if real else gen.random((N, D))).astype(np.float32)).cuda()
    start = torch.from_numpy(gen.normal(size=(N, D)).astype(np.float32) if real else gen.integers(0, 2, size=(N, D)).astype(np.uint8)).cuda()

    def call(same, cap):
        x = start.clone() if same else torch.empty_like(start)
        init, it, code = (x if same else start), torch.full((N,), -1, dtype=torch.int32, device="cuda"), 0
        try:
            if real:
                B.jacobi_sample_real(h, noise, N, init, 0.0, cap, x, it)
            elif kind == "gs":
                B.gs_jacobi_sample(h, noise, N, init, 40, x, it)
            else:
                B.jacobi_sample(h, noise, N, init, cap, x, it)
        except B.MadeError as e:
            code = e.code
            assert code == B.MADE_ERR_NOT_CONVERGED
        torch.cuda.synchronize()
        return x.cpu().numpy(), it.cpu().numpy(), code, B.made_last_stats(h)

    try:
        B.made_set_option(h, B.MADE_OPT_RESIDENT, 0)
        for cap in (0, 2):
            B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 0)
            want = call(False, cap)
            fell_back = 0
            for limit in [1 << 20] + list(range(0, 30)) * 3:
                B.made_set_option(h, B.MADE_OPT_WAIT_LIMIT, limit)
                B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 2)
                got = call(True, cap)
                assert (got[0] == want[0]).all() and (got[1] == want[1]).all() and got[2] == want[2], (limit, cap)
                assert got[3]["kernels"] == 1 or limit < 1 << 20
                fell_back += got[3]["kernels"] > 1
            assert fell_back >= 3, fell_back
            print(kind, cap, "calls that fell back:", fell_back)
    finally:
        B.made_free(h)


def test_more_samples_and_one_hot_models_take_the_other_paths():
    w = S.Workload("xpn", 40, 2, [50], "bf16", 257, "random", "fan_in", S.SEED_BASE + 2190, gain=1.5, real=True)
    h = B.model_from_network(S.make_network(w, with_bias=True))
    try:
        noise = torch.from_numpy(np.random.default_rng(3).logistic(size=(257, 40)).astype(np.float32)).cuda()
        for N, one in ((256, True), (257, False), (256, True)):
            st = _call(h, True, noise, N, None, 0.0, 0, 40)[3]
            assert (st["kernels"] == 1) == one, st
    finally:
        B.made_free(h)
    w = S.workload("small_cat_onehot")
    h = B.model_from_network(S.make_network(w, with_bias=True))
    try:
        B.made_set_option(h, B.MADE_OPT_XCD_RESIDENT, 2)
        st = _call(h, False, torch.from_numpy(S.make_noise(w)).cuda(), w.N, None, 0.0, 0, w.D)[3]
        assert st["kernels"] > 1, st
    finally:
        B.made_free(h)


@pytest.mark.parametrize("persistent", [0, 1])
def test_calls_from_two_threads_do_not_wait_for_each_other(persistent):
    """Two models sampled at once, from two threads on two streams: whichever path a call finds free, its result is the one it
    reaches alone, and no call fails.  persistent: the second one's calls ask for the kernel with one barrier for the whole grid."""
    import threading
    models = []
    for real in (True, False):
        w = S.Workload(f"xpt{real}", 120, 2 if real else 1, [200, 150], "bf16", 60, "random", "fan_in", S.SEED_BASE + 2195, gain=2.0, real=real)
        models.append((real, B.model_from_network(S.make_network(w, with_bias=True))))
    gen = np.random.default_rng(8)
    noises = [torch.from_numpy((gen.logistic(size=(60, 120)) if real else gen.random((60, 120))).astype(np.float32)).cuda() for real, _ in models]
    B.made_set_option(models[1][1], B.MADE_OPT_PERSISTENT, persistent)
    try:
        alone = [_call(h, real, u, 60, None, 0.0, 0, 120)[:2] for (real, h), u in zip(models, noises)]
        wrong, done = [], [0, 0]

        def work(i):
            real, h = models[i]
            x = torch.empty(60, 120, dtype=torch.float32 if real else torch.uint8, device="cuda")
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    for _ in range(20):
                        (B.jacobi_sample_real(h, noises[i], 60, None, 0.0, 0, x) if real else B.jacobi_sample(h, noises[i], 60, None, 0, x))
                        torch.cuda.current_stream().synchronize()
                        if not (x.cpu().numpy() == alone[i][0]).all():
                            wrong.append(i)
                        done[i] += 1
            except Exception as e:                    # (it would end this thread unseen)
                wrong.append((i, repr(e)))

        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong and done == [20, 20], (wrong, done)
        for (real, h), u in zip(models, noises):      # (nothing was switched off on the way)
            assert _call(h, real, u, 60, None, 0.0, 0, 120)[3]["kernels"] == 1
    finally:
        for _, h in models:
            B.made_free(h)
