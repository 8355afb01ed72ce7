"""One-hot first layer where its chunks of units come out ragged: 256 units to a workgroup up to 2048 units, pairs of
512 beyond; layers that end inside a chunk, fewer positions than a round of the waves takes, one sample.  Hidden
activations against float64 (fp32: D sums of weights, 2^-24 each, 1e-5 is ample; bf16 rounding: 2^-8), symbols by the
fixed-point certificate."""
import numpy as np
import pytest

from gpu_util import GpuModel, oracle_models
from oracle import made_oracle as O
from paper_2002_03629_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,C,hidden,N,dtype", [(40, 7, [2048], 1, "f32"), (300, 5, [2049, 60], 3, "bf16"), (70, 9, [257, 90], 33, "f32"),
                                                (17, 256, [2600], 2, "f32"), (131, 20, [31], 5, "bf16"), (520, 3, [3100], 2, "bf16")])
def test_chunks(D, C, hidden, N, dtype):
    w = S.Workload(f"oh{D}", D, C, hidden, dtype, N, "random", "fan_in", S.SEED_BASE + 1300 + D, gain=2.0, onehot=True)
    net = S.make_network(w, with_bias=True)
    ref = oracle_models(net)[1]
    noise = S.make_noise(w)
    with GpuModel(net) as g:
        x, it = g.jacobi(noise)
        act = g.activations(x, 0)
    ok, margin = O.fixed_point_check(ref, x, noise)
    assert (ok | (margin < 1e-3)).all()
    want = np.maximum(O.encode(x, C, True) @ ref.WM[0].T + ref.b[0], 0)
    assert np.abs(act - want).max() <= (1e-5 if dtype == "f32" else 2.0 ** -8) * np.abs(want).max()
