"""The wide kernel's two sources of the padding parameters -- drawn again for
calls of at most 96 steps, loaded for longer ones -- give the oracle's bits in
any mixture of the two, at row lengths around its shapes' limits, with a ragged
row tail, a ragged last block and a global environment offset."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_bit_equal, gpu_run, oracle_run

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [33, 64, 65, 126, 128, 129, 254, 257, 511, 513, 1027, 2051])
def test_drawn_and_loaded_parameters(D):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, schedule, seed, env0 = 261, [1, 96, 97, 3, 600, 2], (1 << 33) + 5, 512
    cfg = workloads.cartpole(pad_a_low=-0.5, pad_a_high=0.99, pad_b_low=-3.0, pad_b_high=0.25)
    T = sum(schedule)
    got = gpu_run(n, T, schedule, D=D, seed=seed, cfg=cfg, env0=env0)
    ref = oracle_run(n, T, schedule, D=D, seed=seed, cfg=cfg, env0=env0)
    assert_bit_equal(got, ref)
    for a, b in zip(got["stats"], ref["stats"]):
        assert np.array_equal(a, b)
