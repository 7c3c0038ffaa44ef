"""The wide kernel's two sources of the padding parameters -- drawn again for
short calls on states too large for the last-level cache, loaded otherwise --
and its block sizes give the oracle's bits in any mixture of the two, at row
lengths around its shapes' limits, with a ragged row tail, a ragged last block
and a global environment offset."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_bit_equal, gpu_run, oracle_run

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [33, 64, 65, 126, 128, 129, 254, 257, 511, 513, 1027, 2051])
def test_loaded_parameters(D):
    """Small states, which load at every call length."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _against_oracle(261, D, [1, 96, 97, 3, 600, 2])


@pytest.mark.parametrize("D,megabytes,schedule", [
    (33, 151, [1, 32]), (64, 151, [32, 33]), (65, 151, [1, 32]), (128, 151, [32, 33]), (129, 151, [1, 32]),
    (254, 151, [32, 33]), (511, 151, [1, 32]), (513, 151, [32, 33]), (2051, 151, [1, 33]), (300, 301, [33])])
def test_drawn_and_loaded_parameters(D, megabytes, schedule):
    """States just above the two sizes (12 bytes a word) from which calls of up
    to 32 and up to 96 steps draw."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Dp = (D + 3) // 4 * 4
    _against_oracle(megabytes * 1000000 // (12 * Dp) + 1, D, schedule)


def _against_oracle(n, D, schedule):
    seed, env0 = (1 << 33) + 5, 512
    cfg = workloads.cartpole(pad_a_low=-0.5, pad_a_high=0.99, pad_b_low=-3.0, pad_b_high=0.25)
    T = sum(schedule)
    got = gpu_run(n, T, schedule, D=D, seed=seed, cfg=cfg, env0=env0)
    ref = oracle_run(n, T, schedule, D=D, seed=seed, cfg=cfg, env0=env0)
    assert_bit_equal(got, ref)
    for a, b in zip(got["stats"], ref["stats"]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n,D", [
    (7, 33), (7, 70), (7, 130), (7, 515), (7, 1030), (2049, 33), (2049, 515), (4097, 70), (4097, 1030), (8192, 130),
    (32768, 33), (32769, 130), (32769, 260), (65537, 33), (65537, 70)])
def test_blocks_of_fewer_environments(n, D):
    """Blocks of 8 to 256 environments (the fewest that give every block its own
    workgroup on 256 CUs), around the sizes where they grow: results and the
    statistics rows that several blocks share, short and long calls mixed."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    schedule = [3, 97] if n < 20000 and D < 500 else [3, 9]
    cfg = workloads.cartpole(max_episode_steps=11)
    got = gpu_run(n, sum(schedule), schedule, D=D, seed=9, cfg=cfg)
    ref = oracle_run(n, sum(schedule), schedule, D=D, seed=9, cfg=cfg)
    assert_bit_equal(got, ref)
    for a, b in zip(got["stats"], ref["stats"]):
        assert np.array_equal(a, b)
