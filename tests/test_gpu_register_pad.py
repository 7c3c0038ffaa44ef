"""Padding words held in registers, at every width of the kernel (4, 8, 16, 20, 24,
28 and 32 words) and one word to either side: the oracle's bits, with episode
ends, a ragged last block and parameters whose states reach both signs of zero."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_bit_equal, gpu_run, oracle_run

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [1, 4, 5, 8, 9, 16, 17, 20, 21, 24, 25, 28, 29, 32])
def test_register_words(D):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, schedule, seed = 300, [1, 70, 9], 4
    cfg = workloads.cartpole(pad_a_low=-0.5, pad_a_high=0.99, pad_b_low=-3.0, pad_b_high=0.25, max_episode_steps=13)
    got = gpu_run(n, sum(schedule), schedule, D=D, seed=seed, cfg=cfg)
    ref = oracle_run(n, sum(schedule), schedule, D=D, seed=seed, cfg=cfg)
    assert_bit_equal(got, ref)
    for a, b in zip(got["stats"], ref["stats"]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("D", [17, 24, 28])
def test_32_register_words_for_fewer(D):
    """A stored rollout long enough for the 32-word form (262,145 environments,
    more than four workgroups per CU of 256, 2^23 rows and more)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_07736_amd.probe import probe_dispatch
    n, K = 262145, 32
    assert probe_dispatch(n, D, K).register_words == 32
    cfg = workloads.cartpole(pad_a_low=-0.5, pad_a_high=0.99, pad_b_low=-3.0, pad_b_high=0.25, max_episode_steps=13)
    got = gpu_run(n, K, [K], D=D, seed=4, cfg=cfg)
    ref = oracle_run(n, K, [K], D=D, seed=4, cfg=cfg)
    assert_bit_equal(got, ref)
    assert np.array_equal(got["stats"][0], ref["stats"][0])
