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


@pytest.mark.parametrize("D", [33, 64, 65, 128, 129, 254, 300, 511, 513, 1027, 2051])
@pytest.mark.parametrize("K", [8, 32, 64, 96])
def test_drawn_and_loaded_parameters(D, K):
    """The smallest state on which calls of K steps draw: calls of K and of one step
    draw and those of 97 load, over environments of the first, a middle and the
    ragged last block."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_07736_amd.probe import probe_dispatch

    def draws(n, k):
        return bool(probe_dispatch(n, D, k).wide_drawn)

    lo, hi = 1, 1 << 20
    if not draws(hi, K):
        # rows that fill their lanes too badly for calls this long
        assert K > 8 and D in (33, 65, 129, 300, 513, 1027, 2051)
        return
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if draws(mid, K) else (mid + 1, hi)
    n = lo + 1 - lo % 2                     # odd: a ragged last block
    schedule = [K, 97, 1]
    assert [draws(n, k) for k in schedule] == [True, False, True]
    _slices_against_oracle(n, D, schedule)


def _slices_against_oracle(n, D, schedule):
    seed, env0 = (1 << 33) + 5, 512
    cfg = workloads.cartpole(pad_a_low=-0.5, pad_a_high=0.99, pad_b_low=-3.0, pad_b_high=0.25)
    slices = [(0, 70), (n // 2, n // 2 + 70), (n - 261, n)]
    got = gpu_run(n, sum(schedule), schedule, D=D, seed=seed, cfg=cfg, env0=env0, slices=slices)
    refs = [oracle_run(b - a, sum(schedule), schedule, D=D, seed=seed, cfg=cfg, env0=env0 + a) for a, b in slices]
    ref = {k: np.concatenate([r[k] for r in refs], axis=-1) for k in ("obs", "action", "reward", "done", "state", "ep")}
    ref["t"] = refs[0]["t"]
    assert_bit_equal(got, ref)


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


@pytest.mark.parametrize("n,D,schedule,blocks", [
    (32769, 33, [160, 5, 161], [128, 128, 128]), (40001, 130, [160, 5, 161], [128, 256, 128]),
    (33000, 400, [160, 3], [128, 256]), (28001, 400, [2, 9, 1], [256, 64, 256]), (32901, 900, [8, 65], [64, 256])])
def test_blocks_that_change_with_the_call(n, D, schedule, blocks):
    """Calls of one handle in blocks of different sizes, their statistics included."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_07736_amd.probe import probe_dispatch
    assert [probe_dispatch(n, D, k).wide_block for k in schedule] == blocks
    cfg = workloads.cartpole(max_episode_steps=11)
    got = gpu_run(n, sum(schedule), schedule, D=D, seed=9, cfg=cfg)
    ref = oracle_run(n, sum(schedule), schedule, D=D, seed=9, cfg=cfg)
    assert_bit_equal(got, ref)
    for a, b in zip(got["stats"], ref["stats"]):
        assert np.array_equal(a, b)
