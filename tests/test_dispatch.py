"""The rules by which a call's sizes choose the form of its kernel, on the CPU: each
rule's edges, and sizes at which the other form was measured slower."""
import pytest

# before the package, whose library binds to the HIP runtime already loaded: the GPU
# tests of the same process share torch's
import torch  # noqa: F401

from paper_2207_07736_amd.probe import probe_dispatch


@pytest.mark.parametrize("D", range(33))
def test_register_words_hold_the_padding_words(D):
    for n, K in ((1, 1), (65536, 1000), (100003, 500), (1 << 30, 7)):
        for traj in (False, True):
            words = probe_dispatch(n, D, K, traj).register_words
            assert words in (0, 4, 8, 16, 20, 24, 28, 32) and words >= D
            assert D > 16 or words - D < (8 if D > 8 else 4)


@pytest.mark.parametrize("D,few", [(17, 20), (20, 20), (21, 24), (24, 24), (25, 28), (28, 28), (29, 32), (32, 32)])
def test_long_stored_rollouts_keep_32_words(D, few):
    """17 to 28 words: the fewest registers while the words set the pace, 32 where
    the stores do (one trajectory row per environment and step)."""
    def words(n, K, traj=True, cus=256):
        return probe_dispatch(n, D, K, traj, cus).register_words
    # one workgroup per CU or fewer: always the fewest
    assert words(1, 1) == words(65536, 100000) == few
    # up to four per CU: below 2^24 rows
    assert words(65537, 255) == words(100003, 128) == words(262144, 63) == few
    assert words(65537, 256) == words(100003, 500) == words(262144, 64) == 32
    # more: below 2^23 rows
    assert words(262145, 31) == words(1048576, 7) == few
    assert words(262145, 32) == words(1048576, 8) == words(1048576, 128) == 32
    # no trajectory: always the fewest
    assert words(1048576, 500, traj=False) == few
    # on a quarter of the CUs the workgroups per CU change with them
    assert words(16385, 2000, cus=64) == 32 and words(16384, 2000, cus=64) == few


def _block(n, D=100, K=200, cus=256):
    return probe_dispatch(n, D, K, cus=cus).wide_block


def test_wide_blocks_give_every_block_a_workgroup():
    """The fewest environments (8 to 256) whose blocks fit one workgroup per CU, two
    from 64 environments a block on."""
    for K in (1, 200):
        assert _block(1, K=K) == _block(2048, K=K) == 8 and _block(2049, K=K) == 16
        assert _block(8192, K=K) == 32 and _block(8193, K=K) == 64 and _block(32768, K=K) == 64
        assert _block(65537, K=K) == _block(1 << 30, K=K) == 256
    assert _block(32769) == _block(65536) == 128
    assert _block(2048, cus=64) == 32 and _block(16384, cus=64) == 128


def test_wide_blocks_of_128_only_for_long_or_drawn_calls():
    """Between 32,769 and 65,536 environments loaded calls whose bytes weigh more than
    their steps were up to 17 % slower in blocks of 128, and few words with a long
    trajectory 10 %."""
    for n in (32769, 36000, 45000, 65536):
        for D, K in ((65, 63), (128, 63), (129, 21), (200, 32), (300, 49), (400, 65), (600, 99), (960, 159),
                     (1000, 159), (4096, 159)):
            assert not _draws(n, D, K) and _block(n, D, K) == 256, (n, D, K)
            assert not _draws(n, D, K + 1) and _block(n, D, K + 1) == 128, (n, D, K)
        assert _block(n, 40, 1) == _block(n, 64, 1) == 128
    assert _block(57000, 100, 294) == 128 and _block(57000, 100, 295) == _block(57000, 128, 400) == 256
    assert _block(57000, 64, 295) == 256
    assert _block(57000, 129, 400) == _block(57000, 4096, 1000) == 128
    for n, block in ((32769, 64), (49152, 64), (49153, 128), (65536, 128)):
        assert _draws(n, 1000, 1) and _block(n, 1000, 1) == block


def test_wide_blocks_of_64_not_for_short_calls_on_large_loaded_states():
    assert _block(32768, 400, 1) == _block(32768, 400, 8) == _block(28000, 400, 8) == 256
    assert _block(32768, 400, 9) == _block(32768, 200, 1) == _block(32768, 1000, 1) == 64
    assert _block(24576, 400, 1) == _block(20011, 1100, 1) == 64


def _draws(n, D, K, cus=256):
    return bool(probe_dispatch(n, D, K, cus=cus).wide_drawn)


@pytest.mark.parametrize("D", [64, 128, 256, 512, 1000, 4096])
def test_wide_parameters_drawn_for_short_calls_on_large_states(D):
    """Full rows: from 180, 190, 300 and 250 MB for calls of up to 8, 32, 64 and 96
    steps (410 MB for up to 96 in batches of up to 192 environments per CU)."""
    for mb, K, cus in ((180, 8, 256), (190, 32, 256), (300, 64, 256), (250, 96, 1), (410, 96, 1 << 20)):
        n = -(-mb * 1000000 // (12 * D))
        slack = 1.03 if D == 1000 else 1.0          # 1,000 of 1,024 words in use
        big, small = int(n * slack) + 1, int(n * 0.99)
        assert _draws(big, D, 1, cus) and _draws(big, D, K, cus) and not _draws(small, D, K, cus)
        assert K == 64 or not _draws(big, D, K + 1, cus)
    assert not _draws(1 << 24, D, 97)


@pytest.mark.parametrize("n,D,K", [
    (131072, 129, 1), (131072, 129, 32), (65536, 300, 32), (131072, 100, 32), (262144, 513, 64), (131072, 65, 1),
    (20011, 1100, 1), (20011, 1100, 32), (50000, 513, 32), (50000, 1100, 64), (50000, 1100, 96), (131072, 1100, 96),
    (262144, 700, 96), (262144, 96, 96), (200000, 129, 1), (33000, 1100, 32), (33000, 513, 1), (36000, 400, 1)])
def test_wide_parameters_loaded_where_rows_fill_their_lanes_badly(n, D, K):
    """Measured 5 to 50 % faster loaded: the last chunk of a row is drawn whole."""
    assert not _draws(n, D, K)


@pytest.mark.parametrize("n,D,K", [
    (262144, 512, 1), (262144, 4096, 1), (131072, 513, 8), (65536, 400, 32), (131072, 512, 64), (65536, 1000, 96),
    (36000, 1000, 8)])
def test_wide_parameters_drawn_where_that_was_measured_faster(n, D, K):
    assert _draws(n, D, K)


def test_policy_forms_follow_the_compute_units():
    def envs(n, cus=256):
        d = probe_dispatch(n, 0, 1, cus=cus)
        return d.policy_envs_bf16, d.policy_envs_f32
    assert envs(1) == envs(49152) == (16, 16)
    assert envs(49153) == envs(98304) == (64, 32)
    assert envs(98305) == envs(1 << 30) == (64, 64)
    # a partition with an eighth of the CUs fills up at an eighth of the batch
    assert envs(6144, 32) == (16, 16) and envs(6145, 32) == envs(12288, 32) == (64, 32)
    assert envs(12289, 32) == (64, 64)
