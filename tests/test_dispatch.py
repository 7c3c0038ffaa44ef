"""The rules by which a call's sizes choose the form of its kernel, on the CPU: each
rule's edges, and sizes at which the other form was measured slower."""
import pytest

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


def test_wide_blocks_give_every_block_a_workgroup():
    """The fewest environments (8 to 256) whose blocks fit one workgroup per CU, two
    from 64 environments a block on."""
    def block(n, cus=256):
        return probe_dispatch(n, 100, 1, cus=cus).wide_block
    assert block(1) == block(2048) == 8 and block(2049) == 16 and block(8192) == 32 and block(8193) == 64
    assert block(32768) == 64 and block(32769) == block(65536) == 128
    assert block(65537) == block(1 << 30) == 256
    assert block(2048, cus=64) == 32 and block(16384, cus=64) == 128


def _draws(n, D, K):
    return bool(probe_dispatch(n, D, K).wide_drawn)


@pytest.mark.parametrize("D", [64, 128, 256, 512, 1000, 4096])
def test_wide_parameters_drawn_for_short_calls_on_large_states(D):
    """Full rows: from 160, 220, 250 and 300 MB for calls of up to 8, 32, 64 and 96
    steps."""
    n = {mb: -(-mb * 1000000 // (12 * D)) for mb in (160, 220, 250, 300)}
    slack = 1.03 if D == 1000 else 1.0          # 1,000 of 1,024 words in use
    for mb, K in ((160, 8), (220, 32), (250, 64), (300, 96)):
        big, small = int(n[mb] * slack) + 1, int(n[mb] * 0.99)
        assert _draws(big, D, 1) and _draws(big, D, K) and not _draws(small, D, K)
        assert not _draws(big, D, K + 1)
    assert not _draws(1 << 24, D, 97)


@pytest.mark.parametrize("n,D,K", [
    (131072, 129, 1), (131072, 129, 32), (65536, 300, 32), (131072, 100, 32), (262144, 513, 64), (262144, 65, 1),
    (20011, 1100, 1), (20011, 1100, 32), (50000, 513, 32), (50000, 1100, 64), (50000, 1100, 96), (131072, 1100, 96),
    (262144, 700, 96), (262144, 96, 96)])
def test_wide_parameters_loaded_where_rows_fill_their_lanes_badly(n, D, K):
    """Measured 5 to 30 % faster loaded: the last chunk of a row is drawn whole."""
    assert not _draws(n, D, K)


@pytest.mark.parametrize("n,D,K", [
    (262144, 512, 1), (262144, 4096, 1), (131072, 513, 8), (65536, 400, 32), (131072, 512, 64), (65536, 1000, 96)])
def test_wide_parameters_drawn_where_that_was_measured_faster(n, D, K):
    assert _draws(n, D, K)
