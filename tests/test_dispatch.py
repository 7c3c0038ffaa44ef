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
