"""The lines of the launch rules (host code of the library, no GPU)."""

import pytest

pytest.importorskip("paper_1705_08210_amd.ps")
import librules


def test_small_3way_tiles_of_unsplit_sums():
    for n_f in (1, 4096, 80000):
        assert [librules.small3(n_f, n_v, 1) for n_v in (3, 96, 97, 208, 209)] == [8, 8, 4, 4, 0]
    assert librules.small3(100, 50, 1, tile=2) == 0


@pytest.mark.parametrize("n_v,n_f,small", [
    # where 32 x 32 tiles ran at least as fast as 64 x 64, and where they were slower
    (64, 80000, True), (97, 28000, True), (110, 20000, True), (120, 16000, True),
    (160, 12000, True), (180, 8192, True), (208, 6000, True),
    (120, 20000, False), (130, 16000, False), (190, 8192, False), (130, 40000, False), (170, 40000, False),
    (180, 12000, False), (208, 12000, False), (208, 40000, False)])
def test_small_3way_tiles_of_split_sums(n_v, n_f, small):
    assert (librules.small3(n_f, n_v, -(-n_f // 4096)) > 0) == small
