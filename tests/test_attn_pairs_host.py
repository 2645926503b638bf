"""The rules that choose between one workgroup per (sequence, head) and ranges with a merge, on the host."""
import pytest

import attn_pairs


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return attn_pairs.build(tmp_path_factory.mktemp("pairs"))


def test_more_pairs_than_a_launch_has_threads_for(rule):
    """A launch holds fewer than 2^32 threads: 2^24 workgroups of 256 are too many, the merge's 64 threads a pair are not."""
    most = (1 << 24) - 1
    assert rule([("p", most, 1, 16, most, 64), ("p", most // 5, 5, 512, 5, 128), ("c", most, 64, 0, 64)]) == [True] * 3
    assert rule([("p", most + 1, 1, 16, most, 64), ("p", 1 << 21, 8, 16, 1 << 21, 128), ("c", most + 1, 64, 0, 64)]) == [False] * 3
