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


def test_a_bound_in_the_place_of_the_tokens(rule):
    """The caller may pass the whole room of the table as the number of tokens.  128 to 256 pairs take a workgroup each then only
    up to a length at which a few long requests among short ones are no slower for it."""
    def full(requests, heads, room, dh):
        return ("p", requests, heads, room, requests * room, dh)
    assert rule([full(8, 32, 1024, 128), full(5, 32, 1024, 128), full(20, 12, 2048, 64)]) == [True] * 3
    assert rule([full(8, 32, 1040, 128), full(8, 32, 4096, 128), full(7, 32, 2000, 128), full(20, 12, 3008, 64)]) == [False] * 4


def test_many_pairs(rule):
    """From 448 pairs on: up to 2048 tokens of head_dim 128 (4096 of 64), and from 2560 pairs on beyond half of that only where the
    lengths are known to differ.  Longer rows lose where one request is long and the others are short."""
    def paged(requests, heads, room, share, dh):
        return ("p", requests, heads, room, int(requests * room * share), dh)
    assert rule([paged(14, 32, 2048, 1.0, 128), paged(32, 72, 2048, 1.0, 128), paged(64, 72, 2048, 0.75, 128), paged(64, 72, 1024, 1.0, 128),
                 paged(128, 32, 4096, 0.5, 64), paged(64, 72, 2048, 0.15, 128)]) == [True] * 6
    assert rule([paged(64, 32, 2064, 0.5, 128), paged(64, 32, 4096, 1.0, 128), paged(64, 72, 4096, 0.5, 128), paged(64, 72, 2048, 1.0, 128),
                 paged(40, 72, 2000, 1.0, 128), paged(128, 32, 4112, 0.5, 64), paged(16, 32, 1040, 0.1, 128)]) == [False] * 7
