"""The rules that choose between one workgroup per (sequence, head) and ranges with a merge, on the host."""
import pytest

import attn_pairs
from test_gpu_attention_pairs import PAGED, SIZES


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


def test_the_compared_sizes_take_both_forms(rule):
    """Which of the sizes that test_gpu_attention_pairs.py compares are cut into ranges; all others take a workgroup per pair."""
    ranges = [(1, 1, 128, 513, 0), (3, 3, 128, 513, 0), (1, 6, 64, 1025, 0), (1, 127, 128, 1000, 0), (1, 128, 128, 1025, 0),
              (1, 257, 64, 1537, 0), (7, 64, 64, 4097, 0), (2, 3, 64, 700, 330)]
    assert [s for s, pair in zip(SIZES, rule([("c", B * H, n0, n1, dh) for B, H, dh, n0, n1 in SIZES])) if not pair] == ranges
    assert {min(attn_steps, 3) for attn_steps in (-(-n0 // 64) - (-n1 // 64) for _, _, _, n0, n1 in SIZES)} == {1, 2, 3}   # one, two, four wavefronts

    in_ranges = [0, 2, 4, 5, 7, 10, 12, 15]                                # of PAGED
    for bt in (16, 128):
        def call(H, dh, lens, spare, wide):
            cols = max(-(-n // bt) for n in lens) + spare + (4097 * 128 // dh // bt if wide else 0)
            return ("p", len(lens), H, cols * bt, sum(lens), dh)
        assert [i for i, pair in enumerate(rule([call(*p, False) for p in PAGED])) if not pair] == in_ranges, bt
        assert not any(rule([call(*p, True) for p in PAGED])), bt          # room for longer rows: cut into ranges
    assert rule([("p", 8, 64, 1008, 8 * 1008, 128), ("p", 8, 64, 2064, 8 * 2064, 128),             # the two tests of single calls
                 ("p", 3, 40, 512, 1138, 128), ("p", 3, 40, 2048, 4122, 128)]) == [True, False, True, False]
