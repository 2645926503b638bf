// One workgroup per (sequence, head), or ranges and a merge?  The rules of the contiguous and of the paged attention: plain
// integer arithmetic, callable from host code, so that they can be checked on a CPU.
//
// Ranges balance any number of pairs over the chip, at the price of a second launch, partials in memory and ranges that end
// inside a pair.  In both rules n counts 16 KB of K and V, what a step of 64 tokens of head_dim 64 reads.
#pragma once
#include <stdint.h>

namespace hk {
namespace pairs {

constexpr int kTile = 64;                                     // tokens of a step
// A launch holds fewer than 2^32 threads and a pair takes up to 256 of them (64 in the merge).
constexpr int64_t kMostPairs = (int64_t(1) << 24) - 1;

// Steps of the two segments of a pair.
inline int steps(int L0, int L1) { return (L0 + kTile - 1) / kTile + (L1 + kTile - 1) / kTile; }

// Measured over 1 to 4608 pairs x 200 to 4096 tokens, both head dimensions and types, one workgroup per pair
// against ranges (us, replayed from a graph, fp16, head_dim 128 unless said):
//   * short contexts: 8 pairs of 400 tokens 6.3 / 8.0, 72 of 200 5.2 / 8.7; at 1000 tokens 8 pairs take 11.4 / 8.9 and 32 take
//     11.9 / 9.7: too few compute units ask for the rows
//   * from 128 pairs on: 128 of 1000 tokens 15.5 / 17.0, of 4096 52.4 / 49.3
//   * 180 to 256 pairs, nearly one per compute unit: 200 of 1000 tokens 19.4 / 25.0, of 4096 68.7 / 75.4; 256: 23.8 / 27.9, 86.4 / 92.7
//   * 257 to 447: some compute units get two: 290 of 700 tokens faster, of 1000 32.1 / 31.8; 352 of 2000 70.7 / 67.4
//   * from 448 on the workgroups' own order evens that out: 480 of 2000 tokens 81.6 / 86.3, 4608 707 / 731; level from 3000
//     tokens on (1100 pairs 273 / 269)
inline bool contiguous(int64_t pairs, int steps, int head_dim)
{
    const int64_t n = (int64_t)steps * (head_dim / 64);
    if (pairs > kMostPairs) return false;
    if (pairs < 128) return n <= 16;
    if (pairs < 180) return n <= 32;
    if (pairs <= 256) return true;
    return n <= (pairs < 448 ? 24 : 64);
}

// With the longest length that the table has room for, and the tokens of all requests as far as the host knows.  Lengths that
// differ make the ranges worse (a wavefront searches its requests, and steps over those that end) and leave compute units to the
// long pairs: half of the requests 16 tokens, half L, 256 pairs, L = 1000: 16.1 us against 27.6; 1024 pairs, L = 2000: 93.5 against
// 122; lengths L/2 to L, 32 requests x 32 heads, L = 1000: 71.7 against 77.0; 2560 pairs, L = 2000: 320 against 326; 864, L = 4000:
// 232 against 230.
// What a workgroup per pair cannot balance is a few long requests among many short ones: beyond short contexts the tokens have to
// be those of 224 pairs of full length, or half of what the table has room for where there are fewer than 448 pairs.
// `tokens` may be a bound, up to the room, whatever the lengths are: the lines for n lie where one long request among short ones
// (16 tokens) is not slower for it either.  256 pairs, L = 1000: 12.5 us against 14.0, L = 2000: 22.2 against 17.6, L = 4096: 41.9
// against 23.7 (and 81 against 89 where all are that long); 240 pairs of head_dim 64, L = 2000 (n = 32): 10.5 against 14.2, L =
// 3000: 17.4 against 14.9.  From 448 pairs on, L = 2000 (n = 64): 448 pairs 25.1 against 26.1, 640 26.3 / 25.5, 2048 26.4 / 27.0, 4608
// 31.2 / 38.6; L = 2500 (n = 80): 448 30.0 / 27.1, 2048 31.4 / 29.7; L = 4096: 2048 46.2 / 35.2, 2880 52.0 / 50.1.
// From 2560 pairs on lengths that are all alike are level up to n = 48 (9216 pairs, L = 1500: 1096 / 1103) and lose a little beyond
// (L = 2000, 2304 pairs: 366 / 371; 2880 480 / 473, 4608 758 / 748, 9216 1514 / 1478); lengths L/2 to L gain 1 to 3 % there, an eighth
// of the requests L and the others 16 tokens a quarter (4608: 108 / 145).
inline bool paged(int64_t requests, int heads, int64_t longest, int64_t tokens, int head_dim)
{
    const int64_t pairs = requests * heads;
    const int64_t n = (longest + kTile - 1) / kTile * (head_dim / 64);
    if (pairs > kMostPairs) return false;
    if (n <= 16) return true;
    const int64_t room = longest * requests;
    if (pairs >= 448)
        return n <= 64 && tokens * heads >= 224 * longest && (pairs < 2560 || n <= 32 || 10 * tokens <= 9 * room);
    if (pairs < 128 || 2 * tokens < room) return false;
    return n <= (pairs <= 256 ? 32 : 24);
}

}  // namespace pairs
}  // namespace hk
