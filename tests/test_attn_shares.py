"""What a batch's lengths make of its columns (attention calls dealt out by length): the kernel's arithmetic from the same header (built
with g++), lane by lane.  Every request, whatever 32-bit values its lengths are, has between one column and eight, and all of them fit."""
import ctypes
import random

import pytest

from attn_plan_util import columns_of, compiled

SOURCE = r"""
#include <algorithm>
#include <cmath>
#include "lengths.hpp"
// the columns of every request, and which length gave them; 0 where none does within `most_steps` steps
extern "C" int deal(const int* prefix, const int* nodes, int B, int nodes_max, int capacity, int columns, int most_ranges,
                    float least_gain, int ulps, int most_steps, int* shares) {
    int rounds[16], total = 0, longest = 0;
    for (int i = 0; i < B; ++i) {
        rounds[i] = (specvlm::keys_of(prefix[i], nodes[i], nodes_max, capacity) + specvlm::kSharesRound - 1) / specvlm::kSharesRound;
        total += rounds[i];
        longest = std::max(longest, rounds[i]);
    }
    auto share = [&](int i, float len) {                  // the device's reciprocal is within an ulp
        float inverse = 1.f / len;
        for (int u = 0; u < ulps; ++u) inverse = std::nextafter(inverse, 2.f);
        for (int u = 0; u < -ulps; ++u) inverse = std::nextafter(inverse, 0.f);
        return specvlm::columns_of(rounds[i], len, inverse);
    };
    float len = std::ceil(std::fmax(total * (1.f / columns), longest * (1.f / most_ranges)) - 0.01f);
    for (int step = 0;; ++step, len += 1.f) {
        if (step == most_steps) return 0;
        int sum = 0;
        for (int i = 0; i < B; ++i) sum += share(i, len);
        if (sum <= columns) break;
    }
    if (longest - len < least_gain) len = longest;
    for (int i = 0; i < B; ++i) shares[i] = share(i, len);
    return static_cast<int>(len);
}
"""
INT_MAX = 2**31 - 1
ANY = [INT_MAX, INT_MAX - 1, INT_MAX - 13, INT_MAX - 63, INT_MAX - 64, 2**30, -1, -2**31, 0]


def deal(P, n, N, cap, columns, D=128, ulps=0):
    B = len(P)
    ints = ctypes.c_int * B
    shares = ints()
    length = compiled(SOURCE).deal(ints(*P), ints(*n), B, N, cap, columns, 8, ctypes.c_float(1.3 if D == 128 else 2.5), ulps, 4 * cap, shares)
    return length, list(shares)


def check(P, n, N, cap, columns, D=128):
    for ulps in (-1, 0, 1):
        length, shares = deal(P, n, N, cap, columns, D, ulps)
        what = (P, n, N, cap, columns, length, shares)
        assert length >= 1 and min(shares) >= 1 and max(shares) <= 8 and sum(shares) <= columns, what
        for p, m, s in zip(P, n, shares):                  # the longest stream is no longer than `length` rounds
            keys = min(max(p, 0) + min(max(m, 1), N), cap)
            assert -(-keys // 128) <= s * length, what


@pytest.mark.parametrize("lengths", [(INT_MAX, 1311, 3000, 777), (1500, 2900, INT_MAX, 900), (2048, 1311, 3000, INT_MAX), (INT_MAX,) * 4])
def test_one_bad_length_leaves_the_others_their_columns(lengths):
    N, cap, columns = 64, 3072, columns_of(4, 32, 8, 128, 64, 3072).columns
    check(list(lengths), [N] * 4, N, cap, columns)


@pytest.mark.parametrize("seed", range(4))
def test_any_lengths(seed):
    rng = random.Random(seed)
    for _ in range(2000):
        B, N = rng.randint(2, 16), rng.choice([1, 13, 60, 64])
        cap, columns = int(16 * 2 ** rng.uniform(0, 20)), rng.randint(B + 1, 256)
        P = [rng.choice(ANY) if rng.random() < 0.2 else int(cap * rng.random() ** rng.choice([0.1, 1, 5])) for _ in range(B)]
        n = [rng.choice(ANY) if rng.random() < 0.2 else rng.randint(1, N) for _ in range(B)]
        check(P, n, N, cap, columns, rng.choice([64, 128]))
