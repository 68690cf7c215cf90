"""Which rounds of the longest request the others' workgroups read ahead (attention calls with a column of workgroups a request): the kernel's
arithmetic from the same header (built with g++), whatever 32-bit values the lengths are."""
import ctypes
import random

import pytest

from attn_plan_util import compiled

SOURCE = r"""
#include <algorithm>
#include <cmath>
#include "lengths.hpp"
// rounds[i], and the rounds from[i] .. to[i] - 1 of the longest request that request i's workgroups read
extern "C" void ahead(const int* prefix, const int* nodes, int B, int nodes_max, int capacity, int* rounds, int* from, int* to) {
    int longest = 0, total = 0, all = 0;
    for (int i = 0; i < B; ++i) {
        rounds[i] = (specvlm::keys_of(prefix[i], nodes[i], nodes_max, capacity) + specvlm::kSharesRound - 1) / specvlm::kSharesRound;
        longest = std::max(longest, rounds[i]);
        total += rounds[i];
    }
    const int mean = static_cast<int>(std::ceil(total * (1.f / B) - 0.01f));
    for (int i = 0; i < B; ++i) all += specvlm::rounds_read_ahead(rounds[i], longest, mean);
    const int first = specvlm::first_read_ahead(longest, all), end = std::min(longest - first, specvlm::kMostReadAhead);
    for (int i = 0, upto = 0; i < B; ++i) {
        from[i] = first + upto;
        upto += specvlm::rounds_read_ahead(rounds[i], longest, mean);
        to[i] = first + std::min(upto, end);
    }
}
"""
ANY = [2**31 - 1, 2**31 - 64, 2**30, -1, -2**31, 0]


def ahead(P, n, N, cap):
    ints = ctypes.c_int * len(P)
    rounds, start, end = ints(), ints(), ints()
    compiled(SOURCE).ahead(ints(*P), ints(*n), len(P), N, cap, rounds, start, end)
    return list(rounds), [list(range(a, b)) for a, b in zip(start, end)]


@pytest.mark.parametrize("prefix,nodes,cap,read", [
    # equal lengths, and a longest request less than two rounds beyond the mean: nothing
    ([443] * 8, 60, 976, [[]] * 8), ([500, 500, 500, 700], 12, 976, [[]] * 4),
    # rounds of 2, 4, 3, 4, 4, 8, 4, 3, four in the mean: seven read one or two each, six of them before the longest request ends
    ([170, 390, 253, 339, 350, 906, 365, 287], 60, 976, [[2, 3], [4], [5], [6], [7], [], [], []]),
    # the longest request's last ones where fewer are read, the first of those shares where eight are too few
    ([1204, 700, 700, 700, 700], 60, 1264, [[], [6], [7], [8], [9]]), ([1204, 1000, 300, 400, 200], 60, 1264, [[], [], [2, 3, 4], [5, 6], [7, 8, 9]]),
    ([2004, 100, 300, 150, 120, 600, 90, 200], 60, 2064, [[], [2, 3, 4], [5, 6], [7, 8, 9], [], [], [], []]),
])
def test_measured_batches(prefix, nodes, cap, read):
    assert ahead(prefix, [nodes] * len(prefix), nodes, cap)[1] == read


@pytest.mark.parametrize("seed", range(2))
def test_any_lengths(seed):
    rng = random.Random(seed)
    some = 0
    for _ in range(4000):
        B, N = rng.randint(1, 16), rng.choice([1, 13, 60, 64])
        cap = int(16 * 2 ** rng.uniform(0, 20))
        P = [rng.choice(ANY) if rng.random() < 0.1 else int(cap * rng.random() ** rng.choice([0.1, 1, 5])) for _ in range(B)]
        n = [rng.choice(ANY) if rng.random() < 0.1 else rng.randint(1, N) for _ in range(B)]
        rounds, read = ahead(P, n, N, cap)
        what = (P, n, N, cap, rounds, read)
        every = [j for r in read for j in r]
        some += bool(every)
        assert every == list(range(every[0], every[0] + len(every))) if every else True, what       # none twice, none left out between
        assert len(every) <= 8 and all(2 <= j < max(rounds) for j in every), what
        for i, r in enumerate(read):
            assert not r or (rounds[i] * B <= sum(rounds) + B and rounds[i] < max(rounds) - 1), what   # at most the mean, rounded up
    assert some > 1000
