"""Which slots and lengths lie inside a cache, from the kernels' own header (built with g++), against arithmetic that cannot wrap."""
import ctypes
import itertools

from attn_plan_util import compiled

SOURCE = r"""
#include "lengths.hpp"
extern "C" int slot_inside(int prefix, int node, int capacity) { return specvlm::slot_inside(prefix, node, capacity); }
extern "C" int length_fits(int prefix, int nodes, int capacity) { return specvlm::length_fits(prefix, nodes, capacity); }
"""
INT_MAX = 2**31 - 1
VALUES = [-2**31, -2**31 + 1, -64, -1, 0, 1, 15, 63, 64, 65, 1000, 2**24, INT_MAX - 64, INT_MAX - 63, INT_MAX - 1, INT_MAX]


def test_slots():
    lib = compiled(SOURCE)
    for prefix, node, capacity in itertools.product(VALUES, VALUES, [c for c in VALUES if c > 0]):
        assert bool(lib.slot_inside(prefix, node, capacity)) == (prefix >= 0 and node >= 0 and prefix + node < capacity), (prefix, node, capacity)


def test_prefix_and_nodes():
    lib = compiled(SOURCE)
    for prefix, nodes, capacity in itertools.product(VALUES, [1, 2, 59, 60, 63, 64], [c for c in VALUES if c > 0]):
        assert bool(lib.length_fits(prefix, nodes, capacity)) == (prefix >= 0 and prefix + nodes <= capacity), (prefix, nodes, capacity)
