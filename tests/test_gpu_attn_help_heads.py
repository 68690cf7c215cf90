"""GPU parity of attention calls in which the shorter requests' workgroups read the longest one's keys ahead, where a head's workgroups lie
across two XCDs: KV heads that are no multiple of 8, with and without shared heads."""
import pytest

import test_gpu_attn_help as help_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,prefix,num_nodes,bad", [
    # (requests, query heads, KV heads, nodes, slots per request)
    ((8, 32, 4, 64, 976), [170, 390, 253, 339, 350, 906, 365, 287], None, None), ((8, 32, 4, 64, 2064), [2000, 100, 300, 150, 120, 600, 90, 200], None, None),
    ((4, 40, 10, 64, 1072), [200, 300, 1000, 0], [64, 1, 33, 2], None), ((5, 28, 28, 60, 1072), [1000, 200, 300, 250, 400], None, (2, 5000)),
])
def test_against_oracle(monkeypatch, shape, prefix, num_nodes, bad):
    monkeypatch.setitem(help_cases.SHAPES, "heads across XCDs", shape)
    help_cases.test_against_oracle("heads across XCDs", prefix, num_nodes, bad)
