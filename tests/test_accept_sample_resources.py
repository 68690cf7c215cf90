"""Registers of the sampling acceptance: a row's chunk is meant to stay in them."""


def test_spills():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("accept_sample.hip").items() if "tree_accept_sample_kernel" in k}
    assert len(usage) == 10, sorted(usage)                     # two types x (32, 64 tokens, whole vectors or not; rows read again)
    for name, u in usage.items():
        # 64 tokens at any alignment need a few more than there are
        most = 164 if "IfLi64ELb0E" in name else 8 if "ItLi64ELb0E" in name else 0
        assert u["scratch"] <= most, (name, u)
