"""Registers of the sampling acceptance: a row's chunk is meant to stay in them."""


def test_spills():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("accept_sample.hip").items() if "tree_accept_sample_kernel" in k}
    assert len(usage) == 4, sorted(usage)                      # two types x (a row in registers, a row read once)
    for name, u in usage.items():
        assert u["scratch"] == 0, (name, u)
