"""The row-dividing attention kernels count outstanding memory operations by hand: no register may spill."""


def test_row_block_kernels_spill_nothing():
    from paper_2509_11815_amd import build
    usage = {k: v for k, v in build.kernel_resource_usage("attn_wave.hip").items() if "attn_wave_kernel" in k}
    assert len(usage) == 8, sorted(usage)                      # two head sizes x two block heights x contiguous / paged
    for name, u in usage.items():
        assert u["scratch"] == 0 and u["lds"] <= 160 * 1024, (name, u)
