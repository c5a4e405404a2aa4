"""The compiler's resource usage of the hot kernels stays where it was measured: a change that makes one of
them spill (a few more live registers under a launch bound) costs a multiple of its run time and no parity
test notices.  CPU only: hipcc cross-compiles the sources with -Rpass-analysis=kernel-resource-usage."""
import functools
import re
import shutil

import pytest

from paper_2410_09397_amd import pmc_summary

# scratch bytes per lane that each kernel is allowed: the d = 64 forward and dQ kernels keep their
# 4-workgroups-per-CU launch bound and spill 7 and 3 registers (measured faster than the build without scratch)
ALLOWED_SCRATCH = {"fwd_kernel<64>": 28, "bwd_dq_kernel<64, 1>": 12}
MIN_OCCUPANCY = {"fwd_kernel<64>": 4, "bwd_dq_kernel<64, 1>": 4, "bwd_dkdv_kernel<64>": 3, "fwd_kernel<128>": 2,
                 "bwd_dq_kernel<128, 1>": 2, "bwd_dkdv_kernel<128>": 2,
                 "fwd_split_kernel<64>": 4, "fwd_split_kernel<128>": 2, "bwd_dq_split_kernel<64>": 3, "bwd_dq_split_kernel<128>": 2}
# fp32-arithmetic kernels, per kind of storage (0: fp32, 3: bf16) and padded width: two waves per SIMD where two workgroups of
# four waves or one of eight fit the LDS, more where the width leaves room
STREAM_OCCUPANCY = {("fwd", 0): {32: 7, 64: 5, 96: 4, 128: 3}, ("bwd", 0): {32: 5, 64: 4, 96: 2, 128: 1},
                    ("fwd", 3): {32: 5, 64: 4, 96: 2, 128: 2, 160: 3, 192: 3, 224: 3, 256: 3},
                    ("bwd", 3): {32: 3, 64: 2, 96: 2, 128: 1, 160: 1, 192: 1, 224: 1, 256: 1}}


@functools.lru_cache(maxsize=None)
def resources():
    return {r["kernel"]: r for r in pmc_summary.kernel_resources()}  # every kernel of the library


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_hot_kernels_keep_their_registers_and_do_not_spill():
    seen = resources()
    assert set(MIN_OCCUPANCY) <= set(seen), sorted(seen)
    for name, r in seen.items():
        assert int(r["ScratchSize [bytes/lane]"]) <= ALLOWED_SCRATCH.get(name, 0), (name, r)
        if name in MIN_OCCUPANCY:
            assert int(r["Occupancy [waves/SIMD]"]) >= MIN_OCCUPANCY[name], (name, r)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_fp32_arithmetic_kernels_keep_their_occupancy():
    seen = {}
    for name, r in resources().items():
        m = re.match(r"stream_(fwd|bwd)_kernel<(\d), (?:true|false), (\d+), ", name)
        if m:
            seen.setdefault((m.group(1), int(m.group(2))), {}).setdefault(int(m.group(3)), []).append(int(r["Occupancy [waves/SIMD]"]))
    assert {k: set(v) for k, v in seen.items()} == {k: set(v) for k, v in STREAM_OCCUPANCY.items()}
    for k, widths in seen.items():
        for width, occupancies in widths.items():
            assert min(occupancies) >= STREAM_OCCUPANCY[k][width], (k, width, occupancies)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_profile_summaries_count_every_kernel():
    """A kernel that belongs to no group is left out of the times and byte counts of attn_fwd and attn_bwd without a word."""
    for name in resources():
        groups = [pmc_summary.is_in(name, g) for g in (pmc_summary.FWD_KERNELS, pmc_summary.BWD_KERNELS, pmc_summary.OTHER_KERNELS)]
        assert sum(groups) == 1, (name, groups)
