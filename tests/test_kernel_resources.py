"""What the kernels of the built library take of a compute unit, where a register more costs a workgroup (tests/kernel_resources.py)."""

import re

import pytest

import kernel_resources as R

METRIC = {"method": 0, "squared differences": 1, "one bit": 2, "three bits": 3}
LARGEST = {"method": 3, "squared differences": 9, "one bit": 1, "three bits": 7}   # distance per dimension


def instances(pattern):
    found = {n: k for n, k in R.kernels().items() if re.fullmatch(pattern, n)}
    assert found, pattern
    return found


@pytest.mark.parametrize("metric,d", [(m, d) for m in METRIC for d in (64, 96, 128) if (m, d) != ("squared differences", 128)])
def test_six_workgroups_of_the_select_kernel_fit_a_compute_unit(metric, d):
    """Contiguous caches, with attention: 256 threads each, so six waves per SIMD.  (Not where the histograms of sixteen tiles are
    longer than a thread per pair of bins takes: these need 90 registers before the attention.)"""
    wide = LARGEST[metric] * d > 511
    tiles = "[48]" if wide else r"\d+"
    for name, k in instances(r"select_kernel<256, true, %d, false, %d, \d+, %s>" % (METRIC[metric], d, tiles)).items():
        assert R.waves_per_simd(k) >= 6 and 6 * k.lds <= 160 * 1024 and k.scratch == 0, (name, k)


def fused_scans(group, waves, metric, d):
    return instances(r"scan_kernel<%d, true, %d, %d, (?:true|false), %d>" % (group, waves, METRIC[metric], d))


@pytest.mark.parametrize("group", range(3, 8))
def test_two_workgroups_of_the_squared_difference_scan_fit_a_compute_unit(group):
    """Sixteen waves each, d = 128: 64 vector registers."""
    for name, k in fused_scans(group, 16, "squared differences", 128).items():
        assert k.vgprs <= 64 and k.scratch == 0, (name, k)


@pytest.mark.parametrize("metric,d,groups,waves", [("three bits", 128, "[3-8]", 6), ("method", 192, "[2-8]", 6), ("squared differences", 192, "[2-7]", 6)])
def test_three_workgroups_of_the_scan_of_query_codes_fit_a_compute_unit(metric, d, groups, waves):
    """Eight waves each: query planes in scalar registers where they would cost the third workgroup."""
    for name, k in instances(r"scan_kernel<%s, false, 8, %d, false, %d>" % (groups, METRIC[metric], d)).items():
        assert R.waves_per_simd(k) >= waves and k.scratch == 0, (name, k)


def test_two_workgroups_of_the_one_bit_scan_of_query_codes_fit_a_compute_unit():
    """Sixteen waves each, d = 192, groups of six to eight: 64 vector registers."""
    for name, k in instances(r"scan_kernel<[678], false, 16, %d, false, 192>" % METRIC["one bit"]).items():
        assert k.vgprs <= 64 and k.scratch == 0, (name, k)


def test_four_workgroups_of_the_smallest_scans_fit_a_compute_unit():
    """Four waves each, the planes of a pass's heads all at once (three at d = 256 with three-bit codes)."""
    for name, k in instances(r"scan_kernel<\d, false, 4, \d, false, \d+>").items():
        assert R.waves_per_simd(k) >= (3 if name.endswith(", 3, false, 256>") else 4) and k.scratch == 0, (name, k)


@pytest.mark.parametrize("group", range(2, 8))
def test_two_workgroups_of_the_three_bit_scan_fit_a_compute_unit(group):
    """Eight waves each, d = 256: 128 vector registers.  And groups of two at d = 64: 80 scalar registers for eight waves per SIMD."""
    for name, k in fused_scans(group, 8, "three bits", 256).items():
        assert k.vgprs <= 128 and k.scratch == 0, (name, k)
    if group == 2:
        for name, k in fused_scans(2, 16, "three bits", 64).items():
            assert k.vgprs <= 64 and k.sgprs <= 80 and k.scratch == 0, (name, k)


def test_the_one_launch_is_built_without_spills_and_where_the_rule_can_ask_for_it():
    for name, k in instances(r"one_launch_kernel<.*>").items():
        assert k.spilled == 0 and k.scratch == 0, (name, k)
    assert not [n for n in R.kernels() if re.fullmatch(r"one_launch_kernel<16, true, 3, \w+, 256>", n)]
