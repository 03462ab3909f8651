"""The library's integer layout and launch rules (csrc/tmm_rules.hpp), compiled for the host."""

import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1410_0204_amd", "csrc")

SHIM = r"""
#include "tmm_rules.hpp"
extern "C" {
int bins_halo(int rows) { return tmm::bins_halo(rows); }
int most_groups(int sweep, int member_kernel, int ntr, int sub, int deep, int lanes, int n) {
    return tmm::most_groups((tmm::Sweep)sweep, member_kernel, ntr, sub, deep, lanes, n);
}
int poll_pause(int sub, int lanes, int ntr, int workgroups, int tangent, int reverse) {
    return tmm::poll_pause(sub, lanes, ntr, workgroups, tangent, reverse);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, out = d / "rules.cpp", d / "librules.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", str(out),
                    str(src)], check=True)
    return ctypes.CDLL(str(out))


@pytest.mark.parametrize("ntr", [1, 2, 3])
def test_binned_lds_buffers_start_on_16_bytes(rules, ntr):
    """The binned kernels keep two buffers one after the other in LDS and access their cells as 16-byte
    vectors: whatever the halo of a grid's domains, a buffer holds it and ends on 16 bytes."""
    for halo in range(0, 513):
        assert halo <= rules.bins_halo(halo) <= 512
        assert (256 + rules.bins_halo(halo)) * ntr * 8 % 16 == 0, halo


def test_poll_pause_goes_by_the_launch(rules):
    """A launch of few workgroups (one member of a 12-domain grid) pauses briefly before its first poll,
    whatever number of members its handle could hold; one of many (21 members of that grid) longer."""
    assert [rules.poll_pause(0, 16, 2, g, 0, 0) for g in (1, 12, 63, 64, 252)] == [3, 3, 3, 7, 7]
    assert [rules.poll_pause(0, 16, 3, g, 0, 0) for g in (12, 252)] == [3, 9]
    assert [rules.poll_pause(0, 32, 2, g, 0, 0) for g in (12, 252)] == [3, 4]
    assert [rules.poll_pause(0, lanes, 2, 252, 1, 0) for lanes in (16, 32)] == [6, 2]
    assert [rules.poll_pause(0, lanes, 2, 252, 0, 1) for lanes in (16, 32)] == [6, 2]
    assert [rules.poll_pause(0, 16, 2, 12, t, r) for t, r in ((1, 0), (0, 1))] == [0, 1]
    assert all(rules.poll_pause(1, 16, 2, g, t, r) == 0 for g in (12, 252) for t in (0, 1) for r in (0, 1))


FORWARD, TANGENT, REVERSE = 0, 1, 2

# (sweep, tracers, internal steps, more than 16 layers, groups, faster as single launches) as measured on
# grids of 52000 points whose members run one per group in the packed layout
PACKED = [
    (TANGENT, 1, 0, 1, 40, True), (TANGENT, 1, 0, 1, 64, False), (TANGENT, 1, 0, 0, 40, True), (TANGENT, 1, 0, 0, 64, False),
    (REVERSE, 1, 0, 1, 8, True), (REVERSE, 1, 0, 1, 25, False), (REVERSE, 1, 0, 0, 25, True), (REVERSE, 1, 1, 1, 25, True),
    (TANGENT, 2, 0, 1, 8, True), (TANGENT, 2, 0, 1, 40, False), (TANGENT, 2, 1, 1, 24, False), (TANGENT, 2, 0, 0, 64, True),
    (REVERSE, 2, 0, 1, 12, True), (REVERSE, 2, 0, 1, 18, False), (REVERSE, 2, 0, 0, 12, True), (REVERSE, 2, 0, 0, 18, False),
    (REVERSE, 2, 1, 1, 18, True), (TANGENT, 3, 0, 1, 4, True), (TANGENT, 3, 0, 1, 8, False), (TANGENT, 3, 0, 1, 24, False),
    (TANGENT, 3, 1, 1, 24, True), (TANGENT, 3, 0, 0, 64, True), (REVERSE, 3, 0, 1, 11, True), (FORWARD, 3, 0, 1, 64, True)]


@pytest.mark.parametrize("sweep,ntr,sub,deep,groups,faster", PACKED)
def test_wide_batches_take_the_faster_kernels(rules, sweep, ntr, sub, deep, groups, faster):
    assert (groups <= rules.most_groups(sweep, int(ntr < 3), ntr, sub, deep, 0, 52000)) == faster


def test_batches_in_bins(rules):
    """In bins single launches were faster at every width measured; years of one or two tracers go over to
    the member kernel."""
    for lanes in (16, 32):
        assert all(rules.most_groups(s, 1, ntr, sub, d, lanes, 52000) >= 64
                   for s in (TANGENT, REVERSE) for ntr in (1, 2, 3) for sub in (0, 1) for d in (0, 1))
        assert rules.most_groups(FORWARD, 0, 3, 0, 0, lanes, 52000) >= 64
        assert [rules.most_groups(FORWARD, 1, 2, 0, 0, lanes, n) for n in (2700, 17000, 52749)] == [6, 7, 11]
    assert rules.most_groups(FORWARD, 1, 2, 0, 0, 0, 52749) == 4
