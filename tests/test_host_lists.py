"""Limits of the matrix filter's closed-form work lists (CPU only): the host
arithmetic of csrc/lists.h, compiled by itself, against plain sums at both
sides of 32-bit entry numbers, and the rule that takes such a list in place
of a traversal.  No list of these sizes is made."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2510_14147_amd", "csrc")
WRAP = """
#include "lists.h"
using namespace fnn;
extern "C" {
long long entries(long long np) { return dense_entries(np); }
int fits(long long np) { return dense_fits(np); }
int rule(long long n, double c) { return dense_rule(n, n / 40 + 1, c, false); }
int sampled(long long n, long long np, double c, double gone)
{
    return dense_sampled(n, np, c, false, gone);
}
int wide_rule(long long n, long long np, double c) { return dense_rule(n, np, c, true); }
int wide_sampled(long long n, long long np, double c, double gone)
{
    return dense_sampled(n, np, c, true, gone);
}
}
"""


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    d = tmp_path_factory.mktemp("lists")
    (d / "wrap.cpp").write_text(WRAP)
    so = str(d / "wrap.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I", CSRC,
                    str(d / "wrap.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.entries.restype = ctypes.c_longlong
    L.entries.argtypes = L.fits.argtypes = [ctypes.c_longlong]
    L.rule.argtypes = [ctypes.c_longlong, ctypes.c_double]
    L.sampled.argtypes = L.wide_sampled.argtypes = [
        ctypes.c_longlong, ctypes.c_longlong, ctypes.c_double, ctypes.c_double]
    L.wide_rule.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_double]
    return L


@pytest.mark.parametrize("np_", [1, 2, 3, 4, 5, 63, 64, 65, 1000, 1023, 15625])
def test_entries(lists, np_):
    assert lists.entries(np_) == sum(np_ - 4 * g for g in range((np_ + 3) // 4))


def test_limit(lists):
    top = max(p for p in range(130000, 132000) if lists.fits(p))
    assert lists.entries(top) < 2**31 - 4096 <= lists.entries(top + 1)
    assert not any(lists.fits(p) for p in range(top + 1, top + 2000))
    assert all(lists.fits(p) for p in range(top - 2000, top + 1))
    # rows in full packs, and the sizes beyond (10M and 2^31 - 1 rows)
    assert top == 131069
    assert not lists.fits(-(-10_000_000 // 64)) and not lists.fits(-(-(2**31 - 1) // 64))


NO, YES, SAMPLE = 0, 1, 2
PRICES = [4.6e-11, 5.7e-11, 8.5e-11, 1.15e-10, 2.5e-10]  # ms per screened pair


@pytest.mark.parametrize("c", PRICES)
def test_rule_never_takes_a_list_without_numbers(lists, c):
    last = 131069 * 64
    assert lists.rule(last, c) == SAMPLE
    for n in (last + 1, 10_000_000, 100_000_000, 2**30, 2**31 - 1):
        # what the tree prunes would be worth less than the traversal
        assert lists.sampled(n, n // 40, c, 0.2) or n > 2**30
        assert lists.rule(n, c) == NO, n


@pytest.mark.parametrize("c", PRICES)
def test_rule_counts_full_packs_not_the_tree_s(lists, c):
    # one point to a pack: the tree's own packs have no list, full ones do
    n = 140_000
    assert not lists.fits(n) and lists.fits(-(-n // 64))
    assert lists.rule(n, c) in (YES, SAMPLE)
    # small sets take the list without a sample
    assert lists.rule(1, c) == lists.rule(20_000, c) == YES
    assert lists.rule(0, c) == NO


@pytest.mark.parametrize("c", PRICES)
def test_sample_decides_by_what_it_prunes(lists, c):
    n, np_ = 1_000_000, 20_000
    take = [lists.sampled(n, np_, c, g / 100) for g in range(101)]
    assert take[0] and not take[100]
    assert take == sorted(take, reverse=True)


@pytest.mark.parametrize("c", PRICES)
def test_wide_margins_take_every_pair_only_where_none_is_prunable(lists, c):
    for n in (1, 1000, 20_000, 1_000_000):
        assert lists.wide_rule(n, 255, c) == NO
        assert lists.wide_rule(n, 256, c) == SAMPLE
        assert lists.wide_sampled(n, 256, c, 0.01)
        assert not lists.wide_sampled(n, 256, c, 0.011)
    assert lists.wide_rule(10_000_000, 200_000, c) == NO
