"""Limits of the matrix filter's closed-form work lists (CPU only): the host
arithmetic of csrc/lists.h, compiled by itself, against plain sums at both
sides of 32-bit entry numbers.  No list of these sizes is made."""
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
