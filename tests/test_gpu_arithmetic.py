"""The fit's short reciprocal, quotient and root against the correctly rounded
operations, on the device, over the ranges that tpcca_kf.h states."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "kf_arithmetic.hip")
LIB = os.path.join(HERE, "native", "libkfarithmetic.so")


def build():
    """Compile the checks with the library's own flags."""
    from paper_1709_00618_amd import build as b
    subprocess.check_call([b._hipcc(), *b.HIPFLAGS, "-shared", "-o", LIB + ".tmp", SRC])
    os.replace(LIB + ".tmp", LIB)
    return LIB


@pytest.mark.gpu
@pytest.mark.parametrize("what, checks", [
    ("reciprocal", 2 ** 23 * 245),  # every significand, exponents -122 to 122
    ("inverse", 2 ** 32),           # every float
    ("root", 2 ** 23 * 217),        # every float from 2^-96 to below 2^121
    ("quotient", 2 ** 31),          # random pairs, significands of many equal bits among them
    ("special", 64 + 8),            # zeros, infinities, NaN and numbers against each other
])
def test_short_forms_are_correctly_rounded(what, checks):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert os.path.exists(LIB), "run __graft_entry__.build() first"
    L = ctypes.CDLL(LIB)
    f = getattr(L, "check_" + what)
    done, wrong = ctypes.c_uint64(), ctypes.c_uint64()
    assert f(ctypes.byref(done), ctypes.byref(wrong)) == 0
    assert (done.value, wrong.value) == (checks, 0)
