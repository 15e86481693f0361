"""The binding's launch path: the entry points it calls once per launch have
plain C argument types (converted without Python code), so their callers check
the 32-bit ranges themselves; the rest of their signature is that of the
checked entry points, and the library's own validation answers through them
(no GPU is touched: every call here is refused or empty)."""
import ctypes

import pytest
import torch

import paper_2308_15152_amd as pkg


def test_plain_entry_points_match_the_checked_ones():
    lib = pkg.load()
    assert len(pkg._fast) == 6
    for name, fn in pkg._fast.items():
        checked = getattr(lib, name)
        assert fn is not checked
        assert len(fn.argtypes) == len(checked.argtypes)
        for a, b in zip(fn.argtypes, checked.argtypes):
            assert ctypes.sizeof(a) == ctypes.sizeof(b)


def test_validation_through_the_plain_entry_points():
    pkg.load()
    one, two, three = 1 << 20, 1 << 22, 1 << 24
    st = pkg.Stride(0, 0, 0)
    gemm = pkg._fast["sgemm_emu_batched"]
    assert gemm(-1, 4, 4, one, 4, two, 4, three, 4, 1, st, None) == -1
    assert gemm(4, 4, 4, one, 3, two, 4, three, 4, 1, st, None) == -2
    assert gemm(4, 4, 4, one, 4, two, 4, None, 4, 1, st, None) == -3
    assert gemm(4, 4, 4, one, 4, two, 4, one, 4, 1, st, None) == -5
    assert gemm(0, 4, 4, None, 4, None, 4, None, 4, 1, st, None) == 0
    acc = pkg._fast["sgemm_emu_batched_acc"]
    st4 = pkg.Stride4(0, 0, 0, 0)
    assert acc(2, 0, 0, 4, 4, 4, one, 4, two, 4, None, 4, three, 4, 1, st4, 1, 1, None) == -8
    assert acc(0, 1, 0, 4, 4, 4, one, 4, two, 4, one, 4, one, 4, 1, st4, 1, 1, None) == -5
    assert pkg._fast["sgemm_emu_scan"](2, 8, one, 7, two, 8, None) == -2
    assert pkg._fast["householder_emu_batched_ex"](32, one, 32, two, 4, 0, 4, three, 4, 0, 1, 0,
                                                   None) == -6
    assert pkg._fast["givens_emu_batched"](64, 3, 3, one, one, 1, two, 4, 0, 4, three, 4, 0, 1, 0,
                                           None) == -1


def test_out_of_range_integers_are_refused():
    pkg._check_ints(0, -(1 << 31), (1 << 31) - 1)
    for bad in ((1 << 31), -(1 << 31) - 1, (1 << 32) + 8):
        with pytest.raises(ctypes.ArgumentError):
            pkg._check_ints(4, bad)


class _OnDevice:
    """A host tensor that passes for a device tensor where only its type,
    shape and strides are looked at."""

    is_cuda = True

    def __init__(self, t):
        self.t = t

    def __getattr__(self, name):
        return getattr(self.t, name)

    def unsqueeze(self, dim):
        return _OnDevice(self.t.unsqueeze(dim))


def test_output_forms_of_a_product():
    """C may be 3-D, 2-D (one item) or, for one row, a contiguous vector;
    anything else is refused."""
    A, B = _OnDevice(torch.zeros(1, 8)), _OnDevice(torch.zeros(8, 5))
    for C in (torch.zeros(5), torch.zeros(1, 5), torch.zeros(1, 1, 5)):
        m, n, k, lda, ldb, ldc, batch, st, out = pkg._gemm_args(A, B, _OnDevice(C))
        assert (m, n, k, batch, ldc, st.c) == (1, 5, 8, 1, 5, 0)
    for C in (torch.zeros(4), torch.zeros(()), torch.zeros(2, 5), torch.zeros(10)[::2],
              torch.zeros(1, 1, 1, 5)):
        with pytest.raises(ValueError):
            pkg._gemm_args(A, B, _OnDevice(C))
    two = _OnDevice(torch.zeros(2, 8))
    with pytest.raises(ValueError):
        pkg._gemm_args(two, B, _OnDevice(torch.zeros(5)))
