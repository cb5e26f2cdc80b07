"""Sizes of the workspace that callers plan with (host code, no GPU)."""
import ctypes as C

import pytest

from paper_2203_15031_amd import spmesl as sp

NOALLOC = 64 << 20


def _size(n, p, prec, data_form=False):
    opt = sp.Context.options(1.0, precision=prec, data_form=data_form)
    prob = sp.Problem(1 << 20, n, p, p)
    sz = C.c_size_t()
    assert sp.load().spmesl_workspace_size(C.byref(prob), C.byref(opt), C.byref(sz)) == 0
    return sz.value


# mixed problems at the edge of what spmesl_solve_noalloc's fixed array took
# when the split was stored variable by variable: the operand order pads it to
# blocks of 16 variables, which must cost no call its place
@pytest.mark.parametrize("n,p", [(441336, 2), (408982, 3), (356678, 5), (299244, 8), (209228, 16), (201632, 17),
                                 (127424, 33), (101606, 44), (73112, 65), (45173, 100), (33663, 129), (20509, 200),
                                 (7372, 500), (3648, 1000), (1912, 1500), (1024, 2048), (735, 2300)])
def test_noalloc_still_holds(n, p):
    assert _size(n, p, "mixed") <= NOALLOC


# the data form's, with the slices of 128 workgroups: more workgroups share them
@pytest.mark.parametrize("n,p,size", [(400, 2048, 1166213296), (400, 2500, 1169961648), (60, 4096, 1157431472),
                                      (400, 5000, 1190681264), (33, 20000, 1205147056),
                                      (2000, 100000, 3853854384), (50, 1000000, 4311505072)])
def test_data_form_workspace(n, p, size):
    assert _size(n, p, "fp64", data_form=True) <= size
