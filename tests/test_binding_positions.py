"""The position lists of a pairwise call as the binding passes them (host code only)."""

import ctypes

import numpy as np
import pytest

from paper_2212_04749_amd import binding as B

LISTS = ([3, 0], [1, 2, 4], [0, 2, 3], [1], [0, 2], [1])  # A m, A k, B k, B n, C m, C n
SIZES = (2, 3, 3, 1, 2, 1)


def read(*lists):
    keep, nm, nn, nk, at = B._positions(*lists)
    assert (nm, nn, nk) == (2, 1, 3)
    return [(ctypes.c_int * n).from_address(a)[:] for n, a in zip(SIZES, at)]


@pytest.mark.parametrize("form", [list, tuple, np.array, lambda x: np.array(x, dtype=np.float64),
                                  lambda x: [float(v) for v in x], lambda x: [np.int64(v) for v in x]])
def test_lists_of_any_kind(form):
    assert read(*(form(x) for x in LISTS)) == list(LISTS)


@pytest.mark.parametrize("which", [2, 4, 5])
def test_surplus_entries_are_ignored(which):
    lists = [list(x) + ([7, 9] if i == which else []) for i, x in enumerate(LISTS)]
    assert read(*lists) == list(LISTS)


@pytest.mark.parametrize("which", [2, 4, 5])
def test_missing_entries_are_refused(which):
    lists = [list(x)[:-1] if i == which else x for i, x in enumerate(LISTS)]
    with pytest.raises(B.MatncError) as e:
        B._positions(*lists)
    assert e.value.code == B.MATNC_E_INVALID


def test_numbers_beyond_32_bits_are_left_to_the_library():
    with pytest.raises(B.MatncError) as e:
        B.matnc_contract_noalloc(0x1000, 0x1000, 0x1000, 1, [0], [1], [0], [1], [1 << 40 | 7], [1], 0, 0)
    assert e.value.code == B.MATNC_E_INVALID  # 7 is no position of a rank-2 tensor
