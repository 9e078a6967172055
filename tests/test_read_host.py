"""Pad.read's choice of a field, on the host: a name, or anything that converts
to its number."""
import numpy as np
import pytest
import torch

import paper_2606_20426_amd as tc


class Library:
    """Fields of n = 2 + field doubles with the value of the field."""

    def tc_field_info(self, h, f, dtype, count, components):
        dtype._obj.value, count._obj.value, components._obj.value = tc._abi.DT_F64, 2 + f, 1
        return 0

    def tc_pad_read(self, h, f, dst, nbytes, device):
        assert nbytes == 8 * (2 + f)
        np.ctypeslib.as_array((tc._abi.C.c_double * (2 + f)).from_address(dst.value))[:] = f
        return 0


@pytest.fixture
def pad():
    p = object.__new__(tc.Pad)
    p.lib, p.h, p._layouts = Library(), None, {}
    return p


@pytest.mark.parametrize("make", [int, np.int64, np.uint8, np.array, torch.tensor, float])
def test_fields_by_number(pad, make):
    for _ in range(2):
        for f in (0, 3):
            assert np.array_equal(pad.read(make(f)), np.full(2 + f, float(f)))


def test_a_number_that_changes_in_place(pad):
    f = torch.tensor(1)
    assert pad.read(f).size == 3
    f += 1
    assert pad.read(f).size == 4


def test_fields_by_name(pad):
    for name in ("positions", "sigma"):
        assert np.array_equal(pad.read(name), np.full(2 + tc.FIELDS[name], float(tc.FIELDS[name])))
    with pytest.raises(KeyError):
        pad.read("nothing")
