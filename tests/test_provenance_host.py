"""A provenance is 32 bytes or any 32 numbers, one byte each."""
import array

import numpy as np
import pytest

from paper_2609_23664_amd import binding as B

VALUES = [(7 * i + 250) % 256 for i in range(32)]


@pytest.mark.parametrize("make", [bytes, bytearray, list, tuple, lambda v: memoryview(bytes(v)), np.uint8,
                                  np.int64, lambda v: array.array("q", v)],
                         ids=["bytes", "bytearray", "list", "tuple", "memoryview", "uint8", "int64", "array"])
def test_forms(make):
    given = np.array(VALUES, dtype=make) if make in (np.uint8, np.int64) else make(VALUES)
    assert list(B._prov(given)) == VALUES
    t = B.Tableau(3)
    assert t.artifact(given)["provenance"] == bytes(VALUES)


@pytest.mark.parametrize("size", [0, 31, 33])
def test_other_lengths_are_refused(size):
    with pytest.raises(AssertionError):
        B._prov([0] * size)
