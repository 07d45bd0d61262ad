"""Row offsets of the attention calls on their way to the C ABI: whatever sequence of numbers they come as."""
import numpy as np
import pytest
import torch

from paper_2511_21317_amd.binding import _row_offsets

WANT = [0, 3, 7, 1 << 40]


@pytest.mark.parametrize("rows", [WANT, tuple(WANT), np.array(WANT), torch.tensor(WANT), [float(x) for x in WANT], [str(x) for x in WANT],
                                  [np.int64(x) for x in WANT], iter(WANT)],
                         ids=["list", "tuple", "numpy", "torch", "floats", "texts", "numpy_ints", "iterator"])
def test_any_sequence_of_numbers_is_taken(rows):
    a = _row_offsets(rows, 4)
    assert a.typecode == "q" and a.itemsize == 8 and list(a) == WANT


def test_the_length_is_that_of_the_call():
    assert list(_row_offsets([0, 5], 4)) == [0, 5, 0, 0]
    with pytest.raises(IndexError):
        _row_offsets([0, 1, 2], 2)
    with pytest.raises((TypeError, ValueError)):
        _row_offsets([0, None], 2)
