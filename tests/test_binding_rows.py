"""The binding's row addresses: what a view of the rows would give, and the same refusals."""

import pytest
import torch

from paper_2504_09590_amd import bros


@pytest.mark.parametrize("shape,dtype", [((7,), torch.int8), ((7,), torch.uint8), ((7,), torch.int32),
                                         ((7, 5), torch.int32), ((7, 1), torch.int8), ((7, 3, 2), torch.bfloat16)])
def test_rows_from_is_the_view_s_address(shape, dtype):
    t = torch.zeros(shape, dtype=dtype)
    for first in range(shape[0]):
        assert bros._rows_from(t, first) == t[first:].data_ptr()


def test_rows_from_refuses_what_a_view_refuses():
    with pytest.raises(TypeError):
        bros._rows_from(None, 1)
    with pytest.raises(ValueError):
        bros._rows_from(torch.zeros(4, 6)[:, :3], 1)


def test_stream_handles_pass_through():
    assert bros._stream(0) == 0 and bros._stream(1234) == 1234
