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


@pytest.mark.parametrize("missing", ["block_tables", "dir", "cls", "ctx_lens"])
@pytest.mark.parametrize("half", ["until", "from"])
def test_halves_of_a_batch_refuse_missing_metadata(monkeypatch, missing, half):
    # what a view of the half's rows refuses is not taken for "by class"
    monkeypatch.setattr(bros, "LIB", type("Calls", (), {"bros_attn_prefill_chunk": staticmethod(lambda *a: 0),
                                                        "bros_attn_decode": staticmethod(lambda *a: 0)}))
    pool = torch.zeros(4, 2, 16, 128)
    meta = {"block_tables": torch.zeros(3, 4, dtype=torch.int32), "dir": torch.ones(3, dtype=torch.int8),
            "cls": torch.zeros(3, dtype=torch.uint8), "ctx_lens": torch.ones(3, dtype=torch.int32)}
    q = torch.zeros(2, 4, 128)

    def call(m):
        if half == "from":
            bros.attn_decode_from(1, q, q, pool, pool, *m.values(), 4, stream=0)
        else:
            bros.attn_prefill_until(2, q, q, torch.zeros(3, dtype=torch.int32), 1, pool, pool, *m.values(), 4, stream=0)

    call(meta)
    with pytest.raises((TypeError, AttributeError)):
        call({**meta, missing: None})


def test_stream_handles_pass_through():
    assert bros._stream(0) == 0 and bros._stream(1234) == 1234
