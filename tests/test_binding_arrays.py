"""Host arguments on their way to the library: every kind of sequence of numbers gives the same C array, every way to name a
stream its handle."""
import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def b():
    from paper_2601_20499_amd import binding
    return binding


@pytest.mark.parametrize("make", [list, tuple, np.array, torch.tensor, lambda v: [float(x) for x in v],
                                  lambda v: [np.int64(x) for x in v], lambda v: [torch.tensor(x) for x in v],
                                  lambda v: [str(x) for x in v], lambda v: np.array(v, dtype=np.float64)])
def test_arrays_of_whole_numbers(b, make):
    for v in ([], [0], [1, 2, 3], list(range(64)), [2**31 - 1, 5]):
        if v or make is not torch.tensor:
            assert b._i32(make(v))[:] == v and b._i64(make(v))[:] == v


def test_numbers_beyond_the_type_and_no_numbers(b):
    assert b._i32([2**31, -2**31 - 1])[:] == [-2**31, 2**31 - 1]      # as ctypes wraps them
    for xs in ([None], ["x"], [[1]]):
        with pytest.raises((TypeError, ValueError)):
            b._i32(xs)


@pytest.mark.parametrize("make", [lambda F: F, tuple, np.array, torch.tensor, lambda F: iter(F), lambda F: [iter(r) for r in F],
                                  lambda F: [[str(x) for x in r] for r in F]])
def test_classify_takes_any_rows(b, make):
    F = [[0.5, 0.25, 0.25], [0.125, 0.5, 0.375], [0.0625, 0.0625, 0.875]]
    assert b.df_classify(make(F), 1, b.DF_CLASSIFY_TWO_CLASS) == b.df_classify(F, 1, b.DF_CLASSIFY_TWO_CLASS)


def test_classify_refuses_rows_that_are_too_long(b):
    with pytest.raises(IndexError):
        b.df_classify([[0.5, 0.25, 0.25, 0.0]], 0, b.DF_CLASSIFY_TWO_CLASS)


@pytest.mark.parametrize("fast", [True, False])
def test_current_stream_with_and_without_the_raw_handle(b, monkeypatch, fast):
    """The raw handle of the current stream comes from a function that torch need not have."""
    class Stream:
        cuda_stream = 0x1230
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    if fast:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x4560 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert b._stream_handle(None) == (0x4563 if fast else 0x1230)
    assert b._stream_handle(Stream) == 0x1230 and b._stream_handle(7) == 7 and b._stream_handle(0) is None
