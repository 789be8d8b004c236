"""Host arrays for logits: which of them lie in pinned memory, and that the memory kept locked for them stays below its limit.  Nothing is pinned
here: torch.empty is replaced by one that notes what was asked for."""
import gc

import numpy as np
import pytest

MB = 1 << 20


@pytest.fixture
def pinned(monkeypatch):
    import torch
    from paper_2408_15766_amd import binding
    real, asked = torch.empty, []

    def empty(shape, dtype=None, pin_memory=False):
        if pin_memory:
            if empty.error is not None:
                raise empty.error
            asked.append(4 * shape[0] * shape[1])
        return real(shape, dtype=dtype)
    empty.error = None
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(binding, "_pinned", {})
    monkeypatch.setattr(binding, "_pinned_gone", type(binding._pinned_gone)())
    return binding._host_floats, asked, empty


def test_small_arrays_are_pageable(pinned):
    floats, asked, _ = pinned
    assert floats(1, 1000).shape == (1, 1000) and asked == []
    assert floats(8, MB // 32).dtype == np.float32 and asked == [MB]


def test_the_limit_counts_whole_blocks(pinned):
    # 64 MiB and a few bytes lie in a block of 128: two of these reach the limit
    floats, asked, _ = pinned
    held = [floats(130, 129056) for _ in range(3)]
    assert len(asked) == 2 and all(x.shape == (130, 129056) for x in held)
    del held
    gc.collect()
    held = [floats(130, 129056) for _ in range(3)]             # the blocks that are kept are given out again
    assert len(asked) == 4


def test_blocks_that_are_kept_count_for_arrays_of_other_sizes(pinned):
    floats, asked, _ = pinned
    sizes = [128, 64, 32, 16, 8, 4, 2, 1]                      # 255 MiB, one block each, one array after the other
    for mb in sizes:
        floats(mb, MB // 4)
        gc.collect()
    assert len(asked) == 8
    held = [floats(2, MB // 4), floats(2, MB // 4)]            # a second one of a size would be one block more: 257
    assert len(asked) == 9
    held.append(floats(1, MB // 4))
    held.append(floats(1, MB // 4))                            # 256
    assert len(asked) == 11


def test_a_view_keeps_the_block(pinned):
    floats, asked, _ = pinned
    rows = [floats(128, MB // 4)[3:5], floats(128, MB // 4)[0]]
    gc.collect()
    floats(128, MB // 4)
    assert len(asked) == 2
    del rows
    gc.collect()
    floats(128, MB // 4)
    assert len(asked) == 3


@pytest.mark.parametrize("error", [RuntimeError("no memory"), MemoryError(), KeyboardInterrupt()])
def test_memory_that_cannot_be_pinned(pinned, error):
    floats, asked, empty = pinned
    for _ in range(5):
        empty.error = error
        if isinstance(error, RuntimeError):
            assert floats(128, MB // 4).shape == (128, MB // 4)   # pageable instead
        else:
            with pytest.raises(type(error)):
                floats(128, MB // 4)
    empty.error = None
    held = [floats(128, MB // 4) for _ in range(3)]
    assert len(asked) == 2 and len(held) == 3                  # none of the failed ones counts


def test_the_streams_handle_without_the_private_name(monkeypatch):
    import torch
    from paper_2408_15766_amd import binding

    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream())
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert binding._stream_ptr() == 103 and binding._stream_ptr(Stream()) == 77
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert binding._stream_ptr() == 77
