"""The binding's argument gathering, without a GPU: what reaches the C call."""
from collections import deque

import numpy as np
import pytest

from paper_1910_10032_amd import binding as B


class Recorder(B.WfstDecoder):
    def __init__(self):
        self.h, self.calls = None, []

    def advance_ptrs(self, *args):
        self.calls.append(args)


@pytest.mark.parametrize("n", [1, 7, 8, 20])                 # (from 8 lanes on, tensors are gathered attribute by attribute)
@pytest.mark.parametrize("kind", [list, tuple, iter, lambda x: (i for i in x), deque, lambda x: dict(enumerate(x)).values()])
def test_advance_takes_any_iterable(n, kind):
    pairs = [(1000 + i, 40 + i) for i in range(n)]
    dec = Recorder()
    dec.advance(range(n), kind(pairs), n_frames=deque(range(5, 5 + n)), stream=0)
    channels, ptrs, strides, frames, stream, every = dec.calls[0]
    assert channels.tolist() == list(range(n)) and ptrs.tolist() == [p for p, _ in pairs]
    assert strides.tolist() == [s for _, s in pairs] and frames.tolist() == list(range(5, 5 + n)) and (stream, every) == (0, 0)
    assert [a.dtype for a in (channels, ptrs, strides, frames)] == [np.int32, np.uint64, np.int32, np.int32]


@pytest.mark.parametrize("n", [3, 12])
def test_advance_refuses_a_wrong_number_of_lanes(n):
    with pytest.raises(AssertionError):
        Recorder().advance(range(n), iter([(1, 2)] * (n - 1)), n_frames=[1] * n, stream=0)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [7, 9])
def test_advance_takes_any_iterable_of_tensors(n):
    import torch
    rows = [torch.zeros((4 + i % 2, 10), device="cuda")[:, :8] for i in range(n)]
    for frames, want in ((None, [4 + i % 2 for i in range(n)]), (deque([1] * n), [1] * n), (range(n + 3), list(range(n)))):
        dec = Recorder()
        dec.advance(range(n), (t for t in rows), n_frames=frames, stream=0)
        _, ptrs, strides, got, _, _ = dec.calls[0]
        assert ptrs.tolist() == [t.data_ptr() for t in rows] and strides.tolist() == [10] * n and got.tolist() == want
