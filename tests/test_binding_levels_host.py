"""The workspace size that the binding looks up for a call, for every kind of
level count the C entry points take: what a size is kept for is the number
itself, not the object that held it."""
import ctypes

import numpy as np
import pytest

import paper_1705_08266_amd as dwt

torch = pytest.importorskip("torch")


def _expect(levels):
    return dwt.workspace_bytes(64, 128, levels) // 4


def test_numbers():
    for levels in (1, 2, 3, 2, 1):
        assert dwt._workspace_size(64, 128, levels) == _expect(levels)


def test_objects_that_stand_for_a_number():
    assert dwt._workspace_size(64, 128, np.int64(3)) == _expect(3)
    assert dwt._workspace_size(64, 128, np.array(3)) == _expect(3)      # not hashable
    for held in (torch.tensor(2), ctypes.c_int32(2)):
        assert dwt._workspace_size(64, 128, held) == _expect(2)
        if isinstance(held, torch.Tensor):
            held.fill_(3)
        else:
            held.value = 3
        assert dwt._workspace_size(64, 128, held) == _expect(3)          # the value it has now


def test_what_was_refused_stays_refused():
    dwt._workspace_size(64, 128, 2)
    for bad in (2.0, "2", None):
        with pytest.raises(ctypes.ArgumentError):
            dwt._workspace_size(64, 128, bad)


def test_sizes_kept_are_bounded():
    for k in range(1, 3 * dwt._CACHE_MAX):
        assert dwt._workspace_size(2 * k, 64, 1) == 0
    assert len(dwt._workspace_floats) <= dwt._CACHE_MAX
