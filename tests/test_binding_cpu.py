"""The native argument marshalling takes only what the ctypes path takes (CPU only: no call here
gets as far as a launch)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2604_16395_amd as s2l
from paper_2604_16395_amd import _lib


class _LooksLikeStream:
    cuda_stream = 0


class _SameSize(ctypes.Structure):
    _fields_ = [("x", ctypes.c_char * ctypes.sizeof(_lib.s2l_plan_opts))]


@pytest.mark.parametrize("opts", [bytearray(ctypes.sizeof(_lib.s2l_plan_opts)), np.zeros(5, np.int32), _SameSize()])
def test_buffers_that_are_no_plan_structs_are_refused(opts):
    assert ctypes.sizeof(_lib.s2l_plan_opts) == 20
    batch = s2l.Batch([16], [4], np.zeros((1, 2), np.int32), device="cpu")
    ws = torch.empty(1 << 16, dtype=torch.uint8)
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        s2l.s2l_attn_plan(batch, 8, 2, ws, opts, 0)
    out = torch.empty((4, 8, 128), dtype=torch.bfloat16)
    info = bytearray(ctypes.sizeof(_lib.s2l_plan_info))
    with pytest.raises(TypeError):
        s2l.s2l_split_reduce(batch, 8, out, None, info, ws, 0)


def test_objects_that_are_no_streams_are_refused():
    batch = s2l.Batch([16], [4], np.zeros((1, 2), np.int32), device="cpu")
    ws = torch.empty(1 << 16, dtype=torch.uint8)
    with pytest.raises(TypeError):
        s2l.s2l_attn_plan(batch, 8, 2, ws, None, _LooksLikeStream())
