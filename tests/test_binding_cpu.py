"""The native argument marshalling takes only what the ctypes path takes (CPU only: no call here
gets as far as a launch)."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2604_16395_amd as s2l
from paper_2604_16395_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


def test_plain_arguments_are_marshalled_natively():
    """Every native function takes plain arguments as far as the library's own checks (which refuse
    these), and holds no reference to them afterwards."""
    native = s2l._load_native()
    batch = s2l.Batch([16, 0], [4, 3], np.zeros((2, 2), np.int32), device="cpu")
    row, q = (torch.empty((7, h, 128), dtype=torch.bfloat16) for h in (2, 8))
    lse, ws, scale = torch.empty((7, 8)), torch.empty(1 << 10, dtype=torch.uint8), torch.ones(2)
    bf16 = torch.empty((2, 2, 32, 128), dtype=torch.bfloat16)      # pages of 32 tokens: not supported
    caches = [s2l.PagedKVCache(bf16, bf16), s2l.PagedKVCache(bf16.view(torch.uint8)[..., :128].contiguous(),
                                                             bf16.view(torch.uint8)[..., :128].contiguous(), scale, scale)]
    info, opts = s2l.s2l_plan_info(), s2l.plan_opts(target_items=4)
    for cache in caches:
        args = [cache, batch, row, q, lse, ws, info, opts]
        before = [sys.getrefcount(a) for a in args]
        for _ in range(50):
            assert native.append(cache, batch, row, row, 0) == -4
            assert native.plan(batch, 8, 3, opts, ws, info, 0) == -1 and native.plan(batch, 8, 3, None, ws, info, 0) == -1
            assert native.attn(0, cache, batch, q, 8, 0.1, q, lse, info, ws, 0) == -4
            assert native.fused(cache, batch, q, 8, 0.1, q, None, info, ws, 0, row, row) == (-4, False)
            assert native.reduce(batch, 8, q, lse, info, ws, 0) == -1
            assert native.append(cache, batch, row, None, 0) is None and native.attn(3, *args) is None
        assert [sys.getrefcount(a) for a in args] == before


def test_a_torch_without_gpu_functions_still_gets_the_library(monkeypatch):
    """Where torch has no device and stream functions, calls with a stream of their own reach the
    library, and the others fail where torch is asked for its current stream."""
    batch = s2l.Batch([16], [4], np.zeros((1, 2), np.int32), device="cpu")
    ws = torch.empty(1 << 10, dtype=torch.uint8)
    try:
        for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
            monkeypatch.delattr(torch._C, name, raising=False)
        monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
        s2l._native = None
        with pytest.raises(s2l.S2LError, match="not a multiple"):
            s2l.s2l_attn_plan(batch, 8, 3, ws, None, 0)
        assert s2l._load_native().plan(batch, 8, 3, None, ws, s2l.s2l_plan_info(), None) is None
    finally:   # the module holds what it was set up with
        monkeypatch.undo()
        s2l._native = None
        s2l._load_native()


def test_without_the_native_module_every_call_goes_through_ctypes():
    """An interpreter that the module was not built for gets a warning and the ctypes path, with the
    same results and errors."""
    code = """
import sys, warnings
import numpy as np, torch
sys.modules["paper_2604_16395_amd._binding"] = None      # as a missing file: ImportError
import paper_2604_16395_amd as s2l
batch = s2l.Batch([16], [4], np.zeros((1, 2), np.int32), device="cpu")
ws = torch.empty(1 << 16, dtype=torch.uint8)
row = torch.empty((4, 2, 128), dtype=torch.bfloat16)
pages = torch.empty((2, 2, 16, 128), dtype=torch.bfloat16)
q, lse = torch.empty((4, 8, 128), dtype=torch.bfloat16), torch.empty((4, 8))
cache, info = s2l.PagedKVCache(pages, pages), s2l.s2l_plan_info()
calls = [lambda: s2l.s2l_attn_plan(batch, 8, 3, ws, None, 0), lambda: s2l.s2l_kv_append(cache, batch, None, row, 0),
         lambda: s2l.s2l_chunk_prefill_attn(cache, batch, q, 8, 0.1, q, lse, info, ws, 0),
         lambda: s2l.s2l_append_chunk_prefill_attn(cache, batch, row, row, q, 8, 0.1, q, lse, info, ws, 0),
         lambda: s2l.s2l_split_reduce(batch, 8, q, lse, info, ws, 0)]
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    for f in calls:
        try:
            f()
        except s2l.S2LError as e:
            print(e)
assert [w.category for w in seen] == [RuntimeWarning], seen
"""
    env = {k: v for k, v in os.environ.items() if k != "S2L_LIBRARY"}   # which may have a module beside it
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    said = p.stdout.strip().splitlines()
    assert len(said) == 5 and all("failed: " in l for l in said), p.stdout
    assert "not a multiple" in said[0] and "k_new/v_new is NULL" in said[1] and "another batch" in said[2]


def test_build_without_python_headers_leaves_the_library(monkeypatch, tmp_path):
    """No Python.h: no module, a warning, and none of an earlier build is left behind."""
    from paper_2604_16395_amd import build
    stale = tmp_path / "_binding.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "BINDING", str(stale))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    with pytest.warns(UserWarning, match="no Python.h"):
        assert build.build_binding() is None
    assert not stale.exists()
