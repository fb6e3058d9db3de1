"""The packed call arguments of the binding hold the same bytes as the ctypes structures of the C header."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2602_14516_amd.binding as b


@pytest.mark.parametrize("scale", [0.125, 1e300])               # (1e300: past a C float, only the structure converts it)
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("n", [0, 1, 5])
def test_packed_arguments_equal_the_structures(n, fp8, scale):
    k, v = torch.zeros(7, 2, 16, 64, dtype=torch.uint8), torch.zeros(7, 2, 16, 64, dtype=torch.uint8)
    ks = torch.ones(7, 2) if fp8 else None
    c = b.KVCache(8, 2, 64, 16, k, v, scale, ks, ks, b.AMPD_KV_FP8_E4M3 if fp8 else b.AMPD_KV_BF16)
    arg = b._cache_arg(c)
    want = bytes(c.c_struct())
    got = arg if isinstance(arg, bytes) else bytes(arg._obj)
    assert len(want) == ctypes.sizeof(b._Cache) and got == want

    table = torch.zeros(n, 3, dtype=torch.int32)
    for writable in (True, False):                              # a read-only array's address comes another way
        C, L = np.arange(n, dtype=np.int32), np.ones(n, np.int32)
        C.flags.writeable = L.flags.writeable = writable
        arg, keep = b._batch_arg(C, L, table)
        s, _ = b._batch(C, L, table)
        got = b._Batch.from_buffer_copy(arg)
        assert len(arg) == ctypes.sizeof(b._Batch)
        assert [getattr(got, f) for f, _ in b._Batch._fields_] == [getattr(s, f) for f, _ in b._Batch._fields_]


def test_the_library_s_own_functions_check_the_structures():
    cache = b.KVCache(8, 2, 64, 16, None, None, 0.125).c_struct()
    batch, keep = b._batch([100, 5], [1, 7], None, max_pages=8)
    want = b.lib.ampd_workspace_bytes(ctypes.byref(cache), ctypes.byref(batch))
    assert want > 0
    assert b.lib.ampd_workspace_bytes(cache, batch) == want                 # a structure itself, as a POINTER argument takes it
    assert b.lib.ampd_workspace_bytes(ctypes.pointer(cache), ctypes.pointer(batch)) == want
    for wrong in ((ctypes.byref(batch), ctypes.byref(cache)), (batch, cache), (bytes(cache), bytes(batch)), (cache, 64)):
        with pytest.raises(ctypes.ArgumentError):
            b.lib.ampd_workspace_bytes(*wrong)
    assert b._packed.ampd_workspace_bytes(bytes(cache), bytes(batch)) == want
