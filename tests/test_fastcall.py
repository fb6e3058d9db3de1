"""The extension module behind the binding's calls fills the same structures as the binding's own path, and leaves every argument of
another kind to that path (a stand-in entry point records what it is given)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2602_14516_amd.binding as b
from paper_2602_14516_amd import _fastcall

VP, I32, SZ = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
KINDS = {10: ctypes.CFUNCTYPE(I32, VP, VP, VP, VP, VP, VP, VP, SZ, VP, VP), 9: ctypes.CFUNCTYPE(I32, VP, VP, I32, I32, VP, VP, VP),
         7: ctypes.CFUNCTYPE(I32, VP, VP, VP, VP, VP)}


@pytest.fixture
def recorder():
    _fastcall.streams(lambda: 0, lambda dev: 0x1230 + dev)
    yield
    b._fastcall = None                                       # the next real call hands torch's functions in again


def _call(args, status=0):
    """(status or None, cache bytes, lengths, rest) of a call whose entry point is the recorder."""
    seen = []

    def record(cache, batch, *rest):
        bt = b._Batch.from_address(batch)
        lens = [np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(I32)), (bt.num_reqs,)).tolist() if bt.num_reqs else [] for p in (bt.h_ctx_len, bt.h_incr_len)]
        seen.append((ctypes.string_at(cache, ctypes.sizeof(b._Cache)), bt.num_reqs, bt.max_pages_per_req, bt.d_block_table, bt.h_block_table, lens, rest))
        return status
    fn = KINDS[len(args) + 1](record)
    return _fastcall.call(ctypes.cast(fn, VP).value, *args), seen


def _usual(fp8=False, n=3):
    k, v = torch.zeros(7, 2, 16, 64, dtype=torch.uint8), torch.zeros(7, 2, 16, 64, dtype=torch.uint8)
    s = torch.ones(7, 2) if fp8 else None
    cache = b.KVCache(8, 2, 64, 16, k, v, 0.125, s, s, b.AMPD_KV_FP8_E4M3 if fp8 else b.AMPD_KV_BF16)
    t = [torch.zeros(4, i + 1) for i in range(5)]
    return [cache, np.arange(n, dtype=np.int32), np.ones(n, np.int32), torch.zeros(n, 3, dtype=torch.int32), *t]


def test_a_table_in_host_memory_takes_the_general_path(recorder):
    st, seen = _call(_usual())
    assert st is None and not seen


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["list", "int64", "strided", "two-dimensional", "unequal", "numpy pool", "subclass", "scale", "no value",
                                  "bool", "past int32", "one-dimensional table"])
def test_other_kinds_take_the_general_path(recorder, what):
    print("case: fastcall", what, flush=True)
    args = _usual()
    args[3] = args[3].cuda()
    if what == "list":
        args[1] = [0, 1, 2]
    elif what == "int64":
        args[1] = np.arange(3)
    elif what == "strided":
        args[2] = np.ones(6, np.int32)[::2]
    elif what == "two-dimensional":
        args[1] = np.zeros((3, 1), np.int32)
    elif what == "unequal":
        args[2] = np.ones(2, np.int32)
    elif what == "numpy pool":
        args[0].k_pool = np.zeros((7, 2, 16, 64), np.uint8)
    elif what == "subclass":
        args[4] = torch.zeros(4).as_subclass(type("T", (torch.Tensor,), {}))
    elif what == "scale":
        args[0].softmax_scale = 1e300
    elif what == "no value":
        args[5] = None
    elif what == "bool":
        args[0].num_kv_heads = True
    elif what == "past int32":
        args[0].page_size = 1 << 40
    elif what == "one-dimensional table":
        args[3] = args[3].reshape(-1)
    st, seen = _call(args)
    assert st is None and not seen


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("n", [0, 1, 5])
def test_the_structures_equal_the_binding_s(recorder, n, fp8):
    print("case: fastcall", n, fp8, flush=True)
    args = _usual(fp8, n)
    args[3] = args[3].cuda()
    args[1].flags.writeable = False
    st, seen = _call(args, status=-2)
    cache, nreq, maxp, table, host, lens, rest = seen[0]
    assert st == -2 and cache == bytes(args[0].c_struct()) and (nreq, maxp, table, host) == (n, 3, args[3].data_ptr() or None, None)
    assert lens == [args[1].tolist(), args[2].tolist()]
    assert [x or 0 for x in rest] == [t.data_ptr() for t in args[4:]] + [args[8].numel() * 4, 0x1230, 0]
    st, seen = _call(args[:4] + [1, 2] + args[4:6])
    assert st == 0 and list(seen[0][6]) == [1, 2, args[4].data_ptr(), args[5].data_ptr(), 0x1230]
    st, seen = _call(args[:6])
    assert st == 0 and list(seen[0][6]) == [args[4].data_ptr(), args[5].data_ptr(), 0x1230]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [10, 9, 7])
@pytest.mark.parametrize("symbol,error", [("_ZSt17__throw_bad_allocv", MemoryError), ("_ZSt20__throw_length_errorPKc", RuntimeError)])
def test_a_cpp_exception_of_the_entry_point_is_raised_once(recorder, symbol, error, n):
    """The entry point throws (a function of the C++ runtime stands in): a Python exception, not None, which would have the binding make
    the call a second time; and the interpreter's lock is held again."""
    print("case: fastcall", symbol, n, flush=True)
    args = _usual()
    args[3] = args[3].cuda()
    rest = {10: args[4:], 9: [0, 1] + args[4:6], 7: args[4:6]}[n]
    entry = ctypes.cast(getattr(ctypes.CDLL("libstdc++.so.6"), symbol), VP).value
    for _ in range(3):
        with pytest.raises(error):
            _fastcall.call(entry, *args[:4], *rest)
    assert _call(args, status=-2)[0] == -2


@pytest.mark.gpu
def test_a_process_forked_from_one_that_used_the_gpu_takes_the_general_path(recorder):
    """There torch refuses to look for the current stream, and the general path with it; the extension asks before it enters the library."""
    print("case: fastcall, forked", flush=True)
    args = _usual()
    args[3] = args[3].cuda()
    for bad, entered in ((lambda: True, 0), (lambda: False, 1)):
        _fastcall.streams(lambda: 0, lambda dev: 0x1230, bad)
        assert len(_call(args)[1]) == entered
    assert hasattr(torch._C, "_cuda_isInBadFork") and torch._C._cuda_isInBadFork() is False


@pytest.mark.parametrize("module", ["none", "another torch's", "this torch's"])
def test_without_a_module_for_this_torch_calls_take_the_general_path(monkeypatch, module):
    """The general path needs nothing of the module: one that was not built, or was built for another torch, costs time, not the call."""
    import sys
    import types
    import warnings
    import paper_2602_14516_amd as A
    calls = []
    stand_in = types.ModuleType("paper_2602_14516_amd._fastcall")
    stand_in.torch_version = torch.__version__ if module == "this torch's" else "0.0"
    stand_in.streams = lambda *functions: None
    stand_in.call = lambda *args: calls.append(args)
    monkeypatch.setitem(sys.modules, "paper_2602_14516_amd._fastcall", None if module == "none" else stand_in)
    monkeypatch.setattr(A, "_fastcall", stand_in, raising=False)
    if module == "none":
        monkeypatch.delattr(A, "_fastcall")
    monkeypatch.setattr(b, "_fastcall", None)
    monkeypatch.setattr(b, "_stream_ptr", lambda stream: 0)
    if module == "this torch's":
        assert b._fast("ampd_kv_append", 1) is None and len(calls) == 1
        return
    cache, ctx, inc, bt, k, v = _usual()[:6]
    inc[:] = 0                                                            # no new tokens: the library returns before it touches the GPU
    with pytest.warns(RuntimeWarning, match="extension"):
        b.kv_append(cache, ctx, inc, bt, k, v)
    with warnings.catch_warnings():
        warnings.simplefilter("error")                                    # said once
        b.kv_append(cache, ctx, inc, bt, k, v)
    assert not calls and b._fastcall is False
    inc[:] = -1
    with pytest.raises(b.AmpdError):
        b.kv_append(cache, ctx, inc, bt, k, v)
