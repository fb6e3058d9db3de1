"""The append / pack / unpack launches find a page's row in the arguments: more rows than a wave has lanes and than a launch
takes, rows without new tokens, pages that get one token, all of theirs or a part, one KV head and several."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, from_dev_bits, to_dev_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,Hkv,d,P", [(1, 1, 128, 16), (64, 2, 64, 16), (65, 3, 128, 32), (130, 1, 64, 64), (130, 8, 128, 16)])
def test_append_pack_unpack_rows_and_pages(n, Hkv, d, P):
    print("case:", n, Hkv, d, P, flush=True)
    g = np.random.default_rng(n * 100 + Hkv)
    C = g.integers(0, 3 * P, n)
    L = g.choice([0, 0, 1, 1, 2, P - 1, P, P + 1, 3 * P], n)
    L[0], L[-1] = max(1, L[0]), 2 * P if n > 1 else 2 * P + 3
    b = W.make_batch(C.tolist(), L.tolist(), 2 * Hkv, Hkv, d, P, seed=n, poison=True)
    db = DevBatch(b)
    # bf16 append: whole pools
    A.kv_append(db.cache, b.ctx_len, b.incr_len, db.bt, db.k_new, db.v_new)
    k_ref, v_ref = oracle.kv_append_reference(b.k_pool, b.v_pool, b.block_table, b.ctx_len, b.incr_len, b.k_new, b.v_new, P)
    assert np.array_equal(from_dev_bits(db.k_pool), k_ref) and np.array_equal(from_dev_bits(db.v_pool), v_ref)
    # pack what was just written, for a share of the heads, and unpack it into clean pools
    for h0, hn in {(0, Hkv), (Hkv - 1, 1)}:
        ko = torch.zeros(int(L.sum()), hn, d, dtype=torch.bfloat16, device="cuda")
        vo = torch.zeros_like(ko)
        A.kv_pack(db.cache, b.ctx_len, b.incr_len, db.bt, h0, hn, ko, vo)
        assert np.array_equal(from_dev_bits(ko), b.k_new[:, h0:h0 + hn]) and np.array_equal(from_dev_bits(vo), b.v_new[:, h0:h0 + hn])
        kp, vp = to_dev_bits(b.k_pool), to_dev_bits(b.v_pool)
        A.kv_unpack(A.KVCache(2 * Hkv, Hkv, d, P, kp, vp, 1.0), b.ctx_len, b.incr_len, db.bt, h0, hn, ko, vo)
        for got, ref, old in ((kp, k_ref, b.k_pool), (vp, v_ref, b.v_pool)):
            want = old.copy()
            want[:, h0:h0 + hn] = ref[:, h0:h0 + hn]
            assert np.array_equal(from_dev_bits(got), want)
    # 8-bit append: the history, then the new tokens at 64 times the size (the exponent of partly filled pages rises)
    pages = len(b.k_pool)
    pools = [np.zeros((pages, Hkv, P, d), np.uint8) for _ in range(2)]
    scales = [np.ones((pages, Hkv), np.float32) for _ in range(2)]
    dk, dv, ds, dt = (torch.from_numpy(a).cuda() for a in pools + scales)
    cache = A.KVCache(2 * Hkv, Hkv, d, P, dk, dv, 1.0, ds, dt, A.binding.AMPD_KV_FP8_E4M3)
    hist = torch.from_numpy(g.standard_normal((2, int(C.sum()), Hkv, d)).astype(np.float32)).cuda().bfloat16()
    new = torch.from_numpy(g.standard_normal((2, int(L.sum()), Hkv, d)).astype(np.float32)).cuda().bfloat16()
    new[0] *= 64
    zero, c32, l32 = np.zeros(n, np.int32), C.astype(np.int32), L.astype(np.int32)
    for c0, l0, x in ((zero, c32, hist), (c32, l32, new)):
        if l0.any():
            A.kv_append(cache, c0, l0, db.bt, x[0].contiguous(), x[1].contiguous())
            for i in range(2):
                oracle.fp8_append_reference(pools[i], scales[i], b.block_table, c0, l0, from_dev_bits(x[i].contiguous()), P, in_place=True)
    for got, want in zip((dk, dv, ds, dt), pools + scales):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n,Hkv,units", [(7, 3, 66), (40, 8, 1024), (42, 8, 1056)])
@pytest.mark.parametrize("P", [16, 32, 64])
@pytest.mark.parametrize("d", [64, 128])
def test_8bit_append_by_one_wave_or_several_a_page(d, P, n, Hkv, units):
    """8-bit append of a launch with few (page, head, K or V) units, which several waves share (up to 1 024), and with more, one
    wave each: pages with one new token, some, all; exponents that stay and that rise; codes and scales bit for bit."""
    print("case:", d, P, units, flush=True)
    g = np.random.default_rng(d + P + n)
    C = np.array([0, 1, P - 1, P, P + P // 2, 3 * P - 1, 2 * P] * 6, np.int32)[:n]
    L = np.array([1, P, 2, 2 * P + 3, P // 2, 1, P // 2 + 1] * 6, np.int32)[:n]
    assert units == 2 * Hkv * int(((C + L - 1) // P - C // P + 1).sum())
    pages = -(-(C + L) // P)
    perm = g.permutation(int(pages.sum()) + 3).astype(np.int32)
    bt = np.full((n, int(pages.max())), -1, np.int32)
    o = 0
    for r in range(n):
        bt[r, :pages[r]] = perm[o:o + pages[r]]
        o += pages[r]
    pools = [np.full((len(perm), Hkv, P, d), 0x7F, np.uint8) for _ in range(2)]
    scales = [np.full((len(perm), Hkv), np.nan, np.float32) for _ in range(2)]
    dk, dv, ds, dt = (torch.from_numpy(a.copy()).cuda() for a in pools + scales)
    cache = A.KVCache(Hkv, Hkv, d, P, dk, dv, 1.0, ds, dt, A.binding.AMPD_KV_FP8_E4M3)
    d_bt = torch.from_numpy(bt).cuda()
    for c0, l0 in ((np.zeros(n, np.int32), C), (C, L)):
        mag = np.exp2(g.integers(-6, 7, size=(2, int(l0.sum()), Hkv, 1)))
        x = torch.from_numpy((g.standard_normal((2, int(l0.sum()), Hkv, d)) * mag).astype(np.float32)).cuda().bfloat16()
        A.kv_append(cache, c0, l0, d_bt, x[0].contiguous(), x[1].contiguous())
        for i in range(2):
            oracle.fp8_append_reference(pools[i], scales[i], bt, c0, l0, from_dev_bits(x[i].contiguous()), P, in_place=True)
    for got, want in zip((dk, dv, ds, dt), pools + scales):
        assert np.array_equal(got.cpu().numpy().view(np.uint8), want.view(np.uint8))
