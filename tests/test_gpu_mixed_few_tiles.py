"""Decode rows next to tiles that fit one round of the CUs: the tiles go first, whole or in a few pieces (chosen by an estimate
that knows the cache's element size); next to more tiles the two kinds alternate."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, TOL_BF16, compare, from_dev_bits, sample_rows, to_dev_bits
from test_gpu_fp8 import Fp8Pool

CASES = {                                  # name: ctx, new tokens, Hq, Hkv, d, P, tiles first
    "cut tiles first": ([900, 2900, 3000, 1700, 64] * 5 + [6000], [1] * 25 + [200], 32, 8, 128, 16, True),
    "whole tiles first": ([1300, 700, 1200, 40] * 8 + [0], [1, 1, 1, 3] * 8 + [2000], 32, 8, 128, 16, True),
    "d 64": ([900, 2900, 3000, 1700] * 12 + [2000, 10], [1] * 48 + [130, 700], 16, 4, 64, 64, True),
    "more tiles than slots": ([900, 2000, 0, 1500], [1, 1500, 2500, 1], 32, 8, 128, 32, False),
}


def _items(name, fp8):
    C, L, Hq, Hkv, d, P, first = CASES[name]
    cache = A.KVCache(Hq, Hkv, d, P, None, None, 0.1, kv_dtype=A.binding.AMPD_KV_FP8_E4M3 if fp8 else A.binding.AMPD_KV_BF16)
    return A.plan_items(cache, C, L, max((c + l + P - 1) // P for c, l in zip(C, L)))


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("name", CASES)
def test_every_key_of_every_token_once(name, fp8):
    C, L, Hq, Hkv, d, P, first = CASES[name]
    it = _items(name, fp8)
    kinds = it[it[:, 1] < 2, 1]
    assert (np.all(np.diff(kinds) >= 0)) == first               # 0: tile, 1: decode rows
    pieces = {}
    for r, kind, kvh, g0, gn, q0, nq, k0, k1, _ in it[it[:, 1] < 2].tolist():
        assert gn == Hq // Hkv
        pieces.setdefault((r, kvh, q0, nq), []).append((k0, k1))
    tokens = {}
    for (r, kvh, q0, nq), ks in pieces.items():
        ks.sort()
        assert ks[0][0] == 0 and ks[-1][1] == C[r] + q0 + nq and all(a[1] == b[0] for a, b in zip(ks, ks[1:]))
        tokens.setdefault((r, kvh), []).append((q0, nq))
    for r in range(len(C)):
        for h in range(Hkv):
            q = sorted(tokens[r, h])
            assert q[0][0] == 0 and sum(n for _, n in q) == L[r] and all(a[0] + a[1] == b[0] for a, b in zip(q, q[1:]))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_against_the_oracle(name):
    print("case:", name, flush=True)
    C, L, Hq, Hkv, d, P, _ = CASES[name]
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=len(name), poison=True)
    db = DevBatch(b)
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new)
    torch.cuda.synchronize()
    compare(b, from_dev_bits(out), rows=sample_rows(b, 3), label=name)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_8bit_cache_against_the_oracle(name):
    """The same batches over an 8-bit cache: the append launch carries the work list, the tiles widen codes; pages bit for bit,
    attention against the oracle on the cache's contents at the bf16 tolerance."""
    print("case: 8-bit,", name, flush=True)
    C, L, Hq, Hkv, d, P, _ = CASES[name]
    C, L = np.array(C, np.int32), np.array(L, np.int32)
    rng = np.random.default_rng(len(name))
    pages = -(-(C.astype(np.int64) + L) // P)
    perm = rng.permutation(int(pages.sum()) + 3).astype(np.int32)
    bt = np.full((len(C), int(pages.max())), -1, np.int32)
    o = 0
    for r in range(len(C)):
        bt[r, :pages[r]] = perm[o:o + pages[r]]
        o += pages[r]
    scale = 1.0 / np.sqrt(d)
    pool = Fp8Pool(len(perm), Hq, Hkv, d, P, scale)
    d_bt = torch.from_numpy(bt).cuda()

    def rows(n, mult):
        return W.f32_to_bf16_bits(rng.standard_normal((n, Hkv, d), dtype=np.float32) * np.float32(mult))

    n1 = int(L.sum())
    for c0, l0, mult in ((np.zeros_like(C), C, 0.25), (C, L, 1.0)):      # new tokens four times the history: exponents rise
        k, v = rows(int(l0.sum()), mult), rows(int(l0.sum()), mult)
        if l0 is L:
            q = W.f32_to_bf16_bits(rng.standard_normal((n1, Hq, d), dtype=np.float32))
            out = A.mixed_batch_attn(pool.cache, C, L, d_bt, to_dev_bits(q), to_dev_bits(k), to_dev_bits(v), block_table_host=bt)
        else:
            A.kv_append(pool.cache, c0, l0, d_bt, to_dev_bits(k), to_dev_bits(v))
        torch.cuda.synchronize()
        pool.reference_append(bt, c0, l0, k, v)
    pool.assert_equal()
    got, off = W.bf16_bits_to_f64(from_dev_bits(out)), np.concatenate([[0], np.cumsum(L)])
    err = []
    for r in range(len(C)):
        pick = sorted({0, int(L[r]) - 1, int(L[r]) // 2, int(L[r]) // 3})           # tokens of the row, each of its tiles' kind
        K, V = (oracle.fp8_dequant_request(h, s, bt[r], int(C[r] + L[r]), P) for h, s in ((pool.h_k, pool.h_ks), (pool.h_v, pool.h_vs)))
        for i in pick:
            t = int(C[r]) + i
            ref = oracle.attn_oracle_request(W.bf16_bits_to_f64(q[off[r] + i:off[r] + i + 1]), K[:t + 1], V[:t + 1], t, 1, scale)
            err.append(np.abs(got[off[r] + i] - ref[0]).ravel())
    err = np.concatenate(err)
    assert np.isfinite(err).all() and err.max() <= TOL_BF16[0] and err.mean() <= TOL_BF16[1], (err.max(), err.mean())
