"""Launches of decode rows alone, whose work list travels in the kernel's arguments: every kernel that the launch may pick and
the edges of the table, the pieces and the pages, against the oracle (the cache image bit for bit, attention on the cache's
contents at the bf16 tolerance, which bounds the rounding of probabilities and outputs whatever the cut)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, compare, from_dev_bits, to_dev_bits, TOL_BF16
from test_gpu_fp8 import Fp8Pool, errs

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(5)
UNEVEN = [int(x) for x in RNG.integers(0, 3200, 40)]      # over 8 KV heads: two or more items per CU

CASES = [
    # name, C, L, Hq, Hkv, d, P
    ("first-token", [0], [1], 8, 2, 128, 16),                                    # one key, nothing cached
    ("table-64-65", [int(x) for x in RNG.integers(0, 600, 65)], [1] * 65, 2, 1, 64, 16),      # both halves of the row lookup
    ("table-full", [int(x) for x in RNG.integers(0, 600, 128)], [1] * 128, 4, 1, 128, 32),    # the largest table ...
    ("list-129", [int(x) for x in RNG.integers(0, 300, 129)], [1] * 129, 4, 1, 128, 16),      # ... and one row more
    ("whole-pieces", [255, 511, 256, 767, 1023], [1] * 5, 16, 8, 128, 16),       # key counts at and around multiples of a piece
    ("small-workgroups", UNEVEN, [1] * 40, 32, 8, 128, 16),                      # 4-wave workgroups, 4 rows per item
    ("small-workgroups-8", UNEVEN, [1] * 40, 64, 8, 128, 32),                    # 8 rows: the most over an 8-bit cache
    ("16-rows", UNEVEN, [2] * 40, 64, 8, 128, 64),                               # 16 rows: the most over a bf16 cache
    ("new-tokens-across-pieces", [250, 506, 0, 1007], [32, 20, 32, 31], 8, 8, 128, 16),       # up to three pages of new tokens
    ("new-tokens-large-pages", [250, 30, 63, 64], [8, 5, 2, 8], 16, 4, 64, 64),
    ("empty-rows-between", [300, 10, 0, 900], [0, 3, 0, 1], 8, 2, 128, 16),
]


@pytest.mark.parametrize("name,C,L,Hq,Hkv,d,P", CASES, ids=[c[0] for c in CASES])
def test_decode_rows_bf16(name, C, L, Hq, Hkv, d, P):
    print(f"case: decode rows bf16, {name}", flush=True)
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=91, poison=True)
    db = DevBatch(b)
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, block_table_host=b.block_table)
    torch.cuda.synchronize()
    k_ref, v_ref = oracle.kv_append_reference(b.k_pool, b.v_pool, b.block_table, b.ctx_len, b.incr_len, b.k_new, b.v_new, b.P)
    assert np.array_equal(from_dev_bits(db.k_pool), k_ref) and np.array_equal(from_dev_bits(db.v_pool), v_ref)
    compare(b, from_dev_bits(out), label=name)


@pytest.mark.parametrize("name,C,L,Hq,Hkv,d,P", CASES, ids=[c[0] for c in CASES])
def test_decode_rows_8bit(name, C, L, Hq, Hkv, d, P):
    print(f"case: decode rows 8-bit, {name}", flush=True)
    rng = np.random.default_rng(17)
    C, L = np.array(C, np.int32), np.array(L, np.int32)
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

    def rows(n, mult):       # magnitudes differ, so that pages get other scales and later tokens raise some of them
        mag = np.exp2(rng.integers(-2, 2, size=(n, Hkv, 1))).astype(np.float32) * np.float32(mult)
        return W.f32_to_bf16_bits(rng.standard_normal((n, Hkv, d), dtype=np.float32) * mag)

    n0, n1 = int(C.sum()), int(L.sum())
    if n0:
        k, v = rows(n0, 0.25), rows(n0, 0.25)
        A.kv_append(pool.cache, np.zeros_like(C), C, d_bt, to_dev_bits(k), to_dev_bits(v))
        pool.reference_append(bt, np.zeros_like(C), C, k, v)
    q = W.f32_to_bf16_bits(rng.standard_normal((n1, Hq, d), dtype=np.float32))
    k, v = rows(n1, 0.5), rows(n1, 0.5)
    out = A.mixed_batch_attn(pool.cache, C, L, d_bt, to_dev_bits(q), to_dev_bits(k), to_dev_bits(v), block_table_host=bt)
    torch.cuda.synchronize()
    pool.reference_append(bt, C, L, k, v)
    pool.assert_equal()
    off = np.concatenate([[0], np.cumsum(L)])
    ref = [None if L[r] == 0 else
           oracle.attn_oracle_request(W.bf16_bits_to_f64(q[off[r]:off[r + 1]]),
                                      oracle.fp8_dequant_request(pool.h_k, pool.h_ks, bt[r], int(C[r] + L[r]), P),
                                      oracle.fp8_dequant_request(pool.h_v, pool.h_vs, bt[r], int(C[r] + L[r]), P),
                                      int(C[r]), int(L[r]), scale) for r in range(len(C))]
    mx, mean = errs(from_dev_bits(out), ref, off)
    assert mx <= TOL_BF16[0] and mean <= TOL_BF16[1], (mx, mean)


@pytest.mark.parametrize("P", [16, 32, 64])
@pytest.mark.parametrize("Hq,Hkv,d", [(32, 8, 128), (32, 8, 64)])
def test_one_new_token_raises_the_page_exponent(Hq, Hkv, d, P):
    """8-bit cache: the token's page also holds cached tokens, in the row's last 32-key block or in the one before it too, and all
    of them are re-encoded while the row is being read (history 2^-6 of the new tokens' size: every exponent rises).  Attention
    in the same launch is bit for bit what attention alone reads from the finished pages with the same cut, and the oracle's."""
    print(f"case: one new token, d {d}, P {P}", flush=True)
    rng = np.random.default_rng(29)
    C = np.array([b * 64 + s for b in (0, 5, 9) for s in (0, 1, 15, 31, 32, 33, 40, 63)], np.int32)   # up to 20 blocks, 8 waves
    L = np.ones_like(C)
    pages = C // P + 1
    perm = rng.permutation(int(pages.sum()) + 2).astype(np.int32)
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

    k, v = rows(int(C.sum()), 2.0 ** -6), rows(int(C.sum()), 2.0 ** -6)
    A.kv_append(pool.cache, np.zeros_like(C), C, d_bt, to_dev_bits(k), to_dev_bits(v))
    pool.reference_append(bt, np.zeros_like(C), C, k, v)
    q = W.f32_to_bf16_bits(rng.standard_normal((len(C), Hq, d), dtype=np.float32))
    k, v = rows(len(C), 1.0), rows(len(C), 1.0)
    out = A.mixed_batch_attn(pool.cache, C, L, d_bt, to_dev_bits(q), to_dev_bits(k), to_dev_bits(v), block_table_host=bt)
    torch.cuda.synchronize()
    pool.reference_append(bt, C, L, k, v)
    pool.assert_equal()
    again = A.paged_attn(pool.cache, C, L, d_bt, to_dev_bits(q))
    assert np.array_equal(from_dev_bits(out), from_dev_bits(again))
    off = np.arange(len(C) + 1)
    ref = [oracle.attn_oracle_request(W.bf16_bits_to_f64(q[r:r + 1]),
                                      oracle.fp8_dequant_request(pool.h_k, pool.h_ks, bt[r], int(C[r] + 1), P),
                                      oracle.fp8_dequant_request(pool.h_v, pool.h_vs, bt[r], int(C[r] + 1), P),
                                      int(C[r]), 1, scale) for r in range(len(C))]
    mx, mean = errs(from_dev_bits(out), ref, off)
    assert mx <= TOL_BF16[0] and mean <= TOL_BF16[1], (mx, mean)
