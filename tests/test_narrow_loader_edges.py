"""The key blocks of decode rows where their loads change: a half block at the end of the range, new tokens inside a block, the last
of the eight blocks whose page ids come together, one and several workgroups per CU; every row against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, TOL_BF16, compare, from_dev_bits, to_dev_bits
from test_gpu_fp8 import Fp8Pool

EDGES = [0, 1, 14, 15, 16, 17, 30, 31, 32, 33, 47, 48, 255, 256, 271, 300, 2031, 2047, 2048, 2063, 2300, 4095, 4111]
CASES = {                              # name: ctx, new tokens, Hq, Hkv, d, P, forced number of key ranges (0: the plan's)
    "whole, d 128": (EDGES, [1] * len(EDGES), 8, 2, 128, 16, 1),
    "whole, d 64": (EDGES, [1] * len(EDGES), 8, 2, 64, 16, 1),
    "whole, pages of 64": (EDGES, [1] * len(EDGES), 8, 2, 64, 64, 1),
    "three tokens": (EDGES, [3] * len(EDGES), 8, 2, 128, 32, 1),
    "31 rows": (EDGES, [7] * len(EDGES), 12, 4, 128, 16, 1),
    "cut": (EDGES, [1] * len(EDGES), 8, 2, 128, 16, 0),
    "small workgroups": ([700 + 13 * i for i in range(70)], [1] * 70, 32, 8, 128, 16, 0),
    "several per CU": ([2900 + 37 * i for i in range(40)], [1] * 40, 32, 8, 128, 16, 0),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_bf16(name):
    print("case: loader edges, bf16,", name, flush=True)
    C, L, Hq, Hkv, d, P, splits = CASES[name]
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=31, poison=True)
    db = DevBatch(b)
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, force_kv_splits=splits)
    torch.cuda.synchronize()
    first = from_dev_bits(out)
    compare(b, first, label=name)
    again = A.paged_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, force_kv_splits=splits)     # all from the pages: the same bits
    assert np.array_equal(from_dev_bits(again), first)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_8bit(name):
    print("case: loader edges, 8-bit,", name, flush=True)
    C, L, Hq, Hkv, d, P, splits = CASES[name]
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=32)
    C, L = b.ctx_len, b.incr_len
    pool = Fp8Pool(b.k_pool.shape[0], Hq, Hkv, d, P, b.scale)
    bt = torch.from_numpy(b.block_table).cuda()
    rng = np.random.default_rng(33)
    k, v = (W.f32_to_bf16_bits(rng.standard_normal((int(C.sum()), Hkv, d), dtype=np.float32)) for _ in range(2))
    A.kv_append(pool.cache, np.zeros_like(C), C, bt, to_dev_bits(k), to_dev_bits(v))
    pool.reference_append(b.block_table, np.zeros_like(C), C, k, v)
    out = A.mixed_batch_attn(pool.cache, C, L, bt, to_dev_bits(b.q), to_dev_bits(b.k_new), to_dev_bits(b.v_new),
                             block_table_host=b.block_table, force_kv_splits=splits)
    torch.cuda.synchronize()
    pool.reference_append(b.block_table, C, L, b.k_new, b.v_new)
    pool.assert_equal()
    got, off, err = W.bf16_bits_to_f64(from_dev_bits(out)), np.concatenate([[0], np.cumsum(L)]), []
    for r in range(len(C)):
        K, V = (oracle.fp8_dequant_request(h, s, b.block_table[r], int(C[r] + L[r]), P) for h, s in ((pool.h_k, pool.h_ks), (pool.h_v, pool.h_vs)))
        err.append(np.abs(got[off[r]:off[r + 1]] - oracle.attn_oracle_request(W.bf16_bits_to_f64(b.q[off[r]:off[r + 1]]), K, V, int(C[r]), int(L[r]), b.scale)).ravel())
    err = np.concatenate(err)
    assert np.isfinite(err).all() and err.max() <= TOL_BF16[0] and err.mean() <= TOL_BF16[1], (err.max(), err.mean())
