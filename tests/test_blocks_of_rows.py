"""Small launches with prefill rows go as blocks of at most 32 query rows: which ones do (host only), every key of every token once,
and every row of such launches against the oracle, over both kinds of cache."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, compare, from_dev_bits, sample_rows

CASES = {
    # name: (C, L, Hq, Hkv, d, P, blocks over a bf16 cache, over an 8-bit cache)
    "one-row-64": ([256], [32], 8, 2, 64, 16, True, True),                           # whole, two rounds of 256 keys
    "first-block-remainder": ([300], [83], 32, 8, 128, 16, True, True),              # 8 tokens a block, the first holds 3
    "group-of-three": ([100, 900], [41, 77], 12, 4, 128, 32, True, True),            # 10 tokens a block, 30 rows
    "cut": ([4000], [40], 8, 1, 128, 32, True, True),                                # pieces and a combine pass
    "new-tokens-alone": ([0, 0], [200, 16], 8, 1, 128, 64, True, True),              # every key is a new token
    "with-decode-rows": ([200, 900, 90], [1, 60, 1], 16, 4, 64, 16, True, True),
    "no-room-in-the-table": ([250 + 7 * i for i in range(20)] + [700], [1] * 20 + [60], 8, 2, 64, 16, True, True),  # with a list in the workspace too
    "long-decode-rows": ([7000, 90, 15000], [1, 60, 1], 16, 4, 64, 16, False, False), # they last longer than the tiles would
    "rows-17": ([20 * i for i in range(17)], [9 + i for i in range(17)], 8, 2, 64, 16, True, True),   # more rows than the table holds
    "blocks-256": ([900], [256], 32, 8, 128, 16, True, True),
    "blocks-264": ([900], [257], 32, 8, 128, 16, False, True),                       # bf16: more than one round
    "blocks-520": ([900], [513], 32, 8, 128, 16, False, False),
    "a-round-and-a-bit": ([0, 0], [222, 239], 32, 8, 128, 16, False, False),         # 464 blocks, each one trip: the second round costs a start
    "many-long-rows": ([6850, 7994, 4209, 621, 6742], [71, 18, 39, 120, 134], 32, 8, 128, 16, False, False),   # 8-bit: 66 us as tiles, 84 as blocks
    "long-tiles": ([16384], [256], 32, 8, 128, 16, False, False),                    # the keys would be read eight times as often
}


def _plan(name, fp8):
    C, L, Hq, Hkv, d, P = CASES[name][:6]
    cache = A.KVCache(Hq, Hkv, d, P, None, None, 0.1, kv_dtype=A.binding.AMPD_KV_FP8_E4M3 if fp8 else A.binding.AMPD_KV_BF16)
    pages = max((c + l + P - 1) // P for c, l in zip(C, L))
    return A.plan_items(cache, C, L, pages), A.plan_describe(cache, C, L, pages)


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "8bit"])
@pytest.mark.parametrize("name", CASES)
def test_plan(name, fp8):
    C, L, Hq, Hkv = CASES[name][:4]
    items, info = _plan(name, fp8)
    assert (info["num_wide_items"] == 0) == CASES[name][7 if fp8 else 6]
    att = items[items[:, 1] < 2]
    assert np.all(att[att[:, 1] == 1][:, 6] * (Hq // Hkv) <= 32)
    seen = {}
    for r, kind, kvh, g0, gn, q0, nq, k0, k1, part in att.tolist():
        assert gn == Hq // Hkv and (part >= 0) == (k0 > 0 or k1 < C[r] + q0 + nq)
        seen.setdefault((r, kvh, q0, nq), []).append((k0, k1))
    tokens = {}
    for (r, kvh, q0, nq), ks in seen.items():
        ks.sort()
        assert ks[0][0] == 0 and ks[-1][1] == C[r] + q0 + nq and all(a[1] == b[0] for a, b in zip(ks, ks[1:]))
        tokens.setdefault((r, kvh), []).append((q0, nq))
    for r in range(len(C)):
        for h in range(Hkv):
            q = sorted(tokens[r, h])
            assert q[0][0] == 0 and sum(n for _, n in q) == L[r] and all(a[0] + a[1] == b[0] for a, b in zip(q, q[1:]))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_bf16_against_the_oracle(name):
    print("case: blocks, bf16,", name, flush=True)
    C, L, Hq, Hkv, d, P = CASES[name][:6]
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=77, poison=True)
    db = DevBatch(b)
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, block_table_host=b.block_table)
    torch.cuda.synchronize()
    k_ref, v_ref = oracle.kv_append_reference(b.k_pool, b.v_pool, b.block_table, b.ctx_len, b.incr_len, b.k_new, b.v_new, b.P)
    assert np.array_equal(from_dev_bits(db.k_pool), k_ref) and np.array_equal(from_dev_bits(db.v_pool), v_ref)
    first = from_dev_bits(out)
    compare(b, first, rows=sample_rows(b, 12) if sum(L) > 200 else None, label=name)
    again = A.paged_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q)        # the same keys, all from the pages: the same bits
    assert np.array_equal(from_dev_bits(again), first)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_8bit_equals_attention_over_the_decoded_pages(name):
    """Against the same batch over a bf16 cache that holds the 8-bit cache's contents: both plans' tiles and blocks see the same bf16
    values, so each is within the bf16 tolerance (2e-2 / 2e-3, doubled: two results) of the other."""
    print("case: blocks, 8-bit,", name, flush=True)
    C, L, Hq, Hkv, d, P = CASES[name][:6]
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=78)
    db = DevBatch(b)
    n = db.k_pool.shape[0]
    k8, v8 = (torch.zeros((n, Hkv, P, d), device="cuda", dtype=torch.uint8) for _ in range(2))
    ks, vs = (torch.ones((n, Hkv), device="cuda") for _ in range(2))
    cache = A.KVCache(Hq, Hkv, d, P, k8, v8, b.scale, ks, vs, A.binding.AMPD_KV_FP8_E4M3)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    Ct = np.asarray(C, np.int32)
    if Ct.any():
        h = [torch.randn((int(Ct.sum()), Hkv, d), device="cuda", dtype=torch.bfloat16, generator=g) for _ in range(2)]
        A.kv_append(cache, np.zeros_like(Ct), Ct, db.bt, *h)
    out = A.mixed_batch_attn(cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new)
    table = torch.tensor([[0 if (c & 0x7f) == 0x7f else
                           (-1) ** (c >> 7) * ((c & 7) / 8 * 2.0 ** -6 if not (c >> 3) & 15 else (1 + (c & 7) / 8) * 2.0 ** (((c >> 3) & 15) - 7))
                           for c in range(256)]], device="cuda").reshape(256)
    kd, vd = ((table[x.long()] * s[:, :, None, None]).to(torch.bfloat16) for x, s in ((k8, ks), (v8, vs)))
    ref = A.paged_attn(A.KVCache(Hq, Hkv, d, P, kd, vd, b.scale), b.ctx_len, b.incr_len, db.bt, db.q, force_kv_splits=1)
    diff = (out.float() - ref.float()).abs()
    assert diff.max().item() <= 4e-2 and diff.mean().item() <= 4e-3, (diff.max().item(), diff.mean().item())
