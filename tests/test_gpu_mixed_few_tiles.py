"""Decode rows next to tiles that fit one round of the CUs: the tiles go first, whole or in a few pieces (chosen by an estimate
that knows the cache's element size); next to more tiles the two kinds alternate."""
import numpy as np
import pytest
import torch

import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, compare, from_dev_bits, sample_rows

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
