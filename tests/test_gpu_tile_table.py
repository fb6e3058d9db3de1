"""Small launches of prefill rows alone over a bf16 cache, whose work list travels in the kernel's arguments, and their neighbours that
do not fit the table: every row of the batch against the oracle, the cache image bit for bit.  Most of these go as blocks of 32 query
rows (TILES: as tiles; tests/test_gpu_tiles.py runs larger batches of the other shapes as tiles)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, compare, from_dev_bits, sample_rows

pytestmark = pytest.mark.gpu

CASES = [
    # name, C, L, Hq, Hkv, d, P
    ("smallest", [0], [9], 4, 1, 64, 16),                                       # 36 query rows: one tile, five waves
    ("rows-16", [40 * i for i in range(16)], [33 + i for i in range(16)], 8, 2, 64, 16),
    ("rows-17", [40 * i for i in range(17)], [33 + i for i in range(17)], 8, 2, 64, 16),
    ("rows-without-tokens", [100, 7, 900, 50], [0, 70, 0, 130], 16, 4, 128, 32),
    ("cut", [4099], [509], 32, 8, 128, 16),                                     # 64 tiles in 256 pieces, 64 append items
    ("cut-ragged-group", [3000, 1111], [100, 77], 12, 4, 128, 16),              # three heads a group: 10 tokens a wave
    ("heads-64", [700], [20], 128, 64, 64, 16),
    ("heads-65", [700], [40], 65, 65, 64, 16),
    ("many-pieces", [60000], [40], 8, 1, 64, 64),
    ("group-32", [1500], [24], 64, 2, 128, 64),
    ("tiles-256", [0], [2048], 32, 8, 128, 16),
    ("tiles-264", [0], [2049], 32, 8, 128, 16),
]

TILES = {"cut", "many-pieces", "tiles-256", "tiles-264"}
WORKSPACE = {"rows-17", "heads-65", "tiles-264"}                                # the list does not fit the arguments


@pytest.mark.parametrize("name,C,L,Hq,Hkv,d,P", CASES, ids=[c[0] for c in CASES])
def test_tile_launches(name, C, L, Hq, Hkv, d, P):
    print("case: tiles,", name, flush=True)
    b = W.make_batch(C, L, Hq, Hkv, d, P, seed=92, poison=True)
    db = DevBatch(b)
    info = A.plan_describe(db.cache, b.ctx_len, b.incr_len, b.block_table.shape[1])
    assert (info["num_wide_items"] > 0) == (name in TILES) and (info["num_narrow_items"] == 0) == (name in TILES)
    assert (info["plan_bytes"] > 0) == (name in WORKSPACE)
    rows = sample_rows(b, 12) if sum(L) > 200 else None
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, block_table_host=b.block_table)
    torch.cuda.synchronize()
    k_ref, v_ref = oracle.kv_append_reference(b.k_pool, b.v_pool, b.block_table, b.ctx_len, b.incr_len, b.k_new, b.v_new, b.P)
    assert np.array_equal(from_dev_bits(db.k_pool), k_ref) and np.array_equal(from_dev_bits(db.v_pool), v_ref)
    first = from_dev_bits(out)
    compare(b, first, rows=rows, label=name)
    # attention alone on the pages as they are now reads the same keys: the same bits
    again = A.paged_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q)
    assert np.array_equal(from_dev_bits(again), first)
