"""Tiles of up to 256 query rows where small launches go as blocks of 32: the shapes of small batches as tiles (cut key ranges on request
take the work list in the workspace), larger batches whose list of tiles travels in the arguments, and those that do not fit it.  Every
test states which kernel it is about and checks that the plan takes it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch, compare, from_dev_bits, sample_rows


def plan(case, splits=0, fp8=False):
    C, L, Hq, Hkv, d, P = case
    cache = A.KVCache(Hq, Hkv, d, P, None, None, 0.1, kv_dtype=A.binding.AMPD_KV_FP8_E4M3 if fp8 else A.binding.AMPD_KV_BF16)
    pages = max((c + l + P - 1) // P for c, l in zip(C, L))
    return A.plan_describe(cache, C, L, pages, splits), A.plan_items(cache, C, L, pages, splits)


def run_and_compare(b, label, splits=0, check_pages=True):
    db = DevBatch(b)
    out = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, block_table_host=b.block_table, force_kv_splits=splits)
    torch.cuda.synchronize()
    if check_pages:
        k_ref, v_ref = oracle.kv_append_reference(b.k_pool, b.v_pool, b.block_table, b.ctx_len, b.incr_len, b.k_new, b.v_new, b.P)
        assert np.array_equal(from_dev_bits(db.k_pool), k_ref) and np.array_equal(from_dev_bits(db.v_pool), v_ref)
    first = from_dev_bits(out)
    compare(b, first, rows=sample_rows(b, 12, seed=2) if int(b.incr_len.sum()) > 400 else None, label=label)
    again = A.paged_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, force_kv_splits=splits)       # the same keys, all from the pages: the same bits
    assert np.array_equal(from_dev_bits(again), first)


SMALL = {                                 # as tiles with a list in the workspace: name: C, L, Hq, Hkv, d, P
    "configuration 1": ([256], [32], 8, 2, 64, 16),
    "ragged, d 128": ([0, 1, 15, 16, 17, 100, 257, 64], [1, 7, 33, 64, 129, 5, 70, 200], 8, 2, 128, 16),
    "ragged, d 64": ([0, 3, 31, 200], [65, 1, 40, 130], 8, 2, 64, 16),
    "groups of 8": ([300, 0, 77], [150, 31, 1], 16, 2, 128, 32),
    "groups of 1": ([50, 129], [140, 9], 4, 4, 128, 16),
    "groups of 16": ([130, 5], [3, 70], 32, 2, 64, 64),
    "groups of 5": ([10, 200], [70, 1], 10, 2, 64, 32),
    "36 query rows": ([0], [9], 4, 1, 64, 16),
}


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("name", SMALL)
def test_small_batches_as_tiles(name, splits):
    print("case: small tiles,", name, splits, flush=True)
    info, _ = plan(SMALL[name], splits)
    assert info["num_wide_items"] > 0 and info["plan_bytes"] > 0
    run_and_compare(W.make_batch(*SMALL[name], seed=61, poison=True), name, splits)


LARGER = {                                # unforced; the last entry: the list fits the arguments
    "16 rows, d 64": ([40 * i for i in range(16)], [133 + i for i in range(16)], 8, 2, 64, 16, True),
    "17 rows, d 64": ([40 * i for i in range(17)], [133 + i for i in range(17)], 8, 2, 64, 16, False),
    "rows without tokens": ([100, 7, 900, 50], [0, 470, 0, 431], 16, 4, 128, 32, True),
    "groups of 3, cut": ([1000, 1111], [700, 771], 12, 4, 128, 16, True),
    "groups of 3, d 64": ([0, 30], [700, 701], 12, 4, 64, 16, True),
    "groups of 32, cut": ([1500, 200], [150, 171], 64, 2, 128, 64, True),
    "groups of 32, d 64, cut": ([7000], [170], 64, 2, 64, 64, True),
    "64 KV heads": ([700], [300], 128, 64, 64, 16, True),
    "65 KV heads": ([700], [300], 65, 65, 64, 16, False),
    "d 64, cut": ([9000, 3000], [309, 77], 12, 2, 64, 16, True),
    "d 64, initial": ([0], [1100], 8, 2, 64, 16, True),
}


@pytest.mark.parametrize("name", LARGER)
def test_larger_batches_stay_tiles(name):
    info, _ = plan(LARGER[name][:6])
    assert info["num_wide_items"] > 0 and info["num_narrow_items"] == 0 and (info["plan_bytes"] == 0) == LARGER[name][6]
    assert (info["num_combine_items"] > 0) >= ("cut" in name)


@pytest.mark.gpu
@pytest.mark.parametrize("name", LARGER)
def test_larger_batches(name):
    print("case: larger tiles,", name, flush=True)
    run_and_compare(W.make_batch(*LARGER[name][:6], seed=92, poison=True), name)


NULLS = {                                 # few K/V streams for 8 dies: queues of unequal length
    "3 streams, list in the arguments": ([700, 0, 333], [1060, 350, 40], 8, 2, 64, 32, 0, True),
    "3 streams, list in the workspace": ([1355, 407, 542], [618, 147, 63], 8, 1, 128, 16, 1, False),
    "3 rows next to a decode row": ([2355, 407, 542, 5000], [918, 447, 263, 1], 8, 1, 128, 16, 0, False),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", NULLS)
def test_null_items_between_tiles_do_nothing(name):
    print("case: null items,", name, flush=True)
    case, splits, in_args = NULLS[name][:6], NULLS[name][6], NULLS[name][7]
    info, items = plan(case, splits)
    assert info["num_wide_items"] > 0 and (items[:, 1] == 2).any() and (info["plan_bytes"] == 0) == in_args
    run_and_compare(W.make_batch(*case, seed=62, poison=True), name, splits)


RISING = {                                # C, L, Hq, Hkv, d, P, forced splits, list in the arguments
    "d 128, mixed": ([900, 3000, 0, 517], [700, 1, 130, 9], 16, 4, 128, 16, 0, False),
    "d 128, alone": ([900, 0], [500, 430], 16, 4, 128, 16, 0, True),
    "d 128, few rows": ([900, 3000, 0, 517], [300, 1, 130, 9], 16, 4, 128, 16, 1, False),
    "d 64, mixed": ([700, 1500, 0, 333], [1060, 1, 350, 40], 8, 2, 64, 32, 0, False),
    "d 64, alone": ([700, 0, 333], [1060, 350, 40], 8, 2, 64, 32, 0, True),
    "groups of 3, mixed": ([700, 1500, 0, 333], [1060, 1, 350, 40], 6, 2, 64, 16, 0, False),
    "groups of 3, alone": ([700, 0, 333], [1060, 350, 40], 6, 2, 64, 16, 0, True),
    "groups of 32, mixed": ([700, 1500, 0, 333], [260, 1, 150, 40], 32, 1, 128, 32, 0, False),
    "groups of 32, alone": ([700], [860], 32, 1, 128, 32, 0, True),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", RISING)
def test_rising_and_sharp_logits_in_tiles(name):
    """The tiles' own rule for raising a row's reference (its sum of exponentials says so): logits that rise with the key position, in
    steps far past the range of exp2 in fp32, and logits with a standard deviation of 16."""
    print("case: rising logits in tiles,", name, flush=True)
    case, splits, in_args = RISING[name][:6], RISING[name][6], RISING[name][7]
    info, _ = plan(case, splits)
    assert info["num_wide_items"] > 0 and (info["plan_bytes"] == 0) == in_args
    for seed, ramp in ((71, (1.0, 37, 400.0)), (72, (0.0, 100, 3000.0)), (73, None)):
        b = W.make_batch(*case, seed=seed, poison=True, **({} if ramp else {"k_mult": 16.0}))
        if ramp:
            W.impose_key_ramp(b, *ramp)
        run_and_compare(b, name, splits, check_pages=False)
