"""What the softmax denominator adds up.  Rows of at most 32 query rows per KV head (decode rows, short chunks) divide by the fp32
probabilities; prefill rows divide by the probabilities rounded to bf16, and by the same ones in a tile and in a block.

Every 32nd key has logit `scale` and the others 0, so that against the first the others have p = exp(-scale), chosen just below a tie
of bf16: it rounds down by 0.0038 of itself.  V is not 0 on every 32nd key alone, so nothing of that cancels in the quotient."""
import math

import numpy as np
import pytest
import torch

import paper_2602_14516_amd as A

SCALE = float(np.float32(-math.log(0.5 * (1 + 0.98 / 256))))


def _call(C, L, Hq, Hkv, d, P, fp8, splits=0):
    n = [(c + l + P - 1) // P for c, l in zip(C, L)]
    bt = np.full((len(C), max(n)), -1, np.int32)
    perm = np.random.default_rng(3).permutation(sum(n)).astype(np.int32)
    for r, k in enumerate(n):
        bt[r, :k] = perm[sum(n[:r]):sum(n[:r]) + k]
    bt = torch.from_numpy(bt).cuda()
    pool = [torch.zeros((sum(n), Hkv, P, d), device="cuda", dtype=torch.uint8 if fp8 else torch.bfloat16) for _ in range(2)]
    scales = [torch.ones((sum(n), Hkv), device="cuda") for _ in range(2)] if fp8 else [None, None]
    cache = A.KVCache(Hq, Hkv, d, P, *pool, SCALE, *scales, A.binding.AMPD_KV_FP8_E4M3 if fp8 else A.binding.AMPD_KV_BF16)
    Ct, Lt = np.asarray(C, np.int32), np.asarray(L, np.int32)
    peak = torch.cat([torch.arange(c, device="cuda") % 32 == 0 for c in C])
    v = 1 + (torch.arange(d, device="cuda") % 8) / 8                    # exact in 8 bits too
    k = torch.zeros((len(peak), Hkv, d), device="cuda", dtype=torch.bfloat16)
    k[peak, :, 0] = 1
    A.kv_append(cache, np.zeros_like(Ct), Ct, bt, k, (peak[:, None] * v).to(torch.bfloat16)[:, None, :].expand(-1, Hkv, -1).contiguous())
    q = torch.zeros((sum(L), Hq, d), device="cuda", dtype=torch.bfloat16)
    q[:, :, 0] = 1
    zero = torch.zeros((sum(L), Hkv, d), device="cuda", dtype=torch.bfloat16)
    out = A.mixed_batch_attn(cache, Ct, Lt, bt, q, zero, zero.clone(), force_kv_splits=splits)
    keys = torch.cat([torch.arange(c + 1, c + l + 1, device="cuda", dtype=torch.float64) for c, l in zip(C, L)])
    peaks = torch.cat([torch.full((l,), c // 32, device="cuda", dtype=torch.float64) for c, l in zip(C, L)])
    return out, lambda p: ((peaks / (peaks + (keys - peaks) * p))[:, None] * v)[:, None, :].expand(-1, Hq, -1), A.plan_describe(
        cache, Ct, Lt, bt.shape[1], splits)


def _is_rounded(out, exact):
    """Whether out is bf16(exact), up to fp32 sums of a few thousand terms."""
    ulp = torch.exp2(torch.floor(torch.log2(exact)) - 7)
    return ((out.double() - exact).abs() <= ulp / 2 + 2e-5 * exact).all().item()


SHORT = {                           # name: ctx, new tokens, Hq, Hkv, d, P
    "one token": ([320, 4096], [1, 1], 8, 2, 128, 16),
    "16 rows": ([320, 4096], [2, 2], 16, 2, 64, 32),
    "17 rows": ([320, 4096], [17, 9], 2, 2, 128, 16),
    "24 rows": ([320, 4096], [3, 3], 16, 2, 128, 16),
    "24 rows, d 64": ([320, 4096], [3, 3], 16, 2, 64, 64),
    "24 rows next to blocks": ([320, 608, 320], [3, 1, 60], 16, 2, 128, 16),
    "24 rows next to tiles": ([320, 4096, 64], [3, 1, 3000], 16, 2, 128, 16),
}


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "8bit"])
@pytest.mark.parametrize("name", SHORT)
def test_short_rows_divide_by_fp32_probabilities(name, fp8):
    print("case: row sums, short,", name, fp8, flush=True)
    C, L, Hq, Hkv = SHORT[name][:4]
    out, exact, info = _call(*SHORT[name], fp8)
    assert (info["num_wide_items"] > 0) == ("tiles" in name)
    short = torch.cat([torch.full((l,), l * Hq // Hkv <= 32, device="cuda") for l in L])
    assert _is_rounded(out[short], exact(math.exp(-SCALE))[short])


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "8bit"])
@pytest.mark.parametrize("geom", [(8, 2, 128, 16), (16, 2, 64, 32)], ids=["d128", "d64"])
def test_prefill_rows_divide_by_the_same_probabilities_in_tiles_and_blocks(geom, fp8):
    """40 new tokens (5 blocks of 8 query tokens, or 10 of 4) and 41 (a first block of one token: at most 16 query rows).  Every wave's
    first block of 32 keys holds one with the highest logit, so tiles and blocks take the probabilities against the same reference."""
    print("case: row sums, prefill,", geom, fp8, flush=True)
    C, L = [512, 640], [40, 41]
    blocks, exact, info = _call(C, L, *geom, fp8)
    tiles, _, info_t = _call(C, L, *geom, fp8, splits=1)
    assert info["num_wide_items"] == info["num_combine_items"] == 0 and info_t["num_wide_items"] > 0
    assert _is_rounded(blocks, exact(0.5)) and torch.equal(blocks, tiles)
