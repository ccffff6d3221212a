"""Batches of few tokens take the fused kernel with 128-row vocabulary tiles and token blocks of 64 to 256: every
block size at the edges of its tiles, against the fp64 oracle.  Entropies to fp32 grade (2e-5 nat, the bar of the
fp32 tests: logits are fp32 sums of d exact products, |z| <= 8 here, so an error of d * 2^-24 * 8 at most)."""
import numpy as np
import pytest

import oracle
from helpers import assert_egtp_close
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (dtype, d, V, T, tokens per block, tiles per range): one token, a block exactly full, one token over, several blocks
# with a ragged last one, more than eight blocks (two groups); a last vocabulary tile of 1, 127 and 128 rows in either
# half of a packed block; ranges of unequal length; K of a single pair of steps and K longer than the ring
CASES = [
    ("bf16", 64, 257, 1, 64, 1),
    ("bf16", 8, 4096, 64, 64, 1),
    ("bf16", 512, 4223, 65, 64, 1),
    ("bf16", 40, 33100, 60, 64, 2),
    ("bf16", 1024, 1025, 579, 64, 1),
    ("bf16", 1024, 32000, 128, 128, 1),
    ("bf16", 264, 66000, 101, 128, 3),
    ("bf16", 2048, 32000, 173, 192, 1),
    ("bf16", 2048, 32000, 256, 256, 1),
    ("bf16", 256, 4000, 2000, 256, 1),
    ("f32", 256, 4096, 309, 64, 1),
    ("f32", 68, 4096, 1000, 128, 1),
]


@pytest.mark.parametrize("dtype,d,V,T,block,per_range", CASES)
def test_every_block_size_against_the_oracle(dtype, d, V, T, block, per_range):
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, V, T)
    assert (plan.tokens_per_block, plan.rows_per_tile, plan.tiles_per_range) == (block, 128, per_range)
    lens = (T,) if T < 3 else (T // 3, 0, T - T // 3)
    base = wl.SPECS["tiny" if dtype == "f32" else "mid"]
    w = wl.make(wl.scaled(base, seed=7000 + T, B=len(lens), d=d, V=V, d_h=16, lengths=lens))
    td = gpu.to_device
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    off = oracle.offsets_from_lengths(lens)
    ws = sc.workspace(T, len(lens))
    runs = []
    for fill in (0, 255):           # whatever the workspace held before, the bits are the same
        ws.fill_(fill)
        out = sc.score(td(w.hidden), torch.from_numpy(off).cuda())
        runs.append({k: v.cpu().numpy() for k, v in out.items()})
    for k in runs[0]:
        assert np.array_equal(runs[0][k], runs[1][k]), k
    want = oracle.egtp(w.hidden, off, w.w_lm, oracle.Head(w.w1, w.w2))
    assert_egtp_close(runs[0], want)
    assert np.abs(runs[0]["entropy"] - want.entropy).max() <= 2e-5
    sc.close()
