"""The fused entropy kernels for small and for very large batches: 128-row vocabulary tiles over 64 or 192 tokens, and
64-row tiles (a fragment per wave) over 128.  Every kind at the edges of its tiles against the fp64 oracle.  Entropies
to fp32 grade (2e-5 nat, the bar of the fp32 tests: logits are fp32 sums of d exact products)."""
import numpy as np
import pytest

import oracle
from helpers import assert_egtp_close
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (dtype, d, V, T, tokens per block, rows per tile, tiles per range): one token, a block exactly full, one token over,
# several blocks with a ragged last one, more than eight blocks; a last vocabulary tile of 1, 127 and 128 rows in either
# half of a packed block; a last range that is shorter; K of a single pair of steps and K longer than the ring.  With
# 64-row tiles every remainder of a range modulo eight fragments a wave (1 to 8, 9, 13, 35), ranges that straddle packed
# blocks, a vocabulary that ends inside a fragment
CASES = [
    ("bf16", 64, 257, 1, 64, 128, 1),
    ("bf16", 8, 4096, 64, 64, 128, 1),
    ("bf16", 512, 4223, 65, 64, 128, 1),
    ("bf16", 40, 33100, 60, 64, 128, 2),
    ("bf16", 1024, 1025, 579, 64, 128, 1),
    ("bf16", 2048, 32000, 173, 192, 128, 1),
    ("f32", 256, 4096, 309, 64, 128, 1),
    ("bf16", 216, 5422, 338, 128, 64, 1),
    ("bf16", 224, 16511, 65, 128, 64, 2),
    ("bf16", 2048, 32000, 128, 128, 64, 2),
    ("bf16", 208, 33136, 66, 128, 64, 3),
    ("bf16", 208, 386, 8981, 128, 64, 4),
    ("f32", 36, 33791, 261, 128, 64, 7),
    ("bf16", 208, 23215, 522, 128, 64, 8),
    ("bf16", 208, 33664, 415, 128, 64, 9),
    ("bf16", 216, 33834, 773, 128, 64, 15),
    ("bf16", 208, 9496, 3359, 128, 64, 17),      # paced, cohorts cut anywhere
    ("bf16", 208, 2052, 43651, 128, 64, 17),     # paced, whole cohorts, the last group of token blocks not full
]


@pytest.mark.parametrize("dtype,d,V,T,block,rows,per_range", CASES)
def test_every_tile_shape_against_the_oracle(dtype, d, V, T, block, rows, per_range):
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, V, T)
    assert (plan.tokens_per_block, plan.rows_per_tile, plan.tiles_per_range) == (block, rows, per_range)
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


def _rows_of_one_lane(rows, per_range, V):
    """Row groups of a tile shape of which a lane folds four fragments' worth at once, or the part of four that is
    left over: what a mask has to tell from rows that do not exist.  64-row tiles: the waves of the first range (16
    per_range rows each); otherwise the last group of the vocabulary."""
    if rows != 64:
        return [((V - 1) // 64 * 64, V)]
    return [(16 * f, 16 * min(f + 4, (wave + 1) * per_range))
            for wave in (0, 3) for f in range(wave * per_range, (wave + 1) * per_range, 4)]


# 64-row tiles with every kind of sweep that masks (1, 2, 3, 7 and 8 + 1, 8 + 7 fragments a wave), and the last,
# partly filled tile of the other two kernels
@pytest.mark.parametrize("dtype,d,V,T,rows,per_range", [
    ("bf16", 216, 5422, 338, 64, 1), ("bf16", 224, 16511, 65, 64, 2), ("bf16", 208, 33136, 66, 64, 3),
    ("f32", 36, 33791, 261, 64, 7), ("bf16", 208, 33664, 415, 64, 9), ("bf16", 216, 33834, 773, 64, 15),
    ("bf16", 512, 4223, 65, 128, 1), ("bf16", 232, 31206, 389, 256, 1)])
def test_nan_reaches_the_entropy(dtype, d, V, T, rows, per_range):
    """Rows of W_lm that are all NaN make every token's entropy NaN, also where they fill all that a lane folds; a NaN
    hidden state makes its own token NaN and leaves the other tokens' bits alone."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, V, T)
    assert (plan.rows_per_tile, plan.tiles_per_range) == (rows, per_range)
    base = wl.SPECS["tiny" if dtype == "f32" else "mid"]
    w = wl.make(wl.scaled(base, seed=7500 + T, B=1, d=d, V=V, d_h=16, lengths=(T,)))
    td = gpu.to_device
    hidden, off = td(w.hidden), torch.tensor([0, T], dtype=torch.int32).cuda()

    def entropies(w_lm, hidden):
        sc = gpu.Scorer(w_lm, gpu.make_head(td(w.w1), td(w.w2)))
        out = sc.score(hidden, off)["entropy"].cpu().numpy()
        sc.close()
        return out

    clean = entropies(td(w.w_lm), hidden)
    assert np.isfinite(clean).all()
    for lo, hi in _rows_of_one_lane(rows, per_range, V):
        broken = td(w.w_lm)
        broken[lo:hi] = float("nan")
        assert np.isnan(entropies(broken, hidden)).all(), (lo, hi)
    for t in (0, T // 2, T - 1):
        broken = hidden.clone()
        broken[t] = float("nan")
        got = entropies(td(w.w_lm), broken)
        assert np.isnan(got[t])
        assert np.array_equal(np.delete(got, t), np.delete(clean, t)), t
