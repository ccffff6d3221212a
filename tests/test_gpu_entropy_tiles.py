"""The fused entropy kernels for small and for very large batches: 128-row vocabulary tiles over 64 or 192 tokens, and
64-row tiles (a fragment per wave) over 128.  Every kind at the edges of its tiles against the fp64 oracle.  Entropies
to fp32 grade (2e-5 nat, the bar of the fp32 tests: logits are fp32 sums of d exact products)."""
import ctypes

import numpy as np
import pytest

import oracle
from helpers import assert_egtp_close
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (dtype, d, V, T, tokens per block, rows per tile, tiles per range): one token, a block exactly full, one token over,
# several blocks with a ragged last one, more than eight blocks; a last vocabulary tile of 1, 127 and 128 rows in either
# half of a packed block; a last range that is shorter; K of a single pair of steps and K longer than the ring; ranges of
# several tiles, so that the ring runs from one tile into the next, with some ranges a tile shorter.  With 64-row tiles every remainder of a range modulo eight fragments a wave (1 to 8, 9, 13, 35), ranges that straddle packed
# blocks, a vocabulary that ends inside a fragment
CASES = [
    ("bf16", 64, 257, 1, 64, 128, 1),
    ("bf16", 8, 4096, 64, 64, 128, 1),
    ("bf16", 512, 4223, 65, 64, 128, 1),
    ("bf16", 40, 33100, 60, 64, 128, 2),
    ("bf16", 1024, 1025, 579, 64, 128, 1),
    ("bf16", 2048, 32000, 173, 192, 128, 1),
    ("f32", 256, 4096, 309, 64, 128, 1),
    ("bf16", 104, 20138, 291, 64, 128, 4),
    ("bf16", 8, 35546, 554, 64, 128, 10),
    ("bf16", 64, 48959, 341, 192, 128, 3),
    ("bf16", 48, 52583, 565, 192, 128, 5),
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


class _Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tb_tokens", "tile_v", "ntb", "ntiles_v", "nsplit", "tiles_per_split")]
    _fields_ += [("whole_cohorts", ctypes.c_bool)]


def _whole_cohorts(dtype, d, V, T):
    """What the queried plan does not say: whether each XCD gets whole cohorts of workgroups."""
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.load_library()._ZN4egtp7k1_planEilii
    plan.restype, plan.argtypes = _Plan, [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    return plan(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, T, d, V).whole_cohorts


@pytest.mark.parametrize("dtype,d,V,T,block,rows,per_range", CASES)
def test_every_tile_shape_against_the_oracle(dtype, d, V, T, block, rows, per_range):
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, V, T)
    assert (plan.tokens_per_block, plan.rows_per_tile, plan.tiles_per_range) == (block, rows, per_range)
    assert plan.paced == (per_range == 17) and _whole_cohorts(dtype, d, V, T) == (per_range == 17 and T > 10000)
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


def test_one_token_block_against_a_large_vocabulary():
    """One token block against a W_lm that the 256 MiB Infinity Cache cannot hold (1.24 GB): the instantiations that read
    it with the non-temporal hint, in the plans of decode steps with few sequences and of single prompts -- 64 and 192
    tokens a block against ranges of 5 tiles of 128 rows, 128 against ranges of 10 of 64.  Every token against the oracle
    and the same bits whatever the workspace held."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    d, V, most = 4096, 151936, 173
    w = wl.make(wl.scaled(wl.SPECS["serving"], seed=7900, B=1, d=d, V=V, d_h=16, lengths=(most,)))
    want = oracle.entropy(w.hidden, w.w_lm)
    td = gpu.to_device
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    hidden = td(w.hidden)
    ws = sc.workspace(most, 1)
    for T, tile in ((1, (64, 128, 5)), (24, (64, 128, 5)), (64, (64, 128, 5)), (100, (128, 64, 10)), (128, (128, 64, 10)),
                    (173, (192, 128, 5))):
        plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16, d, V, T)
        assert (plan.tokens_per_block, plan.rows_per_tile, plan.tiles_per_range, plan.token_blocks) == (*tile, 1)
        off = torch.tensor([0, T], dtype=torch.int32).cuda()
        runs = []
        for fill in (0, 255):
            ws.fill_(fill)
            runs.append({k: v.cpu().numpy() for k, v in sc.score(hidden[:T], off).items()})
        for k in runs[0]:
            assert np.array_equal(runs[0][k], runs[1][k]), (T, k)
        assert np.abs(runs[0]["entropy"] - want[:T]).max() <= 2e-5, T
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
