"""Blocks of 192 tokens on the kernel that loads W_lm straight into registers: sweeps of two and of four fragments a wave in
every mix that the plan makes (1 to 6 tiles a range), last ranges that are shorter, several token blocks with a ragged last
one, contractions of 4 K steps, of more and of a number that is no multiple of 4 (which run two steps ahead, not four).
Against the fp64 oracle, entropies to fp32 grade (2e-5 nat, the bar of the fp32 tests: logits are fp32 sums of d exact
products)."""
import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,V,T,per_range", [
    ("bf16", 96, 22029, 130, 1), ("bf16", 96, 43700, 129, 2), ("bf16", 96, 45703, 259, 3), ("bf16", 96, 50699, 322, 4),
    ("bf16", 96, 43766, 513, 5), ("bf16", 96, 48997, 580, 6), ("bf16", 320, 43938, 258, 3), ("f32", 104, 43680, 259, 3),
    ("f32", 96, 22042, 130, 1)])
def test_every_mix_of_sweeps_against_the_oracle(dtype, d, V, T, per_range):
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, V, T)
    assert (plan.tokens_per_block, plan.rows_per_tile, plan.tiles_per_range) == (192, 128, per_range)
    w = wl.make(wl.scaled(wl.SPECS["tiny" if dtype == "f32" else "mid"], seed=7600 + T, B=1, d=d, V=V, d_h=16, lengths=(T,)))
    td = gpu.to_device
    hidden, off = td(w.hidden), torch.tensor([0, T], dtype=torch.int32).cuda()
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    ws = sc.workspace(T, 1)
    runs = []
    for fill in (0, 255):           # whatever the workspace held before, the bits are the same
        ws.fill_(fill)
        runs.append(sc.score(hidden, off)["entropy"].cpu().numpy())
    sc.close()
    assert np.array_equal(*runs)
    assert np.abs(runs[0] - oracle.entropy(w.hidden, w.w_lm)).max() <= 2e-5
    # rows of the last, partly filled fragment are counted by their numbers: NaN there reaches every token
    broken = td(w.w_lm)
    broken[V - 1] = float("nan")
    sc = gpu.Scorer(broken, gpu.make_head(td(w.w1), td(w.w2)))
    assert np.isnan(sc.score(hidden, off)["entropy"].cpu().numpy()).all()
    sc.close()
