"""fp32 operands read by their pieces (few tokens): the narrow kernel, whose fragments of a piece serve several products, and
one or two token blocks of the stream kernel, which walks the products of a K step in turn; three blocks, which do not.
One K step of pieces, an odd and an even number of them, ranges of one and of several tiles, ragged last blocks.  Entropies
against the fp64 oracle to the fp32 bar (2e-5 nat), of Gaussian operands and of ones whose logits are exact and move the
entropies well past the bar if any of the six piece products is dropped or doubled (test_piece_operands.py)."""
import numpy as np
import pytest

import oracle
from helpers import piece_operands
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    (4, 257, 1, 64, 1), (36, 257, 65, 64, 1), (4, 16500, 65, 64, 2), (100, 33000, 64, 64, 2), (4, 33000, 257, 64, 6), (1024, 1025, 64, 64, 1),
    (96, 16500, 65, 128, 2), (36, 33000, 128, 128, 3), (96, 60001, 65, 128, 4), (36, 16500, 193, 128, 3), (96, 9000, 256, 128, 2),
    (36, 16500, 257, 128, 4),
    (4, 33000, 129, 192, 2), (36, 45001, 257, 192, 3), (4, 60001, 257, 192, 4),
]


@pytest.mark.parametrize("d,V,T,block,per_range", CASES)
def test_against_the_oracle(d, V, T, block, per_range):
    import torch
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.egtp_launch_plan_query(gpu.EGTP_F32, d, V, T)
    assert (plan.tokens_per_block, plan.tiles_per_range) == (block, per_range)
    w = wl.make(wl.scaled(wl.SPECS["tiny"], seed=9500 + T + d, B=1, d=d, V=V, d_h=16, lengths=(T,)))
    off = torch.tensor([0, T], dtype=torch.int32).cuda()
    td = gpu.to_device
    for hidden, w_lm in ((w.hidden, w.w_lm), *piece_operands(np.random.default_rng(9600 + T), T, V, d)):
        sc = gpu.Scorer(td(w_lm), gpu.make_head(td(w.w1), td(w.w2)))
        ws = sc.workspace(T, 1)
        runs = []
        for fill in (0, 255):
            ws.fill_(fill)
            runs.append(sc.score(td(hidden), off)["entropy"].cpu().numpy())
        sc.close()
        assert np.array_equal(*runs)
        assert np.abs(runs[0] - oracle.entropy(hidden, w_lm)).max() <= 2e-5
