"""bf16 hidden states that the fused entropy kernels read where they are, two K steps at a time: rows that begin on and off a line of 128 bytes, K
that ends inside a pair of steps, blocks with one row, all rows and one more, sweeps that begin at any pair of steps; and
the same kernels on packed copies, where the plan keeps them.  Entropies against the fp64 oracle to fp32 grade (2e-5 nat, the bar of the tile
tests), and rows that share a line with a row of NaN and infinities."""
import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl


# (d, V, T, tokens per block, rows per tile, read where they are: tests/sanitize_host.cpp holds the rule to this column)
CASES = [
    (8, 4096, 1, 64, 128, True), (8, 4096, 65, 64, 128, True), (24, 5000, 63, 64, 128, True), (56, 4100, 64, 64, 128, True),
    (64, 33000, 33, 64, 128, True), (72, 4223, 129, 64, 128, True), (1032, 9000, 64, 64, 128, True), (2048, 4096, 40, 64, 128, True),
    (216, 5422, 338, 128, 64, True), (264, 16511, 65, 128, 64, True), (320, 33136, 128, 128, 64, True), (248, 33136, 66, 128, 64, True),
    (512, 17000, 100, 128, 64, True), (4184, 5774, 412, 128, 64, False), (3000, 50000, 127, 128, 64, False),
    (1000, 32000, 191, 192, 128, True), (1024, 32000, 192, 192, 128, True), (40, 52583, 565, 192, 128, True), (904, 70000, 130, 192, 128, True),
    (5216, 5414, 713, 192, 128, False),
    # narrow plans that stream W_lm past the cache, rows off the lines
    (4968, 28800, 11, 64, 128, False), (4968, 28800, 12, 64, 128, True), (4104, 33000, 36, 64, 128, True), (4104, 33000, 37, 64, 128, False),
    (4968, 28800, 64, 64, 128, False), (4968, 28600, 1, 64, 128, True), (4992, 28800, 64, 64, 128, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("d,V,T,block,rows,direct", CASES)
def test_rows_of_every_length_against_the_oracle(d, V, T, block, rows, direct):
    from paper_2602_11812_amd import binding as gpu
    p = gpu.egtp_launch_plan_query(gpu.EGTP_BF16, d, V, T)
    assert (p.tokens_per_block, p.rows_per_tile) == (block, rows)
    w = wl.make(wl.scaled(wl.SPECS["mid"], seed=9100 + T, B=1, d=d, V=V, d_h=16, lengths=(T,)))
    td = gpu.to_device
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    hidden, off = td(w.hidden), td(oracle.offsets_from_lengths((T,)))
    ws = sc.workspace(T, 1)
    runs = []
    for fill in (0, 255):
        ws.fill_(fill)
        runs.append(sc.score(hidden, off)["entropy"].cpu().numpy())
    assert np.array_equal(*runs)
    assert np.abs(runs[0] - oracle.entropy(w.hidden, w.w_lm)).max() <= 2e-5
    # a row that is not finite, its neighbours in memory and everything else bit for bit
    if T > 2:
        import torch
        bad = sorted({0, T // 2, min(T - 1, 63), T - 1})
        broken = hidden.clone()
        flat = broken.view(torch.int16)
        flat[bad] = 0x7fc0
        flat[bad, ::2] = 0x7f80
        got = sc.score(broken, off)["entropy"].cpu().numpy()
        assert not np.isfinite(got[bad]).any()
        assert np.array_equal(np.delete(got, bad), np.delete(runs[0], bad))
    sc.close()


@pytest.mark.gpu
@pytest.mark.parametrize("d,V,T", [(4096, 33000, 64), (4096, 33000, 40), (4096, 33000, 24), (4096, 33000, 5), (2048, 66000, 128), (2048, 66000, 173), (256, 5422, 338), (1024, 32000, 100)])
@pytest.mark.parametrize("shift", [8, 32, 56])
def test_views_that_begin_inside_a_line(d, V, T, shift):
    """Hidden states of whole lines whose first row is 16, 64 or 112 bytes into one, read where they are or packed: the bits of the aligned copy up to the order of the
    fp32 sums (2e-5 nat, the bar against the oracle), rows of NaN before and behind the view notwithstanding."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    torch.manual_seed(T)
    w_lm = (torch.randn(V, d, device="cuda") / d ** 0.5).bfloat16()
    sc = gpu.Scorer(w_lm, gpu.make_head(*(torch.zeros(s, d if s == 8 else 8, dtype=torch.bfloat16, device="cuda") for s in (8, 1))))
    around = torch.full((T * d + 128,), float("nan"), dtype=torch.bfloat16, device="cuda")
    view = around[shift:shift + T * d].view(T, d)
    hidden = torch.randn(T, d, device="cuda").bfloat16()
    view.copy_(hidden)
    off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    want, got = (sc.score(h, off)["entropy"] for h in (hidden, view))
    assert torch.isfinite(want).all() and (got - want).abs().max() <= 2e-5
    sc.close()
