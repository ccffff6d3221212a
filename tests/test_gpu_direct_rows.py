"""bf16 hidden states that the fused entropy kernels read where they are, two K steps at a time: rows that begin on and off a line of 128 bytes, K
that ends inside a pair of steps, blocks with one row, all rows and one more, sweeps that begin at any pair of steps; and
the same kernels on packed copies, where the plan keeps them.  Entropies against the fp64 oracle to fp32 grade (2e-5 nat, the bar of the tile
tests), and rows that share a line with a row of NaN and infinities."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl


class _Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tb_tokens", "tile_v", "ntb", "ntiles_v", "nsplit", "tiles_per_split")]
    _fields_ += [(n, ctypes.c_bool) for n in ("whole_cohorts", "pieces", "direct")]


def _plan(d, V, T, dtype=None):
    from paper_2602_11812_amd import binding as gpu
    plan = gpu.load_library()._ZN4egtp7k1_planEilii
    plan.restype, plan.argtypes = _Plan, [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    return plan(gpu.EGTP_BF16 if dtype is None else dtype, T, d, V)


# (d, V, T, tokens per block, rows per tile, direct)
CASES = [
    (8, 4096, 1, 64, 128, True), (8, 4096, 65, 64, 128, True), (24, 5000, 63, 64, 128, True), (56, 4100, 64, 64, 128, True),
    (64, 33000, 33, 64, 128, True), (72, 4223, 129, 64, 128, True), (1032, 9000, 64, 64, 128, True), (2048, 4096, 40, 64, 128, True),
    (216, 5422, 338, 128, 64, True), (264, 16511, 65, 128, 64, True), (320, 33136, 128, 128, 64, True), (248, 33136, 66, 128, 64, True),
    (512, 17000, 100, 128, 64, True), (4184, 5774, 412, 128, 64, False), (3000, 50000, 127, 128, 64, False),
    (1000, 32000, 191, 192, 128, True), (1024, 32000, 192, 192, 128, True), (40, 52583, 565, 192, 128, True), (904, 70000, 130, 192, 128, True),
    (5216, 5414, 713, 192, 128, False),
]


def test_which_plans_read_directly():
    """The rule on both sides of its lines; never fp32 operands, the 256 x 256 tile or paced plans."""
    for T, d, V, direct in ((24, 4096, 151936, True), (64, 2568, 151936, True), (173, 4096, 151936, True), (173, 3000, 151936, False),
                            (128, 4096, 151936, True), (128, 3000, 50000, False), (100, 1192, 34235, True), (376, 4344, 115887, False),
                            (264, 1736, 104018, True), (412, 4184, 5774, False), (375, 3608, 9865, True), (512, 4096, 151936, False),
                            (137720, 4096, 151936, False), (65088, 5120, 151936, False)):
        assert _plan(d, V, T).direct == direct, (T, d, V)
    rng = np.random.default_rng(5)
    for _ in range(3000):
        d, V, T = 8 * int(2 ** rng.uniform(0, 9.4)), int(2 ** rng.uniform(0, 17.3)), int(2 ** rng.uniform(0, 17.1))
        p = _plan(d, V, T)
        paced = p.tiles_per_split > 16 and p.ntb >= 16
        assert not (p.direct and (p.tile_v == 256 or (p.tile_v == 64 and paced))), (d, V, T)
        assert p.direct or not (p.tile_v == 128 and p.tb_tokens == 64), (d, V, T)
        assert not _plan(d, V, T, 0).direct


@pytest.mark.gpu
@pytest.mark.parametrize("d,V,T,block,rows,direct", CASES)
def test_rows_of_every_length_against_the_oracle(d, V, T, block, rows, direct):
    from paper_2602_11812_amd import binding as gpu
    p = _plan(d, V, T)
    assert (p.tb_tokens, p.tile_v, p.direct) == (block, rows, direct)
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
