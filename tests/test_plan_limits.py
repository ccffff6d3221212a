"""Launch plans at the longest contractions that a context accepts (no device needed)."""
import random

import pytest

from paper_2602_11812_amd import binding as gpu

# the longest contraction the fused kernels address, and the longest of which two packed row tiles still fit 2^31 bytes
LONGEST, LONGEST_PAIR = 4194240, 65535 // 2 * 2 * 32


@pytest.mark.parametrize("dtype,pieces", [(gpu.EGTP_BF16, 1), (gpu.EGTP_F32, 6)])
def test_kernels_are_planned_only_inside_the_contraction_they_address(dtype, pieces):
    def kinds(d):
        return {gpu.egtp_launch_plan_query(dtype, d, V, T).rows_per_tile
                for V in (512, 1000, 4096, 32000) for T in (1, 64, 128, 200, 384, 512, 1000, 5000)}

    inside = LONGEST_PAIR // pieces // 32 * 32
    assert 64 in kinds(inside)
    # 64-row tiles read two packed row tiles under one 32-bit byte offset
    for d in (inside + 96, LONGEST // pieces // 32 * 32):
        assert kinds(d) <= {128, 256}


def test_ranges_fit_the_workspace_and_follow_the_price():
    """Plans over the whole range of sizes: the ranges cover the vocabulary, none is empty, and their partial results stay within what a workspace holds for any batch up to
    theirs (8192 + 9 per block of 256 tokens).  And the lines where ranges of the 256 x 256 tile grow: short contractions only."""
    rng = random.Random(11)
    for _ in range(6000):
        dtype = rng.choice([gpu.EGTP_BF16, gpu.EGTP_F32])
        d, V, T = 8 * int(2 ** rng.uniform(0, 9.4)), int(2 ** rng.uniform(0, 18)), int(2 ** rng.uniform(0, 20))
        p = gpu.egtp_launch_plan_query(dtype, d, V, T)
        blocks = -(-T // 256)
        assert p.token_blocks == -(-T // p.tokens_per_block) and p.vocab_tiles == -(-V // p.rows_per_tile), (dtype, d, V, T)
        assert p.vocab_ranges == -(-p.vocab_tiles // p.tiles_per_range), (dtype, d, V, T)
        assert p.vocab_ranges * T <= (8192 + 9 * blocks) * 256 and p.vocab_ranges * p.token_blocks <= 8192 + 9 * blocks, (dtype, d, V, T)
    for T, d, V, tiles in ((7680, 256, 118784, 14), (9520, 640, 60646, 12), (38353, 1160, 43820, 3), (96402, 4816, 6113, 2), (94324, 936, 28213, 4)):
        p = gpu.egtp_launch_plan_query(gpu.EGTP_BF16, d, V, T)
        assert (p.rows_per_tile, p.tiles_per_range) == (256, tiles), (T, d, V, p.tiles_per_range)
    for T, d, V, rows in ((595, 872, 15403, 128), (1091, 616, 8145, 128), (168, 600, 113504, 128), (389, 232, 31206, 256), (1217, 4096, 151936, 256),
                          (105153, 3344, 65385, 64), (6338, 2608, 78554, 256)):
        assert gpu.egtp_launch_plan_query(gpu.EGTP_BF16, d, V, T).rows_per_tile == rows, (T, d, V)


def test_split_gradient_only_where_its_rows_fit_a_descriptor():
    """W1's gradient of large batches addresses eight samples of 4 d bytes by an offset that has to stay 16 bytes below 2^31: with d = 2^26 the last column of the
    last sample would not.  The workspace shows which kernel a batch takes: one of pieces holds 8 fragments of 3 KiB for each step of 32 samples, 120 KiB from 160 on."""
    def grows(d):
        small, large = (gpu.egtp_head_train_workspace_bytes(B, d, 1, 4) for B in (159, 160))
        return large - small >= 120 * 1024

    assert grows(1 << 20) and grows((1 << 26) - 4) and not grows(1 << 26)
