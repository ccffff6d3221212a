"""Launch plans at the longest contractions that a context accepts (no device needed)."""
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
