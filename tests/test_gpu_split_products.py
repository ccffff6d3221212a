"""fp32 products as bf16 pieces in the head: layer 1 of more than 64 sequences (tiles of 64 and of 128 columns) and W1's
gradient from 192 samples on.  A step each at the edges of their tiles against the fp64 oracle, to the bars of the fp32
training tests: batches one past and one short of a tile, rows of W1 off the 128-row tile, slices of d that end inside a K
step of 32, samples that end inside one."""
import numpy as np
import pytest

from paper_2602_11812_amd import workloads as wl
from test_gpu_training import _run_steps, gpu  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


# layer 1 in tiles of 128 columns (slices of 288) and the gradient; the same with tiles of 64 and one sample past a K step;
# a single K step, two, and columns of W1 that end off every tile
@pytest.mark.parametrize("B,d,d_h,K", [(449, 1028, 2044, 5), (193, 4100, 136, 3), (66, 36, 260, 2), (127, 68, 128, 20),
                                       (223, 2052, 516, 9)])
def test_one_step_at_tile_edges(gpu, B, d, d_h, K):  # noqa: F811
    _run_steps(gpu, wl.make_train(4200 + B, B=B, d=d, d_h=d_h, K=K), 1)


def test_infinite_feature_stays_in_its_sequence(gpu):  # noqa: F811
    """An infinite pooled feature makes its own sequence's prediction non-finite and leaves the others' bits alone."""
    import torch
    rng = np.random.default_rng(8200)
    B, d, d_h = 130, 64, 70
    f32 = lambda *s, std=1.0: (std * rng.standard_normal(s)).astype(np.float32)
    td = gpu.to_device
    sc = gpu.Scorer(td(f32(300, d, std=d ** -0.5)), gpu.make_head(td(f32(d_h, d)), td(f32(1, d_h)), td(f32(d_h)), td(f32(1))))
    hidden, pooled, lse = td(f32(B, d)), td(f32(B, d)), torch.full((B,), 6.0).cuda()
    run = lambda p: sc.step(hidden, p.clone(), lse.clone()).cpu().numpy()
    clean = run(pooled)
    assert np.isfinite(clean).all()
    for b in (0, 64, 129):
        broken = pooled.clone()
        broken[b, b % d] = float("inf")
        got = run(broken)
        assert not np.isfinite(got[b])
        assert np.array_equal(np.delete(got, b), np.delete(clean, b)), b
    sc.close()
