"""The head behind layer 1 at its edges, scoring (layer 2) and training (the samples): rows of hidden units shorter than a
vector, not a multiple of one, at and past a pass of 256 and of 1024 columns; outputs at and past the rows that a round of waves takes;
batches where workgroups take one, two or four sequences with some missing from the last; the longest rows.  Bars: the fp32
bars of the head and training tests (2e-5 of the largest term; fp32 sums of d + d_h products); bf16 weights are exact in
both."""
import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl
from test_gpu_training import _run_steps, gpu  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B,d,d_h,n_out", [(3, 16, 1, 1), (2, 16, 3, 2), (5, 16, 4, 1), (257, 16, 5, 33), (515, 16, 1023, 1),
                                           (514, 24, 1025, 16), (9, 520, 4099, 1), (258, 16, 2050, 65), (2, 16, 16383, 1024),
                                           (515, 16, 2, 1), (259, 16, 3, 33), (65, 2048, 253, 17), (258, 16, 256, 1), (517, 16, 255, 70),
                                           (3, 520, 257, 1)])
def test_scoring(gpu, B, d, d_h, n_out, bf16):  # noqa: F811
    import torch
    rng = np.random.default_rng(9000 + B + d_h)
    f32 = lambda *s, std=1.0: (std * rng.standard_normal(s)).astype(np.float32)
    td = gpu.to_device
    w1, w2 = td(f32(d_h, d, std=d ** -0.5)), td(f32(n_out, d_h, std=d_h ** -0.5))
    if bf16:
        w1, w2 = w1.to(torch.bfloat16), w2.to(torch.bfloat16)
    b1, b2 = f32(d_h, std=0.1), f32(n_out, std=0.1)
    centers = (np.arange(n_out, dtype=np.float32) + 0.5) * 100.0 if n_out > 1 else None
    head = gpu.make_head(w1, w2, td(b1), td(b2), None if centers is None else td(centers))
    sc = gpu.Scorer(td(f32(300, d, std=d ** -0.5)), head)
    pooled, lse = td(f32(B, d)), td(rng.uniform(5.0, 9.0, B).astype(np.float32))
    got = sc.step(td(f32(B, d)), pooled, lse).cpu().numpy().astype(np.float64)
    want = oracle.predict(pooled.cpu().numpy().astype(np.float64),
                          oracle.Head(w1.float().cpu().numpy(), w2.float().cpu().numpy(), b1, b2, centers))
    scale = float(centers.max()) if n_out > 1 else 1.0 + float(np.abs(want).max())
    assert np.abs(got - want).max() <= 2e-5 * scale
    sc.close()


@pytest.mark.parametrize("B,d,d_h,K", [(2, 12, 1, 3), (3, 12, 3, 33), (258, 12, 1027, 21), (514, 12, 6, 40), (5, 12, 2049, 65),
                                       (515, 12, 2, 9), (259, 12, 255, 33), (70, 1024, 256, 21), (601, 12, 253, 90), (2, 12, 257, 5)])
def test_training(gpu, B, d, d_h, K):  # noqa: F811
    _run_steps(gpu, wl.make_train(9200 + B, B=B, d=d, d_h=d_h, K=K), 1)


def test_infinite_weight_meets_its_own_hidden_unit_only(gpu):  # noqa: F811
    """The last four columns of a row are loaded together where its length is no multiple of four: a weight that is infinite
    there makes the prediction infinite, not NaN."""
    rng = np.random.default_rng(9300)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    td = gpu.to_device
    d, d_h = 16, 1027
    w2 = np.abs(f32(1, d_h))
    w2[0, d_h - 4:] = np.inf
    b1 = np.full(d_h, 50.0, np.float32)  # every hidden unit is active
    sc = gpu.Scorer(td(f32(300, d)), gpu.make_head(td(0.1 * f32(d_h, d)), td(w2), td(b1), td(f32(1))))
    got = sc.step(td(f32(3, d)), td(f32(3, d)), td(np.full(3, 6.0, np.float32))).cpu().numpy()
    assert np.all(got == np.inf)
    sc.close()
