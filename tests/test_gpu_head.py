"""The prediction head on its own: predictions against the oracle's head evaluated in fp64 on the GPU's own pooled
states.  Bar 2e-5 of the largest term: fp32 sums of at most d + d_h products (the bar of the fp32 training tests)."""
import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu


# fp32 head weights, states addressed through slots in no order: batch sizes around the tiles of layer 1 (16 / 32 / 64),
# rows of W1 around its 128-row tile, K elements that end inside a chunk of sixteen; one output, and output counts around
# the groups of five that a wave of layer 2 takes
@pytest.mark.parametrize("B,d,d_h,n_out", [(16, 132, 129, 6), (17, 132, 127, 1), (32, 520, 128, 5), (33, 36, 1, 20),
                                           (65, 1000, 257, 21), (130, 64, 66, 64), (3, 8, 5, 65)])
def test_fp32_head_through_slots(B, d, d_h, n_out):
    import torch
    from paper_2602_11812_amd import binding as gpu
    rng = np.random.default_rng(8000 + B)
    w = wl.make(wl.scaled(wl.SPECS["tiny"], seed=8100 + B, B=1, d=d, V=300, d_h=d_h, lengths=(B,)))
    f32 = lambda *s, std=1.0: (std * rng.standard_normal(s)).astype(np.float32)
    w1, w2 = f32(d_h, d, std=d ** -0.5), f32(n_out, d_h, std=d_h ** -0.5)
    b1, b2 = f32(d_h, std=0.1), f32(n_out, std=0.1)
    centers = (np.arange(n_out, dtype=np.float32) + 0.5) * 100.0 if n_out > 1 else None
    td = gpu.to_device
    head = gpu.make_head(td(w1), td(w2), td(b1), td(b2), None if centers is None else td(centers))
    sc = gpu.Scorer(td(w.w_lm), head)
    S = B + 9
    slot = rng.permutation(S)[:B].astype(np.int32)
    pooled, lse = td(f32(S, d)), td(rng.uniform(5.0, 9.0, S).astype(np.float32))
    got = sc.step(td(w.hidden), pooled, lse, slot_dev=td(slot)).cpu().numpy().astype(np.float64)
    x = pooled.cpu().numpy()[slot].astype(np.float64)
    want = oracle.predict(x, oracle.Head(w1, w2, b1, b2, centers))
    scale = float(centers.max()) if n_out > 1 else 1.0 + float(np.abs(want).max())
    assert np.abs(got - want).max() <= 2e-5 * scale
    sc.close()


# bf16 head weights on the matrix cores: batches around tiles of 64 sequences, rows of W1 around 16 and 128, slices of d that end
# inside a K step of 32 (a chunk of eight, three, one step and a chunk), slices past the end of d; fp32 weights
# whose slices fill the compute units' rounds (320 tiles in two rounds became 240 in one)
@pytest.mark.parametrize("wdtype,B,d,d_h", [("bf16", 1, 8, 1), ("bf16", 64, 24, 130), ("bf16", 65, 40, 127),
                                            ("bf16", 129, 264, 17), ("bf16", 3, 4104, 9), ("bf16", 200, 1160, 300),
                                            ("bf16", 513, 544, 129), ("f32", 300, 2564, 1161), ("f32", 513, 1284, 1290)])
def test_layer1_on_matrix_cores_at_tile_edges(wdtype, B, d, d_h):
    import torch
    from paper_2602_11812_amd import binding as gpu
    gen = torch.Generator(device="cuda").manual_seed(8300 + B)
    rnd = lambda *s, std=1.0: torch.randn(*s, generator=gen, device="cuda") * std
    store = torch.bfloat16 if wdtype == "bf16" else torch.float32
    w1, w2 = rnd(d_h, d, std=d ** -0.5).to(store), rnd(1, d_h, std=d_h ** -0.5).to(store)
    sc = gpu.Scorer(rnd(300, d).bfloat16() if d % 8 == 0 else rnd(300, d), gpu.make_head(w1, w2))
    hidden, pooled = rnd(B, d).to(sc.storage), rnd(B, d)
    got = sc.step(hidden, pooled, torch.full((B,), 6.0).cuda()).double()
    want = torch.relu(pooled.double() @ w1.double().T) @ w2.double()[0]
    assert (got - want).abs().max() <= 2e-5 * (1.0 + want.abs().max())
    sc.close()
