"""fp32 products as bf16 pieces in the head: layer 1 of more than 64 sequences (tiles of 64 and of 128 columns; up to 2^24 products,
counted in tiles of 64 x 64, the fp32 instructions) and W1's gradient from 160 samples on (256 where it has at most 128 tiles).  A step each at the edges of their tiles against the fp64 oracle, to the bars of the fp32
training tests: batches one past and one short of a tile, rows of W1 off the 128-row tile, slices of d that end inside a K
step of 32, samples that end inside one.  Sums of a single product, which show every piece product; operands and results that
are not finite."""
import numpy as np
import pytest

import oracle
from helpers import rel_l2
from paper_2602_11812_amd import workloads as wl
from test_gpu_training import (HYPER, NAMES, _Bar, _gpu_step, _oracle_head, _run_steps, _trainer, _weights,  # noqa: F401
                               gpu)  # (the fixture)

pytestmark = pytest.mark.gpu


# layer 1 in tiles of 128 columns (slices of 288) and the gradient; the same with tiles of 64 and one sample past a K step;
# a single K step, two, and columns of W1 that end off every tile; the fp32 instructions with a single slice and at their last size,
# pieces at the next, with two K steps, with slices that end inside one
@pytest.mark.parametrize("B,d,d_h,K", [(449, 1028, 2044, 5), (193, 4100, 136, 3), (66, 36, 260, 2), (127, 68, 128, 20),
                                       (223, 2052, 516, 9), (128, 512, 256, 20), (128, 512, 257, 3), (70, 36, 4100, 2),
                                       (65, 520, 516, 4)])
def test_one_step_at_tile_edges(gpu, B, d, d_h, K):  # noqa: F811
    _run_steps(gpu, wl.make_train(4200 + B, B=B, d=d, d_h=d_h, K=K), 1)


# The samples' kernel leaves d loss / d pre-activation as fragments of pieces: the first batches of the two rules and the last before them;
# samples that end one past and one short of a K step, of the eight of a lane and of the groups of one, two and four of a workgroup; rows off
# the 16 of a fragment and the 128 of a tile, fewer than four; bins off the 32 x 16 tiles of W2's gradient and fewer than four
@pytest.mark.parametrize("B,d,d_h,K", [(160, 4100, 257, 33), (159, 4100, 257, 33), (161, 1044, 1025, 3), (256, 36, 5, 2), (255, 36, 5, 2),
                                       (257, 64, 130, 20), (287, 260, 3, 17), (511, 68, 2, 32), (513, 132, 1, 65), (519, 32, 127, 31),
                                       (1023, 4, 129, 16), (300, 128, 16384, 2)])
def test_one_step_on_ready_pieces(gpu, B, d, d_h, K):  # noqa: F811
    # (the bars of _run_steps, without its share of elements for which they are tight: of a W1 of 20 to 516 elements it
    # counts the two or three whose gradient happens to be near zero)
    ts = wl.make_train(5200 + B, B=B, d=d, d_h=d_h, K=K)
    hp = {k: float(np.float32(v)) for k, v in HYPER.items()}
    tr, oh, bar = _trainer(gpu, ts), _oracle_head(ts), _Bar(_oracle_head(ts).params())
    wgt = _weights(ts)
    loss, gs = oracle.head_loss_grad(ts.x, ts.bins, ts.y, oh, hp["lam"], wgt)
    oracle.train_step(ts.x, ts.bins, ts.y, oh, hp["lam"], hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["weight_decay"], wgt)
    bar.add_step(oh, gs, hp, 1)
    assert np.all(np.abs(_gpu_step(gpu, tr, ts) - loss) <= 2e-5 * np.abs(loss) + 1e-12)
    for i, n in enumerate(NAMES):
        got = tr.grads[n].cpu().numpy()
        assert rel_l2(got, gs[i]) <= 2e-5, n
        assert np.all(got[gs[i] == 0.0] == 0.0), n
        assert (np.abs(tr.params[n].cpu().numpy() - oh.params()[i]) <= bar.tol[i]).all(), n


@pytest.mark.parametrize("B,d,d_h", [(130, 64, 70), (130, 1028, 129)])
def test_infinite_feature_stays_in_its_sequence(gpu, B, d, d_h):  # noqa: F811
    """An infinite pooled feature makes its own sequence's prediction non-finite and leaves the others' bits alone."""
    import torch
    rng = np.random.default_rng(8200)
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


# The fp32 matrix instructions; pieces in tiles of 128 columns, in tiles of 64, and a slice that ends inside a step of 32; bf16
# weights.
@pytest.mark.parametrize("B,d,d_h,bf16", [(64, 64, 70, False), (65, 64, 70, False), (130, 36, 129, False), (449, 1028, 2044, False),
                                          (129, 512, 192, False), (65, 520, 516, False), (70, 36, 4100, False),
                                          (40, 40, 17, True), (129, 264, 130, True)])
def test_operands_that_are_not_finite(gpu, B, d, d_h, bf16):  # noqa: F811
    """An infinite weight or feature gives what IEEE arithmetic gives, whatever the batch size and however few bits the other
    factors have (pieces that are zero); finite values at the end of the range stay finite."""
    import torch
    rng = np.random.default_rng(8700 + B)
    f32 = lambda *s, std=1.0: (std * rng.standard_normal(s)).astype(np.float32)
    td = gpu.to_device
    few_bits = lambda a: (a.view(np.uint32) & 0xffff0000).view(np.float32)
    store = torch.bfloat16 if bf16 else torch.float32
    w_lm, hidden, w2 = td(f32(300, d, std=d ** -0.5)), td(np.zeros((B, d), np.float32)), td(f32(1, d_h)).to(store)
    lse = td(np.full(B + 5, 80.0, np.float32))  # the new tokens add nothing: the states stay as they are
    k, big = d - 3, 3.4e38                  # (past the largest bf16 value)
    for place, value in (("w1", np.inf), ("w1", -np.inf), ("x", np.inf), ("x", -np.inf), ("w1", big), ("x", big)):
        if bf16 and (place, value) == ("w1", big):
            continue  # not a bf16 value
        w1, x = f32(d_h, d, std=d ** -0.5), f32(B, d)
        if place == "w1":
            x[:, k] *= np.float32(2.0 ** -100 if value == big else 1.0)
            w1[d_h - 2, k] = value
        else:
            w1[:, k] *= np.float32(2.0 ** -100 if value == big else 1.0)
            w1 = few_bits(w1)
            x[B - 2, k] = value
        w1 = td(w1).to(store)
        slot = rng.permutation(B + 5)[:B].astype(np.int32)
        sc, states = gpu.Scorer(w_lm, gpu.make_head(w1, w2)), np.zeros((B + 5, d), np.float32)
        states[slot] = x
        states = td(states)
        got = sc.step(hidden, states, lse.clone(), slot_dev=td(slot)).cpu().numpy().astype(np.float64)
        sc.close()
        assert np.array_equal(states.cpu().numpy()[slot], x)
        with np.errstate(all="ignore"):
            want = oracle.predict(x.astype(np.float64), oracle.Head(w1.float().cpu().numpy(), w2.float().cpu().numpy()))
        ok = np.isfinite(want)
        assert ok.all() == (value == big)
        assert np.array_equal(got[~ok], want[~ok], equal_nan=True), (place, value)
        assert (np.abs(got[ok] - want[ok]) <= 2e-5 * (1.0 + np.abs(want[ok]))).all(), (place, value)


@pytest.mark.parametrize("B,d_h", [(66, 260), (257, 516), (70, 4100)])
def test_diverged_head_shows_in_the_loss(gpu, B, d_h):  # noqa: F811
    ts = wl.make_train(4700 + B, B=B, d=36, d_h=d_h, K=3)
    ts.w1[5, 7] = np.inf
    ts.w1[9, 7] = -np.inf
    tr = _trainer(gpu, ts)
    assert np.isnan(_gpu_step(gpu, tr, ts)).all()


def test_gradient_beyond_the_range_is_infinite(gpu):  # noqa: F811
    """A unit's pre-activation gradient that overflows makes its row of W1's gradient infinite, not NaN, where the features
    have few bits, and leaves the other rows alone."""
    B, d, d_h, j = 195, 2052, 516, 77
    ts = wl.make_train(4800, B=B, d=d, d_h=d_h, K=3)
    rng = np.random.default_rng(4801)
    ts.x[:] = rng.choice(np.float32([0.5, 1.0, 2.0]), ts.x.shape)
    ts.y[:] = 1e6
    ts.w1[j] = 0.0
    ts.b1[j], ts.w2[0, j], ts.w2[1:, j] = 1e-38, 3e38, 0.0
    _, gs = oracle.head_loss_grad(ts.x, ts.bins, ts.y, _oracle_head(ts), float(np.float32(0.95)), None)
    assert (gs[0][j] > 1e39).all()
    tr = _trainer(gpu, ts)
    _gpu_step(gpu, tr, ts)
    got = tr.grads["w1"].cpu().numpy().astype(np.float64)
    assert np.all(got[j] == np.inf)
    rest = np.arange(d_h) != j
    assert rel_l2(got[rest], gs[0][rest]) <= 2e-5


def _full(rng, *shape):
    """Values of either sign whose mantissas fill every piece: low bits all set, or any."""
    bits = rng.integers(0, 1 << 23, shape).astype(np.uint32)
    bits = np.where(rng.random(shape) < 0.5, bits | np.uint32(0xffff), bits) | np.uint32(0x3f800000)
    return bits.view(np.float32) * rng.choice(np.float32([-0.5, 1.0, 2.0]), shape)


# A sum of one product shows every piece product: the smallest that is kept is of size 2^-16, and what is dropped and rounded
# may come to 4 x 2^-24 (pieces rounded to nearest drop at most 2^-24 of a product; of six sums few round).
ONE_PRODUCT = 2.0 ** -22


# the fp32 instructions; pieces in tiles of 64 columns; of 128; bf16 weights
@pytest.mark.parametrize("B,d,d_h,bf16", [(65, 64, 260, False), (130, 520, 129, False), (65, 520, 516, False), (70, 36, 4100, False),
                                          (449, 1028, 2044, False),
                                          (66, 264, 130, True)])
def test_single_products_of_layer_1(gpu, B, d, d_h, bf16):  # noqa: F811
    import torch
    rng = np.random.default_rng(8800 + B)
    td = gpu.to_device
    w1 = np.zeros((d_h, d), np.float32)
    at = rng.integers(0, d, d_h)
    w1[np.arange(d_h), at] = np.abs(_full(rng, d_h))
    store = td(w1).to(torch.bfloat16 if bf16 else torch.float32)
    w1 = store.float().cpu().numpy()
    x = np.abs(_full(rng, B, d))
    w_lm, hidden = td(rng.standard_normal((300, d)).astype(np.float32)), td(np.zeros((B, d), np.float32))
    for j in (0, 17, 35, 63, 64, 101, 127, d_h - 1):
        w2 = torch.zeros(1, d_h, device="cuda", dtype=store.dtype)
        w2[0, j] = 1.0
        sc, state = gpu.Scorer(w_lm, gpu.make_head(store, w2)), td(x)
        got = sc.step(hidden, state, td(np.full(B, 80.0, np.float32))).cpu().numpy().astype(np.float64)
        sc.close()
        assert np.array_equal(state.cpu().numpy(), x)
        want = x[:, at[j]].astype(np.float64) * w1[j, at[j]].astype(np.float64)
        assert (np.abs(got - want) <= ONE_PRODUCT * want).all(), (j, np.abs(got / want - 1.0).max())


@pytest.mark.parametrize("B,d,d_h", [(193, 2052, 516), (449, 1028, 1020)])
def test_single_products_of_the_gradient(gpu, B, d, d_h):  # noqa: F811
    """Every hidden unit is active in one sample (which a column of its own names), so that an element of W1's gradient is one
    product, of a feature and of the unit's element of b1's gradient."""
    ts = wl.make_train(4900 + B, B=B, d=d, d_h=d_h, K=5)
    rng = np.random.default_rng(4950 + B)
    own = np.arange(d_h) % B
    rng.shuffle(own)
    ts.x[:, B:] = _full(rng, B, d - B)
    ts.x[:, :B] = np.eye(B)
    ts.w1[:] = 0.0
    ts.w1[np.arange(d_h), own] = 2.0
    ts.b1[:] = -1.0
    tr = _trainer(gpu, ts)
    _gpu_step(gpu, tr, ts)
    b1, w1 = (tr.grads[n].cpu().numpy().astype(np.float64) for n in ("b1", "w1"))
    assert (b1 != 0.0).all()
    want = b1[:, None] * ts.x[own].astype(np.float64)
    assert (np.abs(w1 - want) <= ONE_PRODUCT * np.abs(want)).all(), np.abs(w1 / want - 1.0)[want != 0.0].max()
