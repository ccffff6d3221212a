"""GPU parity of the head's training step (Eq. 5, 7, 9 + AdamW) against the fp64 oracle.

Bars (derived from the arithmetic: the GPU path keeps fp32 parameters, moments and sums):
  * loss terms and gradients: relative L2 <= 2e-5 per tensor;
  * moments after s steps: m relative L2 <= 5e-5, v <= 1e-4 (linear / quadratic in the gradients);
  * parameters: per element  |w_gpu - w_orc| <= sum over steps of (lr * u_tol + 2e-7 |w|), where
    the update u = mhat / (sqrt(vhat) + eps) of a step has the sensitivity-aware tolerance
        u_tol = min(4, 2 dg / (sqrt(vhat) + eps)) + 1e-4,   dg = max over steps so far of
        2e-5 |g| + 2e-6 rms(g):
    Adam divides by the gradient's own magnitude, so an element whose gradient is at the fp32
    noise floor has an update that fp32 cannot determine; everywhere else the bar is ~1e-4 lr.
    The tests also require that bar to be tight (< 1% of lr) for at least 99% of the elements
    and that the step moved the parameters by about lr, so a missing update cannot pass.
"""
import numpy as np
import pytest

import oracle
from helpers import assert_pred_close, rel_l2
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ("w1", "b1", "w2", "b2")
HYPER = dict(lam=0.95, lr=2e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2602_11812_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load_library()
    return binding


def _trainer(gpu, ts, keep_grads=True, **hyper):
    td = gpu.to_device
    hp = dict(HYPER, **hyper)
    return gpu.HeadTrainer(td(ts.w1), td(ts.b1), td(ts.w2), td(ts.b2), td(ts.centers), keep_grads=keep_grads, **hp)


def _oracle_head(ts):
    f = lambda a: np.array(a, dtype=np.float64)
    return oracle.TrainHead(f(ts.w1), f(ts.b1), f(ts.w2), f(ts.b2), f(ts.centers))


def _weights(ts):
    return None if ts.steps is None else 1.0 / (ts.n_seqs * ts.steps.astype(np.float64))


def _gpu_step(gpu, tr, ts, rows=None):
    td = gpu.to_device
    sl = slice(None) if rows is None else rows
    steps = None if ts.steps is None else td(np.ascontiguousarray(ts.steps[sl]))
    loss = tr.step(td(np.ascontiguousarray(ts.x[sl])), td(np.ascontiguousarray(ts.bins[sl])),
                   td(np.ascontiguousarray(ts.y[sl])), steps, ts.n_seqs)
    return loss.cpu().numpy().astype(np.float64)


class _Bar:
    """Running per-element bar of the module docstring: every step adds lr * u_tol + 2e-7 |w|, with
    u_tol from the largest gradient error so far and the oracle's second moment at that step."""

    def __init__(self, params):
        self.dg = [np.zeros_like(p) for p in params]
        self.tol = [np.zeros_like(p) for p in params]
        self.seen = [np.zeros(p.shape, dtype=bool) for p in params]

    def add_step(self, oh, gs, hp, s):
        tight = []
        for i, g in enumerate(gs):
            g_rms = float(np.sqrt(np.mean(np.square(g))))
            self.dg[i] = np.maximum(self.dg[i], 2e-5 * np.abs(g) + 2e-6 * g_rms)
            self.seen[i] |= g != 0.0
            vhat = oh.v[i] / (1.0 - hp["beta2"] ** s)
            u_tol = np.minimum(4.0, 2.0 * self.dg[i] / (np.sqrt(vhat) + hp["eps"])) + 1e-4
            u_tol[~self.seen[i]] = 1e-4     # exact zeros so far (dead units) are exact on both sides
            self.tol[i] += hp["lr"] * u_tol + 2e-7 * np.abs(oh.params()[i])
            tight.append(float(np.mean(u_tol < 1e-2)))
        return tight


def _check_params(tr, oh, bar, tight, gs, hp, w_before):
    for i, n in enumerate(NAMES):
        got = tr.params[n].cpu().numpy().astype(np.float64)
        want = oh.params()[i]
        bad = np.abs(got - want) > bar.tol[i]
        assert not bad.any(), f"{n}: {bad.sum()} elements off, worst {np.abs(got - want).max()}"
        assert tight[i] >= 0.99, f"{n}: bar is tight for only {tight[i]:.4f} of the elements"
        assert rel_l2(tr.m[n].cpu().numpy(), oh.m[i]) <= 5e-5
        assert rel_l2(tr.v[n].cpu().numpy(), oh.v[i]) <= 1e-4
        moved = np.abs(got - w_before[i])
        live = np.abs(gs[i]) > 1e-3 * np.sqrt(np.mean(np.square(gs[i])))
        assert np.median(moved[live]) >= 0.3 * hp["lr"], f"{n} did not move"


def _run_steps(gpu, ts, n_steps, batch=None, **hyper):
    # the C struct carries fp32 hyper-parameters: hand the oracle the same rounded values
    hp = {k: float(np.float32(v)) for k, v in dict(HYPER, **hyper).items()}
    tr = _trainer(gpu, ts, **hyper)
    oh = _oracle_head(ts)
    w_before = [p.copy() for p in oh.params()]
    bar = _Bar(w_before)
    B = ts.x.shape[0]
    for s in range(n_steps):
        rows = None
        if batch is not None:
            lo = (s * batch) % B
            rows = slice(lo, min(lo + batch, B))
        sl = slice(None) if rows is None else rows
        wgt = _weights(ts)
        loss_o, gs = oracle.head_loss_grad(ts.x[sl], ts.bins[sl], ts.y[sl], oh, hp["lam"],
                                           None if wgt is None else wgt[sl])
        loss_o2 = oracle.train_step(ts.x[sl], ts.bins[sl], ts.y[sl], oh, hp["lam"], hp["lr"], hp["beta1"],
                                    hp["beta2"], hp["eps"], hp["weight_decay"], None if wgt is None else wgt[sl])
        assert np.array_equal(loss_o, loss_o2)
        tight = bar.add_step(oh, gs, hp, s + 1)
        loss_g = _gpu_step(gpu, tr, ts, rows)
        assert np.all(np.abs(loss_g - loss_o) <= 2e-5 * np.abs(loss_o) + 1e-12), (loss_g, loss_o)
        for i, n in enumerate(NAMES):
            gg = tr.grads[n].cpu().numpy()
            r = rel_l2(gg, gs[i])
            assert r <= 2e-5, f"step {s}: grad {n} rel L2 {r}"
            assert np.all(gg[gs[i] == 0.0] == 0.0)
        _check_params(tr, oh, bar, tight, gs, hp, w_before)
    return tr, oh


def test_one_step_ragged_shapes(gpu):
    # d_h, B and K leave partial tiles everywhere (64-wide tiles, 16-sample stages)
    ts = wl.make_train(11, B=37, d=256, d_h=96, K=20)
    _run_steps(gpu, ts, 1)


def test_small_batch_ragged_slices_of_d(gpu):
    # at most 16 samples: layer 1 streams W1 in slices of at most 1024 elements of d, 16 head rows per workgroup;
    # d = 2308 leaves a last slice of 260 elements, d_h = 52 a last workgroup of 4 rows, B = 13 three empty columns
    ts = wl.make_train(16, B=13, d=2308, d_h=52, K=11)
    _run_steps(gpu, ts, 2)


def test_several_steps_minibatches(gpu):
    ts = wl.make_train(12, B=64, d=128, d_h=200, K=20)
    _run_steps(gpu, ts, 6, batch=16)


def test_larger_learning_rate_and_no_decay(gpu):
    ts = wl.make_train(13, B=33, d=64, d_h=70, K=7)
    _run_steps(gpu, ts, 4, lr=1e-3, weight_decay=0.0, lam=0.5)


def test_pure_cross_entropy_and_pure_mse(gpu):
    ts = wl.make_train(14, B=20, d=64, d_h=64, K=20)
    _run_steps(gpu, ts, 2, lam=1.0)
    _run_steps(gpu, ts, 2, lam=0.0)


def test_plp_step_average_weights(gpu):
    # Eq. 9: samples are decode steps of 9 sequences; each sequence's steps share its 1/N
    ts = wl.make_train(15, B=41, d=128, d_h=96, K=20, plp_seqs=9)
    assert abs(_weights(ts).sum() - 1.0) < 1e-12
    _run_steps(gpu, ts, 2)


def test_paper_batch_full_width(gpu):
    # batch of 16, d = 4096, d_h = 1024, K = 20: the shape the experimental setup trains at
    ts = wl.make_train(16, B=16, d=4096, d_h=1024, K=20)
    _run_steps(gpu, ts, 2)


def test_single_sample_and_single_bin(gpu):
    ts = wl.make_train(17, B=1, d=64, d_h=32, K=20)
    _run_steps(gpu, ts, 1)
    # K = 1: softmax of one logit is 1, yhat = c_1 whatever the parameters, every gradient is 0
    ts = wl.make_train(18, B=8, d=64, d_h=32, K=1)
    tr = _trainer(gpu, ts, weight_decay=0.0)
    before = {n: tr.params[n].clone() for n in NAMES}
    loss = _gpu_step(gpu, tr, ts)
    want_mse = np.mean((ts.y.astype(np.float64) - float(ts.centers[0])) ** 2)
    assert abs(loss[1]) <= 1e-6 and abs(loss[2] - want_mse) <= 1e-5 * want_mse
    for n in NAMES:
        assert float(tr.grads[n].abs().max()) == 0.0
        assert bool((tr.params[n] == before[n]).all())


def test_bit_reproducible(gpu):
    import torch
    ts = wl.make_train(19, B=50, d=256, d_h=128, K=20)
    outs = []
    for _ in range(2):
        tr = _trainer(gpu, ts)
        for _ in range(3):
            loss = _gpu_step(gpu, tr, ts)
        outs.append((loss, {n: tr.params[n].clone() for n in NAMES}))
    assert np.array_equal(outs[0][0], outs[1][0])
    for n in NAMES:
        assert torch.equal(outs[0][1][n], outs[1][1][n])


def test_loss_goes_down_and_trained_head_scores(gpu):
    # a few hundred steps at a visible learning rate: the joint loss falls, and the trained
    # parameters, used as a K-bin scoring head (Eq. 6), predict what the oracle's head predicts
    import torch
    ts = wl.make_train(20, B=64, d=64, d_h=64, K=20)
    tr = _trainer(gpu, ts, keep_grads=False, lr=2e-3)
    td = gpu.to_device
    x, bins, y = td(ts.x), td(ts.bins), td(ts.y)
    first = tr.step(x, bins, y).cpu().numpy().copy()
    for _ in range(300):
        last = tr.step(x, bins, y)
    last = last.cpu().numpy()
    assert last[0] < 0.7 * first[0] and last[1] < first[1]

    # score a ragged batch whose hidden states are such that pooling is trivial (one token per
    # sequence: pooled = the token), with the trained head; compare with the oracle's head on the
    # GPU-trained parameters
    w = wl.make(wl.scaled(wl.SPECS["tiny"], B=8, d=64, d_h=64, lengths=tuple([1] * 8)))
    p = {n: tr.params[n].cpu().numpy() for n in NAMES}
    sc = gpu.Scorer(td(w.w_lm), tr.as_head())
    off = torch.arange(9, dtype=torch.int32, device="cuda")
    out = sc.score(td(w.hidden), off)
    head = oracle.Head(p["w1"], p["w2"], p["b1"], p["b2"], ts.centers)
    want = oracle.egtp(w.hidden, np.arange(9, dtype=np.int32), w.w_lm, head)
    assert_pred_close(out["pred"].cpu().numpy(), want.pred)
    sc.close()


def test_argument_errors(gpu):
    import torch
    ts = wl.make_train(21, B=8, d=64, d_h=32, K=20)
    td = gpu.to_device
    x, bins, y = td(ts.x), td(ts.bins), td(ts.y)
    for bad, code in ((dict(lam=1.5), 9), (dict(lr=-1.0), 9), (dict(beta1=1.0), 9), (dict(beta2=-0.1), 9),
                      (dict(eps=0.0), 9), (dict(weight_decay=-1.0), 9)):
        tr = _trainer(gpu, ts, **bad)
        with pytest.raises(gpu.EgtpError) as e:
            tr.step(x, bins, y)
        assert e.value.status == code
    tr = _trainer(gpu, ts)
    before = tr.params["w1"].clone()
    h = tr._struct()
    h.t = 0
    ws = torch.empty(gpu.egtp_head_train_workspace_bytes(8, 64, 32, 20), dtype=torch.uint8, device="cuda")
    with pytest.raises(gpu.EgtpError) as e:
        gpu.egtp_head_train_step(h, x, bins, y, None, 0, 8, ws, tr.loss)
    assert e.value.status == 9
    h.t = 1
    with pytest.raises(gpu.EgtpError) as e:                      # workspace too small
        gpu.egtp_head_train_step(h, x, bins, y, None, 0, 8, ws[:256], tr.loss)
    assert e.value.status == 5
    with pytest.raises(gpu.EgtpError) as e:                      # missing targets
        gpu.egtp_head_train_step(h, x, bins, None, None, 0, 8, ws, tr.loss)
    assert e.value.status == 1
    with pytest.raises(gpu.EgtpError) as e:                      # step counts without a sequence count
        gpu.egtp_head_train_step(h, x, bins, y, bins, 0, 8, ws, tr.loss)
    assert e.value.status == 2
    h.d = 62
    with pytest.raises(gpu.EgtpError) as e:
        gpu.egtp_head_train_step(h, x, bins, y, None, 0, 8, ws, tr.loss)
    assert e.value.status == 2
    assert gpu.egtp_head_train_workspace_bytes(8, 62, 32, 20) == 0
    torch.cuda.synchronize()
    assert torch.equal(tr.params["w1"], before)                  # nothing was launched
    h.d = 64
    gpu.egtp_head_train_step(h, x, bins, y, None, 0, 0, None, None)   # B = 0: nothing to do


# The fp32 matrix kernels at the edges of their tiles: 17 and 32 samples (the smallest tile), 33 and 64 (the other one
# exactly full), 65 and 97 (a second tile; one and four samples past a stage of 32); rows of W1 around 64 and 128 and
# off the 16-byte grid, K slices that end inside a chunk of sixteen, bin counts around the four rows of W2 a workgroup takes
@pytest.mark.parametrize("B,d,d_h,K", [(17, 260, 63, 5), (32, 516, 64, 2), (33, 68, 65, 20), (64, 1028, 127, 4),
                                       (65, 252, 129, 33), (97, 4, 130, 9)])
def test_matrix_kernels_at_tile_edges(gpu, B, d, d_h, K):
    _run_steps(gpu, wl.make_train(4000 + B, B=B, d=d, d_h=d_h, K=K), 1)


# W2, b2 and b1: 32 samples of each of four waves at a time -- one chunk less a sample, full, one sample over, two chunks
# and a part; rows of W2 around the four a workgroup takes, columns around 64
@pytest.mark.parametrize("B,d_h,K", [(127, 65, 4), (128, 64, 5), (129, 63, 7), (300, 128, 3)])
def test_small_parameters_at_chunk_edges(gpu, B, d_h, K):
    _run_steps(gpu, wl.make_train(6000 + B, B=B, d=64, d_h=d_h, K=K), 1)


@pytest.mark.parametrize("eps", [1e-8, 1.1e-12, 1e-12, 9e-13, 1e-20, 1e-38])
def test_update_on_both_sides_of_the_quick_arithmetic(gpu, eps):
    """AdamW's update with the hardware's root and reciprocal (eps of 1e-10 and more) and without; gradients over 24 decades, and
    none at all (inactive units).  Against fp64 from the moments that the step left: the weight is rounded twice (2^-22 of it covers
    both), the update ten times within one unit in the last place each (2^-20)."""
    import torch
    B, d, d_h, K = 8, 64, 32, 4
    rng = np.random.default_rng(11)
    x = (rng.standard_normal((B, d)) * 10.0 ** rng.uniform(-12, 12, (1, d))).astype(np.float32)
    w1 = (rng.standard_normal((d_h, d)) * 1e-14).astype(np.float32)
    b1 = np.where(np.arange(d_h) < 16, 5.0, -5.0).astype(np.float32)
    w2, b2 = (rng.standard_normal((K, d_h)) * 0.1).astype(np.float32), np.zeros(K, np.float32)
    td = gpu.to_device
    tr = gpu.HeadTrainer(td(w1), td(b1), td(w2), td(b2), td(np.linspace(1, 4, K, dtype=np.float32)), lr=1e-2, weight_decay=0.1, eps=eps)
    tr.step(td(x), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.ones(B, device="cuda"))
    f = lambda t: t.cpu().numpy().astype(np.float64)
    m, v, got = f(tr.m["w1"]), f(tr.v["w1"]), f(tr.params["w1"])
    beta1, beta2, lr = (float(np.float32(t)) for t in (0.9, 0.999, 1e-2))
    update = lr * m / (1 - beta1) / (np.sqrt(v / (1 - beta2)) + float(np.float32(eps)))
    want = w1 - lr * float(np.float32(0.1)) * w1.astype(np.float64) - update
    assert np.isfinite(got).all() and (m[16:] == 0).all() and (m[:16] != 0).all()
    normal = (v == 0) | (v > 2.0 ** -126)  # a denormal second moment is known to its own step only
    assert normal.mean() > 0.8
    assert (np.abs(got - want) <= 2.0 ** -22 * np.abs(want) + 2.0 ** -20 * np.abs(update))[normal].all()


def _first_update(gpu, x, lr, eps, d_h=64):
    """One step from weights of zero without decay: W1, m, v as fp64, W1 being the negative update alone."""
    import torch
    B, d = x.shape
    K = 4
    rng = np.random.default_rng(12)
    td = gpu.to_device
    tr = gpu.HeadTrainer(td(np.zeros((d_h, d), np.float32)), td(np.full(d_h, 5.0, np.float32)), td((rng.standard_normal((K, d_h)) * 0.1).astype(np.float32)),
                         td(np.zeros(K, np.float32)), td(np.linspace(1, 4, K, dtype=np.float32)), lr=lr, weight_decay=0.0, eps=eps)
    tr.step(td(x), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.ones(B, device="cuda"))
    return [t["w1"].cpu().numpy().astype(np.float64) for t in (tr.params, tr.m, tr.v)]


@pytest.mark.parametrize("lr,eps,decades", [(1e-2, 1e-8, 0), (3e-4, 1e-8, 0), (1e-2, 1e-8, 3), (2e-5, 1e-6, 2), (1e-3, 1.1e-10, 0), (1e-3, 0.9e-10, 0), (1e-3, 0.9e10, 0), (1e-3, 1.1e10, 0)])
def test_update_is_no_less_exact_than_rounded_divisions(gpu, lr, eps, decades):
    """The update alone against fp64, beside lr mhat / (sqrt(vhat) + eps) with every operation of it rounded correctly, which numpy's fp32 is: never further off than the
    roundings of that form allow (5.5 of 2^-24), and no further by the root of the mean square (1 % for the sample of 260000)."""
    rng = np.random.default_rng(31)
    x = (rng.standard_normal((8, 4096)) * 10.0 ** rng.uniform(-decades, decades, (1, 4096))).astype(np.float32)
    got, m, v = _first_update(gpu, x, lr, eps)
    f32 = np.float32
    corr = [1.0 - float(f32(b)) for b in (0.9, 0.999)]
    exact = float(f32(lr)) * m / corr[0] / (np.sqrt(v / corr[1]) + float(f32(eps)))
    mhat, vhat = m.astype(f32) / f32(corr[0]), v.astype(f32) / f32(corr[1])
    rounded = (f32(lr) * mhat / (np.sqrt(vhat) + f32(eps))).astype(np.float64)
    kept = (v > 2.0 ** -126) & (np.abs(exact) > 2.0 ** -100)
    assert kept.mean() > 0.9
    off, off_rounded = ((t - exact)[kept] / exact[kept] * 2.0 ** 24 for t in (-got, rounded))
    assert np.abs(off).max() <= 5.5
    assert np.sqrt(np.mean(off ** 2)) <= 1.01 * np.sqrt(np.mean(off_rounded ** 2))


@pytest.mark.parametrize("eps", [1e-8, 1e-12])
def test_infinite_second_moments_leave_no_update(gpu, eps):
    """Gradients whose square is past fp32's range: the update is divided by infinity, in the quick arithmetic as in the other."""
    x = np.random.default_rng(3).standard_normal((8, 64)).astype(np.float32)
    x[:, 1::4] *= 1e26
    got, m, v = _first_update(gpu, x, 1e-2, eps)
    big = np.isinf(v)
    assert big[:, 1::4].mean() > 0.9 and not big[:, ::4].any() and np.isfinite(m).all()
    assert not got[big].any() and (got[:, ::4] != 0).all()
