"""The pooling merges the fused kernel's partial triples for its units' tokens: from one range to more than a batch of loads per
thread, in units of 16 to 256, with every ragged last unit -- and for tokens that no sequence holds, which get their
entropies all the same.  A batch whose units do not fit behind the triples (many empty sequences) merges them in a launch
of its own.  Against the fp64 oracle, entropies to fp32 grade (2e-5 nat, the bar of the fp32 tests)."""
import numpy as np
import pytest

import oracle
from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _batch(dtype, d, V, lens, seed):
    from paper_2602_11812_amd import binding as gpu
    w = wl.make(wl.scaled(wl.SPECS["tiny" if dtype == "f32" else "mid"], seed=seed, B=len(lens), d=d, V=V, d_h=16,
                          lengths=lens))
    sc = gpu.Scorer(gpu.to_device(w.w_lm), gpu.make_head(gpu.to_device(w.w1), gpu.to_device(w.w2)))
    return w, sc


@pytest.mark.parametrize("dtype,d,V,lens", [
    ("bf16", 64, 200, (5, 0, 37)), ("bf16", 64, 5000, (1,)), ("bf16", 96, 32000, (15, 16, 17, 0, 100)),
    ("f32", 36, 40000, (63, 2)), ("bf16", 64, 151936, (64,)), ("bf16", 32, 9000, (8200, 31, 33)),
    ("f32", 8, 3000, (33, 34001, 129)), ("bf16", 8, 2600, (66001, 255, 257, 0)),
    ("bf16", 8, 700, (1, 0, 0, 0, 0) * 400), ("bf16", 8, 20000, (1, 0, 0, 0, 0) * 400)])
def test_entropies_of_every_unit(dtype, d, V, lens):
    from paper_2602_11812_amd import binding as gpu
    w, sc = _batch(dtype, d, V, lens, 8100 + len(lens) + d)
    hidden, off = gpu.to_device(w.hidden), sc.build_offsets(gpu.to_device(np.asarray(lens, np.int32)), w.T)
    ws = sc.workspace(w.T, len(lens))
    runs = []
    for fill in (0, 255):           # whatever the workspace held before, the bits are the same
        ws.fill_(fill)
        out = sc.score(hidden, off)
        runs.append({k: out[k].cpu().numpy() for k in ("entropy", "pooled", "lse")})
    sc.close()
    for k in runs[0]:
        assert np.array_equal(runs[0][k], runs[1][k]), k
    some = np.unique(np.r_[:min(w.T, 600), max(0, w.T - 600):w.T])
    assert np.abs(runs[0]["entropy"][some] - oracle.entropy(w.hidden[some], w.w_lm)).max() <= 2e-5
    assert np.isfinite(runs[0]["entropy"]).all()


@pytest.mark.parametrize("first,last", [(0, 700), (0, 512), (37, 700), (37, 690), (64, 701), (701, 701), (0, 0), (700, 701)])
def test_tokens_that_no_sequence_holds(first, last):
    """A table may begin after 0 or end before T (rows kept for later): those tokens belong to no sequence and have entropies."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    w, sc = _batch("bf16", 64, 3000, (701,), 8200)
    hidden = gpu.to_device(w.hidden)
    cuts = [first, (first + last) // 2, (first + last) // 2, last]
    out = sc.score(hidden, torch.tensor(cuts, dtype=torch.int32).cuda())
    H = out["entropy"].cpu().numpy()
    assert np.abs(H - oracle.entropy(w.hidden, w.w_lm)).max() <= 2e-5
    for b in range(3):              # the sequences' own pooling is that of their tokens alone
        h = H[cuts[b]:cuts[b + 1]].astype(np.float64)
        want = np.zeros(64) if h.size == 0 else \
            (np.exp(h - h.max())[:, None] * gpu_rows(w.hidden, cuts[b], cuts[b + 1])).sum(0) / np.exp(h - h.max()).sum()
        assert np.linalg.norm(out["pooled"][b].cpu().numpy() - want) <= 1e-5 * max(np.linalg.norm(want), 1e-30)
    sc.close()


def gpu_rows(hidden, a, b):
    """Rows of a batch in fp64, whatever it is stored in."""
    from paper_2602_11812_amd import binding as gpu
    return gpu.to_device(hidden[a:b]).double().cpu().numpy()


@pytest.mark.parametrize("cuts", [(0, 500, 100, 701), (0, 701, 0, 701), (0, 600, 650, 20, 30), (-1000, 300, 701), (-6, 300, 701),
                                  (-2000, -900, -30), (900, 0, 650, 701), (0, 701) + (0,) * 2100, (0,) * 2100 + (701, 690)])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 2052)])
def test_entropies_do_not_depend_on_the_table(dtype, d, cuts):
    """A device table that decreases or begins below 0 gives meaningless sequences (the kernels clamp every index into the batch),
    but the entropies are those of the tokens."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    w, sc = _batch(dtype, d, 3000, (701,), 8300)
    hidden = gpu.to_device(w.hidden)
    good = sc.score(hidden, torch.tensor([0, 701], dtype=torch.int32).cuda())["entropy"].cpu().numpy()
    B = len(cuts) - 1
    out = [torch.full(n, float("nan"), device="cuda") for n in ((701,), (B, d), (B,), (B,))]
    gpu.egtp_score(sc.ctx, hidden, torch.tensor(cuts, dtype=torch.int32).cuda(), None, B, 701, sc.workspace(701, B), *out)
    H = out[0].cpu().numpy()
    sc.close()
    assert np.abs(good - oracle.entropy(w.hidden, w.w_lm)).max() <= 2e-5
    assert np.abs(H - good).max() <= 1e-6  # (units of another size merge the triples in another order)
