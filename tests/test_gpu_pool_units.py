"""Ragged pooling cuts sequences into units of 16 to 256 tokens whose numbers follow from the offsets alone: small
batches of many kinds, in units of 16 to 64 (empty sequences at both ends and in rows, more sequences than are looked
through at once), lengths around the unit in every unit size, and a sequence of more units than the join keeps factors
for at a time; with and without an old state read and replaced through slots.  References in fp64 from the library's
own entropies (which other tests hold to the oracle): pooled 1e-5 relative L2, fp32 sums of at most 300 terms in a row
(a unit's tokens, then a quarter of the units) with weights accurate to a few 2^-24; lse 1e-5 absolute at |lse| < 20."""
import ctypes
import math

import numpy as np
import pytest

from paper_2602_11812_amd import workloads as wl

pytestmark = pytest.mark.gpu

RAGGED = {
    "one": (1,),
    "unit edges": (15, 16, 17, 0, 31, 32, 33, 63, 64, 65),
    "large unit edges": (127, 128, 129, 0, 0, 255, 256, 257, 1, 511, 513),
    "long": (9000, 3),
    "empty ends": (0, 0, 5, 0, 200, 0),
    "many": tuple([1, 0, 2] * 700),
    "very many": tuple([0, 1, 3, 0] * 600),
}


@pytest.mark.parametrize("dtype,d", [("bf16", 2056), ("bf16", 64), ("f32", 1028)])
@pytest.mark.parametrize("name", list(RAGGED))
def test_units_of_ragged_batches(name, dtype, d):
    _check_units(name, RAGGED[name], dtype, d)


def _unit(dtype, d, T, B):
    """Tokens per unit, from the library's own rule.  It may use as many floats of partials as the larger of the merged
    triples' and those of units of 256."""
    from paper_2602_11812_amd import binding as gpu
    lib = gpu.load_library()
    triples, unit = lib._ZN4egtp23k1_partial_floats_boundEl, lib._ZN4egtp9pool_unitEiilim
    triples.restype, triples.argtypes = ctypes.c_size_t, [ctypes.c_int64]
    unit.restype, unit.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.c_size_t]
    cap = max(triples(T), (T // 256 + B) * (d + 2))
    return unit(gpu.EGTP_BF16 if dtype == "bf16" else gpu.EGTP_F32, d, T, B, cap)


# A long sequence in the middle makes the batch large enough for the unit; around it lengths one below, at and one above
# one and two units, starting at multiples of the unit and off them
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 36)])
@pytest.mark.parametrize("unit,long", [(16, 0), (32, 8200), (64, 17001), (128, 34001), (256, 66001)])
def test_lengths_around_every_unit(unit, long, dtype, d):
    edges = [k * unit + e for k in (1, 2) for e in (-1, 0, 1)]
    lens = (*edges, 0, 0, long, *edges[::-1], 1)
    assert _unit(dtype, d, sum(lens), len(lens)) == unit
    _check_units(f"units of {unit}", lens, dtype, d)


# 270 000 tokens are 1055 units of 256; the join keeps the factors of 1024
@pytest.mark.parametrize("dtype,d", [("bf16", 8), ("f32", 4)])
def test_more_units_in_a_sequence_than_factors_are_kept(dtype, d):
    lens = (300, 270000, 5)
    assert _unit(dtype, d, sum(lens), len(lens)) == 256
    _check_units("chunked join", lens, dtype, d)


def _check_units(name, lens, dtype, d):
    import torch
    from paper_2602_11812_amd import binding as gpu
    B, T = len(lens), sum(lens)
    w = wl.make(wl.scaled(wl.SPECS["mid" if dtype == "bf16" else "tiny"], seed=9000 + B, B=B, d=d, V=40, d_h=8, lengths=lens))
    td = gpu.to_device
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    off_dev = td(off.astype(np.int32))
    hidden = td(w.hidden)
    h = hidden.cpu().double().numpy()
    ws = sc.workspace(T, B)

    ws.fill_(255)
    out = {k: v.cpu().numpy().astype(np.float64) for k, v in sc.score(hidden, off_dev).items()}
    H = out["entropy"]
    rng = np.random.default_rng(B)
    S = B + 5
    slot = rng.permutation(S)[:B].astype(np.int32)
    old_p, old_l = rng.standard_normal((S, d)).astype(np.float32), rng.uniform(1.0, 6.0, S).astype(np.float32)
    old_l[slot[::3]] = -math.inf                                  # some states are empty
    new_p, new_l = td(old_p.copy()), td(old_l.copy())
    ws.fill_(255)
    sc.step(hidden, new_p, new_l, offsets_new_dev=off_dev, slot_dev=td(slot))
    new_p, new_l = new_p.cpu().numpy().astype(np.float64), new_l.cpu().numpy().astype(np.float64)

    def fold(b, p_old, l_old):
        a = H[off[b]:off[b + 1]]
        terms = np.append(a, l_old)
        if not np.isfinite(terms.max()):
            return np.zeros(d), -math.inf
        m = terms.max()
        lse = m + math.log(np.exp(terms - m).sum())
        return np.exp(a - lse) @ h[off[b]:off[b + 1]] + (np.exp(l_old - lse) * p_old if l_old > -math.inf else 0.0), lse

    for b in range(B):
        for got_p, got_l, (p, l) in ((out["pooled"][b], out["lse"][b], fold(b, 0.0, -math.inf)),
                                     (new_p[slot[b]], new_l[slot[b]], fold(b, old_p[slot[b]].astype(np.float64),
                                                                           float(old_l[slot[b]])))):
            if l == -math.inf:
                assert got_l == -math.inf and not got_p.any()
            else:
                assert abs(got_l - l) <= 1e-5 and np.linalg.norm(got_p - p) <= 1e-5 * np.linalg.norm(p), (name, b)
    rest = np.setdiff1d(np.arange(S), slot)
    assert np.array_equal(new_p[rest], old_p[rest].astype(np.float64)) and np.array_equal(new_l[rest], old_l[rest])

    for kind, want in ((gpu.EGTP_POOL_AVERAGE, lambda x: x.mean(axis=0)), (gpu.EGTP_POOL_MAX, lambda x: x.max(axis=0)),
                       (gpu.EGTP_POOL_LAST, lambda x: x[-1])):
        ws.fill_(255)
        got = sc.pool_ablation(hidden, off_dev, kind)[0].cpu().numpy().astype(np.float64)
        for b in range(B):
            x = h[off[b]:off[b + 1]]
            p = want(x) if len(x) else np.zeros(d)
            tol = 1e-5 * np.sqrt(np.mean(x * x)) if kind == gpu.EGTP_POOL_AVERAGE and len(x) else 0.0
            assert np.abs(got[b] - p).max() <= tol, (name, b, kind)
    sc.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_hidden_states_near_the_largest_number(dtype):
    """A pooled vector lies between the smallest and the largest hidden state of its sequence, so it is finite whatever
    they are: 3e38 in every token, the same entropy everywhere (W_lm of zeros), on their own and onto an old state.
    Weights are accurate to a few 2^-24 and their sum is one to the same, hence 1e-5 relative."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    d, V, lens = 136, 40, (1000, 1, 37, 256)
    T, B = sum(lens), len(lens)
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    sign = torch.where(torch.arange(d) % 3 == 0, -1.0, 1.0)
    row = (3e38 * sign).to(store)
    hidden = row.expand(T, d).contiguous().cuda()
    zeros = lambda *s: torch.zeros(*s, dtype=store, device="cuda")
    sc = gpu.Scorer(zeros(V, d), gpu.make_head(zeros(8, d), zeros(1, 8)))
    off = sc.build_offsets(torch.tensor(lens, dtype=torch.int32).cuda(), T)
    want = row.double().expand(B, d).numpy()
    got = sc.score(hidden, off)["pooled"].cpu().numpy().astype(np.float64)
    assert np.abs(got / want - 1.0).max() <= 1e-5
    state, lse = row.float().expand(B, d).contiguous().cuda(), torch.full((B,), 5.0, device="cuda")
    sc.step(hidden, state, lse, offsets_new_dev=off)
    assert np.abs(state.cpu().numpy().astype(np.float64) / want - 1.0).max() <= 1e-5
    sc.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 2056), ("f32", 36)])
def test_offsets_past_the_batch_pool_the_tokens_there_are(dtype, d):
    """Device offsets are the caller's word: where a table runs past T, a sequence has the tokens up to T (bit for bit as
    if the table said so), and nothing that the workspace held before gets into a result."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    lens = (40, 200, 3, 57)
    w = wl.make(wl.scaled(wl.SPECS["mid" if dtype == "bf16" else "tiny"], seed=9300, B=4, d=d, V=40, d_h=8, lengths=lens))
    td = gpu.to_device
    sc = gpu.Scorer(td(w.w_lm), gpu.make_head(td(w.w1), td(w.w2)))
    hidden, T = td(w.hidden), sum(lens)
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32).cuda()

    def results(off):
        out = []
        for call in (lambda: sc.score(hidden, off), lambda: sc.pool_ablation(hidden, off, gpu.EGTP_POOL_MAX)[0]):
            sc.workspace(T, 4).fill_(255)
            r = call()
            out += [v.cpu().numpy() for k, v in r.items() if k != "entropy"] if isinstance(r, dict) else [r.cpu().numpy()]
        return out

    for past, cut in (((0, 40, 240, 243, T + 500), (0, 40, 240, 243, T)), ((0, 40, 240, T + 90, T + 700), (0, 40, 240, T, T))):
        for a, b in zip(results(i32(*past)), results(i32(*cut))):
            assert np.array_equal(a, b), past
    sc.close()


# (lengths, d): averages and maxima in units of the sequences' own, the last batch dealt out evenly.  Sequences of a unit's tokens, one more, several units;
# empty ones at both ends and between; more sequences than one workgroup looks through at once; slices of uneven chunks, of one chunk,
# and more slices than one
EVEN = [((17,), 8), ((18,), 136), ((1, 33, 0, 0, 17, 16, 18, 0, 51, 1, 300), 264), ((0, 0, 5000, 0), 2056), ((34, 17, 51, 68, 1, 16), 4104),
        ((40000,), 64), ((16,) * 2100, 40), ((0,) * 900 + (33, 95, 1) * 500, 24), ((70000, 3, 61000), 8)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("lens,d", EVEN)
def test_rows_dealt_out_evenly(lens, d, dtype):
    """Against fp64: maxima exactly, averages to 1e-5 of a feature's root mean square (fp32 sums); the same for tables that leave out the first
    and the last tokens, and for one that runs past the batch."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    B, T = len(lens), sum(lens)
    rng = np.random.default_rng(B + d)
    td = gpu.to_device
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    hidden = td(rng.standard_normal((T, d)).astype(np.float32)).to(store)
    h = hidden.cpu().double().numpy()
    sc = gpu.Scorer(torch.zeros(40, d, dtype=store, device="cuda"), gpu.make_head(torch.zeros(8, d, dtype=store, device="cuda"),
                                                                                   torch.zeros(1, 8, dtype=store, device="cuda")))
    full = np.concatenate([[0], np.cumsum(lens)])
    for off in (full, np.clip(full, 3, T - 2), full + min(5, T)):
        ws = sc.workspace(T, B)
        for kind in (gpu.EGTP_POOL_AVERAGE, gpu.EGTP_POOL_MAX):
            ws.fill_(255)
            got = sc.pool_ablation(hidden, td(off.astype(np.int32)), kind, want_pred=False)[0].cpu().numpy().astype(np.float64)
            for b in range(B):
                x = h[min(off[b], T):min(off[b + 1], T)]
                if len(x) == 0:
                    assert not got[b].any()
                elif kind == gpu.EGTP_POOL_MAX:
                    assert np.array_equal(got[b], x.max(axis=0)), b
                else:
                    assert np.abs(got[b] - x.sum(axis=0) / (off[b + 1] - off[b])).max() <= 1e-5 * np.sqrt(np.mean(x * x)), b
    sc.close()


# Batches that are dealt out: few sequences beside the rows of a workgroup, at least 90 of these.  Short and empty ones side by side, whose ends are closer together than
# the eight rows that are loaded at a time, runs of more than the 64 ends that a wave holds, at both ends of a batch; ends on and beside those
# of a deal; the most sequences of the rule and one more
SKEWED = [((1,) * 20 + (0,) * 8 + (3,) * 4 + (150000,) + (2,) * 3, 8), ((0, 1, 1, 0, 0, 5, 1, 46980, 1, 0, 7, 0, 3), 1032),
          ((0,) * 66 + (1,) * 4 + (249900,) + (0,) * 5 + (30, 8), 8), ((0,) * 130 + (1,) * 70 + (999000,) + (0,) * 50 + (5,), 8),
          ((93, 92, 94, 0, 93, 186, 1, 45000, 1441), 1032), ((1000,) * 22 + (48000,), 24), ((1000,) * 23 + (47000,), 24)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("lens,d", SKEWED)
def test_short_sequences_among_dealt_rows(lens, d, dtype):
    test_rows_dealt_out_evenly(lens, d, dtype)


def test_dealt_rows_of_malformed_tables():
    """Offsets of any value read and write inside the batch and the workspace: what lies behind both, and the next call with a sound table, are unharmed."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    T, B, d, low, high = 70000, 3, 8, -2 ** 31, 2 ** 31 - 1
    hidden = torch.randn(T, d, device="cuda")
    sc = gpu.Scorer(torch.zeros(40, d, device="cuda"), gpu.make_head(torch.zeros(8, d, device="cuda"), torch.zeros(1, 8, device="cuda")))
    table = lambda *o: torch.tensor(o, dtype=torch.int32, device="cuda")
    need, guard = sc.workspace(T, B).numel(), 1 << 16
    ws = torch.full((need + guard,), 255, dtype=torch.uint8, device="cuda")
    sc.workspace = lambda *_: ws[:need]
    for kind in (gpu.EGTP_POOL_AVERAGE, gpu.EGTP_POOL_MAX):
        for o in ((0, low, high, T), (high, low, 5, T), (low,) * 4, (high,) * 4, (-5, T + 5, low + 3, high), (0, low + 299, low + 1, T), (250, 20, high - 1, 3)):
            sc.pool_ablation(hidden, table(*o), kind, want_pred=False)
            torch.cuda.synchronize()
            assert (ws[need:] == 255).all(), o
        got = sc.pool_ablation(hidden, table(0, 100, 101, T), kind, want_pred=False)[0].double()
        parts = hidden.double().split([100, 1, T - 101])
        want = torch.stack([p.mean(0) if kind == gpu.EGTP_POOL_AVERAGE else p.amax(0) for p in parts])
        assert (got - want).abs().max() <= 1e-5
    sc.close()


@pytest.mark.parametrize("lens", [(6_300_000,), (100, 6_299_900), (4_000_000, 2_300_000)])
def test_averages_of_long_batches_do_not_drift(lens):
    """Every token the same value, one that a running sum of a few thousand of them rounds down each time.  A sum has at most 264 terms in a row, 33 of these
    make up what a workgroup adds up, of the 768 of them a wave joins 192, then the four waves and the division: 494 roundings of 2^-24."""
    import torch
    from paper_2602_11812_amd import binding as gpu
    T, d, value = sum(lens), 8, 1.0 + 0.49 * 2.0 ** -11
    hidden = torch.full((T, d), value, dtype=torch.float32, device="cuda")
    sc = gpu.Scorer(torch.zeros(40, d, device="cuda"), gpu.make_head(torch.zeros(8, d, device="cuda"), torch.zeros(1, 8, device="cuda")))
    off = torch.tensor([0, *np.cumsum(lens)], dtype=torch.int32, device="cuda")
    got = sc.pool_ablation(hidden, off, gpu.EGTP_POOL_AVERAGE, want_pred=False)[0].cpu().numpy().astype(np.float64)
    value = float(np.float32(value))
    assert np.abs(got - value).max() <= 494 * 2.0 ** -24 * value
    sc.close()
