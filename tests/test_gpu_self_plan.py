"""The first kernel of a call plans for itself in batches of at most 64 requests: the scores of
unplanned calls, and the plan they leave in the workspace for later calls, equal those of calls
planned by actkv_plan, bit for bit, around that limit; with empty requests, requests without
queries, and several row chunks."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev
from paper_2609_31395_amd import actkv
from paper_2609_31395_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(R, q_hi, seed, kv_heads=2, group=4):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 300, R)
    lens[rng.random(R) < 0.2] = 0
    lens[0] = 0 if R > 2 else 200
    lens[-1] = 257
    n = np.minimum(rng.integers(0, q_hi + 1, R), lens)
    budgets = rng.integers(0, 200, R * kv_heads)
    return W.make_custom(seq_lens=lens, q_lens=n, num_q_heads=kv_heads * group,
                         num_kv_heads=kv_heads, head_dim=64, budgets=budgets, pool_window=3,
                         spike_frac=0.05, seed=seed)


def _lse(pb):
    return torch.from_numpy(oracle.lse(pb).astype(np.float32)).cuda()


@pytest.mark.parametrize("R", [1, 2, 63, 64, 65, 130])
@pytest.mark.parametrize("q_hi", [3, 200])
def test_unplanned_scores_and_what_they_leave(R, q_hi):
    pb = _problem(R, q_hi, seed=R + q_hi, kv_heads=1 if R % 2 else 2, group=4)
    lse = _lse(pb)
    outs = []
    for planned in (False, True):
        bp, t = to_dev(pb)
        ws = actkv.workspace(bp).fill_(0x5A)
        if planned:
            actkv.plan(bp, ws)
        scores = actkv.score(bp.planned() if planned else bp, t["q"], t["kv"], t["bt"], lse=lse,
                             ws=ws)
        kept, pooled = actkv.select(bp.planned(), scores, ws=ws)
        freed, lens = actkv.compact(bp.planned(), t["kv"], t["bt"], kept, t["free"], ws=ws)
        torch.cuda.synchronize()
        outs.append((scores, kept, pooled, freed, lens, t["bt"], t["kv"]))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    ref = oracle.scores(pb, lse_in=lse.cpu().numpy())
    np.testing.assert_allclose(outs[0][0].cpu().numpy(), ref, rtol=2e-3, atol=1e-30)


@pytest.mark.parametrize("lens,n,kv_heads,group", [
    ([1600], [1500], 1, 8),                                # 24 chunks of one head
    ([700], [513], 3, 16),                                 # 17, the last of 16 rows
    ([700, 0, 300, 900], [64, 0, 300, 65], 64, 8),         # 1, 1, 5 and 2 chunks of 64 heads
    ([900, 0, 700], [9, 0, 8], 4, 1),                      # few segments to a request, and more
    ([900, 0, 700], [9, 0, 8], 5, 1),
    ([900, 40, 700], [9, 0, 8], 33, 2),
    ([300] * 31 + [1100] + [0] * 31 + [200], [1] * 31 + [1024] + [0] * 31 + [200], 2, 8),
])
def test_unplanned_scores_of_many_row_chunks_and_heads(lens, n, kv_heads, group):
    """The kernels' own plan, the plan kernel of one wave and, with empty requests up to 65, that of
    larger batches: the same scores and kept entries, bit for bit."""
    outs = []
    for empty in (0, 65 - len(lens)):
        pb = W.make_custom(seq_lens=lens + [0] * empty, q_lens=n + [0] * empty,
                           num_q_heads=kv_heads * group, num_kv_heads=kv_heads, head_dim=64,
                           budgets=100, pool_window=3, spike_frac=0.05, seed=7)
        lse = _lse(pb) if not outs else lse
        for planned in (False, True):
            bp, t = to_dev(pb)
            ws = actkv.workspace(bp).fill_(0x5A)
            if planned:
                actkv.plan(bp, ws)
            scores = actkv.score(bp.planned() if planned else bp, t["q"], t["kv"], t["bt"],
                                 lse=lse, ws=ws)
            kept, _ = actkv.select(bp.planned(), scores, ws=ws)
            torch.cuda.synchronize()
            if not outs:
                ref = oracle.scores(pb, lse_in=lse.cpu().numpy())
                np.testing.assert_allclose(scores.cpu().numpy(), ref, rtol=2e-3, atol=1e-30)
            outs.append((scores, kept))
            if empty:   # its pages lie elsewhere, its values are the same
                assert np.array_equal(pb.q, q)
        q = pb.q
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert torch.equal(a, b)


@pytest.mark.parametrize("R", [1, 5, 64, 65])
def test_unplanned_decode_steps(R):
    pb = _problem(R, 1, seed=R)
    lse = _lse(pb)
    outs = []
    for planned in (False, True):
        bp, t = to_dev(pb)
        ws = actkv.workspace(bp).fill_(0x5A)
        acc = torch.ones(actkv.num_scores(bp), device="cuda")
        if planned:
            actkv.plan(bp, ws)
        for _ in range(2):
            actkv.score_accumulate(bp.planned() if planned else bp, t["q"], t["kv"], t["bt"], acc,
                                   lse=lse, ws=ws)
        o = actkv.select_compact(bp.planned(), acc, t["kv"], t["bt"], t["free"], ws=ws)
        torch.cuda.synchronize()
        outs.append((acc, o["freed"], o["new_lens"], t["bt"], t["kv"]))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("R", [1, 7, 64, 65])
@pytest.mark.parametrize("window", [3, 9])
def test_unplanned_selections_and_their_rewrite(R, window):
    """Selection, LRFU selection, and selection with the compaction behind it (segments too long
    for the fused kernel: rows rewritten beside the selection), first in their calls."""
    rng = np.random.default_rng(R)
    lens = rng.integers(0, 300, R)
    lens[-1] = 29000 if R < 10 else 400
    budgets = rng.integers(0, 1500, R * 2)
    if R > 2:
        budgets[2:4] = lens[1]                       # a request left untouched
    pb = W.make_custom(seq_lens=lens, q_lens=np.zeros(R, int), num_q_heads=2, num_kv_heads=2,
                       head_dim=64, budgets=budgets, pool_window=window, seed=R)
    raw = torch.from_numpy(rng.random(int(lens.sum()) * 2).astype(np.float32)).cuda()
    outs = []
    for planned in (False, True):
        bp, t = to_dev(pb)
        ws = [actkv.workspace(bp).fill_(0x5A) for _ in range(3)]
        pp = bp
        if planned:
            pp = bp.planned()
            for w in ws:
                actkv.plan(bp, w)
        kept, pooled = actkv.select(pp, raw, ws=ws[0])
        ks = torch.ones_like(raw)
        o = actkv.lrfu_select(pp, raw, ks, 0.8, 0.5, ws=ws[1])
        c = actkv.select_compact(pp, raw, t["kv"], t["bt"], t["free"], ws=ws[2])
        freed = c["freed"]
        again = actkv.compact_inplace(bp.planned(), *to_dev_kv(pb), kept, ws=ws[0])
        torch.cuda.synchronize()
        outs.append((kept, pooled, ks, o["kept"], o["ks_kept"], freed, c["new_lens"], t["bt"],
                     t["kv"], again["freed"], again["new_order"]))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    kv_ref, bt_ref, freed_ref, lens_ref = oracle.compact(pb, outs[0][0].cpu().numpy())
    np.testing.assert_array_equal(outs[0][7].cpu().numpy(), bt_ref)
    np.testing.assert_array_equal(outs[0][5].cpu().numpy(), freed_ref)
    np.testing.assert_array_equal(outs[0][6].cpu().numpy(), lens_ref)


def to_dev_kv(pb):
    _, t = to_dev(pb)
    return t["kv"], t["bt"]
