"""Selection of long segments cut into parts over several workgroups, at the edges of its
range, against the oracle (bit-exact).  Besides ordinary scores the inputs are ones whose
sampled bracket is empty, misses the k-th entry or holds more keys than a part can list: those
segments are selected by one workgroup."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_31395_amd import actkv
from paper_2609_31395_amd import workloads as W

pytestmark = pytest.mark.gpu

SAMPLE = 1024   # sampled positions per segment: (2 i + 1) L / 2048


def _scores(kind, L, rng):
    if kind == "softmax":      # probabilities with a few large ones
        s = np.exp(rng.standard_normal(L) * 0.4)
        s[rng.integers(0, L, L // 100)] *= 8
        return s * 1e-3
    if kind == "signed":
        return rng.standard_normal(L)
    if kind == "equal":
        return np.full(L, 0.25)
    if kind == "two_values":   # the k-th entry is one of many equal ones
        return np.where(rng.random(L) < 0.5, 2.0, 1.0)
    if kind == "few_values":
        return rng.integers(0, 40, L) / 64.0
    if kind == "unsampled":    # every sampled entry and its window lies below all the others
        s = 1.0 + rng.random(L)
        at = (2 * np.arange(SAMPLE, dtype=np.int64) + 1) * L // (2 * SAMPLE)
        for d in range(-3, 4):
            s[np.clip(at + d, 0, L - 1)] = rng.random(SAMPLE) * 0.5
        return s
    if kind == "extremes":     # infinities, zeros of both signs, denormals
        s = rng.standard_normal(L)
        s[rng.integers(0, L, L // 5)] = np.inf
        s[rng.integers(0, L, L // 5)] = -np.inf
        s[rng.integers(0, L, L // 5)] = -0.0
        s[rng.integers(0, L, L // 5)] = 1e-42
        return s
    if kind == "sorted":
        return np.sort(rng.standard_normal(L))
    raise ValueError(kind)


def _check(lens, budgets, kinds, window, seed=0, small=False):
    pb = W.make_custom(seq_lens=lens, q_lens=[0] * len(lens), num_q_heads=1, num_kv_heads=1,
                       head_dim=64, budgets=budgets, pool_window=window)
    rng = np.random.default_rng(seed)
    raw = np.concatenate([_scores(k, L, rng) for k, L in zip(kinds, lens)]).astype(np.float32)
    bp = actkv.Problem(seq_lens=pb.seq_lens, q_lens=pb.q_lens, budgets=pb.budgets,
                       num_q_heads=1, num_kv_heads=1, head_dim=64, num_pages=pb.num_pages,
                       bt_stride=pb.bt_stride, pool_window=window).to_device("cuda")
    s = torch.from_numpy(raw).cuda()
    ws = actkv.workspace(bp).fill_(0xA5)
    kept, pooled = actkv.select(bp, s, ws=ws)
    again, none = actkv.select(bp, s, ws=ws, want_pooled=False)
    torch.cuda.synchronize()
    ref = oracle.pool(pb, raw)
    np.testing.assert_array_equal(pooled.cpu().numpy(), ref)
    np.testing.assert_array_equal(kept.cpu().numpy(), oracle.select(pb, ref))
    assert none is None and torch.equal(kept, again)
    np.testing.assert_array_equal(s.cpu().numpy(), raw)


@pytest.mark.parametrize("window", [1, 3, 7])
@pytest.mark.parametrize("L", [8191, 8192, 8193, 12289, 28673, 38401, 65535, 126977, 131072,
                               131073])
def test_lengths_at_the_edges_of_the_parts(L, window):
    for k in (1, L // 4, L - 1):
        _check([L], [k], ["softmax"], window, seed=L + k)


@pytest.mark.parametrize("kind", ["signed", "equal", "two_values", "few_values", "unsampled",
                                  "extremes", "sorted"])
@pytest.mark.parametrize("L", [8197, 40001])
def test_inputs_that_the_sample_cannot_bracket(kind, L):
    for k in (3, L // 10, L // 4, L // 2, L - 2):
        _check([L], [k], [kind], 7 if kind != "few_values" else 1, seed=k)


def test_a_batch_of_short_long_and_uncut_segments():
    lens = [5, 8192, 140000, 0, 20000, 9000, 30000]
    budgets = [3, 8192, 35000, 4, 0, 2250, 29999]   # all of it, none of it, a part of it
    _check(lens, budgets, ["softmax"] * 7, 5)


def test_wide_windows_are_not_cut():
    _check([20000, 45000], [5000, 11000], ["softmax"] * 2, 9)
