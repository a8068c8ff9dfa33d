"""Selection with the keys in registers, at the edges of its register counts and chunks, against
the oracle (bit-exact), TopK and LRFU.  Besides ordinary scores the inputs are ones whose sampled
bracket misses the k-th entry (or the top-p boundary), or whose chosen histogram bin holds more
entries than its list: the passes that narrow it down, and ties taken in index order."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_31395_amd import actkv
from paper_2609_31395_amd import workloads as W
from test_gpu_lrfu import check_stage

pytestmark = pytest.mark.gpu



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
    if kind == "outlier":      # one entry far above: the key range says little about the rest
        s = np.exp(rng.standard_normal(L) * 0.1) * 1e-4
        s[L // 3] = 1e4
        return s
    if kind == "blocks":       # every other 512 entries far below the rest
        return rng.random(L) + 1e3 * ((np.arange(L) // 512) % 2)
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


def _check(lens, budgets, kinds, window, seed=0):
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
@pytest.mark.parametrize("L", [2, 63, 65, 1024, 1025, 6144, 6145, 8193, 16384, 16385, 40960, 40961,
                               64512, 64513])
def test_lengths_at_the_edges_of_the_registers(L, window):
    for k in sorted({1, max(1, L // 4), L - 1}):
        _check([L], [k], ["softmax"], window, seed=L + k)


@pytest.mark.parametrize("kind", ["signed", "equal", "two_values", "few_values", "outlier",
                                  "blocks", "extremes", "sorted"])
@pytest.mark.parametrize("L", [1500, 8197, 40001])
def test_inputs_that_the_sample_cannot_bracket(kind, L):
    for k in (3, L // 10, L // 4, L // 2, L - 2):
        _check([L], [k], [kind], 7 if kind != "few_values" else 1, seed=k)


def test_a_batch_of_short_and_long_segments():
    lens = [5, 8192, 140000, 0, 20000, 9000, 30000]   # one past the registers
    budgets = [3, 8192, 35000, 4, 0, 2250, 29999]     # all of it, none of it, a part of it
    _check(lens, budgets, ["softmax"] * 7, 5)


def test_nan_scores_end():
    """Unspecified selections, but the call returns and every index lies in its segment."""
    L, k = 20000, 5000
    bp = actkv.Problem(seq_lens=[L], q_lens=[0], budgets=[k], num_q_heads=1, num_kv_heads=1,
                       head_dim=64, num_pages=2500, bt_stride=1250, pool_window=1).to_device("cuda")
    for bits in (0x7FC00000, -1):   # a NaN of either sign
        s = torch.full((L,), bits, dtype=torch.int32, device="cuda").view(torch.float32)
        s[: L // 8] = 1.0
        kept = torch.zeros(k, dtype=torch.int32, device="cuda")
        actkv.select(bp, s, kept=kept)
        torch.cuda.synchronize()
        assert int(kept.min()) >= 0 and int(kept.max()) < 64 * 1024


@pytest.mark.parametrize("kind", ["softmax", "two_values", "few_values", "outlier", "blocks"])
@pytest.mark.parametrize("L", [70, 6145, 16384, 40961, 64512])
def test_lrfu_at_the_edges_of_the_registers(L, kind):
    rng = np.random.default_rng(L)
    pb = W.make_custom(seq_lens=[L, L // 2], q_lens=[0, 0], num_q_heads=1, num_kv_heads=1,
                       head_dim=64, budgets=[L // 4, L // 3], pool_window=7 if L % 2 else 1)
    raw = np.concatenate([_scores(kind, n, rng) for n in (L, L // 2)]).astype(np.float32)
    ks = (rng.random(raw.shape[0]) * raw.mean()).astype(np.float32)
    for top_p in (0.2, 0.9, 0.9999):
        check_stage(pb, raw, ks, top_p, 0.5)
