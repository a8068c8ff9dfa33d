"""The confidence monitor where its kernels branch: a wave of a logit chunk with more candidates
than its list, block sizes read a block per thread, percentiles whose histogram cell holds more
keys than the list (repeated histograms) or one key only, traces at odd offsets."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_31395_amd import actkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [20, 64, 511, 512, 513, 600, 2100])
def test_many_equal_logits_in_the_lanes_of_one_wave(count):
    rng = np.random.default_rng(count)
    V = 20000
    x = rng.standard_normal((3, V)).astype(np.float32)
    of_wave = np.nonzero(np.arange(16384) % 256 // 64 == 2)[0]   # logits that wave 2 holds
    x[0, of_wave[:count]] = 9.0
    x[1, rng.choice(of_wave, count, replace=False)] = 9.0
    x[2, rng.choice(of_wave, count, replace=False)] = 9.0 + rng.random(count).astype(np.float32)
    got = actkv.token_confidence(torch.from_numpy(x).cuda(), top_k=20).cpu().numpy()
    np.testing.assert_allclose(got, oracle.token_confidence(x, 20), rtol=1e-6, atol=1e-5)


def _check(seqs, budgets, **params):
    offsets = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    got = actkv.budget_update(torch.from_numpy(np.concatenate(seqs)).cuda(), offsets,
                              torch.from_numpy(budgets).cuda(), **params)
    torch.cuda.synchronize()
    ref = oracle.budget_update(seqs, budgets, **params)
    for name in ("budgets", "retained"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), ref[name])
    np.testing.assert_array_equal(got["slopes"].cpu().numpy().view(np.int64),
                                  ref["slopes"].view(np.int64))
    np.testing.assert_array_equal(got["thresholds"].cpu().numpy(), ref["thresholds"])


@pytest.mark.parametrize("window,stride", [(64, 4), (64, 8), (64, 16), (8, 8), (12, 4), (48, 16),
                                           (20, 12)])
def test_block_sizes_and_odd_offsets(window, stride):
    rng = np.random.default_rng(window * stride)
    lens = [window, window + 1, 997, 16 * 1024 + 3, 8 * 8192 + 5]
    seqs = [(9 + 0.4 * rng.standard_normal(n)).astype(np.float32) for n in lens
            if (n - window) // stride + 1 <= 16384]
    seqs[2][::7] = -0.0
    _check(seqs, np.full(len(seqs), 700, np.int32), window=window, stride=stride)


@pytest.mark.parametrize("pct", [0.0, 10.0, 50.0, 99.0, 100.0])
def test_percentiles_among_ties_and_outliers(pct):
    rng = np.random.default_rng(5)
    n = 20000
    same = np.full(n, 8.25, np.float32)
    two = np.where(np.arange(n) < n // 2, np.float32(8.0), np.float32(9.0))
    far = (8 + 1e-3 * rng.random(n)).astype(np.float32)
    far[0] = 3e30                      # no window's minimum, but the next is
    far[64:128] = 1e30
    near = (8 + 1e-5 * rng.integers(0, 30, n)).astype(np.float32)   # hundreds of keys to a value
    signed = rng.standard_normal(n).astype(np.float32)
    _check([same, two, far, near, signed], np.full(5, 900, np.int32), bottom_pct=pct)
