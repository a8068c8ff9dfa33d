"""The log-sum-exp pass around its work split and its row tiles, against the oracle: balanced over the
chip (several pieces per segment, segments kept whole, both beside empty requests) and one workgroup
per 2,048 keys (small problems, and where a segment would have more pieces than its partials have room
for); query counts around a wave's row tiles and a 512-row chunk; values that raise a row's shift by more than 2^64 late.

Tolerance (natural log): the fp32 dot product of D <= 128 bf16 products, D * 2^-24 * sum |q k| *
sm_scale, is below 1e-4 here; a lane sums at most L / 16 <= 2,100 positive terms one after the other,
2,100 * 2^-24 = 1.3e-4 relative; exponents below 100 round by 100 * 2^-24 = 6e-6."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev
from paper_2609_31395_amd import actkv
from paper_2609_31395_amd import workloads as W

pytestmark = pytest.mark.gpu

ATOL = 3e-4

SPLITS = {   # seq_lens, q_lens, num_q_heads, num_kv_heads (balanced_mixed: with D = 128 only)
    "balanced_long": ([33000, 8001, 20000, 15000] * 4, [3, 1, 2, 3] * 4, 16, 8),
    "balanced_mixed": ([30000, 2049, 600, 29000, 0, 640, 1] * 6, [5, 70, 3, 40, 0, 33, 1] * 6, 16, 8),
    "balanced_uneven_pieces": ([6300, 4200, 0, 640, 1, 4150] * 12, [40, 3, 0, 33, 1, 70] * 12, 16, 8),
    "balanced_whole_segments": ([2048, 2047, 64, 0] * 130, [2, 1, 3, 0] * 130, 8, 8),
    "too_many_pieces": ([8000] + [2100] * 68, [64] + [1] * 68, 64, 8),
    "small": ([2048, 2047, 64, 63, 0, 1, 65] * 6, [2, 1, 3, 1, 0, 1, 2] * 6, 8, 4),
}


def check(pb, atol=ATOL):
    bp, t = to_dev(pb)
    got = actkv.lse(bp, t["q"], t["kv"], t["bt"]).cpu().numpy()
    np.testing.assert_allclose(got, oracle.lse(pb).reshape(got.shape), rtol=0, atol=atol)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("split", sorted(SPLITS))
def test_splits(split, D, causal):
    L, n, Hq, Hkv = SPLITS[split]
    check(W.make_custom(seq_lens=L, q_lens=n, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                        budgets=50, causal=causal, seed=3))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [8, 16])
def test_row_tiles(G, D):
    """Row counts around a wave's tiles and a chunk, beside long requests that make it balanced."""
    n = [-(-rows // G) for rows in (1, 16, 17, 128, 129, 384, 385, 512, 513, 1025)]
    check(W.make_custom(seq_lens=[x + 60 for x in n] + [16000] * 12, q_lens=n + [1] * 12,
                        num_q_heads=8 * G, num_kv_heads=8, head_dim=D, budgets=50, seed=G))


@pytest.mark.parametrize("D", [64, 128])
def test_late_large_values(D):
    """A few late keys 32 times as large (an exact scaling): exponents past 60, so the
    shift taken in a row's first tile is far too low and terms against it overflow."""
    pb = W.make_custom(seq_lens=[20000, 700] * 8, q_lens=[3, 2] * 8, num_q_heads=16,
                       num_kv_heads=8, head_dim=D, budgets=50, spike_frac=0.0, seed=5)
    for r, L in enumerate(int(x) for x in pb.seq_lens):
        for key in (L - 3, L - 70, L // 2):
            k = pb.kv[0, int(pb.block_table[r, key // 16]), key % 16]
            big = (k.astype(np.uint32) << 16).view(np.float32) * np.float32(32)
            k[...] = (big.view(np.uint32) >> 16).astype(np.uint16)
    assert oracle.lse(pb).max() > 60    # the other keys reach 10, and 2^64 is 44 in natural log
    check(pb, atol=32 * ATOL)           # the dot products' bound grows with the keys
