"""MAX_MEAN scoring for every group size it takes (a kernel each; G = 1 runs on SUM's), with query
counts around the row tiles and chunks, against the oracle.  The kernels take the maximum over a
group before the exponential: exp2 keeps the order, so only the fp32 rounding of the exponent (at
most about 2^-18 at the |x| < 40 met here), of exp2 and of the sum of n terms is between the two."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev
from paper_2609_31395_amd import actkv
from paper_2609_31395_amd import workloads as W

pytestmark = pytest.mark.gpu

RTOL = 3e-5   # 2^-18 * ln 2 * 8, for the rounding of an exponent and the fp32 LSE


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_max_mean_groups(G, D):
    for n in (1, 3, 31, 32, 33, 65, 130):
        pb = W.make_custom(seq_lens=[n + 61, n + 300, n], q_lens=[n, max(1, n // 2), n],
                           num_q_heads=2 * G, num_kv_heads=2, head_dim=D, budgets=50,
                           spike_frac=0.02, seed=n)
        bp, t = to_dev(pb, agg="max_mean")
        lse = oracle.lse(pb).astype(np.float32)
        got = actkv.score(bp, t["q"], t["kv"], t["bt"], lse=torch.from_numpy(lse).cuda())
        ref = oracle.scores(pb, lse_in=lse, agg="max_mean")
        np.testing.assert_allclose(got.cpu().numpy(), ref, rtol=RTOL, atol=1e-30)
