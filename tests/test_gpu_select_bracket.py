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
from gpu_util import assert_compaction_matches, to_dev
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
@pytest.mark.parametrize("L", [2, 63, 65, 1024, 1025, 2048, 2049, 4096, 4097, 6144, 6145, 8192, 8193,
                               16384, 16385, 40960, 40961, 64512, 64513])
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


def _nan_problem(segs, budgets, window=1):
    """segs equal segments of one request each; ordinary pages to compact into."""
    pb = W.make_custom(seq_lens=[L for L in segs], q_lens=[0] * len(segs), num_q_heads=1,
                       num_kv_heads=1, head_dim=64, budgets=budgets, pool_window=window)
    return pb, to_dev(pb)


def _assert_ascending_within(pb, kept):
    """k strictly ascending indices of every segment, and nothing written past the last."""
    at = 0
    for L, b in zip(pb.seq_lens, pb.budgets):
        k = min(int(L), int(b))
        idx = kept[at:at + k].astype(np.int64)
        assert (idx >= 0).all() and (idx < L).all() and (np.diff(idx) > 0).all(), (L, k)
        at += k
    assert (kept[at:] == SENTINEL).all(), "entries written past the segments"


SENTINEL = -77
# 0x7FC00000 and 0xFFC00000: NaNs of either sign; 0xFFFFFFFF: the one whose order key is 0, as that
# of a slot without an entry; (its share of a segment, the rest ordinary)
NAN_FILLS = [(0x7FC00000, 0.9), (-0x400000, 0.9), (-1, 0.9), (-1, 1.0), (-1, 0.5)]
# segments whose budgets end inside, before and after slots that hold no entry
NAN_LENS, NAN_KEPT = [70, 20000, 1025, 64512, 9000, 6145], [69, 1500, 1024, 40000, 5, 6000]


def _nan_scores(pb, bits, share, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = int(pb.seq_lens.sum())
    s = torch.rand(n, generator=g, device="cuda")
    nan = torch.full((n,), bits, dtype=torch.int32, device="cuda").view(torch.float32)
    return torch.where(torch.rand(n, generator=g, device="cuda") < share, nan, s)


@pytest.mark.parametrize("bits,share", NAN_FILLS)
def test_nan_scores_end(bits, share):
    """Unspecified selections, but the call returns, every index lies in its segment, each segment
    gets all of its entries, and nothing is written past them.  Where every score is one NaN the
    entries tie, and the first are kept."""
    pb, (bp, t) = _nan_problem(NAN_LENS, NAN_KEPT)
    s = _nan_scores(pb, bits, share)
    n = sum(NAN_KEPT)
    kept = torch.full((n + 4096,), SENTINEL, dtype=torch.int32, device="cuda")
    actkv.select(bp, s, kept=kept)
    torch.cuda.synchronize()
    _assert_ascending_within(pb, kept.cpu().numpy())
    if share == 1.0:
        want = np.concatenate([np.arange(k) for k in NAN_KEPT])
        np.testing.assert_array_equal(kept[:n].cpu().numpy(), want)
    # the keep scores: NaN from the scores of the hits and from the old keep scores
    for scores, ks in ((s, torch.rand_like(s)), (torch.rand_like(s), s.clone())):
        kept.fill_(SENTINEL)
        ks_kept = torch.full((n + 4096,), float(SENTINEL), device="cuda")
        actkv.lrfu_select(bp, scores, ks, 0.9, 0.5, kept=kept, ks_kept=ks_kept)
        torch.cuda.synchronize()
        _assert_ascending_within(pb, kept.cpu().numpy())
        assert (ks_kept[n:] == SENTINEL).all()


@pytest.mark.parametrize("bits,share", NAN_FILLS)
@pytest.mark.parametrize("lens,budgets", [([70], [69]), ([9000, 1025], [500, 300]),
                                          ([20000] * 3, [1500, 9000, 19999]),
                                          ([40000] * 3, [1500, 9000, 39999])])
def test_nan_scores_end_in_the_compaction(lens, budgets, bits, share):
    """The same for the fused kernels and the separate ones: all of a segment's rows are copied."""
    pb, (bp, t) = _nan_problem(lens, budgets)
    n = sum(budgets)
    kept = torch.full((n + 4096,), SENTINEL, dtype=torch.int32, device="cuda")
    kv = t["kv"].cpu().numpy().view(np.uint16)
    o = actkv.select_compact(bp, _nan_scores(pb, bits, share), t["kv"], t["bt"], t["free"],
                             kept=kept)
    torch.cuda.synchronize()
    kept = kept.cpu().numpy()
    _assert_ascending_within(pb, kept)
    assert_compaction_matches(pb, kept[:n], kv, t["kv"].cpu().numpy().view(np.uint16),
                              t["bt"].cpu().numpy(), o["freed"].cpu().numpy(),
                              o["new_lens"].cpu().numpy())


@pytest.mark.parametrize("L", [70, 20000, 1025])
def test_equal_scores_beside_nan_scores(L):
    """One value and NaNs of key 0: the value's entries first, then the first NaNs."""
    pb, (bp, _) = _nan_problem([L] * 3, [L // 4, L // 2 + 5, L - 1])
    nan = np.random.default_rng(L).random(3 * L) < 0.5
    bits = np.where(nan, -1, np.float32(0.25).view(np.int32)).astype(np.int32)
    kept, _ = actkv.select(bp, torch.from_numpy(bits).cuda().view(torch.float32))
    want = []
    for i, k in enumerate(pb.budgets):
        x = nan[i * L:(i + 1) * L]
        want.append(np.sort(np.concatenate([np.nonzero(~x)[0], np.nonzero(x)[0]])[:k]))
    np.testing.assert_array_equal(kept.cpu().numpy(), np.concatenate(want))


def _check_lrfu(lens, raw, top_p, ks=None, window=1):
    pb = W.make_custom(seq_lens=lens, q_lens=[0] * len(lens), num_q_heads=1, num_kv_heads=1,
                       head_dim=64, budgets=[L // 4 + 1 for L in lens], pool_window=window)
    raw = np.concatenate(raw).astype(np.float32)
    check_stage(pb, raw, np.zeros_like(raw) if ks is None else ks, top_p, 0.5)


@pytest.mark.parametrize("top_p", [0.3, 0.9, 1.0])
@pytest.mark.parametrize("value", [0.0, 0.25, -1.0, 3e-45])
def test_lrfu_of_equal_scores(value, top_p):
    lens = [2, 70, 9000, 40001]
    _check_lrfu(lens, [np.full(L, value) for L in lens], top_p)


@pytest.mark.parametrize("scale", [1e-37, 1e-38, 2e-39, 4e-40, 1e-41])
@pytest.mark.parametrize("top_p", [0.05, 0.5, 0.9])
def test_lrfu_of_tiny_scores(scale, top_p):
    """Largest scores around and below the smallest normal float, where 1 / score is infinite."""
    rng = np.random.default_rng(3)
    lens = [70, 9000, 40001]
    _check_lrfu(lens, [(rng.random(L) * scale).astype(np.float32) for L in lens], top_p)


@pytest.mark.parametrize("ties", [2, 63, 64, 65, 66, 900])
@pytest.mark.parametrize("L", [3000, 20001])
def test_ties_at_the_cut_around_the_list(L, ties):
    """The k-th entry, and the top-p boundary, among `ties` equal entries."""
    rng = np.random.default_rng(ties)
    s = rng.random(L).astype(np.float32)
    order = np.argsort(-s, kind="stable")
    at = L // 4
    s[order[at - ties // 2:at - ties // 2 + ties]] = s[order[at]]
    pb = W.make_custom(seq_lens=[L], q_lens=[0], num_q_heads=1, num_kv_heads=1, head_dim=64,
                       budgets=[at])
    bp, _ = to_dev(pb)
    kept, pooled = actkv.select(bp, torch.from_numpy(s).cuda())
    np.testing.assert_array_equal(kept.cpu().numpy(), oracle.select(pb, s))
    mass = np.cumsum(np.sort(s.astype(np.float64))[::-1])
    _check_lrfu([L], [s], float(np.float32((mass[at - ties // 2] + 0.4 * ties * s[order[at]])
                                           / mass[-1])))


@pytest.mark.parametrize("window", [1, 3, 5, 7])
@pytest.mark.parametrize("L", [70, 2048, 20000, 40001])
def test_nan_scores_yield_to_their_window(L, window):
    """A NaN is left out of its window's maximum, on every path: the pooled scores are the host's
    np.fmax, and what is selected is what the small-footprint kernel selects of them."""
    pb, (bp, t) = _nan_problem([L, L // 2 + 1], [L // 4 + 1, L // 3], window)
    rng = np.random.default_rng(L + window)
    raw = rng.standard_normal(int(pb.seq_lens.sum())).astype(np.float32)
    raw[::9] = np.nan
    raw[4::27] = np.uint32(0xFFC00000).view(np.float32)   # and of the other sign, never in a row
    s = torch.from_numpy(raw).cuda()
    kept, pooled = actkv.select(bp, s)
    small_kept, small_pooled = actkv.select(bp.small_select(), s)
    ks = torch.zeros_like(s)
    lrfu_pooled = torch.empty_like(s)
    actkv.lrfu_select(bp, s, ks, 0.9, 0.5, pooled=lrfu_pooled)
    torch.cuda.synchronize()
    want, at = [], 0
    for n in (int(x) for x in pb.seq_lens):
        x, h = raw[at:at + n], window // 2
        m = x.copy()
        for d in range(1, h + 1):
            m[d:] = np.fmax(m[d:], x[:-d])
            m[:-d] = np.fmax(m[:-d], x[d:])
        want.append(m)
        at += n
    want = np.concatenate(want)
    np.testing.assert_array_equal(pooled.cpu().numpy(), want)
    for a, b in ((pooled, small_pooled), (pooled, lrfu_pooled)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert torch.equal(kept, small_kept)


@pytest.mark.parametrize("kind", ["softmax", "two_values", "few_values", "outlier", "blocks"])
@pytest.mark.parametrize("L", [70, 2048, 2049, 4097, 6145, 8192, 8193, 16384, 40961, 64512])
def test_lrfu_at_the_edges_of_the_registers(L, kind):
    rng = np.random.default_rng(L)
    pb = W.make_custom(seq_lens=[L, L // 2], q_lens=[0, 0], num_q_heads=1, num_kv_heads=1,
                       head_dim=64, budgets=[L // 4, L // 3], pool_window=7 if L % 2 else 1)
    raw = np.concatenate([_scores(kind, n, rng) for n in (L, L // 2)]).astype(np.float32)
    ks = (rng.random(raw.shape[0]) * raw.mean()).astype(np.float32)
    for top_p in (0.2, 0.9, 0.9999):
        check_stage(pb, raw, ks, top_p, 0.5)
