"""tri_select_topk on crafted score arrays against the oracle's full stable sort: heavy ties, all-equal scores,
signed zeros, outliers far outside the z-score range, every kernel variant (keys in LDS up to 32768, in memory beyond), ragged
lengths including N <= B and N = 0.  Index sets must match bit for bit (integer work on identical inputs)."""
import zlib

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def make_scores(rng, kind, n):
    if kind == "normal":
        return rng.standard_normal(n).astype(np.float32)
    if kind == "few_values":          # heavy ties: 7 distinct values
        return rng.integers(-3, 4, size=n).astype(np.float32) * 0.5
    if kind == "all_equal":
        return np.full(n, 1.25, dtype=np.float32)
    if kind == "zeros_signed":        # +0.0 and -0.0 tie, a few positives and negatives around them
        x = np.zeros(n, dtype=np.float32)
        x[rng.random(n) < 0.5] = -0.0
        m = rng.random(n) < 0.01
        x[m] = rng.standard_normal(int(m.sum())).astype(np.float32)
        return x
    if kind == "outliers":            # far outside the bin range on both sides, plus a dense normal body
        x = rng.standard_normal(n).astype(np.float32)
        m = rng.random(n) < 0.1
        x[m] = (rng.standard_normal(int(m.sum())) * 1e4).astype(np.float32)
        return x
    if kind == "one_bin_many":        # thousands of distinct scores inside one histogram bin
        return (1.0 + rng.random(n) * 1e-3).astype(np.float32)
    if kind == "huge":                # everything above the top bin
        return (1e6 + rng.integers(0, 50, size=n)).astype(np.float32)
    raise ValueError(kind)


@pytest.mark.parametrize("nmax,budget", [(700, 100), (5000, 512), (8192, 2048), (20000, 2048), (32768, 2048),
                                         (40000, 4096)])
@pytest.mark.parametrize("kind", ["normal", "few_values", "all_equal", "zeros_signed", "outliers", "one_bin_many", "huge"])
def test_select_matches_full_sort(oracle, nmax, budget, kind):
    from paper_2604_04921_amd import binding as T
    rng = np.random.default_rng(zlib.crc32(("%d/%d/%s" % (nmax, budget, kind)).encode()))
    L, S, Hkv = 2, 3, 2
    lens = np.array([nmax, max(1, nmax // 3 + 17), min(budget - 1, nmax)], dtype=np.int32)
    lens[2] = lens[2] if kind != "normal" else 0     # one empty sequence in the 'normal' runs
    final = np.full((L, S, Hkv, nmax), np.nan, dtype=np.float32)
    for l in range(L):
        for s in range(S):
            for h in range(Hkv):
                final[l, s, h, :lens[s]] = make_scores(rng, kind, int(lens[s]))
    dev = "cuda"
    offs = np.array([1], dtype=np.int64)
    model = T.Model(L, Hkv, Hkv, 128, 1e4, offs)
    k = torch.zeros((L, S, Hkv, 1, 128), dtype=torch.bfloat16, device=dev).expand(L, S, Hkv, nmax, 128)
    pos = torch.zeros((L, S, Hkv, nmax), dtype=torch.int32, device=dev)
    seq_len = torch.from_numpy(lens).to(dev)
    cache = T.Cache(k, None, pos, seq_len, torch.zeros(S, dtype=torch.int32, device=dev), nmax)
    kept_idx = torch.full((L, S, Hkv, budget), -7, dtype=torch.int32, device=dev)
    kept_cnt = torch.full((L, S, Hkv), -7, dtype=torch.int32, device=dev)
    T.tri_select_topk(model, torch.from_numpy(final).to(dev), cache, budget, kept_idx, kept_cnt)
    torch.cuda.synchronize()
    idx, cnt = kept_idx.cpu().numpy(), kept_cnt.cpu().numpy()
    for l in range(L):
        for s in range(S):
            for h in range(Hkv):
                n = int(lens[s])
                ref = oracle.topk(final[l, s, h, :n].astype(np.float64), budget)
                assert cnt[l, s, h] == len(ref) == min(n, budget)
                np.testing.assert_array_equal(idx[l, s, h, :len(ref)], ref)
                assert np.all(idx[l, s, h, len(ref):] == -7)     # nothing written past the count
