"""The score kernel that spreads a key over sixteen lanes, on batches that the library's rule sends there (asserted): raw and final
scores against the oracle, kept slots against the oracle's selection on the same scores.  The layers share one layer's keys
(stride 0) and differ in their query statistics, so that thousands of head-instances take little memory."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H
import tri_rules as R
from test_gpu_position_range import KINDS, positions as ends_of_int32

pytestmark = pytest.mark.gpu

SHORT = [1, 15, 16, 17, 31, 33, 64, 127, 129, 255, 300, 0, 48, 113, 96, 272]   # a wave's groups of 16 and their tails


def score_batch(oracle, group, lens, set_positions=None, positions="dense", block=16, budget=40, kv_heads=8):
    from paper_2604_04921_amd import binding as T
    n, S, n_cu = max(lens), len(lens), torch.cuda.get_device_properties(0).multi_processor_count
    chunks = -(-n // 8192)
    layers = -(-8 * n_cu // (S * kv_heads * chunks))   # eight items of 8192 keys per CU
    assert R.sixteen_lane_kernel(group, layers * S * kv_heads, n, n_cu)
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged"], n_layers=1, n_seqs=S, n_q_heads=kv_heads * group, n_kv_heads=kv_heads, seq_len=n,
                        min_seq_len=None, budget=budget, n_calib=64, positions=positions, block_size=block, seed=31 + group)
    w = recipe.generate(cfg)
    w["seq_len"] = np.array(lens, dtype=np.int32)
    if set_positions is not None:
        set_positions(w)
    base = oracle.centers(w["q_samples"])[0]
    stats = np.stack([np.roll(base, 3 * l, axis=0) for l in range(layers)])
    bt, nb = recipe.paged_layout(cfg, w["seq_len"])
    k = H.to_torch(recipe.to_paged(w["k"], w["seq_len"], bt, nb, block), "bf16")
    pos = torch.from_numpy(recipe.to_paged(w["pos"][..., None], w["seq_len"], bt, nb, block)[..., 0].copy()).cuda()
    k, pos = k.expand(layers, *k.shape[1:]), pos.expand(layers, *pos.shape[1:])
    seq_len, cur = torch.from_numpy(w["seq_len"]).cuda(), torch.from_numpy(w["cur_pos"]).cuda()
    model = T.Model(layers, kv_heads * group, kv_heads, 128, cfg.rope_theta, cfg.offsets)
    cache = T.Cache(k, None, pos, seq_len, cur, n, torch.from_numpy(bt).cuda())
    ws = torch.empty(T.tri_workspace_size(model, cache, budget), dtype=torch.uint8, device="cuda")
    final = torch.full((layers, S, kv_heads, n), float("nan"), device="cuda")
    raw = torch.full((layers, S, kv_heads * group, n), float("nan"), device="cuda")
    idx = torch.full((layers, S, kv_heads, budget), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((layers, S, kv_heads), -1, dtype=torch.int32, device="cuda")
    T.tri_score(model, torch.from_numpy(stats).cuda(), cache, final, raw, ws)
    T.tri_select_topk(model, final, cache, budget, idx, cnt, ws)
    torch.cuda.synchronize()
    for l in sorted({0, layers // 2, layers - 1}):
        for s, m in enumerate(lens):
            h = (s + l) % kv_heads
            assert int(cnt[l, s, h]) == min(m, budget)
            assert torch.isnan(raw[l, s, :, m:]).all() and torch.isnan(final[l, s, :, m:]).all()   # nothing past the end
            if m == 0:
                continue
            ref = oracle.head_instance(stats[l, h * group:(h + 1) * group], w["k"][0, s, h, :m], w["pos"][0, s, h, :m],
                                       int(w["cur_pos"][s]), cfg.rope_theta, cfg.offsets, budget, threads=8)
            H.check_raw(raw[l, s, h * group:(h + 1) * group, :m].cpu().numpy(), ref["raw"])
            got = final[l, s, h, :m].cpu().numpy()
            if m > 1:
                H.check_final(got, ref["final"])
            keep = oracle.topk(got.astype(np.float64), budget)
            np.testing.assert_array_equal(idx[l, s, h, :len(keep)].cpu().numpy(), keep)


@pytest.mark.parametrize("positions", ["dense", "sparse"])
@pytest.mark.parametrize("group", [1, 3, 4, 5, 8])
def test_short_ragged_sequences(oracle, group, positions):
    score_batch(oracle, group, SHORT, positions=positions)


@pytest.mark.parametrize("block", [32, 256])
def test_larger_blocks(oracle, block):
    score_batch(oracle, 6, SHORT, block=block)


@pytest.mark.parametrize("group", [5, 8])
def test_two_items_per_sequence(oracle, group):
    """Sequences beyond 8192 keys: a second item, and the shares of an item's waves on either side of their group size."""
    score_batch(oracle, group, [8300, 8192, 8193, 700], kv_heads=2, budget=500)


@pytest.mark.parametrize("group", [4, 8])
def test_wild_positions(oracle, group):
    """Unsorted positions over 2^28 (the direct path), runs of neighbours with jumps (the base moves), equal ones."""
    def set_positions(w):
        rng = np.random.default_rng(11)
        p = w["pos"]
        n = p.shape[-1]
        for s in range(p.shape[1]):
            if s % 3 == 0:
                p[:, s] = rng.integers(0, 1 << 28, size=p[:, s].shape)
            elif s % 3 == 1:
                p[:, s] = np.arange(n) + np.arange(n) // 50 * 5000
            else:
                p[:, s] = np.arange(n) // 37 * 3
        w["cur_pos"][:] = 1 << 28
    score_batch(oracle, group, SHORT, set_positions=set_positions)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("group", [4, 5])
def test_position_range(oracle, group, kind):
    """Negative positions, and both ends of int32 in one group of sixteen keys or in the step of four."""
    def set_positions(w):
        w["pos"][:] = ends_of_int32(kind, w["pos"].shape[-1]).astype(np.int32)
        if kind in ("high_then_low", "low_then_high"):   # the lone end in a step's second key
            w["pos"][:, 1::2] = np.roll(w["pos"][:, 1::2], 1, axis=-1)
        w["cur_pos"][:] = -3
    score_batch(oracle, group, [1000, 1023, 777, 640, 300, 17, 0, 901], set_positions=set_positions)
