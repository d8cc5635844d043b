"""Work items that follow one another in a workgroup: thousands of head-instances of ragged lengths, so that every workgroup takes
several items or stretches, many of the items with fewer tiles than the workgroup has waves, and rows of raw scores that start on cache lines
or do not; and the generic kernel's tiles of one and of two parts.  Raw and final scores of every length against the oracle.  The layers
share one layer's keys (stride 0) and differ in their query statistics."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H

pytestmark = pytest.mark.gpu

LENS = [1, 64, 65, 129, 0, 511, 640, 700, 767, 768, 769, 900, 1023, 1024, 300, 1000]


def check(oracle, lens, per_cu, group, pairs, paged, rotated, n, dtype="bf16", block=16, path=None):
    from paper_2604_04921_amd import binding as T
    kv_heads, S, n_cu = 4, len(lens), torch.cuda.get_device_properties(0).multi_processor_count
    layers = max(1, int(-(-per_cu * n_cu // (S * kv_heads))))
    assert path is None or H.score_path(layers, S, kv_heads, group, n, pairs, paged, rotated) == path
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged"], n_layers=1, n_seqs=S, n_q_heads=kv_heads * group, n_kv_heads=kv_heads, seq_len=n,
                        min_seq_len=None, budget=40, n_calib=64, positions="sparse" if group == 4 else "dense", block_size=block, dtype=dtype, seed=77 + group)
    w = recipe.generate(cfg)
    w["seq_len"] = np.array(lens, dtype=np.int32)
    if pairs:
        for name in ("k", "q_samples"):
            w[name] = np.ascontiguousarray(np.concatenate([w[name][..., 0::2], w[name][..., 1::2]], axis=-1))
    base = oracle.centers(w["q_samples"], pairs=pairs)[0]
    stats = np.stack([np.roll(base, 5 * l, axis=0) for l in range(layers)])
    k = H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, pairs, cfg.dtype) if rotated else w["k"]
    bt = None
    if paged:
        bt, nb = recipe.paged_layout(cfg, w["seq_len"])
        kt = H.to_torch(recipe.to_paged(k, w["seq_len"], bt, nb, block), dtype)
        pos = torch.from_numpy(recipe.to_paged(w["pos"][..., None], w["seq_len"], bt, nb, block)[..., 0].copy()).cuda()
        bt = torch.from_numpy(bt).cuda()
    else:
        kt, pos = H.to_torch(k, dtype), torch.from_numpy(w["pos"]).cuda()
    kt, pos = kt.expand(layers, *kt.shape[1:]), pos.expand(layers, *pos.shape[1:])
    model = T.Model(layers, kv_heads * group, kv_heads, 128, cfg.rope_theta, cfg.offsets, pairs)
    cache = T.Cache(kt, None, pos, torch.from_numpy(w["seq_len"]).cuda(), torch.from_numpy(w["cur_pos"]).cuda(), n, bt, k_rotated=rotated)
    ws = torch.empty(T.tri_workspace_size(model, cache, 40), dtype=torch.uint8, device="cuda")
    final = torch.full((layers, S, kv_heads, n), float("nan"), device="cuda")
    raw = torch.full((layers, S, kv_heads * group, n), float("nan"), device="cuda")
    T.tri_score(model, torch.from_numpy(stats).cuda(), cache, final, raw, ws)
    torch.cuda.synchronize()
    for s, m in enumerate(lens):
        assert torch.isnan(raw[:, s, :, m:]).all() and torch.isnan(final[:, s, :, m:]).all()   # nothing past the end
        if m == 0:
            continue
        for l in {0, layers // 2, layers - 1}:
            h = (s + l) % kv_heads
            ref = oracle.head_instance(stats[l, h * group:(h + 1) * group], k[0, s, h, :m], w["pos"][0, s, h, :m], int(w["cur_pos"][s]),
                                       cfg.rope_theta, cfg.offsets, 40, threads=8, pairs=pairs, rotated=rotated)
            H.check_raw(raw[l, s, h * group:(h + 1) * group, :m].cpu().numpy(), ref["raw"])
            if m > 1:
                H.check_final(final[l, s, h, :m].cpu().numpy(), ref["final"])


@pytest.mark.parametrize("group,pairs,paged,rotated,n", [(4, 0, False, False, 1024), (4, 1, False, False, 1031), (3, 1, True, False, 1028),
                                                         (1, 0, True, False, 1056), (8, 0, False, False, 1025), (6, 1, True, True, 1024),
                                                         (4, 0, False, True, 1030)])
@pytest.mark.parametrize("per_cu,path", [(6, "stretches"), (8, "items")])   # eight head-instances per CU: a large batch
def test_chained_items(oracle, group, pairs, paged, rotated, n, per_cu, path):
    if path == "items" and paged and not pairs and not rotated:
        path = "sixteen"
    check(oracle, LENS, per_cu, group, pairs, paged, rotated, n, path=path)


# three stretches per workgroup and more, all of them its own
@pytest.mark.parametrize("group,pairs,paged,rotated", [(4, 0, False, False), (3, 1, True, False), (8, 0, False, False), (2, 1, True, True)])
def test_chained_stretches(oracle, group, pairs, paged, rotated):
    lens = [2047, 2000, 1999, 1984, 1, 0, 2046, 1900, 1800, 1700, 64, 2047, 1930, 1111, 2045, 2040]
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    layers = int(-(-7.5 * n_cu // (len(lens) * 4)))
    tiles = sum(-(-m // 64) for m in lens) * layers * 4
    assert H.stretches(layers * len(lens) * 4, group, lens, tiles, 2047, pairs, paged, rotated) >= 3 * n_cu
    check(oracle, lens, 7.5, group, pairs, paged, rotated, 2047, path="stretches")


# more than eight: its own two, then the counter's
@pytest.mark.parametrize("group,pairs,paged,rotated", [(4, 0, False, False), (3, 1, True, False), (8, 0, False, False), (2, 1, True, True)])
def test_counted_stretches(oracle, group, pairs, paged, rotated):
    lens = [8100, 8191, 7000, 7936, 1, 0, 8000, 7700, 6400, 8191, 64, 7999, 8190, 1111, 8064, 8129]
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    layers = int(-(-7.5 * n_cu // (len(lens) * 4)))
    tiles = sum(-(-m // 64) for m in lens) * layers * 4
    assert H.stretches(layers * len(lens) * 4, group, lens, tiles, 8191, pairs, paged, rotated) > 8 * n_cu
    check(oracle, lens, 7.5, group, pairs, paged, rotated, 8191, path="stretches")


# many head-instances: tiles of two parts; few: of one, the moments in the phasor table's place
@pytest.mark.parametrize("per_cu", [6, 0])
@pytest.mark.parametrize("group,pairs,paged,rotated,dtype", [(4, 0, False, False, "f32"), (8, 1, False, False, "f32"), (1, 0, True, False, "f32"),
                                                             (5, 1, True, True, "f32"), (4, 0, True, False, "bf16"), (2, 1, True, False, "bf16")])
def test_parts_of_the_generic_kernel(oracle, group, pairs, paged, rotated, dtype, per_cu):
    check(oracle, [1, 127, 128, 129, 0, 255, 256, 257, 300, 383, 385, 511, 512, 513, 64, 600], per_cu, group, pairs, paged, rotated, 600, dtype, block=8)
