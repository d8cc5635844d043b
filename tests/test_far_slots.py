"""Slots far apart (a token's keys of all layers and sequences next to one another): the score kernels address sixteen rows of a block, or a
tile's 64 without blocks, with 32 bits, so bf16 caches with slots up to 2^26, or 2^25, elements apart stay on the matrix kernels.  Which
kernel runs is seen without a GPU; on one, the scores are the oracle's."""
import numpy as np
import pytest
import torch

from workload import recipe

import launch_probe
import tri_harness as H


def test_kernel_by_slot_stride():
    strides = [128, 1 << 24, (1 << 25) - 8, 1 << 25, (1 << 26) - 8, 1 << 26, 1 << 30]
    for block, limit in ((0, 1 << 25), (16, 1 << 26)):
        calls = [dict(entry="score", group=4, kv_heads=2, n=3000, block=block, stride=stride) for stride in strides]
        for stride, (status, launches, _) in zip(strides, launch_probe.run(calls)):
            lane = [name for name, *_ in launches if "score_lane_kernel" in name]
            generic = [name for name, *_ in launches if "12score_kernel" in name]
            assert status == 0 and len(lane) == (stride < limit) and len(generic) == (stride >= limit), (block, stride)


@pytest.mark.gpu
@pytest.mark.parametrize("stride", [(1 << 25) - 8, (1 << 25) + 8, (1 << 26) - 8, 1 << 26])
@pytest.mark.parametrize("paged,pairs", [(False, 0), (False, 1), (True, 0), (True, 1)])
def test_scores(oracle, stride, paged, pairs):
    from paper_2604_04921_amd import binding as T
    n, heads, group, block = 70, 2, 4, 16
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged"], n_layers=1, n_seqs=1, n_q_heads=heads * group, n_kv_heads=heads, seq_len=n,
                        min_seq_len=None, budget=20, n_calib=64, positions="dense", block_size=block, seed=5)
    w = recipe.generate(cfg)
    k = H.to_torch(w["k"], "bf16")   # [1][1][heads][n][128]
    pos = torch.from_numpy(w["pos"]).cuda()
    if paged:   # blocks next to one another within a slot: [1][blocks][heads][block][128]
        blocks = -(-n // block)
        pool = torch.empty(block * stride, dtype=torch.bfloat16, device="cuda")
        kt = pool.as_strided((1, blocks, heads, block, 128), (0, heads * 128, 128, stride, 1))
        pt = torch.zeros((1, blocks, heads, block), dtype=torch.int32, device="cuda")
        for b in range(blocks):
            m = min(block, n - b * block)
            kt[:, b, :, :m] = k[:, 0, :, b * block:b * block + m]
            pt[:, b, :, :m] = pos[:, 0, :, b * block:b * block + m]
        bt = torch.arange(blocks, dtype=torch.int32, device="cuda").view(1, blocks)
    else:
        pool = torch.empty(n * stride, dtype=torch.bfloat16, device="cuda")
        kt, pt, bt = pool.as_strided((1, 1, heads, n, 128), (0, 0, 128, stride, 1)), pos, None
        kt.copy_(k)
    stats = oracle.centers(w["q_samples"], pairs=pairs)
    model = T.Model(1, heads * group, heads, 128, cfg.rope_theta, cfg.offsets, pairs)
    length, cur = torch.from_numpy(w["seq_len"]).cuda(), torch.from_numpy(w["cur_pos"]).cuda()
    cache = T.Cache(kt, None, pt, length, cur, n, bt)
    ws = torch.empty(T.tri_workspace_size(model, cache, 20), dtype=torch.uint8, device="cuda")
    final, raw = torch.zeros((1, 1, heads, n), device="cuda"), torch.zeros((1, 1, heads * group, n), device="cuda")
    T.tri_score(model, torch.from_numpy(stats).cuda(), cache, final, raw, ws)
    torch.cuda.synchronize()
    for h in range(heads):
        ref = oracle.head_instance(stats[0, h * group:(h + 1) * group], w["k"][0, 0, h], w["pos"][0, 0, h], int(w["cur_pos"][0]),
                                   cfg.rope_theta, cfg.offsets, 20, threads=8, pairs=pairs)
        H.check_raw(raw[0, 0, h * group:(h + 1) * group].cpu().numpy(), ref["raw"])
        H.check_final(final[0, 0, h].cpu().numpy(), ref["final"])
    del pool, kt
    torch.cuda.empty_cache()
