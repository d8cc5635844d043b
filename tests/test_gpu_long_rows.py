"""Scores of rows with more moments than the statistics ask for at once (64 tiles), on the kernel for fp32 keys and small blocks: tiles of 128
and of 256 keys, few workgroups and many, lengths around a multiple of 64 tiles, against the oracle; and the fused step's kept set against
the separate calls'."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,group,dtype,block", [
    ([8192, 8193], 4, "f32", 0), ([16384, 16385, 17000], 2, "f32", 0), ([33000], 8, "f32", 0), ([66000, 200], 1, "f32", 0),
    ([140000], 2, "f32", 0), ([33000, 32768], 1, "bf16", 8), ([70001], 4, "bf16", 8)])
def test_long_rows(oracle, lens, group, dtype, block):
    n, budget = max(lens), 300
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged"], n_layers=1, n_seqs=len(lens), n_q_heads=group, n_kv_heads=1, seq_len=n,
                        min_seq_len=None, budget=budget, n_calib=64, positions="dense", block_size=block or 16, dtype=dtype, seed=n)
    w = recipe.generate(cfg)
    w["seq_len"] = np.array(lens, dtype=np.int32)
    run = H.GpuRun(cfg, w, paged=block != 0)
    stats = run.build_centers()
    final, raw = run.score()
    idx, cnt = run.select()
    for s, m in enumerate(lens):
        ref = oracle.head_instance(stats[0], w["k"][0, s, 0, :m], w["pos"][0, s, 0, :m], int(w["cur_pos"][s]), cfg.rope_theta,
                                   cfg.offsets, budget, threads=8)
        H.check_raw(raw[0, s, :, :m], ref["raw"])
        H.check_final(final[0, s, 0, :m], ref["final"])
    run.kept_idx.fill_(-1)
    run.B.tri_compress_step(run.model, run.centers, run.cache, run.cache, budget, run.kept_idx, run.kept_cnt, run.new_len, run.ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.kept_idx.cpu().numpy(), idx)
    np.testing.assert_array_equal(run.kept_cnt.cpu().numpy(), cnt)
