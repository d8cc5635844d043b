"""The selection at the edges of its paths: row and workgroup tails, rows that are no multiple of four entries (scalar loads),
1024- and 256-thread workgroups, keys in LDS up to 32768 and through memory beyond, chunks of the key kernel that begin or
end at a sequence's end.  Integer work on the GPU's own fp32 scores, so the kept sets must equal the oracle's bit for bit,
and those of the fused step those of the separate calls."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,kv_heads,group,lens,budget", [
    (1, 1, 4, [255, 1], 64),                     # one row of 256 slots and its tail
    (1, 2, 1, [1027, 1026, 65, 64], 64),         # scalar loads, N on either side of the budget
    (33, 2, 4, [260, 129], 128),                 # 132 head-instances: 256 threads per workgroup
    (33, 2, 3, [261, 256], 100),                 # the same with scalar loads
    (1, 2, 8, [4096, 4095, 3841], 512),          # the last size of the short kernel's rule
    (1, 2, 5, [4097, 4096, 2000], 512),
    (1, 1, 2, [32768, 32767, 700], 2048),        # the last size whose keys LDS holds
    (1, 1, 4, [32769, 32768, 4096, 4097, 512], 512),   # through memory, scalar loads; sequences that end on a chunk's edge
    (1, 1, 7, [32772, 8192, 8193], 2048),        # through memory, 16-byte loads
    (1, 1, 8, [65540, 61440, 61441], 4096),      # chunks of 8192 keys
])
def test_kept_sets_at_the_edges(oracle, layers, kv_heads, group, lens, budget):
    n = max(lens)
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=layers, n_seqs=len(lens), n_q_heads=kv_heads * group,
                        n_kv_heads=kv_heads, seq_len=n, min_seq_len=None, budget=budget, n_calib=64, positions="dense")
    w = recipe.generate(cfg)
    w["seq_len"] = np.array(lens, dtype=np.int32)
    run = H.GpuRun(cfg, w)
    run.build_centers()
    final, _ = run.score(want_raw=False)
    idx, cnt = run.select()
    for l in (0, layers - 1):
        for s, m in enumerate(lens):
            for h in range(kv_heads):
                ref = oracle.topk(final[l, s, h, :m].astype(np.float64), budget)
                assert cnt[l, s, h] == len(ref) == min(m, budget)
                np.testing.assert_array_equal(idx[l, s, h, :len(ref)], ref)
                assert np.all(idx[l, s, h, len(ref):] == -1)
    run.kept_idx.fill_(-1)
    run.kept_cnt.fill_(-1)
    kd = torch.zeros((layers, len(lens), kv_heads, budget, cfg.head_dim), dtype=run.k.dtype, device="cuda")
    vd, pd = torch.zeros_like(kd), torch.zeros(kd.shape[:-1], dtype=torch.int32, device="cuda")
    dst = run.B.Cache(kd, vd, pd, run.seq_len, run.cur_pos, budget)
    run.B.tri_compress_step(run.model, run.centers, run.cache, dst, budget, run.kept_idx, run.kept_cnt, run.new_len, run.ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.kept_cnt.cpu().numpy(), cnt)
    np.testing.assert_array_equal(run.kept_idx.cpu().numpy(), idx)


@pytest.mark.parametrize("n,kind", [(2176, "ties"), (4100, "ties"), (2176, "bin"), (4100, "bin"), (33001, "bin")])
def test_threshold_bin_longer_than_the_list(oracle, n, kind):
    """More keys in the threshold's bin than its list of 1024 holds: equal scores, or distinct ones within one bin; final scores
    from an address that is no multiple of 16 bytes."""
    from paper_2604_04921_amd import binding as T
    rng = np.random.default_rng(n)
    budget, heads = 1500, 2
    f = np.full((heads, n), 0.5, dtype=np.float32) if kind == "ties" else (1.0 + rng.random((heads, n)) * 1e-3).astype(np.float32)
    m = rng.random((heads, n)) < 0.05
    f[m] = rng.standard_normal(int(m.sum())).astype(np.float32)
    buf = torch.zeros(heads * n + 1, dtype=torch.float32, device="cuda")
    buf[1:] = torch.from_numpy(f).cuda().view(-1)
    model = T.Model(1, heads, heads, 128, 1e4, np.array([1], dtype=np.int64))
    k = torch.zeros((1, 1, heads, 1, 128), dtype=torch.bfloat16, device="cuda").expand(1, 1, heads, n, 128)
    one = torch.full((1,), n, dtype=torch.int32, device="cuda")
    cache = T.Cache(k, None, torch.zeros((1, 1, heads, n), dtype=torch.int32, device="cuda"), one, one, n)
    idx = torch.full((1, 1, heads, budget), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((1, 1, heads), dtype=torch.int32, device="cuda")
    T.tri_select_topk(model, buf[1:].view(1, 1, heads, n), cache, budget, idx, cnt)
    torch.cuda.synchronize()
    for h in range(heads):
        assert int(cnt[0, 0, h]) == budget
        np.testing.assert_array_equal(idx[0, 0, h].cpu().numpy(), oracle.topk(f[h].astype(np.float64), budget))


@pytest.mark.parametrize("layers", [1, 33])   # 4 and 132 head-instances: 1024 and 256 threads per workgroup
@pytest.mark.parametrize("n,budget", [(300, 128), (2176, 2048)])
def test_eviction_at_the_end_of_the_selection(layers, n, budget):
    """The fused step's eviction in place (moves made by the selection's workgroup) against selection and tri_compact_fill."""
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=layers, n_seqs=2, n_q_heads=8, n_kv_heads=2, seq_len=n,
                        min_seq_len=budget - 1, budget=budget, n_calib=64)
    run = H.GpuRun(cfg, recipe.generate(cfg))
    run.build_centers()
    B, before = run.B, [t.clone() for t in (run.k, run.v, run.pos)]
    run.score(want_raw=False)
    run.select()
    B.tri_compact_fill(run.model, run.cache, budget, run.kept_idx, run.kept_cnt, run.new_len)
    torch.cuda.synchronize()
    want = [t.clone() for t in (run.k, run.v, run.pos, run.kept_idx, run.kept_cnt, run.new_len)]
    for t, b in zip((run.k, run.v, run.pos), before):
        t.copy_(b)
    for t in (run.kept_idx, run.kept_cnt, run.new_len):
        t.fill_(-1)
    B.tri_compress_step(run.model, run.centers, run.cache, None, budget, run.kept_idx, run.kept_cnt, run.new_len, run.ws)
    torch.cuda.synchronize()
    for t, w in zip((run.k, run.v, run.pos, run.kept_idx, run.kept_cnt, run.new_len), want):
        assert torch.equal(t, w)
