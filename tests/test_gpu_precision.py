"""The fp32 sums of the score kernels against 64 bits: the kernel that takes most bf16 caches may leave final scores no further from
the oracle's than the sixteen-lane kernel does on the same keys (which that one scores when the batch is large)."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H
import tri_rules as R

pytestmark = pytest.mark.gpu

GROUP, HEADS, LENS, BUDGET, BLOCK = 4, 8, [1000, 1024, 777, 960, 333, 1001, 640, 900], 100, 16


def config(positions):
    return recipe.scaled(recipe.CONFIGS["c4_paged"], n_layers=1, n_seqs=len(LENS), n_q_heads=GROUP * HEADS, n_kv_heads=HEADS,
                         seq_len=max(LENS), min_seq_len=None, budget=BUDGET, n_calib=64, block_size=BLOCK, seed=91,
                         positions="dense" if positions == "scattered" else positions)


@pytest.fixture(scope="module", params=["dense", "sparse", "scattered"])
def case(request, oracle):
    """One layer's workload, its statistics, and how far the sixteen-lane kernel's final scores are from the oracle's."""
    cfg = config(request.param)
    w = recipe.generate(cfg)
    w["seq_len"] = np.array(LENS, dtype=np.int32)
    if request.param == "scattered":
        rng = np.random.default_rng(4)
        w["pos"][:] = rng.integers(0, 40000, size=w["pos"].shape)
        w["cur_pos"][:] = 40000
    stats = oracle.centers(w["q_samples"])
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    layers = -(-8 * n_cu // (len(LENS) * HEADS))
    assert R.sixteen_lane_kernel(GROUP, layers * len(LENS) * HEADS, max(LENS), n_cu)
    assert not R.sixteen_lane_kernel(GROUP, len(LENS) * HEADS, max(LENS), n_cu)
    exact = reference(oracle, cfg, w, stats)
    return request.param, cfg, w, stats, exact, distance(scores(cfg, w, stats, layers), exact)


def reference(oracle, cfg, w, stats, **kw):
    return {(s, h): oracle.head_instance(stats[0, h * GROUP:(h + 1) * GROUP], w["k"][0, s, h, :n], w["pos"][0, s, h, :n],
                                         int(w["cur_pos"][s]), cfg.rope_theta, cfg.offsets, BUDGET, threads=8, **kw)["final"]
            for s, n in enumerate(LENS) for h in range(HEADS)}


def scores(cfg, w, stats, layers=1, paged=True, pairs=0, rotated=False):
    """Final scores of layer 0 (the layers share one layer's keys)."""
    from paper_2604_04921_amd import binding as T
    if paged:
        bt, nb = recipe.paged_layout(cfg, w["seq_len"])
        k = H.to_torch(recipe.to_paged(w["k"], w["seq_len"], bt, nb, BLOCK), "bf16")
        pos = torch.from_numpy(recipe.to_paged(w["pos"][..., None], w["seq_len"], bt, nb, BLOCK)[..., 0].copy()).cuda()
        bt = torch.from_numpy(bt).cuda()
    else:
        k, pos, bt = H.to_torch(w["k"], "bf16"), torch.from_numpy(w["pos"]).cuda(), None
    k, pos = k.expand(layers, *k.shape[1:]), pos.expand(layers, *pos.shape[1:])
    model = T.Model(layers, GROUP * HEADS, HEADS, 128, cfg.rope_theta, cfg.offsets, pairs)
    cache = T.Cache(k, None, pos, torch.from_numpy(w["seq_len"]).cuda(), torch.from_numpy(w["cur_pos"]).cuda(), max(LENS), bt,
                    k_rotated=rotated)
    ws = torch.empty(T.tri_workspace_size(model, cache, BUDGET), dtype=torch.uint8, device="cuda")
    final = torch.zeros((layers, len(LENS), HEADS, max(LENS)), device="cuda")
    centers = torch.from_numpy(stats).cuda().expand(layers, *stats.shape[1:]).contiguous()
    T.tri_score(model, centers, cache, final, None, ws)
    torch.cuda.synchronize()
    return final[0].cpu().numpy().astype(np.float64)


def distance(final, exact):
    num = sum(np.sum((final[s, h, :len(f)] - f) ** 2) for (s, h), f in exact.items())
    return float(np.sqrt(num / sum(np.sum(f ** 2) for f in exact.values())))


def half_split(w):
    return dict(w, k=np.ascontiguousarray(np.concatenate([w["k"][..., 0::2], w["k"][..., 1::2]], axis=-1)))


@pytest.mark.parametrize("paged,pairs", [(True, 0), (True, 1), (False, 1)])   # (contiguous interleaved keys' sums are longer)
def test_no_further_from_64_bits(case, paged, pairs):
    kind, cfg, w, stats, exact, bound = case
    d = distance(scores(cfg, half_split(w) if pairs else w, stats, paged=paged, pairs=pairs), exact)
    print("\n[%s pairs %d paged %d] %.3e, sixteen-lane kernel %.3e" % (kind, pairs, paged, d, bound), flush=True)
    assert d <= 1.02 * bound   # two sets of roundings of some 60000 scores each: their norms differ by about one per cent


@pytest.mark.parametrize("pairs", [0, 1])
def test_post_rope(case, oracle, pairs):
    """Without a rotation there are two roundings less per product: closer than the pre-RoPE scores by a tenth and more (the
    sixteen-lane kernel's post-RoPE variant: by 17 %)."""
    kind, cfg, w, stats, _, bound = case
    if pairs:
        w = half_split(w)
    w = dict(w, k=H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, pairs, "bf16"))
    exact = reference(oracle, cfg, w, stats, pairs=pairs, rotated=True)
    d = distance(scores(cfg, w, stats, pairs=pairs, rotated=True), exact)
    print("\n[%s post-RoPE pairs %d] %.3e, sixteen-lane kernel pre-RoPE %.3e" % (kind, pairs, d, bound), flush=True)
    assert d <= 0.9 * bound
