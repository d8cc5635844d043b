"""The score kernels at the edges of their work items and of their rotation paths, raw scores against the oracle: half-split
batches cut into several items per sequence (and ending inside one), positions in slot order within a tile's table, around it,
and far beyond it."""
import numpy as np
import pytest

from workload import recipe

import tri_harness as H
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,lens,paged,rotated", [
    (4, [1537, 1536, 513, 512, 1], False, False),
    (8, [1153, 1025, 1024, 513, 512], False, False),   # eight waves per workgroup
    (3, [2100, 128, 129], True, False),
    (5, [700, 1664], True, True),
    (4, [3000, 1024], False, True),
])
def test_half_split_items(oracle, group, lens, paged, rotated):
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if paged else "c2_layer"], n_layers=1, n_seqs=len(lens), n_q_heads=2 * group,
                        n_kv_heads=2, seq_len=max(lens), min_seq_len=min(lens), budget=300, n_calib=64, positions="dense",
                        block_size=16 if paged else 0, seed=77 + group)

    assert H.item_keys(2 * len(lens), max(lens)) == 512
    assert H.score_path(1, len(lens), 2, group, max(lens), 1, paged, rotated) == "items"

    def mutate(w):
        for name in ("k", "q_samples"):
            x = w[name]
            w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))
        if rotated:
            w["k"] = H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, 1, cfg.dtype)

    run_and_check(oracle, cfg, paged=paged, inplace=paged, pairs=1, mutate=mutate, rotated=rotated)


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("spread", [1, 2, 3, 4, 40, 1 << 14, 1 << 20])
@pytest.mark.parametrize("shuffled", [False, True])
def test_positions(oracle, pairs, spread, shuffled):
    """A tile of 64 keys spans 63 positions (the table), about 126 (mirrored table or direct), 189 (direct; half-split: mirrored with
    a base per 32 keys), 252 (there either), 2500, 2^20 and 2^26 (direct); shuffled, the whole sequence's range instead."""
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=1, n_seqs=1, n_q_heads=8, n_kv_heads=2, seq_len=700,
                        min_seq_len=700, budget=100, n_calib=64, positions="dense", seed=5)

    def mutate(w):
        rng = np.random.default_rng(spread + shuffled)
        n = w["pos"].shape[-1]
        p = np.arange(n, dtype=np.int64) * spread + rng.integers(0, spread, size=n)
        w["pos"][:] = (rng.permutation(p) if shuffled else p).astype(np.int32)
        w["cur_pos"][:] = min(n * spread, 2 ** 31 - 1)
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))

    run_and_check(oracle, cfg, pairs=pairs, mutate=mutate)


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("dtype,block,group,lens", [
    ("f32", 0, 4, [1025, 1022, 300]),   # rows of an odd length
    ("f32", 0, 8, [513, 256, 1]),    # tile edges, four threads per key
    ("f32", 0, 1, [255]),
    ("bf16", 4, 3, [700, 257]),      # paged blocks below 16: the same kernel on bf16
    ("bf16", 8, 8, [512, 3]),
])
def test_generic_kernel(oracle, dtype, block, group, lens, pairs):
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if block else "c2_layer"], n_layers=1, n_seqs=len(lens), n_q_heads=group,
                        n_kv_heads=1, seq_len=max(lens), min_seq_len=min(lens), budget=100, n_calib=64, positions="dense",
                        block_size=block, dtype=dtype, n_offsets=4, seed=9 + group)

    def mutate(w):
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))

    run_and_check(oracle, cfg, paged=bool(block), inplace=bool(block), pairs=pairs, mutate=mutate)
