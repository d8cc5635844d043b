"""Batches that the score kernel cuts into stretches, raw and final scores against the oracle on head-instances spread over the batch:
stretches that begin and end inside head-instances, hold more of them than a workgroup has tables for at a time, or pass over empty
sequences."""
import numpy as np
import pytest

from workload import recipe

import tri_harness as H
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,layers,heads,lens,pairs,rotated,paged", [
    (4, 5, 8, [2176] * 4, 0, False, False),                                   # pieces of 2 to 32 tiles
    # tiny and empty sequences around one longer one: many pieces to a stretch, listed four (above four heads, two) at a time
    (3, 1, 1, [(37 * i) % 130 if i % 3 else 0 for i in range(500)] + [640] + [0] * 60 + [(29 * i) % 120 for i in range(439)], 0, False, False),
    (6, 1, 1, [0] * 300 + [(41 * i) % 140 if i % 5 else 0 for i in range(699)] + [640], 1, False, True),
    (4, 1, 1, [(31 * i) % 300 if i % 4 else 0 for i in range(1023)], 0, False, False),   # the most sequences that take stretches, and one less
    (4, 1, 1, [(31 * i) % 300 if i % 4 else 0 for i in range(1024)], 0, True, False),
    (8, 3, 4, [2000, 700, 1, 2100, 0, 64, 65, 2101, 900, 1300, 1999], 0, False, False),
    (4, 5, 8, [2100, 300, 2175, 0, 1000], 1, False, False),
    (4, 5, 8, [2100, 300, 2175, 0, 1000], 0, False, True),
    (5, 5, 8, [2100, 300, 2175, 0, 1000], 1, True, False),
    (2, 5, 8, [2100, 300, 2175, 0, 1000], 1, False, True),
])
def test_stretches(oracle, group, layers, heads, lens, pairs, rotated, paged):
    assert H.score_path(layers, len(lens), heads, group, max(lens), pairs, paged, rotated) == "stretches"
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if paged else "c2_layer"], n_layers=layers, n_seqs=len(lens), n_q_heads=heads * group,
                        n_kv_heads=heads, seq_len=max(lens), min_seq_len=0, budget=60 if len(lens) > 100 else 500, n_calib=16,
                        positions="dense", block_size=16 if paged else 0, seed=7 + group)
    rng = np.random.default_rng(3)
    last = layers * len(lens) * heads - 1
    picks = sorted({0, last} | set(rng.integers(0, last, size=22).tolist()))
    instances = [(i // (len(lens) * heads), i // heads % len(lens), i % heads) for i in picks]

    def mutate(w):
        w["seq_len"][:] = lens
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))
        if rotated:
            w["k"] = H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, pairs, cfg.dtype)

    run_and_check(oracle, cfg, instances=instances, paged=paged, pairs=pairs, mutate=mutate, rotated=rotated)


def test_one_sequence_too_many_for_stretches(oracle):
    lens = [(31 * i) % 300 if i % 4 else 0 for i in range(1025)]
    assert H.score_path(1, len(lens), 1, 4, max(lens)) == "items"
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=1, n_seqs=len(lens), n_q_heads=4, n_kv_heads=1, seq_len=max(lens), min_seq_len=0,
                        budget=60, n_calib=16, positions="dense", seed=7)

    def mutate(w):
        w["seq_len"][:] = lens

    run_and_check(oracle, cfg, instances=[(0, s, 0) for s in range(0, 1025, 64)] + [(0, 1023, 0)], mutate=mutate)


@pytest.mark.parametrize("group,lens,n,pairs,rotated,paged", [
    (4, [130, 700, 64, 0, 1, 900], 4096, 0, False, False),    # fewer tiles than eight per CU
    (4, [64, 1, 0, 0, 63, 2], 4096, 1, False, True),          # fewer than one per CU
    (8, [2000, 1500, 0, 1700, 64, 1999], 4096, 0, False, False),
    (2, [3, 4000, 0, 0, 64, 65], 4096, 0, True, True)])
def test_lengths_far_below_the_reserved_one(oracle, group, lens, n, pairs, rotated, paged):
    layers, heads = 3, 8
    assert H.score_path(layers, len(lens), heads, group, n, pairs, paged, rotated) == "stretches"
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if paged else "c2_layer"], n_layers=layers, n_seqs=len(lens), n_q_heads=heads * group,
                        n_kv_heads=heads, seq_len=n, min_seq_len=0, budget=100, n_calib=16, positions="sparse", block_size=16 if paged else 0,
                        seed=17 + group)
    rng = np.random.default_rng(5)
    last = layers * len(lens) * heads - 1
    picks = sorted({0, last} | set(rng.integers(0, last, size=30).tolist()))

    def mutate(w):
        w["seq_len"][:] = lens
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))
        if rotated:
            w["k"] = H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, pairs, cfg.dtype)

    run_and_check(oracle, cfg, instances=[(i // (len(lens) * heads), i // heads % len(lens), i % heads) for i in picks], paged=paged, pairs=pairs,
                  mutate=mutate, rotated=rotated)
