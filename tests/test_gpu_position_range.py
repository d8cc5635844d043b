"""Positions over the whole range of int32, raw and final scores against the oracle: negative ones, ones that cross zero, and tiles
that hold both ends of the range, where a difference of two positions formed in 32 bits would come out small."""
import numpy as np
import pytest

from workload import recipe

from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu

LO, HI = -2 ** 31, 2 ** 31 - 1


def positions(kind, n):
    k = np.arange(n, dtype=np.int64)
    if kind == "negative":           # in slot order, all below zero
        return k - n - 5
    if kind == "around_zero":        # every other tile's base below zero
        return k - n // 2
    if kind == "high_then_low":      # the tile's first slot at the top, the others at the bottom of the range
        return np.where(k % 64 == 0, HI, LO + k % 64 - 1)
    if kind == "low_then_high":
        return np.where(k % 64 == 0, LO, HI - k % 64 + 1)
    if kind == "wrapping":           # k -> HI - 31, ..., HI, LO, LO + 1, ... in every tile
        p = HI - 31 + k % 64
        return np.where(p > HI, p - 2 ** 32, p)
    raise ValueError(kind)


KINDS = ["negative", "around_zero", "high_then_low", "low_then_high", "wrapping"]


def set_positions(w, kind):
    w["pos"][:] = positions(kind, w["pos"].shape[-1]).astype(np.int32)
    w["cur_pos"][:] = np.int32(HI if kind in ("high_then_low", "wrapping") else -3)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("pairs,paged,group", [(0, False, 4), (0, True, 4), (0, False, 8), (1, False, 4), (1, True, 5)])
def test_position_range(oracle, kind, pairs, paged, group):
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if paged else "c2_layer"], n_layers=1, n_seqs=2, n_q_heads=2 * group, n_kv_heads=2,
                        seq_len=333, min_seq_len=200, budget=60, n_calib=64, positions="dense", seed=21)

    def mutate(w):
        set_positions(w, kind)
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))

    run_and_check(oracle, cfg, paged=paged, inplace=paged, pairs=pairs, mutate=mutate)


@pytest.mark.parametrize("kind", KINDS)
def test_position_range_fp32_keys(oracle, kind):
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=1, n_seqs=1, n_q_heads=8, n_kv_heads=2, seq_len=300, min_seq_len=300,
                        budget=60, n_calib=64, positions="dense", dtype="f32", seed=22)
    run_and_check(oracle, cfg, mutate=lambda w: set_positions(w, kind))
