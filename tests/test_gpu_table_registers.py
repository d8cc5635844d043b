"""The score kernel's table, one block of lanes of which a matrix instruction hands to the others: every group size (whole and partial
quads of query heads) in each way of handing out the work, at the edges of tiles and of a workgroup's round of tiles."""
import numpy as np
import pytest

from workload import recipe

import tri_harness as H
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", range(1, 9))
@pytest.mark.parametrize("pairs,rotated,paged", [(0, False, False), (0, False, True), (1, False, False), (0, True, False)])
def test_every_group(oracle, group, pairs, rotated, paged):
    lens = [1, 63, 65, 512, 769]
    cfg = recipe.scaled(recipe.CONFIGS["c4_paged" if paged else "c2_layer"], n_layers=1, n_seqs=len(lens), n_q_heads=2 * group,
                        n_kv_heads=2, seq_len=max(lens), min_seq_len=min(lens), budget=200, n_calib=64, positions="dense",
                        block_size=16 if paged else 0, seed=40 + group)

    def mutate(w):
        w["seq_len"][:] = lens
        if pairs:
            for name in ("k", "q_samples"):
                x = w[name]
                w[name] = np.ascontiguousarray(np.concatenate([x[..., 0::2], x[..., 1::2]], axis=-1))
        if rotated:
            w["k"] = H.to_post_rope(w["k"], w["pos"], cfg.rope_theta, pairs, cfg.dtype)

    run_and_check(oracle, cfg, paged=paged, pairs=pairs, mutate=mutate, rotated=rotated)
