"""Score arrays that start on a float's boundary only: tri_score's final_out and raw_out, the same bits as into aligned arrays and
nothing written beside them."""
import numpy as np
import pytest
import torch

from workload import recipe

import tri_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("final_off,raw_off", [(1, 0), (0, 3), (2, 1), (3, None)])
@pytest.mark.parametrize("dtype,n,group", [("bf16", 1000, 4), ("bf16", 1000, 5), ("bf16", 999, 4), ("f32", 1000, 4)])
def test_unaligned_outputs(dtype, n, group, final_off, raw_off):
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=1, n_seqs=3, n_q_heads=2 * group, n_kv_heads=2, seq_len=n, min_seq_len=n - 70,
                        budget=100, n_calib=64, dtype=dtype)
    run = H.GpuRun(cfg, recipe.generate(cfg))
    run.build_centers()
    run.score()

    def shifted(like, off):
        buf = torch.full((like.numel() + 8,), float("nan"), device="cuda")
        return buf, buf[off:off + like.numel()].view(like.shape)

    fbuf, final = shifted(run.final, final_off)
    rbuf, raw = shifted(run.raw, raw_off or 0)
    run.B.tri_score(run.model, run.centers, run.cache, final, None if raw_off is None else raw, run.ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(final.cpu().numpy(), run.final.cpu().numpy())   # NaN past a sequence's end on both sides
    assert torch.isnan(fbuf[:final_off]).all() and torch.isnan(fbuf[final_off + final.numel():]).all()
    if raw_off is not None:
        np.testing.assert_array_equal(raw.cpu().numpy(), run.raw.cpu().numpy())
        assert torch.isnan(rbuf[:raw_off]).all() and torch.isnan(rbuf[raw_off + raw.numel():]).all()
