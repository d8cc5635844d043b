"""The folded table where a workgroup of the fold has all bands, half of them or a quarter (few layers x heads x sequences), for numbers of
offsets and sequences that fill its threads once, several times and partly: raw scores against the oracle."""
import pytest

from workload import recipe

from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,heads,seqs,group,offsets", [
    (1, 1, 1, 1, 1), (1, 1, 1, 8, 16), (1, 2, 3, 3, 31), (2, 8, 2, 4, 16),      # four parts
    (5, 8, 2, 2, 16), (4, 8, 9, 5, 31),                                         # two
    (9, 8, 1, 4, 31), (3, 8, 17, 7, 2)])                                        # one
def test_parts(oracle, layers, heads, seqs, group, offsets):
    cfg = recipe.scaled(recipe.CONFIGS["c2_layer"], n_layers=layers, n_seqs=seqs, n_q_heads=heads * group, n_kv_heads=heads, seq_len=100,
                        min_seq_len=70, budget=30, n_calib=16, n_offsets=offsets, positions="dense", seed=layers + 10 * seqs)
    last = layers * seqs * heads - 1
    picks = sorted({0, last, last // 2, last // 3, 2 * last // 3, last // 5})
    run_and_check(oracle, cfg, instances=[(i // (seqs * heads), i // heads % seqs, i % heads) for i in picks])
