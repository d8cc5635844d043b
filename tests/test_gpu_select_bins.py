"""The selection where scores lie on the edges of its histogram's bins and next to them: (k - 512) / 128 and the floats around it, ends of
the range, zeros and infinities included, with thresholds inside such a cluster -- all of its ties kept, or some -- against the
oracle's full sort.  Rows in LDS and in memory."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 20000, 33001])
@pytest.mark.parametrize("edge", [0, 1, 511, 512, 513, 777, 2047, 2048])
def test_edges_of_bins(oracle, n, edge):
    from paper_2604_04921_amd import binding as T
    rng = np.random.default_rng(1000 * edge + n)
    at = np.float32((edge - 512) / 128)
    near = [at]
    for way in (np.float32(-np.inf), np.float32(np.inf)):
        x = at
        for _ in range(6):
            x = np.nextafter(x, way)
            near.append(x)
        near += [at + np.float32(d) * (1 if way > 0 else -1) for d in (2.0 ** -24, 2.0 ** -23, 2.0 ** -20, 1 / 256, 1 / 128)]
    near = np.unique(np.array(near + [0.0, -0.0], dtype=np.float32))
    final = rng.uniform(-5, 13, size=n).astype(np.float32)
    final[rng.random(n) < 0.02] = np.float32(np.inf)
    final[rng.random(n) < 0.02] = np.float32(-np.inf)
    spot = rng.random(n) < 0.1
    final[spot] = rng.choice(near, size=int(spot.sum()))
    model = T.Model(1, 1, 1, 128, 1e4, np.array([1], dtype=np.int64))
    k = torch.zeros((1, 1, 1, 1, 128), dtype=torch.bfloat16, device="cuda").expand(1, 1, 1, n, 128)
    cache = T.Cache(k, None, torch.zeros((1, 1, 1, n), dtype=torch.int32, device="cuda"), torch.tensor([n], dtype=torch.int32, device="cuda"),
                    torch.zeros(1, dtype=torch.int32, device="cuda"), n)
    scores = torch.from_numpy(final).cuda().view(1, 1, 1, n)
    reach = int((final >= at).sum())
    for budget in sorted({b for b in (reach - 40, reach - 1, reach, reach + 1, reach + 40) if 0 < b < n}):
        kept = torch.full((1, 1, 1, budget), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((1, 1, 1), -7, dtype=torch.int32, device="cuda")
        T.tri_select_topk(model, scores, cache, budget, kept, cnt)
        ref = oracle.topk(np.clip(final.astype(np.float64), -1e300, 1e300), budget)
        assert int(cnt.item()) == budget
        np.testing.assert_array_equal(kept.view(-1).cpu().numpy(), ref, err_msg="budget %d" % budget)
