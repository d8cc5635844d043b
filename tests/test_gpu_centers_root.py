"""The calibration's moduli in double: sums of one and of a few tokens against numpy, over the magnitudes that fp32 samples can have."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tokens", [1, 3])
def test_moduli(tokens, dtype, pairs):
    from paper_2604_04921_amd import binding as T
    heads = 40
    g = torch.Generator().manual_seed(tokens)
    q = torch.randn((tokens, 1, heads, 128), generator=g, dtype=torch.float64) * torch.logspace(-37, 37, heads, dtype=torch.float64).view(1, 1, heads, 1)
    q[:, :, :, 3] = 0.0
    q[:, :, 5] = 0.0
    q = q.float()
    q = (q.bfloat16() if dtype == "bf16" else q).cuda()
    sums = torch.full((1, heads, 64, 3), float("nan"), dtype=torch.float64, device="cuda")
    T.tri_centers_accumulate(T.Model(1, heads, heads, 128, 1e6, np.array([1], dtype=np.int64), pairs), q, sums, first=True)
    x = q.double().cpu().numpy()[:, 0]
    re, im = (x[..., :64], x[..., 64:]) if pairs else (x[..., 0::2], x[..., 1::2])
    ref = np.sqrt(re.astype(np.longdouble) ** 2 + im.astype(np.longdouble) ** 2).sum(0).astype(np.float64)
    got = sums.cpu().numpy()[0]
    # a rounding in the sum of squares, a unit in the last place of the root, one rounding per addition
    assert np.all(np.abs(got[..., 2] - ref) <= (1.5 + tokens) * 2.3e-16 * ref)
    assert np.all(got[5] == 0.0)
    if tokens == 1:
        assert np.array_equal(got[..., 0], re[0]) and np.array_equal(got[..., 1], im[0])
