"""The calibration where its workgroups own whole heads, a half, a quarter or an eighth of the bands, for token counts around
a workgroup's residues, both storage types and pair layouts; against numpy in double.  Zero vectors, very large and very small
values and infinities included."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads,tokens", [(3, 1), (8, 257), (32, 100), (130, 129), (300, 65), (601, 33), (601, 31)])
def test_centers(heads, tokens, dtype, pairs):
    from paper_2604_04921_amd import binding as T
    g = torch.Generator().manual_seed(heads * 1000 + tokens)
    q = torch.randn((tokens, 1, heads, 128), generator=g) * torch.logspace(-3, 3, heads).view(1, 1, heads, 1)
    q[:, :, 0] = 0.0
    if heads > 2:
        q[:, :, 1] *= 1e30
        q[:, :, 2] = 1e-37
        q[0, :, 2, 4:] = 0.0
    q = (q.bfloat16() if dtype == "bf16" else q).cuda()
    out = torch.full((1, heads, 64, 3), -7.0, device="cuda")
    model = T.Model(1, heads, 1 if heads <= 8 else heads, 128, 1e6, np.array([1], dtype=np.int64), pairs)
    T.tri_build_centers(model, q, out)
    x = q.double().cpu().numpy()[:, 0]
    re, im = (x[..., :64], x[..., 64:]) if pairs else (x[..., 0::2], x[..., 1::2])
    ref = np.stack([re.mean(0), im.mean(0), np.hypot(re, im).mean(0)], axis=-1)
    # one rounding to fp32 (6e-8), and the cancellation of double sums of terms of the mean modulus' size
    tol = 1.2e-7 * np.abs(ref) + 1e-14 * ref[..., 2:] + 1e-44
    assert np.all(np.abs(out.cpu().numpy()[0].astype(np.float64) - ref) <= tol)
    q[0, 0, heads - 1, 5] = float("inf")
    T.tri_build_centers(model, q, out)
    f = 5 if pairs else 2
    got = out.cpu().numpy()[0, heads - 1]
    assert np.isinf(got[f, 2]) and np.isfinite(np.delete(got, f, axis=0)).all()
