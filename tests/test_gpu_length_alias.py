"""The fused step with the new lengths written over the old ones (new_seq_len = seq_len): the same result as into an array of its own.
An eviction that rides along with the selection must not replace a length that other workgroups still read.  In a batch that fills that
path's limit of eight head-instances per compute unit some do so late: a workgroup's 25 KB of LDS let a unit hold six, so a quarter of them begin
when others, those that write the lengths among them, have ended."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# the eviction inside the selection, all head-instances at once and as many as that takes; and in a launch of its own
@pytest.mark.parametrize("layers,n,budget", [(12, 2176, 2048), ("most", 2176, 2048), (3, 5000, 700)])
def test_new_lengths_over_the_old_ones(layers, n, budget):
    from paper_2604_04921_amd import binding as T
    heads, S, i32 = 4, 3, dict(dtype=torch.int32, device="cuda")
    if layers == "most":
        layers = 8 * torch.cuda.get_device_properties(0).multi_processor_count // (heads * S)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k = torch.randn((layers, S, heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    pos = torch.arange(n, **i32).expand(layers, S, heads, n)
    model = T.Model(layers, heads * 2, heads, 128, 1e6, [1, 2, 4, 8])
    centers = torch.randn((layers, heads * 2, 64, 3), generator=g, device="cuda")
    cur = torch.full((S,), n, **i32)
    out = []
    for alias in (False, True):
        kk, vv, pp, seq_len = k.clone(), (k + 1).clone(), pos.contiguous().clone(), torch.tensor([n, n - 9, budget + 1], **i32)
        cache = T.Cache(kk, vv, pp, seq_len, cur, n)
        new_len = seq_len if alias else torch.zeros((S,), **i32)
        idx, cnt = torch.full((layers, S, heads, budget), -1, **i32), torch.full((layers, S, heads), -1, **i32)
        ws = torch.empty(T.tri_workspace_size(model, cache, budget), dtype=torch.uint8, device="cuda")
        T.tri_compress_step(model, centers, cache, None, budget, idx, cnt, new_len, ws)
        torch.cuda.synchronize()
        out.append((kk, vv, pp, new_len, idx, cnt))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert out[0][3].tolist() == [budget] * S
