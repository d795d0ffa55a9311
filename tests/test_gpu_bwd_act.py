"""Attention backward through the projection's activation: bit for bit the attention backward followed by
the pointwise SiLU backward, in both backward forms, at every head_dim, with rows on both sides of a
wave's 32 and a workgroup's 128, with and without a bias (GPU)."""
import numpy as np
import pytest
import torch

from paper_2505_18654_amd import hstu, layer, ops
from tests.gpu_util import custom_layout
from tests.test_gpu_layer import params_for, to_dev

pytestmark = pytest.mark.gpu


def batch(heads, dh, lens=(1, 31, 33, 128, 129, 300)):
    rng = np.random.default_rng(8)
    segs = [np.sort(rng.integers(0, 4, n)) for n in lens]
    L = custom_layout(segs, [rng.integers(0, 5000, len(s)) for s in segs], heads=heads, head_dim=dh)
    return L.total_tokens, ops.Jagged.from_host(L.offsets, L.seg, L.ts)


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("rab_on,bias_on", [(False, True), (True, True), (True, False)])
def test_bits(dh, stored, rab_on, bias_on):
    H = 3
    T, jag = batch(H, dh)
    d = H * dh
    gen = torch.Generator().manual_seed(dh)
    rnd = lambda *s: torch.randn(*s, generator=gen).cuda()
    h = (2 * rnd(T, 4 * d)).bfloat16()
    bias = rnd(4 * d) if bias_on else None
    a = torch.empty_like(h)
    hstu.mtgr_bias_silu_fwd(T, 4 * d, hstu.MTGR_DTYPE_BF16, h, 4 * d, bias, a, 4 * d)
    q, k, v = (a[:, i * d:(i + 1) * d].view(T, H, dh) for i in range(3))
    do, rab = rnd(T, H, dh).bfloat16(), 0.1 * rnd(H, 16) if rab_on else None
    ws = ops.workspace_for(ops.attn_problem(jag, q, k, v, do, rab), "cuda", backward=stored)

    def grads(act):
        da = torch.zeros_like(h)
        g = tuple(da[:, i * d:(i + 1) * d].view(T, H, dh) for i in range(3)) + (
            None if rab is None else torch.empty_like(rab),)
        ops.attn_bwd(q, k, v, do, jag, rab, grads=g, workspace=ws, act=act)
        return da, g[3]

    want, want_drab = grads(None)
    hstu.mtgr_bias_silu_bwd(T, 4 * d, hstu.MTGR_DTYPE_BF16, h, 4 * d, bias, want, 4 * d, want, 4 * d)
    got, drab = grads((h[:, :3 * d], None if bias is None else bias[:3 * d]))
    torch.cuda.synchronize()
    assert torch.equal(got[:, :3 * d], want[:, :3 * d]) and not got[:, 3 * d:].any()
    # (drab is of the bias in both; float atomics: 1e-5 of its size, as in test_gpu_rab_buckets.py)
    if rab is not None:
        assert float((drab - want_drab).abs().max()) <= 1e-5 * float(want_drab.abs().max()) and want_drab.any()


@pytest.mark.parametrize("heads,dh", [(2, 16), (2, 32), (1, 128)])
def test_layer(heads, dh):
    T, jag = batch(heads, dh)
    d = heads * dh
    P = to_dev(params_for(d))
    gen = torch.Generator().manual_seed(1)
    x, dxo = (torch.randn(T, d, generator=gen).bfloat16().cuda() for _ in range(2))
    ctx = layer.layer_fwd(x, jag, P, heads)[1]
    keep = {}
    two = layer.layer_bwd(dxo, ctx, jag, P, heads, keep=keep)       # da kept: the pointwise kernel
    one = layer.layer_bwd(dxo, ctx, jag, P, heads)
    torch.cuda.synchronize()
    assert torch.equal(one["w_in"], two["w_in"]) and torch.equal(one["b_in"], two["b_in"])


def test_refused():
    T, jag = batch(2, 32)
    q = torch.zeros(T, 2, 32, device="cuda", dtype=torch.bfloat16)
    h, b = torch.zeros(T, 192, device="cuda", dtype=torch.bfloat16), torch.zeros(192, device="cuda")
    for act in ((h[:, :64], b), (h.float(), b), (h, b[:64]), (h, b.double())):
        with pytest.raises(ValueError):
            ops.attn_bwd(q, q, q, q, jag, act=act)
    with pytest.raises(hstu.MtgrError):      # the vector kernels have no such epilogue
        ops.attn_bwd(q.float(), q.float(), q.float(), q.float(), jag, act=(h.float(), b))
