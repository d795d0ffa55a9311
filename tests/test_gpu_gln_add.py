"""Group-LN backward that adds a residual's gradient to dx in the same pass: against the oracle, at
widths on both sides of a full row of chunks and of each register plan, with a strided or an in-place
residual; and the layer's one-pass dX against its two-pass form (GPU)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_18654_amd import hstu, layer, ops
from tests.gpu_util import TOL, bf16_half_ulp, custom_layout, rel_err, tensor_err
from tests.test_gpu_layer import params_for, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype", [(8, torch.bfloat16), (256, torch.bfloat16), (520, torch.bfloat16),
                                     (1024, torch.bfloat16), (2048, torch.bfloat16), (4096, torch.bfloat16),
                                     (4, torch.float32), (516, torch.float32), (2048, torch.float32)])
@pytest.mark.parametrize("T,form", [(1, "dense"), (331, "strided"), (331, "in place")])
def test_residual(d, dtype, T, form):
    gen = torch.Generator().manual_seed(d + T)
    rnd = lambda *s: torch.randn(*s, generator=gen).to(dtype).cuda()
    x, dy = rnd(T, d), rnd(T, d)
    res = rnd(T, 2 * d)[:, d:] if form == "strided" else rnd(T, d)
    gid = (torch.arange(T) // 7 % 3).to(torch.int8).cuda()
    gamma, beta = torch.randn(3, d, generator=gen).cuda(), torch.zeros(3, d).cuda()
    _, mean, rstd = ops.gln_fwd(x, None, gid, gamma, beta)
    f = lambda t: t.float().cpu().numpy()
    rdx, _, rdg, rdb = oracle.gln_bwd(f(x), None, gid.cpu().numpy(), f(gamma), f(dy))
    want = rdx + f(res)
    grads = (res, None, torch.empty_like(gamma), torch.empty_like(gamma)) if form == "in place" else None
    dx, _, dgamma, dbeta = ops.gln_bwd(dy, x, None, gid, gamma, mean, rstd, grads=grads, residual=res)
    torch.cuda.synchronize()
    key = "bf16" if dtype == torch.bfloat16 else "fp32"
    assert tensor_err(f(dx), want, key, TOL[key])["checked"] <= TOL[key]
    assert rel_err(f(dgamma), rdg) <= TOL[key] and rel_err(f(dbeta), rdb) <= TOL[key]


def test_refused():
    x = torch.zeros(4, 8, device="cuda", dtype=torch.bfloat16)
    gid, st = torch.zeros(4, dtype=torch.int8, device="cuda"), torch.zeros(4, device="cuda")
    gamma = torch.ones(1, 8, device="cuda")
    for res, u in ((x[:, :4], None), (x.float(), None), (x, x)):
        with pytest.raises(ValueError):
            ops.gln_bwd(x, x, u, gid, gamma, st, st, residual=res)
    with pytest.raises(hstu.MtgrError):
        p = hstu.gln_problem(4, 8, 1, hstu.MTGR_DTYPE_BF16)
        hstu.mtgr_group_layernorm_bwd_add(p, x, x, None, gid, gamma, st, st, x, gamma, gamma, x, 1 << 20)


def test_layer_one_pass():
    rng = np.random.default_rng(5)
    segs = [np.sort(rng.integers(0, 4, n)) for n in (1, 70, 200)]
    L = custom_layout(segs, [rng.integers(0, 50, len(s)) for s in segs], heads=2, head_dim=32)
    T, d = L.total_tokens, 64
    jag, P = ops.Jagged.from_host(L.offsets, L.seg, L.ts), to_dev(params_for(d))
    wide = torch.randn(T, 2 * d, generator=torch.Generator().manual_seed(1)).bfloat16().cuda()
    dxo = torch.randn(T, d, generator=torch.Generator().manual_seed(2)).bfloat16().cuda()
    x = wide[:, :d].contiguous()
    keep = {}
    two = layer.layer_bwd(dxo, layer.layer_fwd(x, jag, P, 2)[1], jag, P, 2, keep=keep)["x"]
    one = layer.layer_bwd(dxo, layer.layer_fwd(x, jag, P, 2)[1], jag, P, 2)["x"]
    view = layer.layer_bwd(dxo, layer.layer_fwd(wide[:, :d], jag, P, 2)[1], jag, P, 2)["x"]
    torch.cuda.synchronize()
    # two roundings of the two-pass form (dX_gln, then the sum) and one of this one
    f = lambda t: t.double().cpu().numpy()
    bound = bf16_half_ulp(f(keep["dx_gln"])) + bf16_half_ulp(f(two)) + bf16_half_ulp(f(one))
    assert (np.abs(f(one) - f(two)) <= bound * (1 + 2.0 ** -10)).all()
    assert torch.equal(view, two) and view.is_contiguous() and one.is_contiguous()
