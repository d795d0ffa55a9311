"""The vector-ALU kernels around their steps of four keys and tiles of 64: user lengths on both sides
of them, fp32 against the oracle (relative to the RMS, 1e-4 as in test_gpu_parity.py), and infinite
values in rows that the mask hides from everyone else (0 contribution, not 0 times infinity)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_18654_amd import ops
from synth import make_values
from tests.gpu_util import TOL, custom_layout, jagged, make_inputs, per_user_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rab", [0, 64])
@pytest.mark.parametrize("dh", [16, 32, 64, 128])
def test_lengths(dh, rab):
    rng = np.random.default_rng(dh)
    lens = [1, 3, 4, 5, 63, 64, 65, 67, 130]
    segs = [np.sort(rng.integers(0, 4, n)) for n in lens]
    L = custom_layout(segs, [rng.integers(0, 50, n) for n in lens], heads=2, head_dim=dh, dtype="fp32", rab_buckets=rab)
    inp, vals = make_inputs(L, all_exact=True), make_values(L)
    jag, rb = jagged(inp), inp["rab"]
    q, k, v, do = (inp[n] for n in ("q", "k", "v", "do"))
    o = ops.attn_fwd(q, k, v, jag, rb)
    got = (o, *ops.attn_bwd(q, k, v, do, jag, rb)[:3])
    torch.cuda.synchronize()
    args = (L.offsets, L.seg, L.ts, vals["q"], vals["k"], vals["v"])
    want = (oracle.attn_fwd(*args, inp["rab_np"]), *oracle.attn_bwd(*args, vals["do"], inp["rab_np"])[:3])
    for name, g, w in zip(("o", "dq", "dk", "dv"), got, want):
        e = per_user_err(L, list(range(len(lens))), to_np(g), w, "fp32", TOL["fp32"])
        assert e["checked"] <= TOL["fp32"], (name, e)


def test_hidden_infinities():
    L = custom_layout([[1] * 70 + [3] * 5], [[0] * 75], heads=1, head_dim=16, dtype="fp32")
    inp = make_inputs(L, all_exact=True)
    jag = jagged(inp)
    q, k, v, do = (inp[n] for n in ("q", "k", "v", "do"))
    clean = ops.attn_fwd(q, k, v, jag), *ops.attn_bwd(q, k, v, do, jag)[:3]
    v2, do2 = v.clone(), do.clone()
    v2[72], do2[73] = float("inf"), float("inf")       # candidates: seen by themselves only
    o = ops.attn_fwd(q, k, v2, jag)
    dq = ops.attn_bwd(q, k, v2, do, jag)[0]
    dk, dv = ops.attn_bwd(q, k, v, do2, jag)[1:3]
    rest = [i for i in range(75) if i not in (72, 73)]
    cand = [i for i in range(70, 75) if i != 73]      # (a candidate's dO reaches the static keys)
    assert torch.equal(o[rest], clean[0][rest]) and torch.equal(dq[rest], clean[1][rest])
    assert torch.equal(dk[cand], clean[2][cand]) and torch.equal(dv[cand], clean[3][cand])
