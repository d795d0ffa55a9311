"""The relative bias at the edges of its buckets: time gaps one below, at and one above every
2^e and 1.5 2^e up to 2^32 - 1 (from 2^24 on the gap does not fit a float), tables of 1, 2, 3, 9,
32 and 64 buckets, on the matrix-core kernels and both backward forms, against the oracle.  Bias values of
order 1 make a wrong bucket an error of order 1 in its rows.

Bound: the operands P and dS and the results are each rounded to bf16 (relative error at most 2^-9
each).  The errors of the many terms are independent, so in the 2-norm an output is off by at most
about sqrt(2) 2^-9 = 2.8e-3 of its size, times the cancellation of its sums (the 2-norm of the terms
over that of the sum, below 3 for values of either sign); 1e-2 is asked for.  drab is summed in fp32
from unrounded dS: 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_18654_amd import ops
from synth import make_values
from synth.torch_inputs import device_inputs
from tests.gpu_util import custom_layout, jagged, say, to_np

pytestmark = pytest.mark.gpu


def gaps():
    g = {0, 1, 2 ** 32 - 1}
    for e in range(1, 32):
        for m in (1 << e, 3 << (e - 1)):
            g |= {m - 1, m, m + 1}
    return np.array(sorted(x for x in g if x < 2 ** 32), np.int64)


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("buckets", [1, 2, 3, 9, 32, 64])
def test_bucket_edges(buckets, dh):
    ts = np.concatenate([[-2 ** 31], -2 ** 31 + gaps()]).astype(np.int32)
    segs = [np.ones(len(ts), np.int8), np.concatenate([np.ones(5, np.int8), np.full(len(ts) - 5, 2, np.int8)])]
    L = custom_layout(segs, [ts, ts], heads=2, head_dim=dh, rab_buckets=buckets)
    inp = device_inputs(L, "cuda", all_exact=True)
    rab = np.random.default_rng(buckets).standard_normal((2, buckets)).astype(np.float32)
    rab_d = torch.from_numpy(rab).cuda()
    vals = make_values(L)
    jag = jagged(inp)
    q, k, v, do = (inp[n] for n in ("q", "k", "v", "do"))
    o = ops.attn_fwd(q, k, v, jag, rab_d)
    want_o = oracle.attn_fwd(L.offsets, L.seg, L.ts, vals["q"], vals["k"], vals["v"], rab)
    want = oracle.attn_bwd(L.offsets, L.seg, L.ts, vals["q"], vals["k"], vals["v"], vals["do"], rab)
    rel = lambda g, w: float(np.linalg.norm(to_np(g).reshape(-1) - w.reshape(-1)) / np.linalg.norm(w))
    for form in ("stored", "recomputed"):
        ws = ops.workspace_for(ops.attn_problem(jag, q, k, v, o, rab_d), "cuda", form == "stored")
        got = ops.attn_bwd(q, k, v, do, jag, rab_d, workspace=ws)
        torch.cuda.synchronize()
        errs = {"o": rel(o, want_o), **{n: rel(g, w) for n, g, w in zip(("dq", "dk", "dv", "drab"), got, want)}}
        say(f"[rab edges] {buckets} buckets dh {dh} {form}: " + " ".join(f"{n}={e:.1e}" for n, e in errs.items()))
        for n, e in errs.items():
            assert e <= (1e-5 if n == "drab" else 1e-2), (n, e)
