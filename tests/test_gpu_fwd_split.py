"""Forward with the keys split over two wave groups (few work items) against the oracle, and against
the unsplit forward of the same users in a batch with many more: 1 to 5 visible key tiles (odd
counts end with a hidden tile), RT keys that leave tiles fully masked, candidates only, cached keys
of 0 to 4 tiles.  The bar of test_gpu_parity.py; the two forwards differ in the order of fp32
sums only, so their bf16 results differ by at most one rounding of a value (2^-8 of it) in few."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_18654_amd import ops
from synth import make_values
from tests.gpu_util import TOL, custom_layout, jagged, make_inputs, per_user_err, say, to_np

pytestmark = pytest.mark.gpu
U, S, R, C = 0, 1, 2, 3


def users(rng):
    segs, tss = [], []
    for n_s, n_r, n_c in ((1, 0, 0), (64, 0, 0), (65, 0, 3), (128, 10, 70), (190, 70, 130), (250, 40, 5), (0, 0, 90),
                          (0, 200, 60), (300, 0, 0)):
        segs.append([S] * n_s + [R] * n_r + [C] * n_c)
        tss.append(sorted(rng.integers(-1000, 0, n_s).tolist()) + sorted(rng.integers(0, 5000, n_r).tolist())
                   + rng.integers(0, 5000, n_c).tolist())
    return segs, tss


@pytest.mark.parametrize("dh,rab", [(32, 0), (64, 64), (128, 0), (128, 64)])
def test_split_forward(dh, rab):
    segs, tss = users(np.random.default_rng(dh + rab))
    few = custom_layout(segs, tss, heads=2, head_dim=dh, rab_buckets=rab)
    many = custom_layout(segs + [[S] * 30] * 250, tss + [[0] * 30] * 250, heads=2, head_dim=dh, rab_buckets=rab)
    sel = list(range(len(segs)))
    T = few.total_tokens
    vals = make_values(few, tensors=("q", "k", "v"))
    outs = {}
    for name, L in (("few", few), ("many", many)):
        inp = make_inputs(L, all_exact=True)
        outs[name] = ops.attn_fwd(inp["q"], inp["k"], inp["v"], jagged(inp), inp["rab"])[:T]
        if name == "few":
            cand = ops.attn_fwd(inp["q"], inp["k"], inp["v"], jagged(inp), inp["rab"], out=torch.zeros_like(inp["q"]),
                                cand_rows=True)
            is_c = torch.from_numpy(L.seg == C).cuda()
            want = oracle.attn_fwd(L.offsets, L.seg, L.ts, vals["q"], vals["k"], vals["v"], inp["rab_np"])
    torch.cuda.synchronize()
    assert torch.equal(cand[is_c], outs["few"][is_c]) and not cand[~is_c].any()
    e = per_user_err(few, sel, to_np(outs["few"]), want, "bf16", TOL["bf16"])
    say(f"[split] dh {dh} rab {rab} vs oracle: checked {e['checked']:.2e}")
    assert e["checked"] <= TOL["bf16"]
    a, b = to_np(outs["few"]), to_np(outs["many"])
    off = np.abs(a - b) > 2.0 ** -7 * np.maximum(np.abs(a), np.abs(b)) + 1e-6 * np.sqrt(np.mean(b ** 2))
    say(f"[split] dh {dh} rab {rab} vs unsplit: {np.mean(a != b):.1e} differ, {int(off.sum())} by more than a rounding")
    assert not off.any() and np.mean(a != b) < 0.02


@pytest.mark.parametrize("dh,rab", [(32, 0), (64, 0), (128, 0), (128, 64)])
@pytest.mark.parametrize("heads,lens,last", [(2, [(64, 0), (128, 0), (192, 0), (320, 0)], [40, 100, 150, 300]),
                                             (1, [(192, 64 * 62)], [150])])
def test_split_infinite_values(dh, rab, heads, lens, last):
    """An infinity in V of the last visible tile (token `last` of each user): the same infinities and NaNs
    as the unsplit forward, with 1, 2, 3 and 5 fully visible tiles, and with 62 fully masked ones, which
    reach past the tile walker's first window of 64, behind three visible."""
    segs = [[S] * n_s + [C] * n_c for n_s, n_c in lens]
    rng = np.random.default_rng(dh)
    tss = [sorted(rng.integers(-1000, 0, len(s)).tolist()) for s in segs]
    few = custom_layout(segs, tss, heads=heads, head_dim=dh, rab_buckets=rab)
    many = custom_layout(segs + [[S] * 30] * 250, tss + [[0] * 30] * 250, heads=heads, head_dim=dh, rab_buckets=rab)
    T = few.total_tokens
    at = torch.from_numpy(few.offsets[:-1].astype(np.int64) + np.array(last)).cuda()
    outs = []
    for L in (few, many):
        inp = make_inputs(L, all_exact=True)
        v = inp["v"].clone()
        v[at, 0, 1], v[at, heads - 1, dh - 1] = float("inf"), float("-inf")
        outs.append(ops.attn_fwd(inp["q"], inp["k"], v, jagged(inp), inp["rab"])[:T].float())
    torch.cuda.synchronize()
    split, whole = outs
    inf, fin = torch.isinf(whole), torch.isfinite(whole)
    say(f"[split] infinite V dh {dh} rab {rab}: {int(inf.sum())} infinities, {int(torch.isnan(whole).sum())} NaN")
    assert int(inf.sum()) > T // 2
    assert torch.equal(torch.isnan(split), torch.isnan(whole)) and torch.equal(torch.isinf(split), inf)
    assert torch.equal(split[inf], whole[inf])
    a, b = to_np(split[fin]), to_np(whole[fin])
    off = np.abs(a - b) > 2.0 ** -7 * np.maximum(np.abs(a), np.abs(b)) + 1e-6 * np.sqrt(np.mean(b ** 2))
    assert not off.any()


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("cached", [[0, 1, 64, 65], [128, 150, 200, 256]])
def test_split_cached(dh, cached):
    rng = np.random.default_rng(dh)
    segs = [[S] * n + [C] * (40 + 50 * i) for i, n in enumerate(cached)]
    tss = [[0] * n + rng.integers(0, 99, 40 + 50 * i).tolist() for i, n in enumerate(cached)]
    L = custom_layout(segs, tss, heads=2, head_dim=dh)
    inp = make_inputs(L, all_exact=True)
    c = torch.from_numpy(L.seg == C).cuda()
    side = ops.Jagged.from_host(np.concatenate([[0], np.cumsum(cached)]), L.seg[L.seg != C], L.ts[L.seg != C])
    cl = np.array([40 + 50 * i for i in range(len(cached))])
    req = ops.Jagged.from_host(np.concatenate([[0], np.cumsum(cl)]), L.seg[L.seg == C], L.ts[L.seg == C])
    q, k, v = inp["q"], inp["k"], inp["v"]
    got = ops.attn_fwd_cached(q[c], k[c], v[c], req, ops.user_cache(k[~c], v[~c], side))
    full = ops.attn_fwd(q, k, v, jagged(inp))[c]
    torch.cuda.synchronize()
    a, b = to_np(got), to_np(full)
    off = np.abs(a - b) > 2.0 ** -7 * np.maximum(np.abs(a), np.abs(b)) + 1e-6 * np.sqrt(np.mean(b ** 2))
    say(f"[split] cached {cached} dh {dh}: {np.mean(a != b):.1e} differ, {int(off.sum())} by more than a rounding")
    assert not off.any()
