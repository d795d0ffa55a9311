"""The embedding table's kernels at the sizes where their split of the work changes: batches on both
sides of the one-ID-per-thread limit, IDs whose positions fill several workgroups of the SGD step,
end on their edge or are the whole batch, and widths with few and many column blocks.  Against
the dict oracle, with its tolerances: gathers of untouched rows exact, an SGD step within one
rounding of the dtype (the fp32 sums of k terms within k 2^-24 of their absolute sum)."""
import numpy as np
import pytest
import torch

from oracle.embedding import DictTable
from paper_2505_18654_amd.embedding import DynamicEmbedding
from tests.gpu_util import bf16_half_ulp, say

pytestmark = pytest.mark.gpu


def to_dev(ids):
    return torch.from_numpy(ids.astype(np.uint64).view(np.int64).copy()).cuda()


@pytest.mark.parametrize("n", [255, 257, 65536, 65537, 262145])
def test_dedup_sizes(n):
    rng = np.random.default_rng(n)
    ids = rng.integers(0, n // 2 + 1, n).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    unique, occ, inverse, num = DynamicEmbedding(16, 8).dedup(to_dev(ids))
    nu = int(num.item())
    u = unique.cpu().numpy().view(np.uint64)[:nu]
    want, counts = np.unique(ids, return_counts=True)
    assert nu == len(want)
    np.testing.assert_array_equal(u[inverse.cpu().numpy()[:n]], ids)
    order = np.argsort(u)
    np.testing.assert_array_equal(u[order], want)
    np.testing.assert_array_equal(occ.cpu().numpy()[:nu][order], counts)


# positions per ID: one workgroup takes 1024 places (512 at cpb = 16 column chunks, 32 at dim 1024 fp32)
@pytest.mark.parametrize("counts", [[1], [1024], [1023, 1, 1024, 1], [5000], [1] * 40 + [3000] + [2] * 700 + [1024]])
@pytest.mark.parametrize("dim,dtype", [(64, torch.bfloat16), (8, torch.bfloat16), (24, torch.float32),
                                       (128, torch.bfloat16), (1024, torch.float32)])
def test_sgd_runs(counts, dim, dtype):
    rng = np.random.default_rng(len(counts) + dim)
    ids = np.repeat(np.arange(1, len(counts) + 1, dtype=np.uint64), counts)
    rng.shuffle(ids)
    t, ref = DynamicEmbedding(4096, dim, dtype=dtype), DictTable(4096, dim)
    lr = 0.125
    for step in range(2):
        out, b = t.lookup(to_dev(ids), now=step)
        u, occ, _ = ref.dedup(ids)
        ref.lookup(u, occ, now=step, insert=True)
        grad = torch.from_numpy(rng.standard_normal((len(ids), dim)).astype(np.float32)).to(dtype)
        g64 = grad.float().numpy().astype(np.float64)
        before = t.gather(b).float().cpu().numpy().astype(np.float64)
        t.sgd(b, grad.cuda(), lr)
        got = t.gather(b).float().cpu().numpy().astype(np.float64)
        sums, mags = np.zeros((len(counts) + 1, dim)), np.zeros((len(counts) + 1, dim))
        np.add.at(sums, ids.astype(np.int64), g64)
        np.add.at(mags, ids.astype(np.int64), np.abs(g64))
        want = before - lr * sums[ids.astype(np.int64)]
        # half an ulp of the stored result (bf16: half the spacing of 8-bit significands)
        half = bf16_half_ulp(got) if dtype == torch.bfloat16 else np.spacing(np.abs(got).astype(np.float32)) / 2
        bound = half + lr * (max(counts) + 2) * 2.0 ** -24 * mags[ids.astype(np.int64)] + 1e-30
        ratio = float((np.abs(got - want) / bound).max())
        say(f"[embedding] runs {len(counts)} ids dim {dim} {dtype} step {step}: max err / bound {ratio:.3f}")
        assert ratio <= 1.0


@pytest.mark.parametrize("cap,old,new", [(1000, 500, 1100), (2000, 1, 300), (60000, 30000, 65536), (150000, 70001, 200000)])
def test_insertion_from_freed_rows_and_the_tail_together(cap, old, new):
    """More new IDs than freed rows, in one and in many workgroups of both widths: the rest comes from the
    never-used rows, then nothing is left.  Every row is handed out once."""
    t = DynamicEmbedding(cap, 8)
    t.lookup(to_dev(np.arange(1, old + 1)), now=1, gather=False)
    assert t.evict(2) == old
    _, b = t.lookup(to_dev(np.arange(old + 1, old + 1 + new)), now=3, gather=False)
    got = min(cap, new)
    rows = b.rows.cpu().numpy()[:int(b.num_unique.item())]
    st = t.stats()
    assert st["num_keys"] == got and st["free_top"] == 0 and st["next_row"] == (cap if new > cap - old else max(old, got))
    assert bool(st["overflow"] & 1) == (new > cap)
    live = np.sort(rows[rows >= 0])
    assert len(live) == got and (np.diff(live) > 0).all() and live[-1] < cap and (rows == -1).sum() == new - got
    counts, seen = t.counts.cpu().numpy(), t.last_ts.cpu().numpy()
    assert (counts[live] == 1).all() and (seen[live] == 3).all()
    again = t.lookup(to_dev(np.arange(old + 1, old + 1 + new)), now=4, insert=False, gather=False)[1]
    # (the unique list has an order of its own in each call: compared by ID)
    by_id = lambda x: x.rows.cpu().numpy()[:new][np.argsort(x.unique.cpu().numpy()[:new])]
    np.testing.assert_array_equal(by_id(again), by_id(b))
