"""The 256 x 256 tiles of the large dense products where they can go wrong: ragged rows, columns
and k steps of 64, one to four k steps (the copies' prologue), more tiles than the chip has CUs (a
workgroup's second tile starts under the first one's epilogue), and K splits that end in a ragged
step.  Same references and bounds as test_gpu_gemm.py."""
import numpy as np
import pytest
import torch

from paper_2505_18654_amd import ops
from tests.dense_ref import bf16_half_ulp
from tests.test_gpu_gemm import U, assert_within, f64, product_ref, rand_bf16, splits_of
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


# (bias + SiLU takes these tiles at every size with K <= 512, and up to K = 768 from 128 of the narrow ones on)
@pytest.mark.parametrize("M, N, K", [(1, 8, 32), (257, 264, 64), (256, 256, 96), (300, 520, 128), (255, 248, 160),
                                     (513, 256, 192), (700, 1000, 512), (700, 1000, 736), (4100, 1000, 736),
                                     (256 * 23 + 5, 256 * 12 + 8, 224)])
def test_bias_silu(M, N, K):
    say(f"[gemm wide] bias+silu M={M} N={N} K={K}")
    A, B = rand_bf16((M, K), 5, cols=K + 8), rand_bf16((K, N), 6, scale=K ** -0.5 * 2)
    bias = torch.randn(N, generator=torch.Generator().manual_seed(7)).cuda() * 0.5
    h = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    full = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    a = full[:M, :N]
    ops.gemm(A, B, "nn", out=h, bias=bias, silu_out=a)
    torch.cuda.synchronize()
    ref, S = product_ref("nn", A, B)
    g = (K + 5) * U
    got_h, got_a = f64(h), f64(a)
    assert_within("pre-activation", got_h, ref, bf16_half_ulp(got_h) + g * S + 1e-30)
    z = ref + f64(bias[None, :])
    silu = z / (1.0 + np.exp(-z))
    bound = bf16_half_ulp(got_a) + 1.1 * (g * S + 2 * U * np.abs(z)) + 16 * U * (np.abs(z) + 1) * np.abs(silu)
    assert_within("silu", got_a, silu, bound + 1e-30)
    assert bool((full[M:] == 7.0).all()) and bool((full[:, N:] == 7.0).all())


# (the last three are on these tiles, one of them with two tiles per workgroup, the first two on the narrow ones)
@pytest.mark.parametrize("M, N, K", [(256 * 32 - 3, 256 * 8 - 8, 96), (256 * 33 + 1, 256 * 16, 64),
                                     (256 * 32 - 3, 256 * 8 - 8, 448), (256 * 32 - 3, 256 * 8 - 8, 800),
                                     (256 * 64 - 3, 256 * 8, 448)])
@pytest.mark.parametrize("layout", ["nn", "nt"])
def test_plain(layout, M, N, K):
    say(f"[gemm wide] {layout} M={M} N={N} K={K}")
    A = rand_bf16((M, K), 1)
    B = rand_bf16((K, N) if layout == "nn" else (N, K), 2)
    C = ops.gemm(A, B, layout)
    torch.cuda.synchronize()
    ref, S = product_ref(layout, A, B)
    got = f64(C)
    assert_within(layout, got, ref, bf16_half_ulp(got) + (K + 5) * U * S + 1e-30)


def test_bias_residual_in_place():
    M, N, K = 256 * 32 - 9, 256 * 8 - 8, 160
    A, B = rand_bf16((M, K), 8), rand_bf16((K, N), 9, scale=K ** -0.5)
    R = rand_bf16((M, N), 10)
    bias = torch.randn(N, generator=torch.Generator().manual_seed(11)).cuda() * 0.1
    ref, S = product_ref("nn", A, B)
    br = f64(bias[None, :]) + f64(R)
    C = ops.gemm(A, B, "nn", out=R, bias=bias, residual=R)
    torch.cuda.synchronize()
    got, want = f64(C), ref + br
    bound = bf16_half_ulp(got) + (K + 5) * U * S + 2 * U * (np.abs(br) + np.abs(want))
    assert_within("bias+residual", got, want, bound + 1e-30)


# 64 and 66 tiles in splits of 8 to 12 k steps (one split ends 58, 1 or 0 k short of a whole step)
@pytest.mark.parametrize("M, N, K", [(1024, 4096, 1030), (1024, 4096, 1535), (776, 4104, 1152)])
def test_weight_gradient(M, N, K):
    say(f"[gemm wide] tn M={M} N={N} K={K}")
    A, B = rand_bf16((K, M), 1), rand_bf16((K, N), 2)
    cs = torch.full((N,), float("nan"), device="cuda")
    C = ops.gemm(A, B, "tn", colsum=cs)
    torch.cuda.synchronize()
    ref, S = product_ref("tn", A, B)
    got = f64(C)
    g = (K + splits_of(2, M, N, K) + 4) * U
    assert_within("tn", got, ref, bf16_half_ulp(got) + g * S + 1e-30)
    b = f64(B)
    assert_within("colsum", cs.cpu().numpy().astype(np.float64), b.sum(0), g * np.abs(b).sum(0) + 1e-30)
