"""The fp32 product in 64- and 128-wide tiles, and with leading dimensions
beyond the tiles' 32-bit byte ranges, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import partir_oracle as O
from paper_2401_11202_amd import inputs as I
from paper_2401_11202_amd import partir as P
from tests.gpu_common import accum_bound, host, say

pytestmark = pytest.mark.gpu


# one element, edges of both tiles and of the 32-wide K tile, K shorter than
# the LDS pipeline, one and several workgroups a CU
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("M,N,K,tile", [(1, 4, 4, 64), (63, 68, 36, 64), (65, 132, 100, 64), (200, 520, 132, 64),
                                        (1800, 2056, 68, 128), (1793, 2052, 264, 128)])
def test_ragged_products(M, N, K, tile, layout):
    A = I.gaussian(211, 0, (M, K), 1.0, "f32")
    B = I.gaussian(211, 1, (K, N), K ** -0.5, "f32")
    text = P.plan_loop_matmul(M, N, K, ab=P.F32, b_layout=P.B_KN if layout == "kn" else P.B_NK)["text"]
    assert f"workgroup tiles of {tile}" in text, text
    say(f"f32 tile {M}x{N}x{K} {layout}")
    big = torch.full((M + 4, N + 8), 7.25, dtype=torch.float32, device="cuda")
    Bd = (B if layout == "kn" else I.transposed(B)).to_device()
    P.loop_matmul(A.to_device(), Bd, b_layout=layout, out=big[:M, :N])
    torch.cuda.synchronize()
    ref, norm = O.matmul(A.f64(), B.f64()), O.abs_product(A.f64(), B.f64())
    assert O.normalised_error(host(big[:M, :N]), ref, norm) <= accum_bound(K)
    assert torch.all(big[M:] == 7.25) and torch.all(big[:, N:] == 7.25)


# a short K on many workgroups: one K step of 16, parts of one, the longest and
# one past it, with and without a #sum
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("M,N,K,R", [(1299, 2004, 4, 1), (1299, 2004, 112, 1), (1299, 2004, 116, 1), (899, 732, 96, 8),
                                     (2173, 408, 384, 8)])
def test_short_contractions(M, N, K, R, layout):
    A = I.gaussian(213, 0, (M, K), 1.0, "f32")
    B = I.gaussian(213, 1, (K, N), K ** -0.5, "f32")
    summ = "K" if R > 1 else None
    text = P.plan_loop_matmul(M, N, K, ab=P.F32, b_layout=P.B_KN if layout == "kn" else P.B_NK, sum=summ, R=R)["text"]
    assert ("register-staged" in text) == (K // R <= 112), text
    say(f"f32 short K {M}x{N}x{K} R={R} {layout}")
    big = torch.full((M + 4, N + 8), 7.25, dtype=torch.float32, device="cuda")
    Bd = (B if layout == "kn" else I.transposed(B)).to_device()
    P.loop_matmul(A.to_device(), Bd, sum=summ, R=R, b_layout=layout, out=big[:M, :N])
    torch.cuda.synchronize()
    ref, norm = O.matmul(A.f64(), B.f64()), O.abs_product(A.f64(), B.f64())
    assert O.normalised_error(host(big[:M, :N]), ref, norm) <= accum_bound(K)
    assert torch.all(big[M:] == 7.25) and torch.all(big[:, N:] == 7.25)


@pytest.mark.parametrize("summ,R,impl", [(None, 1, "auto"), ("K", 5, "splitk"), ("K", 5, "fused")])
def test_rows_further_apart_than_a_byte_range_holds(summ, R, impl):
    """lda = 2^24 + 4: views whose rows lie 64 MiB apart."""
    M, N, K, ld = 5, 8, 140, (1 << 24) + 4
    A = I.small_ints(212, 0, (M, K), dtype="f32")
    B = I.small_ints(212, 1, (K, N), dtype="f32")
    wide = torch.zeros(M * ld, dtype=torch.float32, device="cuda").view(M, ld)
    wide[:, :K] = A.to_device()
    C = P.loop_matmul(wide[:, :K], B.to_device(), sum=summ, R=R, sum_impl=impl)
    torch.cuda.synchronize()
    assert np.array_equal(host(C), O.matmul(A.f64(), B.f64()))
