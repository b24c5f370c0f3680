"""The bf16 product in 128- and 64-wide workgroup tiles: edges of the tiles,
remainders, K splits and both load pipelines, against the oracle and against
the 256-wide tiles bit for bit."""
import numpy as np
import pytest
import torch

from oracle import partir_oracle as O
from paper_2401_11202_amd import inputs as I
from paper_2401_11202_amd import partir as P
from tests.gpu_common import accum_bound, host, say

pytestmark = pytest.mark.gpu


def product(A, B, layout, out=torch.float32, **kw):
    Bd = (B if layout == "kn" else I.transposed(B)).to_device()
    C = P.loop_matmul(A.to_device(), Bd, b_layout=layout, out_dtype=out, **kw)
    torch.cuda.synchronize()
    return C


# (M, N, K, words of the plan): one element, one past and one short of a tile,
# several tiles, K shorter than the LDS pipeline, one and many workgroups a CU
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("M,N,K,words", [
    (1, 8, 8, "tiles of 64 x 64"),
    (63, 56, 72, "tiles of 64 x 64"),
    (65, 72, 136, "tiles of 64 x 64"),
    (192, 264, 448, "tiles of 64 x 64"),
    (130, 4104, 200, "tiles of 64 x 64"),
    (1000, 2200, 328, "tiles of 128 x 128"),         # one workgroup a CU: the four-stage pipeline
    (2100, 2312, 264, "tiles of 128 x 128"),         # 323 workgroups: the two-stage pipeline
    (300, 520, 4104, "as 4 K parts of 17 K tiles"),  # the last part ends inside a K tile
    (200, 2056, 8200, "K parts"),
])
def test_ragged_products(M, N, K, words, layout):
    A = I.gaussian(201, 0, (M, K), 1.0, "bf16")
    B = I.gaussian(201, 1, (K, N), K ** -0.5, "bf16")
    text = P.plan_loop_matmul(M, N, K, b_layout=P.B_KN if layout == "kn" else P.B_NK)["text"]
    assert words in text, text
    ref, norm = O.matmul(A.f64(), B.f64()), O.abs_product(A.f64(), B.f64())
    for out in (torch.float32, torch.bfloat16):
        say(f"bf16 tile {M}x{N}x{K} {layout} out={out}")
        err = O.normalised_error(host(product(A, B, layout, out)), ref, norm)
        assert err <= accum_bound(K) + (2.0 ** -8 if out == torch.bfloat16 else 0.0)


@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("rows", [60, 200, 900, 1700])
def test_small_tiles_give_the_bits_of_the_large_ones(rows, layout):
    """Without a K split every tile size forms an output's sum in the same
    order: the first rows of a product computed alone (64- or 128-wide tiles)
    are the rows of the whole product (256-wide tiles)."""
    M, N, K = 8192, 2048, 448
    A = I.gaussian(202, 0, (M, K), 1.0, "bf16")
    B = I.gaussian(202, 1, (K, N), K ** -0.5, "bf16")
    lay = P.B_KN if layout == "kn" else P.B_NK
    assert "workgroup tiles" not in P.plan_loop_matmul(M, N, K, b_layout=lay)["text"]
    text = P.plan_loop_matmul(rows, N, K, b_layout=lay)["text"]
    assert "workgroup tiles" in text and "K parts" not in text, text
    Ad = A.to_device()
    Bd = (B if layout == "kn" else I.transposed(B)).to_device()
    whole = P.loop_matmul(Ad, Bd, b_layout=layout, out_dtype=torch.float32)
    part = P.loop_matmul(Ad[:rows], Bd, b_layout=layout, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(part, whole[:rows])


def test_shards_of_a_tile_loop_may_end_inside_a_tile():
    """#tile shards of 50 rows / 88 columns share 64-wide tiles: the result is
    the unpartitioned one bit for bit and nothing outside [M, N] is written."""
    M, N, K = 200, 352, 200
    A = I.gaussian(203, 0, (M, K), 1.0, "bf16")
    B = I.gaussian(203, 1, (K, N), K ** -0.5, "bf16")
    plain = product(A, B, "kn")
    for tile in ("M", "N"):
        big = torch.full((M + 8, N + 16), 7.25, dtype=torch.float32, device="cuda")
        P.loop_matmul(A.to_device(), B.to_device(), tile=tile, R=4, b_layout="kn", out_dtype=torch.float32,
                      out=big[:M, :N])
        torch.cuda.synchronize()
        assert torch.equal(big[:M, :N], plain)
        assert torch.all(big[M:] == 7.25) and torch.all(big[:, N:] == 7.25)


def test_k_parts_equal_their_ordered_sum():
    """Integer inputs: the K parts and their sum are exact."""
    M, N, K = 300, 520, 4104
    A = I.small_ints(204, 0, (M, K), dtype="bf16")
    B = I.small_ints(204, 1, (K, N), dtype="bf16")
    assert "K parts" in P.plan_loop_matmul(M, N, K)["text"]
    for layout in ("kn", "nk"):
        assert np.array_equal(host(product(A, B, layout)), O.matmul(A.f64(), B.f64()))


@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("rows,R", [(304, 3), (200, 9), (1000, 3)])
def test_a_fused_sum_is_one_accumulator(rows, R, layout):
    """Short grids, where the planner would cut K: a fused #sum has the bits of
    the unsplit 256-wide tiles."""
    M, N, K = 8192, 2048, 4104
    A = I.gaussian(205, 0, (M, K), 1.0, "bf16")
    B = I.gaussian(205, 1, (K, N), K ** -0.5, "bf16")
    lay = P.B_KN if layout == "kn" else P.B_NK
    whole_text = P.plan_loop_matmul(M, N, K, b_layout=lay)["text"]
    assert "workgroup tiles" not in whole_text and "K parts" not in whole_text
    plan = P.plan_loop_matmul(rows, 512, K, b_layout=lay, sum="K", R=R, sum_impl=P.SUM_FUSED)
    assert plan["n_launches"] == 1 and plan["n_sum_splitk"] == 0
    Ad = A.to_device()
    Bd = (B if layout == "kn" else I.transposed(B)).to_device()
    few = Bd[:, :512] if layout == "kn" else Bd[:512]
    say(f"bf16 fused #sum {rows}x512x{K} R={R} {layout}")
    whole = P.loop_matmul(Ad, Bd, b_layout=layout, out_dtype=torch.float32)
    part = P.loop_matmul(Ad[:rows], few, sum="K", R=R, sum_impl="fused", b_layout=layout, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(part, whole[:rows, :512])


# the weight gradients: both operands stored [K, .], K = T ending inside a K
# tile, ragged in both directions; words of both products' plans
@pytest.mark.parametrize("T,D,F,words", [
    (136, 136, 200, "grid 12 WGs; read in place: A as [K, M] B as [K, N]; workgroup tiles of 64 x 64"),
    (136, 2312, 392, "grid 259 WGs; read in place: A as [K, M] B as [K, N]; workgroup tiles of 64 x 64"),
    (2056, 136, 392, "21 tiles as 4 K parts of 9 K tiles each; workgroup tiles of 64 x 64"),
    (136, 1032, 2312, "grid 171 WGs; read in place: A as [K, M] B as [K, N]; workgroup tiles of 128 x 128"),
    (136, 1544, 3080, "grid 325 WGs; read in place: A as [K, M] B as [K, N]; workgroup tiles of 128 x 128"),
    (4104, 136, 3080, "50 tiles as 4 K parts of 17 K tiles each; workgroup tiles of 128 x 128"),
])
def test_operands_stored_k_m(T, D, F, words):
    """Entries in {-1, 0, 1} and the identity activation: Z and dH are integers
    that bf16 holds, so the gradients are exact."""
    X, W1 = I.small_ints(206, 0, (T, D), -1, 1), I.small_ints(206, 1, (D, F), -1, 1)
    W2, dY = I.small_ints(206, 2, (F, D), -1, 1), I.small_ints(206, 3, (T, D), -1, 1)
    Z, dH = X.f64() @ W1.f64(), dY.f64() @ W2.f64().T
    assert max(np.abs(Z).max(), np.abs(dH).max()) <= 256
    say(f"A [K, M], B [K, N]: T={T} D={D} F={F}")
    _, dW1, dW2 = P.mlp_block_backward(*(t.to_device() for t in (X, W1, W2, dY)), act="none")
    torch.cuda.synchronize()
    text = P.lib().partir_last_plan_text().decode()
    for name in ("bwd.dw1", "bwd.dw2"):
        line = next(l for l in text.splitlines() if name in l)
        assert words in line, line
    assert np.array_equal(host(dW1), X.f64().T @ dH) and np.array_equal(host(dW2), Z.T @ dY.f64())
