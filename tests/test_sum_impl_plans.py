"""How a #sum over K is realised, as the plan states it (host only)."""
import pytest

from paper_2401_11202_amd import partir as P


@pytest.mark.parametrize("ab", [P.BF16, P.F32])
@pytest.mark.parametrize("M,N,K,R", [
    (256, 256, 65536, 8),     # one 256-wide tile, a long K
    (304, 520, 4104, 3),      # few tiles
    (200, 4096, 16384, 8),
    (8192, 4352, 4096, 2),    # 544 tiles of 256, 32 past two waves
    (8192, 5120, 5120, 2),    # two whole waves and a half
])
def test_fused_is_one_accumulator(M, N, K, R, ab):
    for bl in (P.B_KN, P.B_NK):
        p = P.plan_loop_matmul(M, N, K, ab=ab, b_layout=bl, sum="K", R=R, sum_impl=P.SUM_FUSED)
        assert p["n_sum_loops"] == 1 and p["n_sum_splitk"] == 0
        assert p["n_launches"] == 1 and p["workspace_bytes"] == 0
        assert "fused in accumulator" in p["text"] and "K parts" not in p["text"]


def test_split_is_one_partial_per_shard():
    for ab in (P.BF16, P.F32):
        p = P.plan_loop_matmul(304, 520, 4104, ab=ab, sum="K", R=3, sum_impl=P.SUM_SPLITK)
        assert p["n_sum_splitk"] == 1 and p["n_launches"] == 2 and p["workspace_bytes"] == -(-3 * 304 * 520 * 4 // 256) * 256
        assert "sum_{r=0..2} partial[r]" in p["text"]


def test_fused_says_nothing_about_a_product_without_a_sum():
    a, f = (P.plan_loop_matmul(304, 520, 4104, tile="M", R=2, sum_impl=i) for i in (P.SUM_AUTO, P.SUM_FUSED))
    assert a["text"] == f["text"] and a["n_launches"] == 2
