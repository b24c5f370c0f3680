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


@pytest.mark.parametrize("M,N,K,tiles,edge,parts,kt", [
    (512, 512, 4096, 64, 64, 4, 16),
    (300, 520, 4104, 45, 64, 4, 17),
    (200, 4096, 16384, 64, 128, 4, 64),
])
@pytest.mark.parametrize("R", [1, 8])
def test_k_parts_are_counted_in_the_tiles_that_run(M, N, K, tiles, edge, parts, kt, R):
    """A short grid: every output tile in K parts whose fp32 partials a
    reduction adds, with or without a #sum."""
    R = R if K % (8 * R) == 0 else 3
    p = P.plan_loop_matmul(M, N, K, sum="K" if R > 1 else None, R=R)
    t = p["text"]
    assert f"; {tiles} tiles as {parts} K parts of {kt} K tiles each; workgroup tiles of {edge} x {edge}" in t, t
    assert f"grid {tiles * parts} WGs" in t and "the last" not in t and ".fixup" not in t
    assert f"splitk_reduce: C[{M},{N}] = sum of the {parts} K parts in ascending order" in t
    assert p["n_launches"] == 2 and p["n_sum_splitk"] == (R > 1)
    assert p["workspace_bytes"] >= parts * M * N * 4


def test_fused_says_nothing_about_a_product_without_a_sum():
    a, f = (P.plan_loop_matmul(304, 520, 4104, tile="M", R=2, sum_impl=i) for i in (P.SUM_AUTO, P.SUM_FUSED))
    assert a["text"] == f["text"] and a["n_launches"] == 2
