"""How many ordered parts a causal key shard runs as (host only): under 64 key
blocks a part only while the grid has fewer than 768 workgroups."""
import pytest

from paper_2401_11202_amd import partir as P


@pytest.mark.parametrize("B,S,H,R,parts", [
    (1, 8192, 5, 2, 2),      # 640 workgroups, then 1280
    (1, 8192, 6, 2, 1),      # 768
    (1, 4096, 11, 2, 2),     # 704
    (1, 4096, 12, 2, 1),     # 768
    (1, 8192, 1, 2, 4),      # 128: parts of 16 blocks, the shortest
    (1, 3840, 1, 2, 1),      # 30 key blocks: no two parts of 16
    (1, 16384, 4, 2, 2),     # 1024: parts of 64 blocks, up to 2048 workgroups
    (1, 16384, 8, 2, 1),     # 2048
])
def test_parts(B, S, H, R, parts):
    text = P.plan_attention(B, S, H, 128, True, R)["text"]
    if parts == 1:
        assert "ordered parts" not in text
    else:
        assert f"each as {parts} ordered parts of {S // R // parts}" in text
