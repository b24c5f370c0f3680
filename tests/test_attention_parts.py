"""How many ordered parts a causal key shard runs as, and which attention kernel
a launch takes (host only): parts under 64 key blocks only while the grid has
fewer than 768 workgroups; two key groups a workgroup on short grids."""
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


@pytest.mark.parametrize("B,S,H,R,causal,block,groups", [
    (1, 384, 2, 1, 1, 64, 1),      # under 512 keys
    (1, 512, 2, 1, 1, 64, 2),
    (2, 1152, 1, 2, 0, 64, 2),     # shards of 576 keys
    (1, 1024, 32, 1, 1, 64, 2),    # 256 workgroups ...
    (1, 1024, 33, 1, 1, 32, 1),    # ... and 264
    (1, 1024, 33, 1, 0, 32, 1),
    (1, 2048, 32, 1, 1, 64, 2),    # 512 under a causal mask from 2048 keys on ...
    (1, 2048, 32, 1, 0, 32, 1),    # ... not without one ...
    (1, 2048, 33, 1, 1, 32, 1),    # ... and not 528
    (1, 1920, 34, 1, 1, 32, 1),    # 510 workgroups over 1920 keys
    (1, 3072, 8, 2, 1, 64, 2),     # 384 over causal shards of 1536 keys ...
    (1, 3072, 8, 2, 0, 32, 1),
    (1, 3072, 9, 2, 1, 32, 1),     # ... and 432
])
def test_attention_kernel(B, S, H, R, causal, block, groups):
    text = P.plan_attention(B, S, H, 128, bool(causal), R)["text"]
    assert f"; key blocks of {block}" in text and ("two key groups" in text) == (groups == 2), text
