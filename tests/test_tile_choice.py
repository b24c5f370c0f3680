"""Which workgroup tile the planner takes for a bf16 product (host only), at
sizes where the measured times of the tiles are well apart."""
import pytest

from paper_2401_11202_amd import partir as P


@pytest.mark.parametrize("M,N,K,layout,tile", [
    # a little over one round of 256-wide tiles, or over two of 128-wide pairs
    (4457, 4440, 3816, P.B_NK, 256),     # us in 256 / 128 wide tiles: 158 / 194
    (5612, 4344, 7536, P.B_NK, 256),     # 317 / 403
    (4103, 4456, 2808, P.B_NK, 256),     # 117 / 143
    (6205, 2888, 3848, P.B_KN, 256),     # 139 / 182
    (5869, 4168, 5968, P.B_KN, 256),     # 261 / 321
    (6582, 1200, 11528, P.B_NK, 256),    # 214, in two K parts of 128-wide ones 293
    (3936, 2336, 288, P.B_NK, 256),      # 16.0 / 21.9
    (2261, 7072, 2512, P.B_KN, 256),     # one round: 66 / 93
    # half a round, and many short tiles
    (1166, 2768, 1672, P.B_KN, 128),     # 35 / 20
    (3279, 10544, 80, P.B_KN, 128),      # 33 / 26
    # few tiles
    (18, 14448, 2408, P.B_KN, 64),       # 44 / 20 / 13 in 64-wide ones
    (62, 15552, 2560, P.B_KN, 64),       # 47 / 21 / 15
])
def test_the_faster_tile_is_taken(M, N, K, layout, tile):
    text = P.plan_loop_matmul(M, N, K, b_layout=layout)["text"]
    assert ("workgroup tiles of" not in text) if tile == 256 else (f"workgroup tiles of {tile} x" in text), text
    assert "0 split-K" in text


def test_few_residual_tiles_are_not_tail_split():
    """The fixup of a residual product over device-local arrays takes as long
    for 22 tiles as for 128: 114 us against 67 in 64-wide tiles."""
    text = P.plan_decoder_layer_sharded(1, 1152, 1024, 8, 128, 10240, R_batch=1, R_model=2)["text"]
    down = next(l for l in text.splitlines() if "ffn_down" in l)
    assert "the last" not in down and "workgroup tiles of 64 x 64" in down, down


@pytest.mark.parametrize("M,N,K,R,staged", [
    (2173, 408, 384, 8, True),      # 8 shards of 48, 7.4 workgroups a CU: us pipelined / register-staged 26.3 / 22.1
    (1070, 640, 320, 8, True),      # 23.6 / 20.9
    (896, 728, 64, 8, True),        # 20.3 / 17.8
    (1921, 2280, 80, 1, True),      # 14.2 / 13.0
    (1300, 2000, 112, 1, True),     # the last short K ...
    (1300, 2000, 116, 1, False),    # ... and past it
    (1800, 2056, 68, 1, False),     # one round of 128-wide tiles
    (1255, 2576, 120, 1, False),    # 14.1 / 15.8
    (1266, 232, 288, 4, False),     # 1.2 workgroups a CU: 11.8 / 12.1
    (256, 256, 512, 4, False),
])
def test_short_fp32_contractions_on_many_workgroups_are_register_staged(M, N, K, R, staged):
    for layout in (P.B_KN, P.B_NK):
        text = P.plan_loop_matmul(M, N, K, ab=P.F32, b_layout=layout, sum="K" if R > 1 else None, R=R)["text"]
        assert ("tiles of 64, register-staged" in text) == staged, text
