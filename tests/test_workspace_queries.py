"""Every entry point runs in exactly the workspace that its size query returns
and refuses one byte less (host only: the calls stop at PARTIR_FAIL_LAUNCH).

The sizes spread over small blocks, ragged ones, and wide ones whose products
have few output tiles, where the planner splits K."""
import ctypes

import pytest

from paper_2401_11202_amd import partir as P

D_ = ctypes.c_void_p(0x10000)      # 16-byte aligned, never dereferenced


@pytest.fixture(autouse=True)
def _never_launch(monkeypatch):
    monkeypatch.setenv("PARTIR_FAIL_LAUNCH", "1")


def arr(n):
    return (ctypes.c_void_p * n)(*([0x10000] * n))


def fits(call, need):
    """call(ws_bytes) reaches the launch with `need` bytes, not with fewer."""
    assert need != ctypes.c_size_t(-1).value
    assert P.STATUS[call(need)] == "PARTIR_E_HIP", P.lib().partir_last_error().decode()
    if need:
        assert P.STATUS[call(need - 1)] == "PARTIR_E_WORKSPACE"


MLP = [(2048, 8192, 4096, 1, 8), (1024, 8192, 8192, 1, 8), (4096, 8192, 2048, 1, 8), (8192, 7168, 1024, 1, 8),
       (512, 7168, 16384, 1, 1), (256, 8192, 32768, 1, 1), (512, 256, 1024, 1, 8), (200, 4096, 16384, 1, 8),
       (1536, 2560, 10240, 2, 4), (8192, 4096, 16384, 1, 8), (8, 8, 8, 1, 1), (2056, 520, 336, 1, 2),
       (3000, 12288, 4104, 1, 1), (0, 64, 64, 1, 1), (64, 64, 0, 1, 2)]


@pytest.mark.parametrize("T,D,F,Rb,Rm", MLP)
@pytest.mark.parametrize("out", [P.F32, P.BF16])
def test_mlp_forward_and_train(T, D, F, Rb, Rm, out):
    L = P.lib()
    need = L.partir_mlp_block_workspace(T, D, F, out, Rb, Rm)
    fits(lambda n: L.partir_mlp_block(D_, D_, None, D_, None, D_, T, D, F, P.BF16, out, P.ACT_GELU, Rb, Rm, D_, n,
                                      None), need)
    fits(lambda n: L.partir_mlp_block_train(D_, D_, None, D_, None, D_, D_, T, D, F, P.BF16, out, P.ACT_GELU, Rb, Rm,
                                            D_, n, None), need)


@pytest.mark.parametrize("T,D,F,Rb,Rm", [m for m in MLP if all(m[:3]) and m[0] % (8 * m[3]) == 0])
@pytest.mark.parametrize("bias", [0, 1])
def test_mlp_backward(T, D, F, Rb, Rm, bias):
    L = P.lib()
    db = D_ if bias else None

    def call(Z):
        return lambda n: L.partir_mlp_block_backward(D_, D_, None, D_, D_, Z, D_, D_, db, D_, db, T, D, F, P.ACT_GELU,
                                                     Rb, Rm, D_, n, None)
    need = L.partir_mlp_block_backward_workspace(T, D, F, P.ACT_GELU, bias, Rb, Rm)
    fits(call(None), need)
    assert P.STATUS[call(D_)(need)] == "PARTIR_E_HIP"   # the query assumes a recomputed Z


ATTN = [(2, 256, 1024, 8, 1, 8), (4, 2048, 4096, 32, 1, 8), (1, 128, 128, 1, 1, 1), (1, 1024, 8192, 64, 1, 8),
        (2, 384, 7168, 56, 2, 1), (1, 512, 12288, 96, 1, 4), (3, 640, 1280, 10, 3, 2)]


@pytest.mark.parametrize("B,S,D,H,Rb,Rm", ATTN)
def test_attention_block(B, S, D, H, Rb, Rm):
    L = P.lib()
    need = L.partir_attn_block_workspace(B, S, D, H, 128, Rb, Rm)
    for out in (P.F32, P.BF16):
        fits(lambda n: L.partir_attn_block(D_, D_, D_, D_, D_, D_, B, S, D, H, 128, 1, 0.0, P.BF16, out, Rb, Rm, D_, n,
                                           None), need)
    st = L.partir_attn_block_train(D_, D_, D_, D_, D_, D_, D_, B, S, D, H, 128, 1, 0.0, P.BF16, P.F32, Rb, Rm, D_,
                                   need, None)
    assert P.STATUS[st] == "PARTIR_E_HIP"               # Q, K, V and A live in `saved`: needs less
    need = L.partir_attn_block_backward_workspace(B, S, D, H, 128, Rb, Rm)
    fits(lambda n: L.partir_attn_block_backward(D_, D_, D_, D_, D_, D_, D_, D_, D_, D_, D_, D_, B, S, D, H, 128, 1,
                                                0.0, Rb, Rm, D_, n, None), need)


@pytest.mark.parametrize("B,S,D,H,F,Rb,Rm", [a[:4] + (f,) + a[4:] for a in ATTN for f in (1024, 13312, 0)])
def test_decoder_layer(B, S, D, H, F, Rb, Rm):
    F -= F % (8 * Rm)
    L = P.lib()
    need = L.partir_decoder_layer_workspace(B, S, D, H, 128, F, Rb, Rm)
    fits(lambda n: L.partir_decoder_layer(D_, D_, D_, 1e-6, D_, D_, D_, D_, D_, D_, B, S, D, H, 128, F, Rb, Rm, D_, n,
                                          None), need)


@pytest.mark.parametrize("B,S,H,R", [(1, 8192, 2, 4), (1, 128, 1, 1), (4, 4096, 5, 2), (1, 3840, 1, 2)])
@pytest.mark.parametrize("causal", [0, 1])
def test_attention(B, S, H, R, causal):
    L = P.lib()
    need = L.partir_attention_workspace(B, S, H, 128, R)
    call = lambda n: L.partir_attention(D_, D_, D_, D_, B, S, H, 128, causal, 0.0, R, D_, n, None)
    train = lambda n: L.partir_attention_train(D_, D_, D_, D_, D_, B, S, H, 128, causal, 0.0, R, D_, n, None)
    for f in (call, train):
        if causal:
            fits(f, need)
        else:
            assert P.STATUS[f(need)] == "PARTIR_E_HIP"  # one query for both masks; causal shards take more parts
    need = L.partir_attention_backward_workspace(B, S, H, 128)
    fits(lambda n: L.partir_attention_backward(D_, D_, D_, D_, D_, D_, D_, D_, D_, B, S, H, 128, causal, 0.0, D_, n,
                                               None), need)


@pytest.mark.parametrize("T,D,F,Rb,Rm", [(1024, 256, 1024, 2, 4), (2048, 4096, 4096, 2, 4), (512, 7168, 8192, 1, 8)])
def test_mlp_sharded(T, D, F, Rb, Rm):
    L = P.lib()
    a = arr(Rb * Rm)
    fits(lambda n: L.partir_mlp_block_sharded(a, a, None, a, None, a, T, D, F, P.F32, P.ACT_GELU, Rb, Rm, D_, n, None),
         L.partir_mlp_block_sharded_workspace(T, D, F, Rb, Rm))


@pytest.mark.parametrize("B,S,D,H,F,Rb,Rm", [(2, 1024, 2048, 16, 5632, 2, 4), (4, 2048, 5120, 40, 13824, 2, 4),
                                             (1, 512, 8192, 64, 8192, 1, 4), (2, 128, 1024, 8, 0, 2, 4)])
def test_decoder_sharded(B, S, D, H, F, Rb, Rm):
    L = P.lib()
    a = arr(Rb * Rm)
    fits(lambda n: L.partir_decoder_layer_sharded(a, D_, D_, 1e-6, a, a, a, a, a, a, B, S, D, H, 128, F, Rb, Rm, D_, n,
                                                  None),
         L.partir_decoder_layer_sharded_workspace(B, S, D, H, 128, F, Rb, Rm))


@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (300, 520, 4104), (2048, 2048, 8192), (256, 256, 65536),
                                   (1000, 304, 4112), (8192, 5120, 5120), (200, 16384, 4096)])
@pytest.mark.parametrize("ab", [P.F32, P.BF16])
@pytest.mark.parametrize("summ,R", [(P.AXIS_NONE, 1), (P.AXIS_K, 1), (P.AXIS_K, 2)])
@pytest.mark.parametrize("impl", [P.SUM_AUTO, P.SUM_FUSED, P.SUM_SPLITK])
def test_loop_matmul(M, N, K, ab, summ, R, impl):
    if K // R % 8:
        R = 1
    L = P.lib()
    for bl in (P.B_KN, P.B_NK):
        need = L.partir_loop_matmul_workspace(M, N, K, ab, P.F32, bl, P.AXIS_NONE, summ, R, impl)
        fits(lambda n: L.partir_loop_matmul(D_, D_, D_, M, N, K, K, N if bl == P.B_KN else K, N, ab, P.F32, bl,
                                            P.AXIS_NONE, summ, R, impl, D_, n, None), need)
