"""The plan text of a call that executes is built when it is asked for; it is
the text the plan query gives for the same arguments.  Host only: the calls
stop at PARTIR_FAIL_LAUNCH."""
import ctypes
import threading

import pytest

from paper_2401_11202_amd import partir as P

D = ctypes.c_void_p(0x10000)


@pytest.fixture(autouse=True)
def _never_launch(monkeypatch):
    monkeypatch.setenv("PARTIR_FAIL_LAUNCH", "1")


def last():
    return P.lib().partir_last_plan_text().decode()


def parts(n):
    return (ctypes.c_void_p * n)(*([0x10000] * n))


CALLS = [
    (lambda L: L.partir_loop_matmul(D, D, D, 1000, 304, 4112, 4112, 304, 304, P.BF16, P.F32, P.B_KN, -1, 2, 2,
                                    P.SUM_AUTO, D, 1 << 34, None),
     lambda: P.plan_loop_matmul(1000, 304, 4112, b_layout=P.B_KN, sum="K", R=2)),
    (lambda L: L.partir_mlp_block(D, D, None, D, None, D, 512, 256, 1024, P.BF16, P.F32, P.ACT_GELU, 1, 8, D, 1 << 34,
                                  None),
     lambda: P.plan_mlp_block(512, 256, 1024, R_model=8)),
    (lambda L: L.partir_attn_block(D, D, D, D, D, D, 2, 256, 1024, 8, 128, 1, 0.0, P.BF16, P.F32, 1, 8, D, 1 << 34,
                                   None),
     lambda: P.plan_attn_block(2, 256, 1024, 8, 128, 1, 8)),
    (lambda L: L.partir_decoder_layer(D, D, D, 1e-6, D, D, D, D, D, D, 2, 256, 1024, 8, 128, 1728, 2, 4, D, 1 << 34,
                                      None),
     lambda: P.plan_decoder_layer(2, 256, 1024, 8, 128, 1728, 2, 4)),
    (lambda L: L.partir_mlp_block_sharded(parts(8), parts(8), None, parts(8), None, parts(8), 1024, 256, 1024, P.F32,
                                          P.ACT_GELU, 2, 4, D, 1 << 34, None),
     lambda: P.plan_mlp_block_sharded(1024, 256, 1024, R_batch=2, R_model=4)),
]


# every entry point that executes (the device pointers of one call alike)
ENTRY = {
    "loop_matmul": CALLS[0][0],
    "mlp_block": CALLS[1][0],
    "attn_block": CALLS[2][0],
    "decoder_layer": CALLS[3][0],
    "mlp_block_sharded": CALLS[4][0],
    "mlp_block_train": lambda L: L.partir_mlp_block_train(D, D, D, D, D, D, D, 1000, 8200, 4104, P.BF16, P.F32,
                                                          P.ACT_GELU, 1, 1, D, 1 << 34, None),
    "mlp_block_backward": lambda L: L.partir_mlp_block_backward(D, D, D, D, D, D, D, D, D, D, D, 1536, 2560, 10240,
                                                                P.ACT_GELU, 2, 4, D, 1 << 34, None),
    "mlp_block_backward, Z recomputed, no bias gradients": lambda L: L.partir_mlp_block_backward(
        D, D, None, D, D, None, D, D, None, D, None, 520, 200, 336, P.ACT_GELU, 5, 2, D, 1 << 34, None),
    "attn_block_train": lambda L: L.partir_attn_block_train(D, D, D, D, D, D, D, 2, 256, 1024, 8, 128, 1, 0.0, P.BF16,
                                                            P.F32, 1, 8, D, 1 << 34, None),
    "attn_block_backward": lambda L: L.partir_attn_block_backward(D, D, D, D, D, D, D, D, D, D, D, D, 4, 2048, 4096, 32,
                                                                  128, 1, 0.0, 2, 8, D, 1 << 34, None),
    "attention": lambda L: L.partir_attention(D, D, D, D, 1, 8192, 2, 128, 1, 0.0, 4, D, 1 << 34, None),
    "attention_train": lambda L: L.partir_attention_train(D, D, D, D, D, 1, 512, 2, 128, 0, 0.0, 1, D, 1 << 34, None),
    "attention_backward": lambda L: L.partir_attention_backward(D, D, D, D, D, D, D, D, D, 1, 512, 2, 128, 1, 0.0, D,
                                                                1 << 34, None),
    "decoder_layer_sharded": lambda L: L.partir_decoder_layer_sharded(
        parts(8), D, D, 1e-6, parts(8), parts(8), parts(8), parts(8), parts(8), parts(8), 2, 1024, 2048, 16, 128, 5632,
        2, 4, D, 1 << 34, None),
}


@pytest.mark.parametrize("name", ENTRY)
def test_deferred_text_is_the_text_of_the_plan_that_runs(name, monkeypatch, capfd):
    """PARTIR_DUMP_PLAN formats the plan that is executed, pointers and all;
    without it the text is planned again from the sizes alone."""
    call = ENTRY[name]
    monkeypatch.setenv("PARTIR_DUMP_PLAN", "1")
    assert P.STATUS[call(P.lib())] == "PARTIR_E_HIP", P.lib().partir_last_error().decode()
    want = last()
    assert want.startswith(name.split(",")[0] + ":") and want in capfd.readouterr().err
    monkeypatch.delenv("PARTIR_DUMP_PLAN")
    P.plan_loop_matmul(8, 8, 8)
    assert P.STATUS[call(P.lib())] == "PARTIR_E_HIP"
    assert last() == want and capfd.readouterr().err == ""


@pytest.mark.parametrize("call,plan", CALLS)
def test_text_of_a_call_is_the_plan_querys(call, plan):
    want = plan()["text"]
    P.plan_loop_matmul(8, 8, 8)
    assert last() != want
    assert P.STATUS[call(P.lib())] == "PARTIR_E_HIP"
    assert last() == want and last() == want


def test_text_is_kept_per_thread_and_by_failing_calls():
    call, plan = CALLS[1]
    want = plan()["text"]
    call(P.lib())
    got = {}

    def other():
        CALLS[2][0](P.lib())
        got["t"] = last()

    t = threading.Thread(target=other)
    t.start()
    t.join()
    assert got["t"].startswith("attn_block:")
    assert P.STATUS[P.lib().partir_mlp_block(None, D, None, D, None, D, 512, 256, 1024, P.BF16, P.F32, P.ACT_GELU, 1, 8,
                                             D, 1 << 34, None)] == "PARTIR_E_NULL"
    assert last() == want
