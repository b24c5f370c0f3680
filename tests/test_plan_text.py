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
