"""The memory-bound passes of the MLP backward at the edges of their tiles.

The activation backward works on 64-row tiles of 64 columns, from 2^26
elements on of 128; bias gradients sum 64-row blocks (four quarters, 512
columns a workgroup) and then the blocks, 32 and 8 at a time.  Sampled rows
and hidden units against the oracle, normalised as in the other backward tests.
"""
import numpy as np
import pytest

from oracle import partir_oracle as O
from paper_2401_11202_amd import inputs as I
from tests.gpu_common import say
from tests.test_gpu_backward import check, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,F", [(8, 8, 8),            # one partial quarter, one lane of columns
                                   (2056, 520, 336),     # 33 row blocks, the last of 8 rows; columns past 512
                                   (2632, 1032, 72),     # 42 row blocks: 32, 8 and 2
                                   (8200, 64, 8264)])    # 128-wide tiles, ragged in rows and columns
def test_backward_pass_edges(T, D, F):
    x = {"X": I.gaussian(131, 0, (T, D), 1.0), "W1": I.gaussian(131, 1, (D, F), D ** -0.5),
         "W2": I.gaussian(131, 2, (F, D), F ** -0.5), "dY": I.gaussian(131, 3, (T, D), 1.0),
         "b1": I.gaussian(131, 4, (F,), 0.5, "f32")}
    say(f"mlp backward passes T={T} D={D} F={F}")
    got = run(x, 1, 1)
    rows = sorted({0, T - 1, T // 2})
    units = sorted({0, F - 1, F // 2, min(F - 1, 64), max(F - 57, 0)})
    ref, norm = O.mlp_block_backward_sampled(x["X"].f64(), x["W1"].f64(), x["W2"].f64(), x["dY"].f64(),
                                             x["b1"].f64(), "gelu", 1, 1, rows, units)
    picked = {"dX": got["dX"][rows], "dW1": got["dW1"][:, units], "dW2": got["dW2"][units],
              "db1": got["db1"][units], "db2": got["db2"]}
    check(picked, ref, norm)
