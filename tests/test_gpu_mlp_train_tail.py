"""mlp_block_train where the up-projection that keeps its pre-activation is
split: 1000 x 4104 outputs over K = 8200 are 68 ragged 256-wide tiles, each
run as two K parts (the second ends inside a K tile); the fixup launch adds
them and stores Z and H."""
import numpy as np
import pytest
import torch

from oracle import partir_oracle as O
from paper_2401_11202_amd import inputs as I
from paper_2401_11202_amd import partir as P
from tests.gpu_common import TOL_BF16, accum_bound, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["gelu", "none"])
def test_kept_preactivation_through_the_tail_split(act):
    T, D, F = 1000, 8200, 4104
    X, W1 = I.gaussian(161, 0, (T, D), 1.0), I.gaussian(161, 1, (D, F), D ** -0.5)
    W2 = I.gaussian(161, 2, (F, D), F ** -0.5)
    b1, b2 = I.gaussian(161, 3, (F,), 0.5, "f32"), I.gaussian(161, 4, (D,), 0.5, "f32")
    ws = torch.full((P.lib().partir_mlp_block_workspace(T, D, F, P.F32, 1, 1),), 255, dtype=torch.uint8, device="cuda")
    Zbig = torch.full((T + 8, F), 7.25, dtype=torch.bfloat16, device="cuda")
    say(f"mlp_block_train T={T} D={D} F={F} act={act}")
    args = [t.to_device() for t in (X, W1, W2)]
    kw = dict(b1=b1.to_device(), b2=b2.to_device(), act=act)
    Y, Z = P.mlp_block_train(*args, Z=Zbig[:T], workspace=ws, **kw)
    text = P.lib().partir_last_plan_text().decode()
    assert "the last 68 tiles as 2 K parts of 65 K tiles" in text and "mlp.up.fixup" in text, text
    again, _ = P.mlp_block_train(*args, **kw)      # the workspace of the size query
    torch.cuda.synchronize()
    assert torch.equal(again, Y) and torch.all(Zbig[T:] == 7.25)
    rows = sorted({0, 255, 256, T - 1} | set(np.random.default_rng(161).integers(0, T, 28).tolist()))
    Xr, W1f, b1f = X.f64()[rows], W1.f64(), b1.f64()
    norm = O.abs_product(Xr, W1f) + np.abs(b1f)
    err = O.normalised_error(host(Z)[rows], O.matmul(Xr, W1f) + b1f, norm)
    say(f"    Z: max normalised error {err:.3e}")
    assert err <= accum_bound(D) + 2.0 ** -8        # fp32 sums of D products, one rounding to bf16
    ref, norm = O.mlp_block(X.f64(), W1f, W2.f64(), b1f, b2.f64(), act, rows=rows, return_norm=True)
    err = O.normalised_error(host(Y)[rows], ref, norm)
    say(f"    Y: max normalised error {err:.3e}")
    assert err <= TOL_BF16
