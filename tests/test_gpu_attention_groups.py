"""The attention forward with two key groups a workgroup: both sides of the
choice (512 keys; one workgroup a CU, two or one and a half under a causal mask), odd block counts, groups that see no
key, the training statistics, and determinism, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import partir_oracle as O
from paper_2401_11202_amd import partir as P
from tests.gpu_common import TOL_BF16, host, say
from tests.test_gpu_attention import make_qkv, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
# key groups of the launch with and without a causal mask
@pytest.mark.parametrize("B,S,H,R,groups", [
    (1, 384, 2, 1, (1, 1)),
    (1, 512, 2, 1, (2, 2)),      # the first query block has one block for each group
    (1, 640, 3, 1, (2, 2)),
    (2, 1152, 1, 2, (2, 2)),     # shards of 9 blocks of 64: the second group has one less
    (1, 1024, 2, 2, (2, 2)),     # shards past a query block, and blocks past a wave's queries
    (1, 1024, 32, 1, (2, 2)),    # 256 workgroups ...
    (1, 1024, 33, 1, (1, 1)),    # ... and 264
    (1, 1024, 64, 1, (1, 1)),
    (1, 1024, 65, 1, (1, 1)),
    (1, 2048, 32, 1, (2, 1)),    # 512 workgroups ...
    (1, 2048, 33, 1, (1, 1)),    # ... and 528
    (1, 3072, 8, 2, (2, 1)),     # 384 workgroups over shards of 1536
])
def test_key_groups(B, S, H, R, groups, causal):
    Q, K, V = make_qkv(140 + H, B, S, H)
    rng = np.random.default_rng(140)
    rows = np.unique(np.concatenate([[b * S + r for b in range(B) for r in (0, 63, 64, 127, 128, 191, S - 1)],
                                     rng.choice(B * S, 40, replace=False)]))
    say(f"attention B={B} S={S} H={H} R_kv={R} causal={causal}")
    q, k, v = Q.to_device(), K.to_device(), V.to_device()
    o, lse = P.attention_train(q, k, v, B=B, S=S, n_heads=H, causal=causal, R_kv=R)
    text = P.lib().partir_last_plan_text().decode()
    assert ("two key groups" in text) == (groups[0 if causal else 1] == 2), text
    again, lse2 = P.attention_train(q, k, v, B=B, S=S, n_heads=H, causal=causal, R_kv=R)
    torch.cuda.synchronize()
    assert torch.equal(o, again) and torch.equal(lse, lse2)
    ref, nrm = reference(Q, K, V, B, S, H, causal, rows)
    assert O.normalised_error(host(o)[rows], ref, nrm) <= TOL_BF16
    # the log-sum-exp of the same scores by torch, one head in fp32
    D, c = 128, 128 ** -0.5 * np.log2(np.e)
    s = c * (q[:S, :D].float() @ k[:S, :D].float().t().contiguous())
    if causal:
        s.masked_fill_(torch.ones_like(s, dtype=torch.bool).triu_(1), float("-inf"))
    want = torch.logsumexp(s * np.log(2.0), dim=1) / np.log(2.0)
    assert float((lse[:S, 0] - want).abs().max()) < 1e-4


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,many", [(2048, 40), (1024, 40)])
def test_two_key_groups_are_as_exact_as_one(S, many, causal):
    """The same heads alone (two key groups) and among many (one): the two
    results round the weights against different maxima, so they differ, but
    neither is further from the 64-bit result."""
    Q, K, V = make_qkv(150, 1, S, many)
    q, k, v = Q.to_device(), K.to_device(), V.to_device()
    few = [t[:, :256].contiguous() for t in (q, k, v)]
    say(f"attention S={S} causal={causal}: 2 heads, {many} heads")
    two = P.attention(*few, B=1, S=S, n_heads=2, causal=causal)
    assert "two key groups" in P.lib().partir_last_plan_text().decode()
    one = P.attention(q, k, v, B=1, S=S, n_heads=many, causal=causal)[:, :256]
    assert "two key groups" not in P.lib().partir_last_plan_text().decode()
    torch.cuda.synchronize()
    err = {"one": 0.0, "two": 0.0}
    for h in range(2):
        a = slice(128 * h, 128 * h + 128)
        s = few[0][:, a].double() @ few[1][:, a].double().t().contiguous() * 128 ** -0.5
        if causal:
            s.masked_fill_(torch.ones_like(s, dtype=torch.bool).triu_(1), float("-inf"))
        ref = torch.softmax(s, dim=1) @ few[2][:, a].double()
        for name, o in (("one", one), ("two", two)):
            err[name] += float((o[:, a].double() - ref).norm() / ref.norm()) / 2
    say(f"    relative error: one group {err['one']:.3e}, two {err['two']:.3e}")
    # weights and outputs rounded to bf16 (2^-9 each); 2% for the luck of the roundings
    assert err["two"] <= 1.02 * err["one"] and err["one"] <= 2 * 2.0 ** -9
