"""fp32 cross-entropy where one point's logit lies far from the mean's.

A logit 800 below the row's largest at the mean and 10 below it at one of the
two points (half difference 790) has e^-800 as its factor at the mean, which
fp64 rounds to zero, and e^790 as its factor between the points, which overflows.
"""
import numpy as np
import pytest

from oracle import hvp as OH
from oracle import model as M
from tests import micro
from tests.gpu_util import need_gpu, rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drop", [0.0, 60.0, 800.0])
def test_fp32_logits_far_apart(drop):
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    w = dict(family="llama", n_layers=1, d_model=64, n_heads=4, n_kv_heads=4, d_ff=128, vocab=64, max_seq=16,
             rope_base=10000.0, dtype="f32")
    cfg = micro.cfg_of(w)
    lay = {e.name: e for e in M.layout(cfg)}
    rng = np.random.default_rng(5)
    theta = (0.02 * rng.standard_normal(M.num_params(cfg))).astype(np.float32)
    for e in lay.values():
        if e.numel == 64:
            theta[e.offset:e.offset + 64] = 1.0
    # every normed row is close to sqrt(64) along the first coordinate
    emb, head = list(lay.values())[0], list(lay.values())[-1]
    assert emb.numel == head.numel == 64 * 64
    theta[emb.offset:emb.offset + emb.numel].reshape(64, 64)[:, 0] = 10.0
    rows = theta[head.offset:head.offset + head.numel].reshape(64, 64)
    rows[:] = 0.0
    rows[1:, 0] = -drop / 8 + 0.05 * rng.standard_normal(63)
    v = np.zeros_like(theta)
    eps = 1e-3
    v[head.offset:head.offset + head.numel].reshape(64, 64)[1:, 0] = max(0.0, drop - 10) / 8 / eps + rng.standard_normal(63)
    tok = rng.integers(0, 64, (2, 16)).astype(np.int32)
    say(f"fp32 cross-entropy, logits {drop} apart at the mean")
    mod = fd.Model.from_workload(w)
    mod.set_workspace(2, 16)
    got = mod.hvp(torch.from_numpy(theta).cuda(), torch.from_numpy(v).cuda(), eps, torch.from_numpy(tok).cuda()).cpu().numpy()
    want = OH.lm_hvp(cfg, theta, v.astype(np.float64), eps, tok)
    # the head's own block: its products drop no term of the pair form here (the
    # normed rows are the same at both points).  Logits of magnitude `drop` carry
    # a few fp32 roundings of it into the exponent.
    b = slice(head.offset, head.offset + head.numel)
    err = rel_l2(got[b], want[b])
    say(f"  rel_l2 of the head block {err:.2e}")
    assert err <= 1e-5 + 16 * drop * 2.0 ** -24
