"""Attention on sequence lengths that are no multiple of the fused kernels' blocks.

The fused kernels for 128-wide heads take 32-key blocks, 64 queries and 64 keys
per workgroup; here the last of each is partly past the sequence, in a batch of
two so that the rows after the first sequence are the second one's.  The
reference is the unfused path on the same inputs, with the bars of the aligned
comparison (bf16 rounding of the probabilities that the unfused path stores),
and float64.  64-wide heads keep the unfused path at such lengths.
"""
import math

import numpy as np
import pytest

from tests.gpu_util import need_gpu, rel_l2, say
from tests.test_gpu_attention import _both_paths

pytestmark = pytest.mark.gpu

MODELS = {
    "llama dh 128, grouped": dict(family="llama", n_layers=1, d_model=512, n_heads=4, n_kv_heads=2, d_ff=256),
    "llama dh 128": dict(family="llama", n_layers=1, d_model=256, n_heads=2, n_kv_heads=2, d_ff=256),
}
NARROW = {
    "gpt2 dh 64": dict(family="gpt2", n_layers=1, d_model=256, n_heads=4, n_kv_heads=4, d_ff=256),
    "llama dh 64": dict(family="llama", n_layers=1, d_model=256, n_heads=4, n_kv_heads=1, d_ff=256),
}


@pytest.mark.parametrize("seq", [8, 40, 72, 136, 200, 456, 1000])
@pytest.mark.parametrize("name", list(MODELS))
def test_ragged_fused_matches_unfused(name, seq):
    w = dict(MODELS[name], vocab=512, max_seq=seq, rope_base=10000.0, dtype="bf16")
    say(f"ragged fused attention: {name}, 2x{seq}")
    fused, unfused, layout = _both_paths(w, 2, seq)
    assert np.all(np.isfinite(fused))
    err = rel_l2(fused, unfused)
    say(f"  rel_l2 {err:.3e}")
    assert err <= 2e-2
    for e in layout:
        ref = unfused[e.offset:e.offset + e.numel]
        if e.numel >= 4096 and np.linalg.norm(ref) > 1e-3 * np.linalg.norm(unfused):
            assert rel_l2(fused[e.offset:e.offset + e.numel], ref) <= 5e-2, e.name


@pytest.mark.parametrize("seq", [8, 72, 200, 1000])
@pytest.mark.parametrize("name", list(NARROW))
def test_ragged_narrow_heads_keep_the_score_matrices(name, seq):
    """The row sums and the softmax gradient of these lengths are formed in fp64
    from stored scores: the same bits as with the unfused path asked for."""
    w = dict(NARROW[name], vocab=512, max_seq=seq, rope_base=10000.0, dtype="bf16")
    say(f"ragged attention of 64-wide heads: {name}, 2x{seq}")
    default, unfused, _ = _both_paths(w, 2, seq)
    assert np.array_equal(default, unfused)


@pytest.mark.parametrize("seq,plan", [(200, 200), (456, 456), (256, 264)])
def test_ragged_fused_is_no_further_from_float64(seq, plan):
    """Error against float64 of the fused and the unfused path over 24 seeds, in a
    workspace for sequences of `plan` tokens.

    Both round the same operands and probabilities to bf16, with different
    roundings: the logarithm of their errors' ratio scatters by 0.025 (q and k
    rows, measured) from seed to seed, so its mean over 24 by 0.005.  The bar is
    four times that."""
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    from perf import cases
    c = dict(family="llama", layers=1, d=512, heads=4, kv=2, ff=768, vocab=512, dtype="bf16", rope=10000.0, op="hvp",
             B=2, S=seq)
    say(f"ragged fused attention against float64: 2x{seq} in a plan for {plan}")
    qk = c["d"] + c["kv"] * 128
    off = c["vocab"] * c["d"] + c["d"]
    logs = []
    for seed in range(24):
        want = cases.exact(c, seed)
        theta, tok = cases._params(c, seed), cases._batches(c, seed)[0][0]
        v = cases._unit(theta.numel(), seed)
        err = []
        for unfused in (False, True):
            m = fd.Model("llama", 1, c["d"], c["heads"], c["kv"], c["ff"], c["vocab"], plan, "bf16", rope_base=c["rope"])
            m.unfused_attention(unfused)
            m.set_workspace(2, plan)
            d = m.hvp(theta, v, 1e-3, tok).double() - want
            w = slice(off, off + qk * c["d"])
            err.append((float(d.norm() / want.norm()), float(d[w].norm() / want[w].norm())))
        logs.append([math.log(a / b) for a, b in zip(*err)])
    mean = np.mean(logs, axis=0)
    say(f"  mean log ratio: all {mean[0]:+.4f}, q and k {mean[1]:+.4f}; per seed +-{np.std(logs, axis=0)[1]:.4f}")
    assert max(mean) <= 0.02


def test_smaller_ragged_batch_in_a_ragged_plan():
    """A workspace planned for a ragged length takes any shorter multiple of 8."""
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    w = dict(MODELS["llama dh 128, grouped"], vocab=512, max_seq=200, rope_base=10000.0, dtype="bf16")
    got = []
    for plan in (200, 104):
        mod = fd.Model.from_workload(w)
        mod.set_workspace(2, plan)
        th = mod.init_params(1)
        tok = mod.make_tokens(2, 104, 2, "zipf")
        got.append(mod.hvp(th, mod.random_vector(3, "rademacher"), 1e-3, tok).cpu())
    assert torch.equal(got[0], got[1])
