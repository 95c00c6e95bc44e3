"""Fused attention on sequence lengths that are no multiple of its blocks.

The fused kernels take 32-key blocks, 64 or 128 queries and 64 keys per
workgroup; here the last of each is partly past the sequence, in a batch of
two so that the rows after the first sequence are the second one's.  The
reference is the unfused path on the same inputs, with the bars of the aligned
comparison (bf16 rounding of the probabilities that the unfused path stores).
"""
import numpy as np
import pytest

from tests.gpu_util import need_gpu, rel_l2, say
from tests.test_gpu_attention import _both_paths

pytestmark = pytest.mark.gpu

MODELS = {
    "llama dh 128, grouped": dict(family="llama", n_layers=1, d_model=512, n_heads=4, n_kv_heads=2, d_ff=256),
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
