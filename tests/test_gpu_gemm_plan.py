"""A product's bits do not depend on the workspace that it runs in.

Contractions are cut by a rule on the product alone, and every workspace holds
the parts of whatever smaller batch runs in it."""
import pytest

from tests.gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

# (model, planned B x S, batch B x S)
PAIRS = [
    (dict(family="llama", n_layers=1, d_model=512, n_heads=4, n_kv_heads=2, d_ff=1984, vocab=13648, dtype="f32"),
     (1, 528), (1, 328)),
    (dict(family="llama", n_layers=1, d_model=256, n_heads=2, n_kv_heads=1, d_ff=368, vocab=7896, dtype="f32"),
     (1, 400), (1, 376)),
    (dict(family="gpt2", n_layers=1, d_model=512, n_heads=8, n_kv_heads=8, d_ff=2048, vocab=8192, dtype="f32"),
     (3, 456), (1, 8)),
    (dict(family="llama", n_layers=1, d_model=512, n_heads=8, n_kv_heads=4, d_ff=1504, vocab=3984, dtype="bf16"),
     (1, 304), (1, 248)),
    (dict(family="llama", n_layers=1, d_model=1024, n_heads=8, n_kv_heads=4, d_ff=3208, vocab=8448, dtype="bf16"),
     (2, 640), (1, 512)),
    (dict(family="gpt2", n_layers=1, d_model=256, n_heads=4, n_kv_heads=4, d_ff=1024, vocab=4032, dtype="bf16"),
     (4, 328), (2, 104)),
]


@pytest.mark.parametrize("case", range(len(PAIRS)))
def test_same_bits_in_a_larger_workspace(case):
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    w, big, (B, S) = PAIRS[case]
    w = dict(w, rope_base=10000.0, max_seq=big[1])
    say(f"{w['family']} {w['dtype']} {B}x{S} in its own workspace and in one for {big[0]}x{big[1]}")
    got = []
    for plan in ((B, S), big):
        m = fd.Model.from_workload(w)
        m.set_workspace(*plan)
        th = m.init_params(1)
        tok = m.make_tokens(B, S, 2, "zipf")
        got.append(m.hvp(th, m.random_vector(3, "rademacher"), 1e-3, tok).cpu())
    assert torch.equal(got[0], got[1])
