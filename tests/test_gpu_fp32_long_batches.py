"""fp32 products over thousands of tokens against float64.

What is left is the fp32 rounding of the stored activations and of the sums: 7e-8
to 2.5e-7 of the product over 32 models of 32 to 512 columns and 4200 to 16,384
tokens, at most 2e-5 of the root mean square (or of the value, where larger) in
any element.  The bars are twice that.
"""
import pytest

from tests.gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

MODELS = [
    dict(family="gpt2", layers=2, d=128, heads=4, kv=4, ff=384, vocab=5216, B=84, S=168),
    dict(family="gpt2", layers=1, d=160, heads=4, kv=4, ff=640, vocab=7720, B=28, S=424),
    dict(family="llama", layers=3, d=96, heads=4, kv=2, ff=256, vocab=1888, B=49, S=224),
    dict(family="gpt2", layers=2, d=512, heads=8, kv=8, ff=2048, vocab=8192, B=9, S=512),
]


@pytest.mark.parametrize("model", range(len(MODELS)))
def test_long_batches(model):
    need_gpu()
    from perf import cases
    c = dict(MODELS[model], dtype="f32", rope=10000.0, op="hvp")
    say(f"fp32 product, {c['family']} d {c['d']}, {c['B']}x{c['S']} tokens")
    for seed in range(2):
        got = cases.run(cases.prepare(c, seed)).double()
        want = cases.exact(c, seed)
        rms = want.norm() / want.numel() ** 0.5
        rel = float((got - want).norm() / want.norm())
        most = float(((got - want).abs() / want.abs().clamp_min(rms)).max())
        say(f"  rel_l2 {rel:.2e}, largest element {most:.2e}")
        assert rel <= 5e-7 and most <= 4e-5
