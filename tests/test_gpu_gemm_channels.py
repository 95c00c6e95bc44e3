"""The two channel products of a linear layer in one launch, whole and cut into parts.

The reference is the float64 product of the same operands.  For fp32 operands
the error bar is the worst-case rounding of a K-term fp32 sum taken 16 terms
at a time in six partial products, K/16 * 6 additions of half an ulp each on
the sum of magnitudes; for bf16 the same without the split (K/16 additions).
That worst case grows past 2^-16, the size of a lost partial product, so the
root-mean-square error, relative to the root of the sum of the terms' squares, is
held to the random walk of its 2K/16 additions too (test_gpu_gemm_epilogue.py).
"""
import numpy as np
import pytest

from tests.gpu_util import need_gpu, say
from tests.test_gpu_gemm_epilogue import rms_bar

pytestmark = pytest.mark.gpu

# (M, N, K, batch): tile edges and remainders in every dimension, one tile, long
# contractions over few tiles, the shapes of the small workloads
# (fp32 operands need multiples of 4, bf16 ones of 8)
SHAPES = [(4, 4, 4, 1), (8, 8, 8, 1), (128, 128, 32, 1), (136, 72, 40, 2), (64, 64, 200, 3), (256, 512, 1024, 1),
          (1200, 512, 2816, 1), (520, 192, 1000, 1), (96, 4096, 1200, 1), (16, 24, 4096, 1), (2056, 2312, 264, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_channel_products(dtype, ak, bk, shape):
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    M, N, K, batch = shape
    if dtype == "bf16" and (M % 8 or N % 8 or K % 8):
        pytest.skip("bf16 operands come in 16-byte vectors of 8")
    say(f"gemm channels {dtype} {shape} layouts {ak}{bk}")
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    # magnitudes over several decades, so that no operand's low bits are idle
    ops = [(rng.standard_normal((batch, r, K)) * 10.0 ** rng.integers(-3, 3, (batch, r, 1))).astype(np.float32)
           for r in (M, N, M, N)]
    if dtype == "bf16":
        ops = [torch.from_numpy(x).to(torch.bfloat16).float().numpy() for x in ops]
    A, B, A2, B2 = ops
    one = A.astype(np.float64) @ B.astype(np.float64).transpose(0, 2, 1)
    two = one + A2.astype(np.float64) @ B2.astype(np.float64).transpose(0, 2, 1)
    mag1 = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64).transpose(0, 2, 1)
    mag2 = mag1 + np.abs(A2).astype(np.float64) @ np.abs(B2).astype(np.float64).transpose(0, 2, 1)
    sq = [x.astype(np.float64) ** 2 for x in ops]
    walk = np.sqrt(sq[0] @ sq[1].transpose(0, 2, 1) + sq[2] @ sq[3].transpose(0, 2, 1))

    def up(x, kmajor):
        return torch.from_numpy(np.ascontiguousarray(x if kmajor else x.transpose(0, 2, 1))).cuda().to(
            torch.bfloat16 if dtype == "bf16" else torch.float32)

    dA, dB, dA2, dB2 = up(A, ak), up(B, bk), up(A2, ak), up(B2, bk)
    for nbytes in (0, 64 << 20):
        scratch = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
        C2 = torch.full((batch, M, N), float("nan"), device="cuda")
        C1 = torch.full_like(C2, float("nan"))
        fd.testing_gemm_channels(dtype, M, N, K, batch, ak, bk, dA, dB, dA2, dB2, C2, C1, 0.5, scratch)
        bar = (6 if dtype == "f32" else 1) * (K / 16 + 2) * 2.0 ** -24
        e1 = (np.abs(2 * C1.cpu().numpy().astype(np.float64) - one) / mag1).max()
        e2 = (np.abs(2 * C2.cpu().numpy().astype(np.float64) - two) / mag2).max()
        rms = np.sqrt((((2 * C2.cpu().numpy().astype(np.float64) - two) / walk) ** 2).mean())
        say(f"  scratch {nbytes >> 20} MB: one pair {e1:.2e}, two pairs {e2:.2e} of the magnitudes (bar {bar:.1e}); rms {rms:.2e}")
        assert e1 <= bar and e2 <= 2 * bar
        assert rms <= rms_bar(2 * K)
