"""Products with their whole epilogue, causal products and long fp32 contractions,
against the float64 product of the same operands.

Bars.  A K-term fp32 sum of magnitudes m (the sum of |a b|) rounds once per 16 k
in the matrix instructions, six times where fp32 operands are split, each time by
at most 2^-24 m; the epilogue adds three roundings of the result's terms, an output
in bf16 half an ulp, 2^-9.  The
worst case grows with K and hides a lost partial product (2^-16), so the
root-mean-square error of fp32 results is held as well.  Each of n additions
rounds the partial sum by at most 2^-24, 2^-24 / sqrt(3) in the mean square, and
with terms of random sign no partial sum has more than the result's mean square, the
sum of the terms' squares: n additions come to at most 2^-24 sqrt(n / 3) of it,
with one more rounding for the epilogue.  A lost partial product is above 4e-6.
"""
import numpy as np
import pytest

from tests.gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu


def rms_bar(k):
    return 2.0 ** -24 * (np.sqrt(k / 16 / 3) + 1)


def _operands(torch, rng, dtype, M, N, K, batch, n):
    """n pairs of operands as float64 arrays and as device tensors, both layouts"""
    out = []
    for r in (M, N) * n:
        x = rng.standard_normal((batch, r, K)).astype(np.float32)
        if dtype == "bf16":
            x = torch.from_numpy(x).to(torch.bfloat16).float().numpy()
        out.append(x)
    return out


def _up(torch, x, kmajor, dtype):
    y = torch.from_numpy(np.ascontiguousarray(x if kmajor else x.transpose(0, 2, 1))).cuda()
    return y.to(torch.bfloat16) if dtype == "bf16" else y


def _product(ops):
    return sum(a.astype(np.float64) @ b.astype(np.float64).transpose(0, 2, 1) for a, b in zip(ops[::2], ops[1::2]))


def _steps(dtype, K):
    return (6 if dtype == "f32" else 1) * (K / 16 + 2)


# (M, N, K, parts wanted): one tile and edges, cut and whole
CUT = [(16, 24, 4096, True), (136, 264, 2048, True), (520, 192, 1000, True), (128, 128, 64, False), (1032, 776, 72, False)]


@pytest.mark.parametrize("M,N,K,cut", CUT)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["bias, residual", "bias of both kinds, operand type", "accumulate", "wide rows, residual"])
def test_epilogue(kind, dtype, M, N, K, cut):
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    say(f"gemm epilogue {dtype} {M}x{N}x{K} ({kind})")
    rng = np.random.default_rng(M + N + K)
    ops = _operands(torch, rng, dtype, M, N, K, 1, 2)
    mag = _product([np.abs(x) for x in ops])[0]
    ldc = N + 8 if kind.startswith("wide") else N
    odt = torch.bfloat16 if dtype == "bf16" and "operand" in kind else torch.float32
    bth = (4 * rng.standard_normal(N)).astype(np.float32)
    if dtype == "bf16":
        bth = torch.from_numpy(bth).to(torch.bfloat16).float().numpy()
    bv, res, old = (s * rng.standard_normal(shape).astype(np.float32) for s, shape in ((5, N), (20, (M, ldc)), (10, (M, ldc))))
    args, want = {}, 0.5 * _product(ops)[0]
    extra = np.zeros((M, N))
    if "bias" in kind:
        args["bias_theta"] = _up(torch, bth.reshape(1, 1, N), True, dtype)
        want = want + bth
        extra = extra + np.abs(bth)
    if "both" in kind:
        args.update(bias_v=torch.from_numpy(bv).cuda(), bias_v_scale=0.25)
        want = want + 0.25 * bv.astype(np.float64)
        extra = extra + np.abs(bv)
    if "residual" in kind:
        args["resid"] = torch.from_numpy(res).cuda()
        want = want + res[:, :N]
        extra = extra + np.abs(res[:, :N])
    if kind == "accumulate":
        args["beta"] = 1.0
        want = want + old[:, :N]
        extra = extra + np.abs(old[:, :N])
    dev = [_up(torch, x, True, dtype) for x in ops]
    two, one = fd.testing_gemm_plan(dtype, M, N, K, 1, 64 << 20)[2:]
    assert (two > 1) == cut
    for nbytes in (0, 64 << 20):
        scratch = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
        C = torch.from_numpy(old).cuda().to(odt)
        before = C.clone()
        fd.testing_gemm_epilogue(dtype, M, N, K, 1, 1, 1, *dev, C, ldc=ldc, alpha=0.5, scratch=scratch, **args)
        got = C.float().cpu().numpy().astype(np.float64)[:, :N]
        bar = 0.5 * mag * _steps(dtype, 2 * K) * 2.0 ** -24 + 3 * (np.abs(want) + extra) * 2.0 ** -24
        rms = np.linalg.norm(got - want) / np.linalg.norm(want)
        say(f"  scratch {nbytes >> 20} MB: rel L2 {rms:.2e}")
        if odt == torch.bfloat16:
            assert np.all(np.abs(got - want) <= bar + np.abs(want) * 2.0 ** -8)
        else:
            assert np.all(np.abs(got - want) <= bar)
            assert rms <= rms_bar(2 * K)
        assert torch.equal(C[:, N:], before[:, N:])


@pytest.mark.parametrize("S", [8, 120, 320, 584])
@pytest.mark.parametrize("causal", [1, 2, 3])
@pytest.mark.parametrize("dtype,tile", [("f32", 0), ("bf16", 0), ("bf16", 9)])
def test_causal(dtype, tile, causal, S):
    """Tiles above the diagonal left out (1); contractions of triangular matrices (2, 3), whose
    other half is not read: it holds NaN beyond the tiles that touch the diagonal."""
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    if tile == 9 and S % 32:
        pytest.skip("asked for by number, the kernel takes K in multiples of 32")
    say(f"gemm causal {causal} {dtype} tile {tile} S {S}")
    rng = np.random.default_rng(8)
    M, N, K = (S, S, 64) if causal == 1 else (S, 64, S)
    ops = _operands(torch, rng, dtype, M, N, K, 2, 1)
    if causal != 1:
        ops[0] = (ops[0] * (np.tril(np.ones((S, S))) if causal == 2 else np.triu(np.ones((S, S))))).astype(np.float32)
    want, mag = _product(ops), _product([np.abs(x) for x in ops])
    A = ops[0].copy()
    if causal != 1:   # (both kernels' tiles are 128 or 256 rows)
        i, k = np.indices((S, S))
        far = k >= (i // 256 + 1) * 256 if causal == 2 else k < (i // 256) * 256
        A[:, far] = np.nan
    C = torch.zeros((2, M, N), device="cuda")
    fd.testing_gemm_epilogue(dtype, M, N, K, 2, 1, 1, _up(torch, A, True, dtype), _up(torch, ops[1], True, dtype), None, None,
                             C, causal=causal, tile=tile)
    err = np.abs(C.cpu().numpy().astype(np.float64) - want) - mag * _steps(dtype, K) * 2.0 ** -24
    if causal == 1:
        err = err[:, np.tril(np.ones((S, S), bool))]
    assert err.max() <= 0


@pytest.mark.parametrize("K", [8192, 66000, 131072])
def test_long_fp32_contraction(K):
    """Parts of at most 4096 k, added in fp64, keep the error of a long sum that of a short one."""
    torch = need_gpu()
    from paper_2602_00816_amd import fdhvp as fd
    M, N = 64, 72
    say(f"gemm fp32 {M}x{N}x{K}")
    rng = np.random.default_rng(K)
    # terms of one sign: every rounding is one of the whole partial sum
    ops = [np.abs(x) for x in _operands(torch, rng, "f32", M, N, K, 1, 2)]
    want = _product(ops)
    C = torch.empty((1, M, N), device="cuda")
    scratch = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    fd.testing_gemm_epilogue("f32", M, N, K, 1, 1, 1, *[_up(torch, x, True, "f32") for x in ops], C, scratch=scratch)
    rms = np.linalg.norm(C.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want)
    say(f"  rel L2 {rms:.2e}")
    # 256 additions of a part's leading products round by 2^-25 on average of a
    # sum that grows to 4096 terms, in one direction or the other: 2^-25 sqrt(256) at most
    assert rms <= 2.0 ** -25 * 16
