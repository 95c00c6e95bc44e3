"""CPU checks of how contractions are cut into parts (no call launches GPU work)."""
import pytest

fd = pytest.importorskip("paper_2602_00816_amd.fdhvp")

LONGEST = 128   # slices of 32 k in one part of an fp32 product


@pytest.mark.parametrize("K", [4096, 8192, 32000, 65536, 66000, 128256, 262136])
@pytest.mark.parametrize("M,N", [(64, 256), (512, 512), (512, 1024)])
def test_long_fp32_contractions_are_cut_to_the_limit(M, N, K):
    """With scratch for them, no part is longer than the limit, and the parts
    cover the contraction (two operand pairs, and one) without an empty one."""
    width, length, two, one = fd.testing_gemm_plan("f32", M, N, K, 1, 512 << 20)
    assert width in (64, 128)
    assert length <= LONGEST
    slices = (K + 31) // 32
    for parts, total in ((two, 2 * slices), (one, slices)):
        assert (parts - 1) * length < total <= parts * length


@pytest.mark.parametrize("K", [65536, 66000, 128256])
def test_small_scratch_still_cuts_where_that_is_faster(K):
    """512 x 512 outputs are 16 tiles on 256 CUs: with room for six parts of each
    product, which is too few for the limit, the contraction is still cut."""
    M = N = 512
    room = 12 * M * N * 4
    width, length, two, one = fd.testing_gemm_plan("f32", M, N, K, 1, room)
    assert length > LONGEST and two > 1
    assert (two + (one if one > 1 else 0)) * M * N * 4 <= room


def test_no_scratch_keeps_contractions_whole():
    for dtype in ("f32", "bf16"):
        assert fd.testing_gemm_plan(dtype, 512, 512, 128256)[2:] == (1, 1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(512, 3968), (4096, 512), (1504, 512), (28976, 2944)])
def test_one_plan_for_all_rows_of_a_tile_count(dtype, N, K):
    """The workspace reserves parts for one row count per 128-row tile count."""
    for tiles in (1, 2, 3, 5, 9):
        plans = {fd.testing_gemm_plan(dtype, 128 * tiles - cut, N, K, 1, 512 << 20) for cut in (0, 8, 56, 120)}
        assert len(plans) == 1, (tiles, plans)
