"""Which prefill kernel the library takes, on both sides of the lines that were measured (no GPU needed): 64 and 65 the 64 x
64 tiles with a ring of steps and with roles, 128, 256 and 257 the 128 x 128 and 256 x 128 ones, 1000 + parts the 256 x 256 ones."""
import random

import pytest

from paper_2512_19720_amd import binding as pd

ROW, COL, GROUP = 0, 1, 2


def route(M, d_out, d_in, axis, dtype=pd.BF16, may_split=1):
    return pd.lib().pdelta_probe_prefill_kernel(M, d_out, d_in, dtype, axis, may_split)


# a step of the kernel with roles takes longer with column and blockwise scales, so those calls are split earlier than row
# calls: (row, column and blockwise)
@pytest.mark.parametrize("M,d_out,d_in,dtype,row,other", [
    (65, 3072, 8192, pd.F16, 65, 1016), (128, 3072, 8192, pd.F16, 65, 1016), (128, 4096, 8192, pd.F16, 65, 1016), (128, 4096, 8192, pd.BF16, 65, 1016),
    (128, 3072, 7168, pd.BF16, 65, 1014), (448, 2048, 8192, pd.BF16, 65, 1016), (128, 384, 5760, pd.F16, 65, 1015),
    (251, 4096, 4096, pd.F16, 65, 65), (100, 1024, 1024, pd.BF16, 65, 65), (256, 1024, 4096, pd.BF16, 65, 65), (128, 8192, 8192, pd.F16, 65, 65),
    (256, 512, 8192, pd.BF16, 1016, 1016), (256, 4096, 11008, pd.F16, 1015, 1015), (777, 4096, 11008, pd.BF16, 1004, 1004), (512, 4096, 4096, pd.F16, 1008, 1008)])
def test_split_or_roles(M, d_out, d_in, dtype, row, other):
    assert [route(M, d_out, d_in, axis, dtype) for axis in (ROW, COL, GROUP)] == [row, other, other]
    need = pd.lib().pdelta_linear_workspace_bytes(M, d_out, d_in, dtype)
    assert (need > 0) == (other > 1001)                                  # room for whichever kind of scales splits
    assert route(M, d_out, d_in, COL, dtype, 0) < 1002                   # the entry points without a workspace split nothing


@pytest.mark.parametrize("M,d_out,d_in,kernel", [
    (70, 11008, 4096, 64), (65, 130, 192, 64), (300, 300, 448, 64), (200, 100, 96, 256), (128, 100, 96, 128), (65, 8256, 128, 64), (65, 8192, 128, 65),
    (2048, 4096, 11008, 256), (2048, 11008, 4096, 1002), (4096, 4096, 4096, 1001), (129, 16512, 160, 256)])
def test_other_kernels(M, d_out, d_in, kernel):
    for axis in (ROW, COL, GROUP):
        assert route(M, d_out, d_in, axis) == kernel, axis


# more than one 64 x 64 tile per CU: the busiest CU's tiles count, not the tiles by 256 (312 and 405 tiles cost two whole ones)
@pytest.mark.parametrize("M,d_out,d_in,dtype,kernel", [
    (140, 6656, 8192, pd.BF16, 1008), (107, 8588, 15360, pd.F16, 1007), (488, 2104, 6656, pd.BF16, 1013), (196, 4384, 7936, pd.F16, 1013),
    (1117, 1024, 7808, pd.BF16, 1011), (284, 3328, 11264, pd.F16, 1009), (643, 1536, 7552, pd.F16, 1012), (65, 16320, 1024, pd.F16, 64)])
def test_more_tiles_than_cus(M, d_out, d_in, dtype, kernel):
    for axis in (ROW, COL, GROUP):
        assert route(M, d_out, d_in, axis, dtype) == kernel, axis


def test_workspace_holds_the_parts_of_every_kind_of_scales():
    """The size that callers ask for does not know the scales: whichever kinds split a call split it alike, and the size is
    that of its parts (256 x 256 fp32 sums each) where any of them does."""
    rng = random.Random(5)
    for _ in range(4000):
        M, d_out = (int(2 ** rng.uniform(lo, hi)) for lo, hi in ((6.03, 12.5), (5, 14.5)))
        d_in, dtype = 128 * rng.randint(1, 120), rng.choice((pd.F16, pd.BF16))
        kernels = [route(M, d_out, d_in, axis, dtype) for axis in (ROW, COL, GROUP)]
        parts = {k - 1000 for k in kernels if k > 1001}
        tiles = -(-M // 256) * -(-d_out // 256) % 256
        assert len(parts) <= 1, (M, d_out, d_in, dtype, kernels)
        need = pd.lib().pdelta_linear_workspace_bytes(M, d_out, d_in, dtype)
        assert need == sum(parts) * tiles * 256 * 256 * 4 and need <= 64 << 20, (M, d_out, d_in, dtype, kernels)


def test_argument_errors():
    probe = pd.lib().pdelta_probe_prefill_kernel
    assert probe(0, 64, 64, pd.F16, ROW, 0) == pd.EINVAL and probe(65, 64, 64, pd.F16, 3, 0) == pd.EINVAL and probe(65, 64, 64, pd.F16, ROW, 2) == pd.EINVAL
    assert probe(64, 64, 64, pd.F16, ROW, 0) == pd.ESHAPE and probe(65, 64, 48, pd.F16, ROW, 0) == pd.ESHAPE and probe(65, 64, 64, pd.F32, ROW, 0) == pd.EDTYPE


# the cases of the GPU tests that are there for one kernel reach it
@pytest.mark.parametrize("M,d_out,d_in,kernel", [
    (65, 128, 256, 65), (130, 257, 1024, 65), (300, 384, 512, 65), (200, 100, 96, 256), (65, 130, 192, 64), (100, 70, 448, 64), (300, 300, 320, 64)])
def test_blockwise_cases_of_the_gpu_tests(M, d_out, d_in, kernel):
    for dtype in (pd.F16, pd.BF16):
        assert route(M, d_out, d_in, GROUP, dtype) == kernel
