"""Which decode kernel the library takes, on both sides of the lines that were measured (no GPU needed): 0 the register
kernel, 1 to 3 the one with direct loads and that many row tiles, 8 the staged one."""
import pytest

from paper_2512_19720_amd import binding as pd

ROW, COL, GROUP = 0, 1, 2


def route(M, d_out, d_in, axis, dtype=pd.BF16, group=128):
    return pd.lib().pdelta_probe_decode_kernel(M, d_out, d_in, dtype, axis, group)


# row scales, 5 to 16 tokens on many rows
@pytest.mark.parametrize("M,d_out,d_in,kernel", [
    (5, 11008, 4096, 0), (8, 12288, 4096, 0), (12, 12288, 4096, 0), (6, 14336, 2048, 0), (8, 16384, 2048, 0), (5, 28672, 8192, 0), (12, 32000, 4096, 0),
    (6, 10240, 6144, 0), (5, 6144, 4096, 0), (8, 12288, 11008, 0), (12, 10240, 512, 0), (6, 8192, 512, 0), (10, 18432, 6144, 0),
    (12, 11008, 4096, 3), (16, 12288, 4096, 3), (10, 14336, 2048, 2), (8, 6144, 2048, 2), (8, 10240, 8192, 3), (8, 5120, 5120, 2), (8, 14336, 512, 2), (8, 12288, 1024, 3),
    (16, 18432, 1024, 2), (16, 4096, 4096, 1), (1, 4096, 4096, 1), (4, 4097, 128, 0), (17, 8192, 4096, 2)])
def test_row_scales(M, d_out, d_in, kernel):
    for dtype in (pd.F16, pd.BF16):
        assert route(M, d_out, d_in, ROW, dtype) == kernel


# few inputs: one round of workgroups with up to three units, any scales
@pytest.mark.parametrize("M,d_out,d_in,kernel", [
    (1, 1152, 256, 0), (16, 4096, 384, 0), (16, 4096, 512, 1), (17, 4096, 256, 0), (17, 4096, 384, 1), (64, 1536, 128, 0), (64, 4112, 128, 2)])
def test_few_inputs(M, d_out, d_in, kernel):
    assert [route(M, d_out, d_in, axis, dtype) for axis in (ROW, COL, GROUP) for dtype in (pd.F16, pd.BF16)] == 6 * [kernel]


# row scales, rounds of workgroups that come out badly, and waves without a unit (other scales: the kernel with direct loads)
@pytest.mark.parametrize("M,d_out,d_in,row,other", [
    (16, 22784, 256, 0, 2), (16, 21760, 896, 2, 2), (12, 8605, 896, 3, 3), (8, 8192, 896, 0, 2), (6, 7680, 1152, 0, 2), (6, 7680, 1280, 2, 2),
    (6, 17408, 2688, 0, 2), (6, 20224, 4352, 0, 2), (8, 20736, 1024, 2, 2), (8, 11492, 7168, 3, 3), (5, 11904, 6784, 3, 3)])
def test_thin_rounds(M, d_out, d_in, row, other):
    assert [route(M, d_out, d_in, axis) for axis in (ROW, COL, GROUP)] == [row, other, other]


# column scales: one to three tokens on rows of 8 KB, one bf16 token on rows of 4 KB, two tiles that do not meet at one channel
@pytest.mark.parametrize("M,d_out,d_in,dtype,kernel", [
    (3, 8192, 4096, pd.BF16, 8), (3, 14336, 4096, pd.F16, 8), (3, 32000, 4096, pd.BF16, 8), (2, 8192, 4096, pd.F16, 8), (1, 14336, 2048, pd.BF16, 8),
    (1, 4096, 2048, pd.BF16, 8), (1, 2048, 2048, pd.BF16, 8), (1, 1024, 2048, pd.BF16, 1), (1, 4096, 2048, pd.F16, 1), (1, 2048, 4096, pd.BF16, 1),
    (3, 11008, 4096, pd.BF16, 3), (4, 8192, 4096, pd.BF16, 1), (4, 6144, 4096, pd.BF16, 2), (3, 8192, 6144, pd.BF16, 2), (3, 14336, 2048, pd.BF16, 2),
    (6, 20480, 4096, pd.BF16, 3), (6, 20480, 4096, pd.F16, 1), (2, 8192, 8192, pd.BF16, 1), (8, 23232, 9216, pd.F16, 2), (8, 14336, 10240, pd.BF16, 2)])
def test_column_scales(M, d_out, d_in, dtype, kernel):
    assert route(M, d_out, d_in, COL, dtype) == kernel


# blockwise scales (0: one scale per row)
@pytest.mark.parametrize("M,d_out,d_in,dtype,group,kernel", [
    (1, 8192, 4096, pd.BF16, 128, 8), (1, 32000, 4096, pd.BF16, 128, 8), (3, 32000, 4096, pd.BF16, 0, 8), (2, 14336, 4096, pd.F16, 0, 8),
    (1, 12288, 4096, pd.F16, 0, 8), (2, 8192, 6144, pd.BF16, 128, 8), (3, 28672, 6144, pd.F16, 128, 8), (1, 12288, 6144, pd.BF16, 0, 8),
    (1, 6144, 8192, pd.BF16, 128, 8), (1, 12288, 11008, pd.BF16, 128, 1),
    (2, 8192, 4096, pd.BF16, 128, 1), (1, 8192, 4096, pd.F16, 128, 1), (1, 32000, 4096, pd.F16, 128, 1), (1, 12288, 4096, pd.BF16, 128, 3),
    (2, 12288, 4096, pd.BF16, 0, 3), (1, 10240, 4096, pd.BF16, 0, 3), (1, 5120, 4096, pd.BF16, 128, 2), (3, 14336, 6144, pd.BF16, 128, 2),
    (1, 8192, 8192, pd.BF16, 128, 1), (1, 14336, 2048, pd.BF16, 128, 2), (1, 4096, 4096, pd.F16, 128, 1), (1, 8192, 4096 + 32, pd.F16, 32, 0)])
def test_blockwise_scales(M, d_out, d_in, dtype, group, kernel):
    assert route(M, d_out, d_in, GROUP, dtype, group or d_in) == kernel


def test_routes_that_do_not_fit_are_not_taken(monkeypatch):
    """A workgroup's LDS: a few long rows are never staged, and every route is one of the kernels."""
    for axis in (ROW, COL, GROUP):
        for dtype in (pd.F16, pd.BF16):
            for M in (1, 2, 3, 8, 16, 17, 64):
                for d_in in (32, 128, 4096, 8192, 28672, 1 << 22):
                    for d_out in (1, 4096, 6000, 8192, 12288, 1 << 22):
                        assert route(M, d_out, d_in, axis, dtype, 32) in (0, 1, 2, 3, 8)
                        if d_in > 28672:
                            assert route(M, d_out, d_in, axis, dtype, 32) < 8
    monkeypatch.setenv("PDELTA_TUNE", "skinny_staged=1")
    assert route(16, 64, 28672, COL) in (1, 2, 3) and route(1, 64, 4096, COL) == 8


def test_argument_errors():
    probe = pd.lib().pdelta_probe_decode_kernel
    assert probe(0, 64, 64, pd.F16, ROW, 0) == pd.EINVAL and probe(1, 64, 64, pd.F16, 3, 0) == pd.EINVAL
    assert probe(65, 64, 64, pd.F16, ROW, 0) == pd.ESHAPE and probe(1, 64, 48, pd.F16, ROW, 0) == pd.ESHAPE
    assert probe(1, 64, 128, pd.F16, GROUP, 48) == pd.ESHAPE and probe(1, 64, 128, pd.F32, ROW, 0) == pd.EDTYPE
