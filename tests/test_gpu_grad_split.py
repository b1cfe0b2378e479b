"""The 256 x 256 gradient kernel, whole and in parts of the contraction, at the edges of its tiles, steps and
parts, against the fp64 oracle under the rule of test_gpu_grad_v.py, and its workspace sizes."""
import pytest
import torch

from oracle import pdelta_oracle as orc
from paper_2512_19720_amd import binding as pd
from paper_2512_19720_amd import synth
from parity_util import to_dev, words_dev
from test_gpu_grad_v import check_grad, make


# one step pair; a short last group of signs (contraction % 256 = 128); tiles cut in both directions
@pytest.mark.gpu
@pytest.mark.parametrize("M,d_out,d_in", [(1, 128, 128), (257, 128, 384), (300, 384, 640), (64, 640, 1152)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("axis", [orc.ROW, orc.COL])
@pytest.mark.parametrize("parts", [1, 2, 3])
def test_whole_and_split_contraction(M, d_out, d_in, dtype, axis, parts, monkeypatch):
    monkeypatch.setenv("PDELTA_TUNE", f"grad_big={parts}")
    X, dY, B = make(M, d_out, d_in, dtype, 31 * M + d_in + parts)
    ref = orc.grad_v(X, dY, B, axis, dtype)
    got = pd.pdelta_grad_v(to_dev(X, dtype), to_dev(dY, dtype), words_dev(B), axis)
    check_grad(got, ref, f"grad big M={M} {d_out}x{d_in} dt={dtype} axis={axis} parts={parts}")


# the transposition of the signs, by ballots and (above 2^23 signs, from 2^24 on with d_out % 128 != 0) at the edges of its 128 x 2048 tiles (d_out % 128 != 0:
# rows of the result that are not 16-byte aligned), and sums over many partial rows (9 token tiles in 5 parts; 64 x 9 outputs of a reduction block)
@pytest.mark.gpu
@pytest.mark.parametrize("M,d_out,d_in", [(2, 4096, 2080), (1, 2080, 4128), (2, 128, 2048), (5, 288, 64), (2304, 640, 576), (2, 4160, 4064), (1, 2080, 8160)])
@pytest.mark.parametrize("axis", [orc.ROW, orc.COL])
def test_transposed_signs_and_many_partial_rows(M, d_out, d_in, axis):
    X, dY, B = make(M, d_out, d_in, synth.BF16, 5 * M + d_out + d_in)
    ref = orc.grad_v(X, dY, B, axis, synth.BF16)
    got = pd.pdelta_grad_v(to_dev(X, synth.BF16), to_dev(dY, synth.BF16), words_dev(B), axis)
    check_grad(got, ref, f"M={M} {d_out}x{d_in} axis={axis}")


# exactly the least workspace where the call would rather run in parts: the 256 x 128 kernel, which needs no more, and
# nothing behind the workspace is written; and a byte less than the parts take
@pytest.mark.gpu
@pytest.mark.parametrize("M,d_out,d_in", [(64, 128, 1024), (300, 640, 256), (513, 256, 384)])
@pytest.mark.parametrize("axis", [orc.ROW, orc.COL])
def test_least_workspace(M, d_out, d_in, axis):
    least, parts = (f(M, d_out, d_in, axis) for f in (pd.pdelta_grad_v_workspace_bytes, pd.pdelta_grad_v_split_workspace_bytes))
    X, dY, B = make(M, d_out, d_in, synth.BF16, 3 * M + d_out + d_in)
    ref = orc.grad_v(X, dY, B, axis, synth.BF16)
    Xd, dYd, Bd = to_dev(X, synth.BF16), to_dev(dY, synth.BF16), words_dev(B)
    for size in sorted({least, max(least, parts - 1), parts}):
        memory = torch.full((parts + 4096,), 0xCD, dtype=torch.uint8, device=Xd.device)
        got = pd.pdelta_grad_v(Xd, dYd, Bd, axis, workspace=memory[:size])
        torch.cuda.synchronize()
        check_grad(got, ref, f"workspace of {size} bytes M={M} {d_out}x{d_in} axis={axis}")
        assert bool((memory[size:] == 0xCD).all()), f"written behind a workspace of {size} bytes"


def test_split_workspace_sizes():
    L = pd.lib()
    assert L.pdelta_grad_v_split_workspace_bytes(256, 4096, 4096, pd.ROW) == 8 * 4096 * 4        # 16 tiles in 8 parts
    assert L.pdelta_grad_v_split_workspace_bytes(0, 64, 96, pd.ROW) == 64 * 4
    assert L.pdelta_grad_v_split_workspace_bytes(5, 0, 96, pd.ROW) == 0
    for M in (1, 64, 300, 2048, 4096):
        for d_out, d_in in ((32, 32), (256, 640), (4096, 4096), (14336, 4096), (4096, 11008)):
            for axis in (pd.ROW, pd.COL):
                assert L.pdelta_grad_v_split_workspace_bytes(M, d_out, d_in, axis) >= pd.pdelta_grad_v_workspace_bytes(M, d_out, d_in, axis)


def test_cases_of_the_least_workspace_would_run_in_parts():
    for M, d_out, d_in in ((64, 128, 1024), (300, 640, 256), (513, 256, 384)):
        for axis, k in ((pd.ROW, d_in), (pd.COL, d_out)):
            assert (pd.pdelta_grad_v_split_workspace_bytes(M, d_out, d_in, axis) > pd.pdelta_grad_v_workspace_bytes(M, d_out, d_in, axis)) == (k > 128)


def test_parts_of_few_tiles():
    """One to sixteen tokens, where the epilogue is short: sixteen parts for at most 128 workgroups, and the 256 x 128 kernel
    (no parts) for one or two units of the contraction, and for three to five where there is room for two parts only."""
    L = pd.lib()
    for M, d_out, d_in, axis, parts in ((1, 1024, 4096, pd.ROW, 16), (16, 8192, 1024, pd.COL, 16), (1, 2048, 8192, pd.ROW, 16), (1, 2560, 2560, pd.ROW, 10),
                                        (1, 3072, 8192, pd.ROW, 10), (16, 4096, 4096, pd.ROW, 8), (1, 512, 256, pd.ROW, 1), (16, 256, 512, pd.COL, 1),
                                        (17, 512, 256, pd.ROW, 2), (1, 512, 384, pd.ROW, 3),
                                        (1, 22784, 384, pd.ROW, 1), (16, 21888, 640, pd.ROW, 1), (17, 22784, 384, pd.ROW, 2), (16, 21760, 384, pd.ROW, 3),
                                        (16, 22784, 768, pd.ROW, 2)):
        n, signs = (d_out, 0) if axis == pd.ROW else (d_in, d_in * d_out // 8)
        assert L.pdelta_grad_v_split_workspace_bytes(M, d_out, d_in, axis) == parts * n * 4 + signs, (M, d_out, d_in, axis)
