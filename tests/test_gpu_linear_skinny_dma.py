"""The decode kernel with direct loads into LDS at the edges of its tiles (16 tokens; 16, 32, 48 output rows), units (128
inputs, dealt to 8 waves) and ring of stages, against the fp64 oracle under the rule of parity_util.py, and bit for bit
against the register-staged kernel, which adds the same sums in the same order."""
import pytest
import torch

from oracle import pdelta_oracle as orc
from paper_2512_19720_amd import binding as pd
from paper_2512_19720_amd import synth
from parity_util import DEV, check_y, f16_dev, make_case

pytestmark = pytest.mark.gpu


# one unit (seven waves without work); nine (one wave with two); 41 (a ring that wraps, waves of unequal length)
@pytest.mark.parametrize("M,d_out,d_in", [(1, 17, 128), (16, 49, 1152), (17, 33, 128), (32, 47, 5248), (33, 16, 1152), (48, 95, 640), (49, 50, 5248), (64, 96, 1152)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("rows", [1, 2, 3])
def test_row_and_token_tiles(M, d_out, d_in, dtype, rows, monkeypatch):
    L = make_case(d_out, d_in, M, dtype, "row", 3 * M + d_out + d_in)
    d = L["d"]
    kinds = [("row", d["v_row"], lambda v, y: pd.pdelta_linear_row(d["X"], d["W_b"], d["B"], v, out=y),
              lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_row"], orc.ROW, L["dtype"])),
             ("col", d["v_col"], lambda v, y: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], v, out=y),
              lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_col"], orc.COL, L["dtype"]))]
    for group, shared in ((32, False), (128, True), (d_in, True)):
        v_bits = orc.pack_group(L["dW"], L["dW"] * 0, group, shared, dtype)[1]
        kinds.append((f"group {group}", f16_dev(v_bits), lambda v, y, group=group: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], v, group, out=y),
                      lambda v_bits=v_bits, group=group: orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, group, dtype)))
    for name, v, call, oracle in kinds:
        ref = oracle()
        for y_dtype in (torch.float32, d["X"].dtype):
            Y, Z = (torch.full((M, d_out), float("nan"), dtype=y_dtype, device=DEV) for _ in range(2))
            monkeypatch.setenv("PDELTA_TUNE", f"skinny_dma={rows}")
            call(v, Y)
            monkeypatch.setenv("PDELTA_TUNE", "skinny_dma=0")
            call(v, Z)
            check_y(Y, ref, f"{name} M={M} {d_out}x{d_in} dt={dtype} rows={rows}")
            assert torch.equal(Y.view(torch.uint8), Z.view(torch.uint8)), f"{name} M={M} {d_out}x{d_in} dt={dtype} rows={rows}"


# an infinity or a NaN in one row of W_b, one token or one scale stays in the outputs that it belongs to
@pytest.mark.parametrize("M", [5, 40])
def test_infinities_stay_in_their_outputs(M, monkeypatch):
    d_out, d_in = 70, 384
    L = make_case(d_out, d_in, M, synth.BF16, "row", 8)
    d = L["d"]
    W, X, v = d["W_b"].clone(), d["X"].clone(), d["v_row"].clone()
    W[-1, 200], X[-1, 5], v[3] = float("inf"), float("nan"), float("inf")
    got = []
    for tune in ("skinny_dma=3", "skinny_dma=0"):
        monkeypatch.setenv("PDELTA_TUNE", tune)
        got.append(pd.pdelta_linear_row(X, W, d["B"], v, out_dtype=torch.float32))
    finite = torch.ones((M, d_out), dtype=torch.bool, device=DEV)
    finite[:, -1], finite[-1, :], finite[:, 3] = False, False, False
    assert torch.equal(torch.isfinite(got[0]), finite) and torch.equal(torch.nan_to_num(got[0]), torch.nan_to_num(got[1]))


# a few tokens on more than 4096 outputs, and row scales on rows of 8 KB, run the register kernels: the same sums
@pytest.mark.parametrize("M,d_out,d_in", [(1, 4097, 128), (2, 4112, 1152), (3, 4097, 640), (4, 4100, 256), (5, 4100, 256), (2, 4097, 8064), (9, 8190, 4096), (16, 5121, 4096)])
@pytest.mark.parametrize("axis", ["row", "col"])
def test_routes_of_few_tokens(M, d_out, d_in, axis, monkeypatch):
    g = torch.Generator(device=DEV).manual_seed(M + d_out + d_in)
    X = torch.randn((M, d_in), device=DEV, generator=g).half()
    W = torch.randn((d_out, d_in), device=DEV, generator=g).half()
    B = torch.randint(-2**31, 2**31, (d_out, d_in // 32), device=DEV, generator=g, dtype=torch.int64).to(torch.int32)
    v = torch.rand(d_out if axis == "row" else d_in, device=DEV, generator=g).half()
    call = pd.pdelta_linear_row if axis == "row" else pd.pdelta_linear_col
    here = call(X, W, B, v, out_dtype=torch.float32)
    monkeypatch.setenv("PDELTA_TUNE", "skinny_dma=1")
    assert torch.equal(here, call(X, W, B, v, out_dtype=torch.float32))


# the staged kernel (column and blockwise scales): one unit, seven waves without work; rows past the end; the same sums in
# the same order as the kernel with direct loads
@pytest.mark.parametrize("M,d_out,d_in", [(1, 17, 128), (2, 49, 1152), (3, 33, 4096), (4, 16, 640), (1, 15, 8192)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_staged_kernel(M, d_out, d_in, dtype, monkeypatch):
    L = make_case(d_out, d_in, M, dtype, "row", 5 * M + d_out + d_in)
    d = L["d"]
    calls = [("col", lambda y: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], d["v_col"], out=y),
              lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_col"], orc.COL, L["dtype"]))]
    for group, shared in ((32, False), (128, True), (d_in, False)):
        v_bits = orc.pack_group(L["dW"], L["dW"] * 0, group, shared, dtype)[1]
        v = f16_dev(v_bits)
        calls.append((f"group {group}", lambda y, v=v, group=group: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], v, group, out=y),
                      lambda v_bits=v_bits, group=group: orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, group, dtype)))
    for name, call, oracle in calls:
        ref = oracle()
        for y_dtype in (torch.float32, d["X"].dtype):
            got = []
            for tune in ("skinny_staged=1", "skinny_dma=1"):
                monkeypatch.setenv("PDELTA_TUNE", tune)
                got.append(torch.full((M, d_out), float("nan"), dtype=y_dtype, device=DEV))
                call(got[-1])
            check_y(got[0], ref, f"staged {name} M={M} {d_out}x{d_in} dt={dtype}")
            assert torch.equal(got[0].view(torch.uint8), got[1].view(torch.uint8)), f"staged {name} M={M} {d_out}x{d_in} dt={dtype}"
