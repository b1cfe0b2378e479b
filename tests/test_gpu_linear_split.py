"""The 256 x 256 prefill kernel, whole tiles and tiles in parts of d_in, at the edges of its tiles, steps
and parts, against the fp64 oracle under the rule of parity_util.py, and its workspace rules."""
import pytest
import torch

from oracle import pdelta_oracle as orc
from paper_2512_19720_amd import binding as pd
from paper_2512_19720_amd import synth
from parity_util import DEV, check_y, f16_dev, gpu_linear, make_case

GB = 1 << 30


# one step pair; a short last group of signs (d_in % 256 = 128); tiles cut in both directions; parts of
# unequal length; more parts than the call has steps for fall back to whole tiles
@pytest.mark.gpu
@pytest.mark.parametrize("M,d_out,d_in", [(65, 40, 128), (256, 256, 256), (257, 300, 384), (300, 264, 640), (129, 513, 1152)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("parts", [1, 2, 3])
def test_whole_and_split_tiles(M, d_out, d_in, dtype, parts, monkeypatch):
    monkeypatch.setenv("PDELTA_TUNE", f"gemm_big={parts}")
    L = make_case(d_out, d_in, M, dtype, "row", 77 * M + d_out + d_in)
    d = L["d"]
    for axis, v_bits, v_dev in ((orc.ROW, L["v_row"], d["v_row"]), (orc.COL, L["v_col"], d["v_col"])):
        ref = orc.linear(L["X"], L["W_b"], L["B"], v_bits, axis, L["dtype"])
        for y in (torch.float32, torch.float16 if dtype == synth.F16 else torch.bfloat16):
            check_y(gpu_linear(axis, d["X"], d["W_b"], d["B"], v_dev, y), ref, f"big M={M} {d_out}x{d_in} dt={dtype} axis={axis} parts={parts}")


# an output of a whole tile is the same sum in the same order in every prefill kernel, and it is what the entry points
# without a workspace compute
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("M,d_out,d_in", [(300, 264, 640), (1024, 4096, 4096)])
def test_whole_tiles_have_the_bits_of_the_other_kernels(M, d_out, d_in, dtype, monkeypatch):
    L = make_case(d_out, d_in, M, dtype, "row", 31 * M + d_out)
    d = L["d"]
    for axis, v in ((orc.ROW, d["v_row"]), (orc.COL, d["v_col"])):
        got = []
        for tune in ("gemm_big=1", "gemm_big=0,gemm_small=0", "gemm_big=0,gemm_small=1"):
            monkeypatch.setenv("PDELTA_TUNE", tune)
            got.append(gpu_linear(axis, d["X"], d["W_b"], d["B"], v, torch.float32))
        monkeypatch.delenv("PDELTA_TUNE")
        Y = torch.full((M, d_out), float("nan"), dtype=torch.float32, device=DEV)
        fn = pd.lib().pdelta_linear_row if axis == orc.ROW else pd.lib().pdelta_linear_col
        assert fn(d["X"].data_ptr(), d["W_b"].data_ptr(), d["B"].data_ptr(), v.data_ptr(), Y.data_ptr(), M, d_out, d_in,
                  pd.F16 if dtype == synth.F16 else pd.BF16, pd.F32, torch.cuda.current_stream().cuda_stream) == pd.OK
        for other in got[1:] + [Y]:
            assert torch.equal(other, got[0]), f"axis={axis}"


# the 64 x 64 kernel with roles: one pair of steps, as many as are held in registers and in LDS, one more, and many; tiles
# cut in both directions; 35 tiles, whole columns of them per XCD, and 200, of which that would give one XCD 40.  Bit for bit the 256 x 256 kernel's whole tiles
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("M,d_out,d_in", [(65, 63, 128), (66, 65, 256), (128, 64, 384), (97, 130, 512), (129, 72, 640), (70, 200, 4224), (444, 300, 256), (1224, 628, 128)])
def test_roles_kernel(M, d_out, d_in, dtype, monkeypatch):
    L = make_case(d_out, d_in, M, dtype, "row", 11 * M + d_out + d_in)
    d = L["d"]
    v_bits = orc.pack_group(L["dW"], L["dW"] * 0, 32, False, dtype)[1]
    vg = f16_dev(v_bits)
    calls = [(lambda y: pd.pdelta_linear_row(d["X"], d["W_b"], d["B"], d["v_row"], out=y), lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_row"], orc.ROW, L["dtype"])),
             (lambda y: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], d["v_col"], out=y), lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_col"], orc.COL, L["dtype"])),
             (lambda y: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], vg, 32, out=y), lambda: orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, 32, dtype))]
    for k, (call, oracle) in enumerate(calls):
        ref = oracle()
        for y_dtype in (torch.float32, d["X"].dtype):
            got = []
            for tune in ("gemm_big=0,gemm_small=1,gemm_roles=1", "gemm_big=1"):
                monkeypatch.setenv("PDELTA_TUNE", tune)
                got.append(torch.full((M, d_out), float("nan"), dtype=y_dtype, device=DEV))
                call(got[-1])
            check_y(got[0], ref, f"roles kind {k} M={M} {d_out}x{d_in} dt={dtype}")
            assert torch.equal(got[0].view(torch.uint8), got[1].view(torch.uint8)), f"kind {k} M={M} {d_out}x{d_in} dt={dtype}"


@pytest.mark.gpu
@pytest.mark.parametrize("group,shared", [(32, False), (64, False), (128, True), (640, False), (640, True)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_blockwise_scales(group, shared, dtype, monkeypatch):
    M, d_out, d_in = 130, 264, 640
    L = make_case(d_out, d_in, M, dtype, "row", 9 + group)
    d = L["d"]
    _, v_bits = orc.pack_group(L["dW"], L["dW"] * 0, group, shared, dtype)
    v_dev = f16_dev(v_bits)
    ref = orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, group, dtype)
    for parts in (1, 2):
        monkeypatch.setenv("PDELTA_TUNE", f"gemm_big={parts}")
        Y = pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], v_dev, group, out_dtype=torch.float32)
        check_y(Y, ref, f"big group={group} shared={shared} dt={dtype} parts={parts}")


# parts that begin inside a group of scales: 1280 inputs in 3 parts begin at 384 and 768, 768 in 2 at 384, 1536 in 5 at
# 256, 512, 896 and 1152; at the groups' own ends: 1536 in 3 at 512 and 1024; and groups of 128, which no part cuts
@pytest.mark.gpu
@pytest.mark.parametrize("group,d_in,parts", [(256, 1280, 3), (256, 768, 2), (512, 1536, 5), (512, 1536, 3), (128, 640, 3)])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_parts_that_begin_inside_a_group(group, d_in, parts, shared, dtype, monkeypatch):
    M, d_out = 130, 264
    monkeypatch.setenv("PDELTA_TUNE", f"gemm_big={parts}")
    L = make_case(d_out, d_in, M, dtype, "row", 19 + group + d_in)
    d = L["d"]
    v_bits = orc.pack_group(L["dW"], L["dW"] * 0, group, shared, dtype)[1]
    # scales that differ from group to group by more than the tolerance: one taken from a neighbour shows
    v_dev = f16_dev(v_bits) * (1 + torch.arange(d_in // group, device=DEV) % 3).to(torch.float16)
    v_bits = synth.torch_to_bits(v_dev)
    Y = torch.full((M, d_out), float("nan"), dtype=torch.float32, device=DEV)
    pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], v_dev, group, out=Y)
    check_y(Y, orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, group, dtype), f"group={group} d_in={d_in} parts={parts} shared={shared}")


def test_workspace_rules_without_a_gpu():
    L = pd.lib()
    A = 1 << 40
    M, d_out, d_in = 1024, 4096, 4096                                   # 64 tiles in 4 parts
    need = L.pdelta_linear_workspace_bytes(M, d_out, d_in, pd.F16)
    assert need == 256 * 256 * 256 * 4
    assert L.pdelta_linear_workspace_bytes(64, d_out, d_in, pd.F16) == 0            # decode
    assert L.pdelta_linear_workspace_bytes(M, d_out, 4096 + 32, pd.F16) == 0        # another kernel's d_in
    assert L.pdelta_linear_workspace_bytes(M, d_out, 100, pd.F16) == 0 and L.pdelta_linear_workspace_bytes(M, d_out, d_in, pd.F32) == 0
    for m in (65, 251, 777, 2048, 4096):
        for o in (1, 256, 4096, 11008, 14336):
            for k in (128, 640, 4096, 11008):
                assert L.pdelta_linear_workspace_bytes(m, o, k, pd.BF16) <= 64 << 20

    def call(ws=A + 5 * GB, n=need, axis=pd.ROW):
        return L.pdelta_linear_ws(A, A + GB, A + 2 * GB, A + 3 * GB, axis, A + 4 * GB, M, d_out, d_in, pd.F16, pd.F16, ws, n, None)

    assert call(n=need - 1) == pd.EWORKSPACE
    assert call(ws=A + 5 * GB + 8) == pd.EALIGN
    assert call(ws=None) == pd.EINVAL
    for k in range(5):
        assert call(ws=A + k * GB) == pd.EINVAL                         # on X, W_b, B_packed, v, Y
    assert call(axis=2) == pd.EINVAL
    assert L.pdelta_linear_group_ws(A, A + GB, A + 2 * GB, A + 3 * GB, 128, 0, A + 4 * GB, M, d_out, d_in, pd.F16, pd.F16,
                                    A + 5 * GB, need - 1, None) == pd.EWORKSPACE


def test_small_grids_stay_with_the_small_tiles():
    """Few tiles in many parts were measured slower than the 64 x 64 kernel on the first shapes (26 against 35 us on
    256 x 1024 x 4096 fp16) and faster on the last ones (58 against 36 us on 256 x 512 x 8192 bf16)."""
    need = pd.lib().pdelta_linear_workspace_bytes
    for M, d_out, d_in in ((129, 1024, 4096), (200, 1024, 4096), (256, 1024, 4096), (256, 300, 3968), (512, 300, 3968), (251, 4096, 4096)):
        assert need(M, d_out, d_in, pd.F16) == 0, (M, d_out, d_in)
    assert need(256, 1024, 4096, pd.BF16) == 0
    for M, d_out, d_in in ((256, 512, 8192), (1024, 4096, 4096), (256, 4096, 11008), (777, 4096, 11008)):
        assert need(M, d_out, d_in, pd.F16) > 0 and need(M, d_out, d_in, pd.BF16) > 0, (M, d_out, d_in)
