"""A prefill call has the same bits whether or not there is memory for the parts' sums, and without it they are
within the rule of parity_util.py of the fp64 oracle."""
import pytest
import torch

from oracle import pdelta_oracle as orc
from paper_2512_19720_amd import binding as pd
from paper_2512_19720_amd import synth
from parity_util import DEV, check_y, f16_dev, make_case

pytestmark = pytest.mark.gpu


def without_memory(monkeypatch, fn):
    """fn() while every allocation of a workspace fails."""
    real, refused = torch.empty, []

    def empty(*args, **kw):
        if kw.get("dtype") == torch.uint8:
            refused.append(args)
            raise torch.cuda.OutOfMemoryError("no memory for the workspace")
        return real(*args, **kw)

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", empty)
        Y = fn()
    return Y, len(refused)


# one part per unit of 128 inputs; parts of unequal length; tiles cut in both directions; (1024, 4096, 4096) is the
# library's own choice of 4 parts
@pytest.mark.parametrize("M,d_out,d_in,parts", [(256, 256, 256, 2), (300, 264, 640, 3), (130, 513, 1152, 5), (1024, 4096, 4096, 0)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_same_bits_without_memory(M, d_out, d_in, parts, dtype, monkeypatch):
    if parts:
        monkeypatch.setenv("PDELTA_TUNE", f"gemm_big={parts}")
    L = make_case(d_out, d_in, M, dtype, "row", 5 * M + d_out + d_in)
    d = L["d"]
    vg = torch.rand((d_out, d_in // 128), device=DEV).mul_(2e-3).sub_(1e-3).to(torch.float16)
    calls = [lambda y: pd.pdelta_linear_row(d["X"], d["W_b"], d["B"], d["v_row"], out_dtype=y),
             lambda y: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], d["v_col"], out_dtype=y),
             lambda y: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], vg, 128, out_dtype=y)]
    for k, call in enumerate(calls):
        for y in (torch.float32, d["X"].dtype):
            want = call(y)
            got, refused = without_memory(monkeypatch, lambda: call(y))
            assert refused == 1
            assert torch.equal(got.view(torch.uint8), want.view(torch.uint8)), f"kind {k} {M}x{d_out}x{d_in} dt={dtype} y={y}"


# 289 tiles: a whole round of 256 and 33 tiles in parts
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
def test_whole_round_and_split_rest(dtype, monkeypatch):
    M, d_out, d_in = 4200, 4200, 384
    monkeypatch.setenv("PDELTA_TUNE", "gemm_big=2")
    L = make_case(d_out, d_in, M, dtype, "row", 4242)
    d = L["d"]
    _, v_bits = orc.pack_group(L["dW"], L["dW"] * 0, 128, False, dtype)
    vg = f16_dev(v_bits)
    calls = [(lambda: pd.pdelta_linear_row(d["X"], d["W_b"], d["B"], d["v_row"], out_dtype=torch.float32),
              lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_row"], orc.ROW, L["dtype"])),
             (lambda: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], d["v_col"], out_dtype=torch.float32),
              lambda: orc.linear(L["X"], L["W_b"], L["B"], L["v_col"], orc.COL, L["dtype"])),
             (lambda: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], vg, 128, out_dtype=torch.float32),
              lambda: orc.linear_group(L["X"], L["W_b"], L["B"], v_bits, 128, dtype))]
    for k, (call, oracle) in enumerate(calls):
        ref = oracle()
        want = call()
        check_y(want, ref, f"289 tiles, kind {k}, dt={dtype}")
        got, refused = without_memory(monkeypatch, call)
        assert refused == 1 and torch.equal(got, want), f"kind {k} dt={dtype}"


def test_a_callers_workspace(monkeypatch):
    """The caller's workspace is the one that is used, nothing is allocated beside it, and an empty one asks for none."""
    M, d_out, d_in = 1024, 4096, 4096
    L = make_case(d_out, d_in, M, synth.F16, "row", 99)
    d = L["d"]
    vg = torch.full((d_out, d_in // 128), 1e-3, dtype=torch.float16, device=DEV)
    need = pd.pdelta_linear_workspace_bytes(M, d_out, d_in, torch.float16)
    own, none = torch.empty(need, dtype=torch.uint8, device=DEV), torch.empty(0, dtype=torch.uint8, device=DEV)
    plan = pd.pdelta_linear_batch_plan([(d["X"], d["W_b"], d["B"], d["v_row"], pd.ROW)])
    assert pd.pdelta_linear_batch_workspace_bytes(plan) == need
    Y = torch.empty((M, d_out), dtype=torch.float16, device=DEV)
    for call in (lambda ws: pd.pdelta_linear_row(d["X"], d["W_b"], d["B"], d["v_row"], out=Y, workspace=ws),
                 lambda ws: pd.pdelta_linear_col(d["X"], d["W_b"], d["B"], d["v_col"], out=Y, workspace=ws),
                 lambda ws: pd.pdelta_linear_group(d["X"], d["W_b"], d["B"], vg, 128, out=Y, workspace=ws),
                 lambda ws: pd.pdelta_linear_batch(plan, workspace=ws)[0]):
        want = call(None).clone()
        for ws in (own, none):
            own.zero_()
            got, refused = without_memory(monkeypatch, lambda: call(ws))
            assert refused == 0 and torch.equal(got, want)
            assert bool(own.any()) == (ws is own)
        with pytest.raises(pd.PdeltaError) as e:
            call(own[:need - 16])
        assert e.value.status == pd.EWORKSPACE
