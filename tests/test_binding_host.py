"""Host side of the Python binding, without a GPU."""
import torch

from paper_2512_19720_amd import binding as pd


def test_prefill_workspace_belongs_to_the_device_whose_stream_runs_the_call(monkeypatch):
    """Kernels go to the current device's current stream.  Memory from another device's pool would go back to that
    pool when the call returns and could be handed out there while the kernel still runs here."""
    seen = []

    def empty(*args, **kw):
        seen.append(torch.device(kw["device"]))
        return "workspace"

    monkeypatch.setattr(torch, "empty", empty)

    assert pd._prefill_workspace(1024) == "workspace"
    assert seen == [torch.device("cuda")]                     # no index: the current device


def test_batch_workspace_rules():
    L, A, M = pd.lib(), 1 << 40, 1024
    GB = 1 << 30
    arr = (pd.Layer * 2)()
    for k, (d_out, d_in) in enumerate([(256, 640), (4096, 4096)]):
        base = A + k * 8 * GB
        arr[k] = pd.Layer(base, base + GB, base + 2 * GB, base + 3 * GB, base + 4 * GB, d_out, d_in, k, -1)
    assert L.pdelta_linear_batch_plan(arr, 2) == pd.OK
    need = L.pdelta_linear_batch_workspace_bytes(arr, 2, M, pd.F16)
    assert need == L.pdelta_linear_workspace_bytes(M, 4096, 4096, pd.F16) > 0
    assert L.pdelta_linear_batch_workspace_bytes(arr, 2, 16, pd.F16) == 0            # decode
    assert L.pdelta_linear_batch_workspace_bytes(None, 2, M, pd.F16) == 0

    def call(ws, n):
        return L.pdelta_linear_batch_ws(arr, A + 32 * GB, 2, M, pd.F16, pd.F16, ws, n, None)

    assert call(A + 33 * GB, need - 1) == pd.EWORKSPACE
    assert call(A + 33 * GB + 8, need) == pd.EALIGN
    assert call(None, need) == pd.EINVAL
    for k in range(5):
        assert call(A + 8 * GB + k * GB, need) == pd.EINVAL                          # on a tensor of the second layer


def test_a_decode_call_is_one_library_call(monkeypatch):
    """The smallest decode call is host time only: one call into the library and one look at each shape, whatever
    the prefill path needs beside that."""
    class FakeTensor:
        def __init__(self, *shape):
            self.size, self.dtype, self.is_cuda, self.reads = shape, torch.float16, True, 0

        @property
        def shape(self):
            self.reads += 1
            return self.size

        def dim(self):
            return len(self.size)

        def is_contiguous(self):
            return True

        def data_ptr(self):
            return 16

    calls = []

    class FakeLibrary:
        def __getattr__(self, name):
            return lambda *args: calls.append(name) or pd.OK

    monkeypatch.setattr(pd, "_lib", FakeLibrary())
    monkeypatch.setattr(pd, "_stream", lambda: 0)
    for fn in (pd.pdelta_linear_row, pd.pdelta_linear_col):
        X, W_b, Y = FakeTensor(4, 512), FakeTensor(256, 512), FakeTensor(4, 256)
        assert fn(X, W_b, FakeTensor(256, 16), FakeTensor(256), out=Y) is Y
        assert X.reads == 1 and W_b.reads == 1
    X, W_b, Y = FakeTensor(4, 512), FakeTensor(256, 512), FakeTensor(4, 256)
    assert pd.pdelta_linear_group(X, W_b, FakeTensor(256, 16), FakeTensor(256, 4), 128, out=Y) is Y
    assert X.reads == 1 and W_b.reads == 1
    assert calls == ["pdelta_linear_row", "pdelta_linear_col", "pdelta_linear_group"]
    del calls[:]                                              # a short prompt that uses no workspace: its size, then the same call
    pd.pdelta_linear_row(FakeTensor(65, 512), W_b, FakeTensor(256, 16), FakeTensor(256), out=FakeTensor(65, 256))
    pd.pdelta_linear_group(FakeTensor(65, 512), W_b, FakeTensor(256, 16), FakeTensor(256, 4), 128, out=FakeTensor(65, 256))
    assert calls == ["pdelta_linear_workspace_bytes", "pdelta_linear_row", "pdelta_linear_workspace_bytes", "pdelta_linear_group"]


def test_group_workspace_rules():
    L, A, GB = pd.lib(), 1 << 40, 1 << 30
    M, d_out, d_in = 1024, 4096, 4096
    need = L.pdelta_linear_workspace_bytes(M, d_out, d_in, pd.BF16)

    def call(ws=A + 5 * GB, n=need, group=128, shared=0, M=M):
        return L.pdelta_linear_group_ws(A, A + GB, A + 2 * GB, A + 3 * GB, group, shared, A + 4 * GB, M, d_out, d_in, pd.BF16, pd.F32,
                                        ws, n, None)

    assert call(n=need - 1) == pd.EWORKSPACE
    assert call(ws=A + 5 * GB + 4) == pd.EALIGN
    assert call(ws=None) == pd.EINVAL
    for k in range(5):
        assert call(ws=A + k * GB) == pd.EINVAL                          # on X, W_b, B_packed, v, Y
    # the last bytes of the tensors, whose sizes depend on the call: 4 bytes an output, 2 a scale
    assert call(ws=A + 4 * GB + M * d_out * 4 - 16) == pd.EINVAL
    assert call(ws=A + 3 * GB + d_out * (d_in // 128) * 2 - 16) == pd.EINVAL
    assert call(group=100) != pd.OK and call(group=3) != pd.OK           # refused with a workspace as without
    assert call(M=0) == pd.OK


def test_gradient_without_memory_for_the_parts(monkeypatch):
    """A call whose parts' sums cannot be allocated runs with the least workspace, as it did before parts were used."""
    M, d_out, d_in = 2048, 4096, 4096
    least, parts = (f(M, d_out, d_in, pd.ROW) for f in (pd.pdelta_grad_v_workspace_bytes, pd.pdelta_grad_v_split_workspace_bytes))
    assert parts > least
    X, dY, B = torch.zeros((M, d_in), dtype=torch.bfloat16), torch.zeros((M, d_out), dtype=torch.bfloat16), torch.zeros((d_out, d_in // 32), dtype=torch.int32)
    real, calls = torch.empty, []

    def empty(n, *args, **kw):
        if n == parts:
            raise torch.cuda.OutOfMemoryError("no memory for the parts")
        return real(n, *args, **kw)

    class Lib:
        def pdelta_grad_v_workspace_bytes(self, *args): return least
        def pdelta_grad_v_split_workspace_bytes(self, *args): return parts

        def pdelta_grad_v(self, *args):
            calls.append(args[-2])
            return pd.OK

    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(pd, "lib", lambda: Lib())
    monkeypatch.setattr(pd, "_dev", lambda t, name: t.data_ptr())
    monkeypatch.setattr(pd, "_stream", lambda: None)
    assert pd.pdelta_grad_v(X, dY, B, pd.ROW).shape == (d_out,)
    assert calls == [least]
