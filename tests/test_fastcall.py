"""The binding's plain calls in native code: what is not plain goes the Python way, and both ways give the same."""
import subprocess
import sys

import pytest
import torch

from paper_2604_27124_amd import binding as A
from paper_2604_27124_amd import build


def test_what_is_not_plain_is_left_to_python():
    fast = A._fastcalls()
    assert fast.__name__.endswith("_fastcall")                        # built, and bound to the loaded library
    x, n, b = torch.zeros(1, 8, 1, 64, dtype=torch.bfloat16), torch.zeros(1, dtype=torch.int32), torch.zeros(1)
    for args in ((x, x, x, n, b, 0.125), (x, x, x, n, b), (1, 2, 3, 4, 5, 6.0), (None,) * 6):
        assert fast.fwd(*args) is None and fast.bwd(args[0], *args) is None
    with pytest.raises(ValueError):
        A.sigmoid_attn_fwd(x, x, x, n, b, 0.125)


@pytest.mark.parametrize("lacks", ["torch", "g++"])
def test_the_library_builds_without_what_only_the_extension_needs(monkeypatch, tmp_path, capsys, lacks):
    made = []
    monkeypatch.setattr(build, "_compile", lambda lib, sources, verbose: made.append(lib) or lib)
    monkeypatch.setattr(build, "FASTCALL", str(tmp_path / "_fastcall.so"))
    (tmp_path / "_fastcall.so").write_text("of an earlier build")
    if lacks == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    else:
        monkeypatch.setattr(subprocess, "run", lambda cmd, **kw: (_ for _ in ()).throw(FileNotFoundError(cmd[0])))
    assert build.build_library() == build.LIB
    assert made == [build.PROBE_LIB, build.LIB] and not list(tmp_path.iterdir())
    assert "_fastcall.so was not built" in capsys.readouterr().err


def test_scratch_belongs_to_the_stream_it_is_used_on(monkeypatch):
    """Memory for a call is taken only where torch hands it out by the order of the stream the kernels run on."""
    from types import SimpleNamespace as NS
    made = []
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0, raising=False)
    monkeypatch.setattr(torch, "empty", lambda n, dtype, device: made.append((n, device)) or "memory")
    here, there = (NS(device=torch.device("cuda", i)) for i in (0, 1))
    for stream in (None, NS(cuda_stream=0)):                           # default streams of all devices have the same handle
        assert A._scratch(64, here, stream) == "memory" and A._scratch(64, there, stream) is None
    assert A._scratch(64, here, NS(cuda_stream=5)) is None             # torch does not know it
    assert made == [(64, here.device)] * 2


def test_workspaces_the_kernels_may_write_to():
    from types import SimpleNamespace as NS
    def tensor(**kw):
        t = dict(is_cuda=True, device=torch.device("cuda", 0), is_contiguous=lambda: True, data_ptr=lambda: 4096, numel=lambda: 10, element_size=lambda: 2)
        return NS(**{**t, **kw})
    q = tensor()
    assert A._workspace_args(tensor(), q) == (4096, 20)
    for bad in (None, torch.empty(1 << 20), torch.empty(1).expand(1 << 20), tensor(is_contiguous=lambda: False), tensor(device=torch.device("cuda", 1))):
        assert A._workspace_args(bad, q) == (0, 0)


@pytest.mark.gpu
def test_a_workspace_of_another_kind_is_left_alone():
    B, N, H = 16, 1030, 12
    need = A.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, H, 64)
    q, k, v, g = (torch.randn(B, N, H, 64, device="cuda").bfloat16() for _ in range(4))
    n, b = torch.full((B,), N, dtype=torch.int32, device="cuda"), torch.full((B,), -5.0, device="cuda")
    want = (A.sigmoid_attn_bwd_dq(q, k, v, g, n, b, 0.125), *A.sigmoid_attn_bwd_dkdv(q, k, v, g, n, b, 0.125))
    host, small = torch.full((need,), 3, dtype=torch.uint8), torch.full((256,), 3, dtype=torch.uint8, device="cuda")
    strided = torch.full((need, 2), 3, dtype=torch.uint8, device="cuda")
    for ws in (host, small[:1].expand(need), strided[:, 0]):
        got = A.sigmoid_attn_bwd(q, k, v, g, n, b, 0.125, workspace=ws)
        torch.cuda.synchronize()
        for x, y in zip(got, want):                                    # two passes, as without a workspace
            assert torch.equal(x.view(torch.int16), y.view(torch.int16))
    assert bool((host == 3).all()) and bool((small == 3).all()) and bool((strided == 3).all())


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,H,d", [(2, 256, 2, 64), (16, 1030, 12, 64), (3, 200, 2, 128)])      # pairs; one pass; d = 128
def test_same_results_as_the_python_way(B, N, H, d):
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, g = (torch.empty(B, N, H, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    n, b = torch.tensor([N - 3 * i for i in range(B)], dtype=torch.int32, device="cuda"), torch.full((B,), -5.0, device="cuda")
    stream = torch.cuda.current_stream()
    assert A._fastcalls().fwd(q, k, v, n, b, 0.125) is not None
    plain = (A.sigmoid_attn_fwd(q, k, v, n, b, 0.125), *A.sigmoid_attn_bwd(q, k, v, g, n, b, 0.125))
    other = (A.sigmoid_attn_fwd(q, k, v, n, b, 0.125, stream=stream), *A.sigmoid_attn_bwd(q, k, v, g, n, b, 0.125, stream=stream))
    for x, y in zip(plain, other):
        assert x.is_contiguous() and not x.requires_grad and torch.equal(x.view(torch.int16), y.view(torch.int16))
    # refused as before: shape, layout, type, a lengths tensor of another kind, an argument the library refuses
    for bad in ((q, k[:, :-1], v, n, b, 0.125), (q, k, v.transpose(1, 2).contiguous().transpose(1, 2), n, b, 0.125),
                (q.float(), k, v, n, b, 0.125), (q, k, v, n.long(), b, 0.125), (q, k, v, n, b[:-1], 0.125)):
        with pytest.raises(ValueError):
            A.sigmoid_attn_fwd(*bad)
    with pytest.raises(A.SigAttnError):
        A.sigmoid_attn_fwd(q, k, v, n, b, float("nan"))
    with pytest.raises(RuntimeError):                                  # a wrapped tensor has no memory to give
        torch.vmap(lambda t: A.sigmoid_attn_fwd(t, k, v, n, b, 0.125))(q[None])
    with torch.cuda.stream(torch.cuda.Stream()) as _:                  # the current stream, whichever it is
        torch.cuda.current_stream().wait_stream(stream)
        side = A.sigmoid_attn_fwd(q, k, v, n, b, 0.125)
    torch.cuda.synchronize()
    assert torch.equal(side.view(torch.int16), plain[0].view(torch.int16))
