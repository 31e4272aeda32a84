"""The C++ half of the binding against its ctypes half: the same results for what it takes, and the
ctypes half's errors for what it does not."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa
from paper_2409_04431_amd import binding


class _CtypesOnly:
    """Stands in for the C++ half and takes nothing."""

    def __getattr__(self, name):
        return lambda *args: None


def _calls(g, layout):
    B, H, N, d, Hkv, Nk = 2, 4, 70, 64, 2, 1100
    # B, N, H, d views have permuted strides; the odd head stride of a slice leaves rows contiguous
    def t(h=H, n=N):
        x = torch.randn(B, n, h + 1, d, generator=g, device="cuda").bfloat16()[:, :, 1:]
        return x.transpose(1, 2) if layout == "bnhd" else x.transpose(1, 2).contiguous()
    q, k, v, do = (t() for _ in range(4))
    kg, vg, kl, vl = t(Hkv), t(Hkv), t(n=Nk), t(n=Nk)
    e = torch.empty_like
    f = lambda *s: torch.empty(*s, device="cuda")
    slopes = torch.rand(H, generator=g, device="cuda")
    pk = [torch.randn(N, H, d, generator=g, device="cuda").bfloat16() for _ in range(4)]
    cu = torch.tensor([0, 30, N], dtype=torch.int32, device="cuda")
    bv = torch.tensor([-3.0, -4.0], device="cuda")
    b = -math.log(N)
    yield lambda: [sa.sigmoid_attn_fwd(q, k, v, e(q), b, True, slopes)]
    yield lambda: sa.sigmoid_attn_bwd(q, k, v, do, e(q), e(k), e(v), b, 1)
    yield lambda: sa.sigmoid_attn_bwd_bias_grad(q, k, v, do, e(q), e(k), e(v), f(B, H, N), b, db=f(B, H))
    yield lambda: sa.sigmoid_attn_bwd_bias_grad(q, k, v, do, e(q), e(k), e(v), f(B, H, N), b)[:4]
    yield lambda: [sa.sigmoid_attn_varlen_fwd(*pk[:3], e(pk[0]), cu, 40, 0, True, slopes, bv)]
    yield lambda: sa.sigmoid_attn_varlen_bwd(*pk, *(e(x) for x in pk[:3]), cu, 40, b)
    yield lambda: sa.sigmoid_attn_varlen_bwd_bias_grad(*pk, *(e(x) for x in pk[:3]), f(H, N), cu, 40, b, bias_per_seq=bv, db=f(2, H))
    yield lambda: [sa.sigmoid_attn_mqa_fwd(q, kg, vg, e(q), b, True)]
    yield lambda: sa.sigmoid_attn_mqa_bwd_split(q, kg, vg, do, e(q), e(kg), e(vg), b, True)
    yield lambda: [sa.sigmoid_attn_cross_aligned_fwd(q[:, :, :1], kl, vl, e(q[:, :, :1]), b, False, slopes)]  # takes a workspace
    yield lambda: [sa.sigmoid_attn_cross_fwd(q, kl, vl, e(q), b)]
    def norm(kind):
        x, y, dx, st = q, e(q), e(q), f(B, N, 2)
        sa.sattn_headconcat_norm_fwd(x, y, st, kind=kind)
        sa.sattn_headconcat_norm_bwd(x, do, st, dx, kind=kind)
        return y, st, dx
    yield lambda: norm("layer")
    yield lambda: norm("rms")


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
def test_native_calls_equal_ctypes_calls(monkeypatch, layout):
    g = torch.Generator(device="cuda").manual_seed(5)
    sa.load_library()
    native = binding._native
    taken = []
    class Count:
        def __getattr__(self, name):
            def call(*args):
                rc = getattr(native, name)(*args)
                taken.append((name, rc))
                return rc
            return call
    for call in _calls(g, layout):
        monkeypatch.setattr(binding, "_native", Count())
        got = [x.clone() for x in call()]
        monkeypatch.setattr(binding, "_native", _CtypesOnly())
        for x, y in zip(got, call()):
            assert torch.equal(x, y)
    assert len(taken) == 15 and all(rc == 0 for _, rc in taken)


@pytest.mark.gpu
def test_what_the_native_half_does_not_take_raises_as_before():
    q = torch.zeros(1, 2, 8, 64, device="cuda", dtype=torch.bfloat16)
    ok = [q] * 4
    bad = [ok[:3] + [q.cpu()], ok[:3] + [q.float()], ok[:3] + [q[:, :1]], [q.transpose(2, 3)] * 4, [q.half()] * 4, [q[0]] * 4,
           [q[..., :32].contiguous()] * 4]
    for args in bad:
        with pytest.raises(sa.SattnError):
            sa.sigmoid_attn_fwd(*args, 0.0)
    for slopes in (torch.zeros(3, device="cuda"), torch.zeros(2), torch.zeros(2, device="cuda").double()):
        with pytest.raises(sa.SattnError):
            sa.sigmoid_attn_fwd(*ok, 0.0, False, slopes)
    with pytest.raises(ValueError):
        sa.sigmoid_attn_fwd(*ok, "x")
    with pytest.raises(KeyError):
        sa.sattn_headconcat_norm_fwd(q, q.clone(), torch.zeros(1, 8, 2, device="cuda"), kind="other")


def test_native_half_takes_no_cpu_tensor_and_no_other_object():
    sa.load_library()
    x = torch.zeros(1, 1, 4, 64)
    assert binding._native.fwd(x, x, x, x, 0.0, False, None) is None
    assert binding._native.fwd(1, x, None, "y", 0.0, False, None) is None
    with pytest.raises(TypeError):
        binding._native.fwd(x)


@pytest.mark.gpu
def test_calls_on_a_side_stream_and_under_capture():
    """The calls go to torch's current stream: captured there, every replay gives the eager result."""
    B, H, N, d = 2, 12, 333, 64
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v, do = (torch.randn(B, H, N, d, generator=g, device="cuda").bfloat16() for _ in range(4))
    kl, vl = (torch.randn(B, H, 1200, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    pk = [torch.randn(N, H, d, generator=g, device="cuda").bfloat16() for _ in range(4)]
    cu = torch.tensor([0, 100, N], dtype=torch.int32, device="cuda")
    e, f = torch.empty_like, lambda *s: torch.empty(*s, device="cuda")
    out = [e(q), e(q), e(q), e(q), e(q[:, :, :1]), e(q), f(B, N, 2)] + [e(x) for x in pk[:3]] + [f(B, H, N), f(B, H)]

    def work():
        o, dq, dk, dv, o1, y, st, pq, pk_, pv, rows, db = out
        sa.sigmoid_attn_fwd(q, k, v, o, -5.0, True)
        sa.sigmoid_attn_bwd_bias_grad(q, k, v, do, dq, dk, dv, rows, -5.0, True, db=db)
        sa.sigmoid_attn_cross_aligned_fwd(q[:, :, :1], kl, vl, o1, -7.0)   # takes a workspace
        sa.sattn_headconcat_norm_fwd(o, y, st)
        sa.sigmoid_attn_varlen_bwd(*pk, pq, pk_, pv, cu, 233, -5.0)

    work()
    torch.cuda.synchronize()
    want = [x.clone() for x in out]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for x in out:
            x.zero_()
        work()
    side.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(out, want))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        work()
    for _ in range(3):
        for x in out:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want))
        q.copy_(q.flip(0).contiguous())  # eager work between the replays, undone at once
        q.copy_(q.flip(0).contiguous())


def test_library_loads_without_the_native_half(monkeypatch):
    import sys
    sa.load_library()
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.delattr(sa, "_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2409_04431_amd._native", None)
    with pytest.warns(RuntimeWarning, match="C\\+\\+ half"):
        lib = sa.load_library()
    assert lib.sattn_version() == sa.sattn_version()
    with pytest.raises(sa.SattnError, match="must live on the GPU"):  # the ctypes half's checks answer
        x = torch.zeros(1, 1, 4, 64)
        sa.sigmoid_attn_fwd(x, x, x, x.clone(), 0.0)
