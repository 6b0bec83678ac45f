"""The C++ marshalling of the tensor functions against their Python checks:
the same outputs for what both take (given or allocated outputs and
workspaces, every option), the same errors for what they refuse, the current
stream, and calls from several threads."""

import threading

import numpy as np
import pytest
import torch

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import alibi_slopes, random_tensors

pytestmark = pytest.mark.gpu


def _qkv(B=2, Hq=4, Hkv=2, Lq=70, Lk=90, D=64, dt="f16"):
    return [t.cuda() for t in random_tensors([(B, Hq, Lq, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], dt, seed=5)]


def _in_python(monkeypatch, f):
    """f() with every call going through the Python checks and ctypes."""
    with monkeypatch.context() as m:
        m.setattr(pa, "_BINDING", pa._NotBuilt)
        return f()


FWD = [dict(), dict(causal=True), dict(causal=True, scale=0.3), dict(scale=1), dict(causal=True, softcap=5.0),
       dict(causal=True, softcap=5, window=20), dict(causal=True, softcap=0, window=0), dict(causal=1, window=True)]


@pytest.mark.parametrize("kw", FWD, ids=str)
@pytest.mark.parametrize("alibi", [False, True])
def test_prefill(monkeypatch, kw, alibi):
    q, k, v = _qkv()
    if alibi and kw.get("softcap"):
        alibi = False
    kw = dict(kw, alibi_slopes=alibi_slopes(4).cuda() if alibi else None)
    for fn in (pa.attn_fwd, pa.attn_fwd_mod):
        o = torch.full_like(q, float("nan"))
        a, b = fn(q, k, v, **kw), fn(q, k, v, o, **kw)
        c = _in_python(monkeypatch, lambda: fn(q, k, v, **kw))
        assert b is o and torch.equal(a, c) and torch.equal(b, c) and a.dtype == q.dtype


def test_decode_and_norms(monkeypatch):
    q, k, v = _qkv(Lq=1, Lk=700, D=128, dt="bf16")
    ws = torch.empty(1 << 16, dtype=torch.float32, device="cuda")
    for kw in (dict(), dict(num_splits=3), dict(scale=0.2, softcap=4.0), dict(alibi_slopes=alibi_slopes(4).cuda()),
               dict(workspace=ws)):
        for fn in (pa.attn_decode, pa.attn_decode_mod, pa.attn_decode_noalloc):
            if fn is pa.attn_decode_noalloc and "workspace" in kw:
                continue
            o = torch.full_like(q, float("nan"))
            a, b = fn(q, k, v, **kw), fn(q, k, v, o, **kw)
            c = _in_python(monkeypatch, lambda: fn(q, k, v, **kw))
            assert b is o and torch.equal(a, c) and torch.equal(b, c)
    for dt in (torch.float16, torch.bfloat16, torch.float32):
        x = torch.randn(40, 9000, device="cuda").to(dt)
        for kw in (dict(), dict(chunks=3), dict(workspace=ws)):
            out, y, m = torch.empty(40, device="cuda"), torch.empty_like(x), torch.empty(40, device="cuda")
            assert pa.norm_l2(x, out, **kw) is out
            yy, mm = pa.rmsnorm_rowmax(x, y, m, eps=1e-5, **kw)
            assert yy is y and mm is m
            y2, m2 = pa.rmsnorm_rowmax(x, eps=1e-5, **kw)
            y3, m3 = _in_python(monkeypatch, lambda: pa.rmsnorm_rowmax(x, eps=1e-5, **kw))
            n3 = _in_python(monkeypatch, lambda: pa.norm_l2(x, **kw))
            assert torch.equal(out, n3) and torch.equal(pa.norm_l2(x, **kw), n3)
            assert torch.equal(y, y3) and torch.equal(y2, y3) and torch.equal(m, m3) and torch.equal(m2, m3)


def test_what_is_refused_stays_refused(monkeypatch):
    q, k, v = _qkv()
    qd, x = q[:, :, :1].contiguous(), torch.randn(8, 64, device="cuda")
    bad = [
        lambda: pa.attn_fwd(q.cpu(), k, v), lambda: pa.attn_fwd(q.float(), k, v), lambda: pa.attn_fwd(q, k[:, :, :9], v),
        lambda: pa.attn_fwd(q.transpose(1, 2), k, v), lambda: pa.attn_fwd(q[0], k, v), lambda: pa.attn_fwd(q[:1], k, v),
        lambda: pa.attn_fwd(q, k.bfloat16(), v.bfloat16()), lambda: pa.attn_fwd(q, k, v, q[:, :, :5].contiguous()),
        lambda: pa.attn_fwd(q, k, v, scale=float("nan")), lambda: pa.attn_fwd(q, k, v, scale="a"),
        lambda: pa.attn_fwd(q, k, v, softcap=3.0), lambda: pa.attn_fwd(q, k, v, causal=True, softcap=-3.0),
        lambda: pa.attn_fwd(q, k, v, causal=True, window=-1), lambda: pa.attn_fwd(q, k, v, window=5),
        lambda: pa.attn_fwd(q, k, v, alibi_slopes=alibi_slopes(4)), lambda: pa.attn_fwd(q, k, v, alibi_slopes=alibi_slopes(3).cuda()),
        lambda: pa.attn_fwd(q[:, :, :0], k, v), lambda: pa.attn_fwd(q[..., :32].contiguous(), k[..., :32].contiguous(), v[..., :32].contiguous()),
        lambda: pa.attn_decode(q, k, v), lambda: pa.attn_decode(qd, k, v, num_splits=-1),
        lambda: pa.attn_decode(qd, k, v, num_splits=None), lambda: pa.attn_decode_noalloc(q, k, v),
        lambda: pa.attn_decode(qd, k, v, workspace=torch.empty(16, dtype=torch.uint8, device="cuda")),
        lambda: pa.attn_decode_noalloc(qd, k, v, num_splits=100000),
        lambda: pa.norm_l2(x.double()), lambda: pa.norm_l2(x[0]), lambda: pa.norm_l2(x.t()), lambda: pa.norm_l2(x.cpu()),
        lambda: pa.norm_l2(x[:, :62].contiguous()), lambda: pa.norm_l2(x, chunks=None), lambda: pa.norm_l2(x, chunks=-2),
        lambda: pa.norm_l2(x, torch.empty(7, device="cuda")), lambda: pa.rmsnorm_rowmax(x, x.half()),
        lambda: pa.rmsnorm_rowmax(x, eps=-1.0), lambda: pa.rmsnorm_rowmax(x, eps=None),
    ]
    for i, f in enumerate(bad):
        with pytest.raises(Exception) as here:
            f()
        with pytest.raises(Exception) as there:
            _in_python(monkeypatch, f)
        assert type(here.value) is type(there.value) and str(here.value) == str(there.value), (i, here.value, there.value)


def test_current_stream_and_threads():
    q, k, v = _qkv(Lq=300, Lk=300)
    ref = pa.attn_fwd(q, k, v, causal=True)
    torch.cuda.synchronize()
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                got[i] = pa.attn_fwd(q, k, v, causal=True)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(torch.equal(g, ref) for g in got)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    x = torch.randn(8, 4096, device="cuda")
    with torch.cuda.graph(g, stream=s):       # the call lands on the capturing stream
        y, m = pa.rmsnorm_rowmax(x)
    x.normal_()
    g.replay()
    torch.cuda.synchronize()
    y2, m2 = pa.rmsnorm_rowmax(x)
    assert torch.equal(y, y2) and torch.equal(m, m2)


def test_key_ranges_on_every_path(monkeypatch):
    """A call whose keys are divided over workgroups takes the same kernels,
    and so has the same bits, however it comes: marshalled in C++, through the
    Python checks, with a stream, with scalars of other types."""
    q, k, v = _qkv(B=1, Hq=8, Hkv=2, Lq=33, Lk=5000, D=128, dt="bf16")
    S = pa.load_library().attn_fwd_num_splits(1, 8, 2, 33, 5000, 128, 1, 0)
    assert S > 1
    ref = pa.attn_fwd(q, k, v, causal=True)
    one = torch.empty_like(q)                                # one range: other bits
    rc = pa.load_library().attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), one.data_ptr(), 1, 8, 2, 33, 5000, 128, 1,
                                    128 ** -0.5, None, 1, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and not torch.equal(ref, one)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    for fn in (pa.attn_fwd, pa.attn_fwd_mod):
        got = [_in_python(monkeypatch, lambda: fn(q, k, v, causal=True)), fn(q, k, v, causal=1),
               fn(q, k, v, causal=True, scale=np.float64(128 ** -0.5)), fn(q, k, v, causal=True, stream=s),
               fn(torch.nn.Parameter(q, requires_grad=False), k, v, causal=True)]
        s.synchronize()
        for i, g in enumerate(got):
            assert torch.equal(g, ref), i


def test_key_ranges_without_memory_in_python(monkeypatch):
    """The Python path does without the workspace too where it doesn't fit."""
    q, k, v = _qkv(B=1, Hq=8, Hkv=2, Lq=33, Lk=5000, D=128)
    ref = pa.attn_fwd(q, k, v, causal=True)
    empty, o = torch.empty, torch.empty_like(q)

    def refuse(*a, **kw):
        if kw.get("dtype") is torch.uint8:
            raise torch.cuda.OutOfMemoryError("no memory")
        return empty(*a, **kw)

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", refuse)
        _in_python(monkeypatch, lambda: pa.attn_fwd(q, k, v, o, causal=True))
    torch.cuda.synchronize()
    assert (o.float() - ref.float()).abs().max() < 2e-3 and not torch.equal(o, ref)


def test_workspaces_belong_to_the_stream_of_the_call(monkeypatch):
    """With stream= the workspace, which is dropped before the kernels have
    run, comes from that stream's pool: from another one it could be handed
    out again at once.  The results are those of plain calls."""
    q, k, v = _qkv(Lq=1, Lk=3000, D=128)
    x = torch.randn(8, 40000, device="cuda")
    calls = [lambda s: pa.attn_decode(q, k, v, stream=s), lambda s: pa.attn_decode_mod(q, k, v, softcap=5.0, stream=s),
             lambda s: pa.norm_l2(x, stream=s), lambda s: pa.rmsnorm_rowmax(x, stream=s)[0]]
    ref = [f(None) for f in calls]
    s, empty, seen = torch.cuda.Stream(), torch.empty, []

    def record(*a, **kw):
        if kw.get("dtype") is torch.uint8:
            seen.append(torch.cuda.current_stream())
        return empty(*a, **kw)

    s.wait_stream(torch.cuda.current_stream())
    with monkeypatch.context() as m:
        m.setattr(torch, "empty", record)
        got = [f(s) for f in calls]
    s.synchronize()
    assert seen == [s] * len(calls)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
