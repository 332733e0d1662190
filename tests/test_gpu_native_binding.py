"""The C++ marshalling of the frequent calls against the Python code it stands in for: same results,
same errors, and forms it does not take (fp32, tensor subclasses, odd argument types) still work."""
import numpy as np
import pytest
import torch

import sdvg_inputs as si
from gpu_util import to_dev_bf16

pytestmark = pytest.mark.gpu


def tensors(H=3, T=40, c_len=33, extra=50):
    q, kc, vc, kb, vb = si.attn_inputs(H, T, c_len, seed=8, cache_capacity=c_len + extra)
    return [to_dev_bf16(a) for a in (q, kc, vc, kb, vb)] + [c_len]


def both(monkeypatch, call):
    """call() through the C++ marshalling (which has to take it) and through Python alone."""
    import paper_2604_17397_amd as P
    b = P.binding
    P.lib()
    assert b._NATIVE is not None
    taken = []

    class Spy:
        def __getattr__(self, name):
            def f(*args):
                r = getattr(native, name)(*args)
                taken.append(r is not None)
                return r
            return f
    native = b._NATIVE
    monkeypatch.setattr(b, "_NATIVE", Spy())
    got = call(P)
    monkeypatch.setattr(b, "_NATIVE", b._PythonOnly)
    want = call(P)
    monkeypatch.setattr(b, "_NATIVE", native)
    torch.cuda.synchronize()
    return got, want, taken


@pytest.mark.parametrize("form", ["new", "out", "no_cache", "scale", "stream", "head_major", "strided_out", "parameter"])
def test_attention_forms(monkeypatch, form):
    q, kc, vc, kb, vb, n = tensors()
    kw = {}
    if form == "no_cache":
        kc = vc = None
        n = 0
    if form == "scale":
        kw["scale"] = 0.2
    if form == "stream":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        kw["stream"] = side
    if form == "head_major":
        kc, vc = (t.transpose(0, 1).contiguous().transpose(0, 1) for t in (kc, vc))
    if form == "parameter":
        q = torch.nn.Parameter(q, requires_grad=True)

    def call(P):
        out = None
        if form == "out":
            out = torch.zeros_like(q)
        if form == "strided_out":
            out = torch.zeros((40, 3, 136), dtype=torch.bfloat16, device="cuda")[:, :, :128]
        r = P.block_attn(q, kc, vc, kb, vb, n, out=out, **kw)
        torch.cuda.synchronize()
        assert out is None or r is out
        assert not r.requires_grad
        return r
    got, want, taken = both(monkeypatch, call)
    assert taken == [True] and torch.equal(got, want) and got.stride() == want.stride()


def test_fused_commit_and_rope_and_route(monkeypatch):
    q, kc, vc, kb, vb, n = tensors()

    def commit(P):
        k, v = kc.clone(), vc.clone()
        return [P.block_attn_commit(q, k, v, kb, vb, n), k, v]
    got, want, taken = both(monkeypatch, commit)
    assert taken == [True] and all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(got, want))
    angle = torch.rand(40, 64, device="cuda") * 6
    got, want, taken = both(monkeypatch, lambda P: P.rope(q, angle.cos(), angle.sin()))
    assert taken == [True] and torch.equal(got, want)
    for scores in ([0.5, -0.2, 0.1], [0.5, float("nan")], [-0.0, 0.0], [float("inf"), float("-inf")]):
        s = torch.tensor(scores, device="cuda")
        for mode in ("min", "mean"):
            got, want, taken = both(monkeypatch, lambda P: P.worst_frame_route(s, -0.7, 3, mode=mode))
            assert taken == [True] and got[0] == want[0] and type(got[0]) is int
            assert type(got[1]) is type(want[1]) is np.float32 and got[1].view(np.uint32) == want[1].view(np.uint32)


def test_forms_left_to_python_still_work(monkeypatch):
    class Sub(torch.Tensor):
        pass
    q, kc, vc, kb, vb, n = tensors()
    for call in (lambda P: P.block_attn(q.as_subclass(Sub), kc, vc, kb, vb, n),
                 lambda P: P.block_attn(q, kc, vc, kb, vb, np.int64(n)),
                 lambda P: P.block_attn(q, kc, vc, kb, vb, n, scale=1),
                 lambda P: P.block_attn(q.float(), kc[:n].float(), vc[:n].float(), kb.float(), vb.float(), n)):
        got, want, taken = both(monkeypatch, call)
        assert taken == [False] and torch.equal(torch.as_tensor(got), torch.as_tensor(want))


def test_errors_are_those_of_the_python_code():
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb, n = tensors()
    for bad in (dict(cache_len=-1), dict(cache_len=1000), dict(v_cache=None), dict(k_blk=kb[:, :2]), dict(q=q.cpu()),
                dict(out=torch.zeros(40, 3, 128, device="cuda")), dict(v_blk=vb[:7]), dict(k_cache=None, v_cache=None)):
        args = dict(q=q, k_cache=kc, v_cache=vc, k_blk=kb, v_blk=vb, cache_len=n)
        args.update(bad)
        with pytest.raises(ValueError):
            P.block_attn(**args)
    with pytest.raises(ValueError):
        P.block_attn_commit(q, kc[:n + 3], vc[:n + 3], kb, vb, n)     # no room for the block
    with pytest.raises(P.SdvgError) as e:
        P.block_attn(q, kc, vc, kb, vb, n, scale=-1.0)
    assert e.value.status == -3
    with pytest.raises(P.SdvgError):
        P.worst_frame_route(torch.zeros(3, device="cuda"), float("nan"), 1)
    with pytest.raises(KeyError):
        P.worst_frame_route(torch.zeros(3, device="cuda"), 0.0, 1, mode="max")
    with pytest.raises(ValueError):
        P.rope(q, torch.zeros(39, 64, device="cuda"), torch.zeros(39, 64, device="cuda"))
