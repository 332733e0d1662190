"""The C++ marshalling of the batched attention call, commit, rollback and snapshot against the Python code it stands in
for: same results, same errors, and the forms it leaves to Python still work."""
import numpy as np
import pytest
import torch

from test_gpu_native_binding import both, tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["new", "outs", "tuples", "no_cache", "scale", "stream", "workspace", "static", "one_item"])
def test_batch_forms(monkeypatch, form):
    items = [tensors() for _ in range(1 if form == "one_item" else 3)]
    lists = [[it[i] for it in items] for i in range(5)]
    n, kw = items[0][5], {}
    if form == "tuples":
        lists = [tuple(x) for x in lists]
    if form == "no_cache":
        lists[1] = lists[2] = None
        n = 0
    if form == "scale":
        kw["scale"] = 0.2
    if form == "stream":
        kw["stream"] = torch.cuda.Stream()
        kw["stream"].wait_stream(torch.cuda.current_stream())
    if form == "workspace":  # of another type, too small: the plain launch
        kw.update(workspace=torch.empty(16, dtype=torch.float64, device="cuda"), split="always")

    def call(P):
        outs = [torch.zeros_like(q) for q in lists[0]] if form in ("outs", "static") else None
        f = P.block_attn_batch_static if form == "static" else P.block_attn_batch
        r = f(*lists, n, outs=outs, **kw)
        torch.cuda.synchronize()
        assert type(r) is list and (outs is None or r is outs)
        return r
    got, want, taken = both(monkeypatch, call)
    assert taken == [True] and len(got) == len(want) == len(items)
    assert all(torch.equal(a, b) and a.stride() == b.stride() for a, b in zip(got, want))


def test_batch_with_a_split(monkeypatch):
    import paper_2604_17397_amd as P
    d = [torch.randn(33, 4, 128, device="cuda").bfloat16() for _ in range(3)] + \
        [torch.randn(65500, 4, 128, device="cuda").bfloat16() for _ in range(2)]
    args = [[d[0]], [d[3]], [d[4]], [d[1]], [d[2]], 65500]
    ws = torch.empty(P.block_attn_workspace_bytes(d[0], d[3], d[4], d[1], d[2], 65500, split="always"), dtype=torch.uint8, device="cuda")
    got, want, taken = both(monkeypatch, lambda P: P.block_attn_batch(*args, workspace=ws, split="always")[0])
    assert taken == [True] and torch.equal(got, want) and not torch.equal(got, P.block_attn_batch(*args)[0])


def cache_calls(P, head_major):
    L, T, H = 3, 17, 2
    shape = (L, H, 3 * T, 128) if head_major else (L, 3 * T, H, 128)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k, v = (torch.randn(shape, generator=gen, device="cuda").bfloat16() for _ in range(2))
    kv = [t.transpose(1, 2) for t in (k, v)] if head_major else [k, v]
    kb, vb = (torch.randn((L, T, H, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    angle = torch.rand((T, 64), generator=gen, device="cuda") * 6
    cache = P.KVCache(*kv, T, cache_len=T)
    P.kv_commit(cache, kb, vb, 1)
    P.kv_commit_rope(cache, kb, vb, 2, angle.cos(), angle.sin())
    lens = [cache.cache_len]
    snap = torch.zeros(k.numel() * 2 + 5, dtype=torch.uint8, device="cuda")
    P.buffer_snapshot(snap, k)
    P.buffer_snapshot(snap[3 * 16:], v, n_bytes=37)
    P.kv_rollback(cache, 2 * T)
    return [k, v, snap.view(torch.uint8), torch.tensor(lens + [cache.cache_len])]


@pytest.mark.parametrize("head_major", [False, True])
def test_cache_calls(monkeypatch, head_major):
    got, want, taken = both(monkeypatch, lambda P: cache_calls(P, head_major))
    assert taken == [True] * 5
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b)


def test_forms_left_to_python(monkeypatch):
    q, kc, vc, kb, vb, n = tensors()
    one = ([q], [kc], [vc], [kb], [vb])
    for call in (lambda P: P.block_attn_batch(*one, np.int64(n))[0], lambda P: P.block_attn_batch(*one, n, scale=1)[0],
                 lambda P: P.block_attn_batch(*([x[0].float()] for x in one[:1]), [kc.float()], [vc.float()], [kb.float()], [vb.float()], n)[0]):
        got, want, taken = both(monkeypatch, call)
        assert taken == [False] and torch.equal(got, want)

    def snapshot(P):
        dst = torch.zeros(64, dtype=torch.uint8, device="cuda")
        P.buffer_snapshot(dst, torch.arange(64, dtype=torch.uint8, device="cuda"), n_bytes=np.int64(33))
        return dst
    got, want, taken = both(monkeypatch, snapshot)
    assert taken == [False] and torch.equal(got, want) and int(got[32]) == 32 and int(got[33]) == 0


def test_errors_are_those_of_the_python_code():
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb, n = tensors()
    one = dict(qs=[q], k_caches=[kc], v_caches=[vc], k_blks=[kb], v_blks=[vb], cache_len=n)
    for bad in (dict(v_blks=[]), dict(k_blks=[kb[:, :2]]), dict(cache_len=1000), dict(qs=[q.cpu()]), dict(workspace=q.cpu()),
                dict(workspace=torch.zeros(8, 8, device="cuda")[:, :4]), dict(outs=[kb[:7]])):
        with pytest.raises(ValueError):
            P.block_attn_batch(**{**one, **bad})
    with pytest.raises(KeyError):
        P.block_attn_batch(**one, split="sometimes")
    with pytest.raises(P.SdvgError) as e:
        P.block_attn_batch(**one, scale=-1.0)
    assert e.value.status == -3 and "sdvg_block_attn_batch failed" in str(e.value)
    L, T, H = 2, 8, 2
    k, v, b = (torch.zeros((L, t, H, 128), dtype=torch.bfloat16, device="cuda") for t in (2 * T, 2 * T, T))
    cache = P.KVCache(k, v, T)
    for call, error in ((lambda: P.kv_commit(cache, b[:, :4], b, 0), ValueError), (lambda: P.kv_commit(cache, b.float(), b.float(), 0), TypeError),
                        (lambda: P.kv_commit(cache, b, b, 1), P.SdvgError), (lambda: P.kv_rollback(cache, 1), P.SdvgError),
                        (lambda: P.kv_commit_rope(cache, b, b, 0, torch.zeros(T, 63, device="cuda"), torch.zeros(T, 64, device="cuda")), ValueError),
                        (lambda: P.buffer_snapshot(b[:, :, :1], k), ValueError), (lambda: P.buffer_snapshot(b, k), ValueError),
                        (lambda: P.buffer_snapshot(b, k, n_bytes=-1), P.SdvgError)):
        with pytest.raises(error):
            call()
    assert cache.cache_len == 0
