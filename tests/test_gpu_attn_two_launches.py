"""An unsplit attention call whose 256-row workgroups fill some rounds and a small part of another is launched in two
parts, by heads or by query rows: which calls are cut and where, and parity of both cuts with the oracle and with the
two calls that they stand for."""
import ctypes
import os
import subprocess

import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, MI355X_CUS, attn_errors, bits_of, to_dev_bf16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("cut") / "attn_cut.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2604_17397_amd", "csrc"), os.path.join(ROOT, "tests", "host", "attn_cut.cpp"),
                    "-o", out], check=True)
    lib = ctypes.CDLL(out)

    def call(H, n_q, n_k, n_items=1, n_cu=MI355X_CUS):
        r = (ctypes.c_double * 4)()
        lib.attn_cut(n_items, n_q, H, ctypes.c_int64(n_k), n_cu, r)
        return int(r[0]), int(r[1]), r[2], r[3]
    return call


def test_cut_by_size(cut):
    assert [cut(*a)[:2] for a in [(16, 4680, 14040), (14, 4680, 23400), (30, 3044, 12176)]] == [(13, 0), (13, 0), (21, 0)]
    assert cut(1, 65836, 1500)[:2] == (0, 65536) and cut(70, 410, 897, n_items=2)[:2] == (64, 0)
    # 256-row workgroups below or at whole rounds, or a last round more than half full: one launch
    for a in [(12, 4680, 14040), (18, 1800, 10800), (256, 200, 9000), (40, 4680, 32760), (20, 4680, 14040)]:
        assert cut(*a)[:2] == (0, 0), a
    assert cut(16, 4680, 14040, n_cu=0)[:2] == (0, 0)
    n_cut = 0
    for H in list(range(1, 41)) + [128, 255, 256, 257, 300, 1000]:
        for n_q in (1, 33, 256, 257, 312, 1031, 2048, 3100, 4680, 65535):
            for n_k in (n_q, 3 * n_q, 7 * n_q, 20000):
                for n_items in (1, 2, 8):
                    heads, rows, one, two = cut(H, n_q, n_k, n_items)
                    wgs = n_items * H * -(-n_q // 256)
                    if wgs <= MI355X_CUS or wgs % MI355X_CUS == 0:
                        assert (heads, rows) == (0, 0)
                    if heads or rows:
                        assert 0 <= heads < H and 0 <= rows < n_q and not (heads and rows) and rows % 256 == 0
                        first = n_items * (heads * -(-n_q // 256) if heads else H * (rows // 256))
                        assert first <= wgs // MI355X_CUS * MI355X_CUS and 1.02 * two + 8 < one + 1e-9
                        n_cut += 1
    assert n_cut > 100


def parts(cut, n_heads, n_q):
    heads, rows = cut[:2]
    return [(slice(0, heads or n_heads), slice(0, rows or n_q)), (slice(heads, n_heads), slice(rows, n_q))]


# (items, heads, queries, cached keys, block keys): by heads; with rows that end within a tile; two items; by rows, the
# rest 300 rows, no cache and a seam
@pytest.mark.gpu
@pytest.mark.parametrize("head_major", [False, True])
@pytest.mark.parametrize("n,H,n_q,c_len,n_blk", [(1, 139, 410, 487, 410), (1, 259, 183, 2000, 77), (2, 70, 410, 487, 410),
                                                 (1, 1, 65836, 0, 1500), (1, 1, 65836, 1001, 499)])
def test_both_cuts_match_the_oracle_and_their_parts(cut, n, H, n_q, c_len, n_blk, head_major):
    import paper_2604_17397_amd as P
    at = cut(H, n_q, c_len + n_blk, n)
    if torch.cuda.get_device_properties(0).multi_processor_count == MI355X_CUS:
        assert at[0] or at[1]
    sets, host = [], []
    for i in range(n):
        q, kc, vc, kb, vb = si.attn_inputs(H, max(n_q, n_blk), c_len, seed=700 + H + i, jitter=True, cache_capacity=max(c_len, 1))
        host.append((q[:n_q], kc, vc, kb[:n_blk], vb[:n_blk]))
        d = [to_dev_bf16(x) for x in host[-1]]
        if head_major:
            d = [x.transpose(0, 1).contiguous().transpose(0, 1) for x in d]
        sets.append(d)
    outs = [torch.full_like(d[0], float("nan")) for d in sets]
    P.block_attn_batch(*[list(x) for x in zip(*sets)], c_len, outs=outs)
    piecewise = [torch.full_like(d[0], float("nan")) for d in sets]
    for h, r in parts(at, H, n_q):
        P.block_attn_batch([d[0][r, h] for d in sets], *[[d[j][:, h] for d in sets] for j in range(1, 5)], c_len,
                           outs=[o[r, h] for o in piecewise])
    (_, h), (_, r) = [(0, s) for s in parts(at, H, n_q)[1]]
    rows = sorted({0, 31, 32, n_q - 1, max(r.start - 1, 0), r.start, min(r.start + 33, n_q - 1)})
    heads = sorted({0, max(h.start - 1, 0), h.start, H - 1})
    for o, w, x in zip(outs, piecewise, host):
        assert torch.equal(o, w)
        q, kc, vc, kb, vb = [t[:, heads] for t in x]
        max_abs, rel = attn_errors(bits_of(o[:, heads].contiguous())[rows], oracle.block_attn(q, kc, vc, kb, vb, c_len, rows=rows))
        assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,c_len,n_blk", [(139, 410, 487, 410), (1, 65836, 1001, 499)])
def test_commit_and_capture_of_a_cut_call(cut, H, n_q, c_len, n_blk):
    import paper_2604_17397_amd as P
    g = torch.Generator(device="cuda").manual_seed(5)
    mk = lambda t: torch.randn((t, H, 128), device="cuda", generator=g).bfloat16()
    q, kb, vb, kc, vc = mk(n_q), mk(n_blk), mk(n_blk), mk(c_len + n_blk + 3), mk(c_len + n_blk + 3)
    k0, v0, plain, out = kc.clone(), vc.clone(), torch.empty_like(q), torch.empty_like(q)
    P.block_attn(q, kc, vc, kb, vb, c_len, out=plain)
    P.block_attn_commit(q, kc, vc, kb, vb, c_len, out=out)
    assert torch.equal(out, plain)
    for cache, before, blk in ((kc, k0, kb), (vc, v0, vb)):
        assert torch.equal(cache[c_len:c_len + n_blk], blk)
        assert torch.equal(cache[:c_len], before[:c_len]) and torch.equal(cache[c_len + n_blk:], before[c_len + n_blk:])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.block_attn(q, kc, vc, kb, vb, c_len, out=out)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        assert torch.equal(out, plain)
        q.add_(0)  # work of another kind between the replays
