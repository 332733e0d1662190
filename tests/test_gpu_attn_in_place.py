"""Attention that writes its result over its query rows: on the CPU, that no two workgroups share query rows then; on the GPU,
the same bits as with an output of its own, for every kernel and way of launching."""
import pytest
import torch

from gpu_util import MI355X_CUS, attn_plan, attn_plan_halves


def test_no_shared_query_rows_in_place():
    packed = torch.empty((312, 3, 12, 128), dtype=torch.bfloat16)
    q, out = packed[:, 0], torch.empty((312, 12, 128), dtype=torch.bfloat16)
    assert attn_plan_halves(936, q, out) and attn_plan_halves(936, out, torch.empty_like(out))
    assert not attn_plan_halves(936, out, out) and not attn_plan_halves(936, q, q)
    both = torch.empty((2 * 312, 12, 128), dtype=torch.bfloat16)  # neighbours, and one row shared
    assert attn_plan_halves(936, both[:312], both[312:]) and attn_plan_halves(936, both[312:], both[:312])
    assert not attn_plan_halves(936, both[:312], both[311:623]) and not attn_plan_halves(936, both[311:623], both[:312])


# (items, heads, queries, cached keys, block keys), query rows per workgroup: each kernel, two workgroups per 32 rows with a
# separate output, two launches by heads and by rows (0), a key split (always)
CASES = [(1, 3, 300, 97, 83, 256), (1, 36, 460, 200, 100, 128), (1, 20, 500, 300, 100, 64), (1, 43, 97, 100, 160, 32),
         (1, 5, 300, 330, 300, 32), (1, 12, 33, 0, 312, 32), (2, 3, 129, 64, 257, 32), (1, 139, 410, 487, 410, 0),
         (1, 1, 65836, 1001, 499, 0), (1, 128, 40, 2100, 40, -1)]


@pytest.mark.gpu
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("n,H,n_q,c_len,n_blk,rows", CASES)
def test_out_is_q(n, H, n_q, c_len, n_blk, rows, packed):
    import paper_2604_17397_amd as P
    if rows > 0:
        assert attn_plan(H, n_q, c_len + n_blk, n, n_cu=MI355X_CUS).rows == rows
    g = torch.Generator(device="cuda").manual_seed(n_q + H)
    mk = lambda t: torch.randn((t, H, 128), device="cuda", generator=g).bfloat16()
    sets = [[mk(n_q), mk(c_len + n_blk), mk(c_len + n_blk), mk(n_blk), mk(n_blk)] for _ in range(n)]
    if packed:
        for s in sets:
            s[0] = torch.stack([s[0], torch.zeros_like(s[0])], 1)[:, 0]
    split, ws = "never", None
    if rows < 0:
        split, ws = "always", torch.empty(attn_plan(H, n_q, c_len + n_blk, n, split=2).workspace, dtype=torch.uint8, device="cuda")
        assert ws.numel() > 0
    lists = [list(x) for x in zip(*sets)]
    want = P.block_attn_batch(*lists, c_len, outs=[torch.empty((n_q, H, 128), dtype=torch.bfloat16, device="cuda") for _ in sets],
                              workspace=ws, split=split)
    if n == 1 and rows >= 0:  # the fused commit, on copies of the cache and the query
        q, kc, vc = sets[0][0].clone(), sets[0][1].clone(), sets[0][2].clone()
        assert torch.equal(P.block_attn_commit(q, kc, vc, *sets[0][3:], c_len, out=q), want[0])
        assert torch.equal(kc[c_len:], sets[0][3]) and torch.equal(vc[c_len:], sets[0][4])
    P.block_attn_batch(*lists, c_len, outs=lists[0], workspace=ws, split=split)
    for q, w in zip(lists[0], want):
        assert torch.equal(q, w)


@pytest.mark.gpu
def test_out_is_q_in_fp32():
    import paper_2604_17397_amd as P
    g = torch.Generator(device="cuda").manual_seed(2)
    q, kc, vc, kb, vb = (torch.randn((t, 3, 128), device="cuda", generator=g) for t in (200, 90, 90, 70, 70))
    want = P.block_attn(q, kc, vc, kb, vb, 90)
    assert torch.equal(P.block_attn(q, kc, vc, kb, vb, 90, out=q), want)
