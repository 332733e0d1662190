"""GPU parity of the key split's merge kernel where its pieces can go wrong: many pieces per query
tile (more than the loops are unrolled by), query tiles of unequal and of partly filled wave tiles,
query tiles that one workgroup finished beside others that need the merge."""
import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, attn_errors, bits_of, to_dev_bf16

pytestmark = pytest.mark.gpu


# (heads, queries, cached keys): 64 pieces of 16 key tiles; 2 query tiles with a last row of its own
# and some 42 pieces; 9 wave tiles over 2 query tiles; 260 query tiles over two rounds
@pytest.mark.parametrize("H,n_q,c_len", [(4, 33, 65500), (3, 257, 45003), (7, 270, 20011), (130, 257, 2000)])
def test_merge_matches_oracle_and_unsplit(H, n_q, c_len):
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb = si.attn_inputs(H, n_q, c_len, seed=500 + H, jitter=True, cache_capacity=c_len)
    d = [to_dev_bf16(x) for x in (q, kc, vc, kb, vb)]
    need = P.block_attn_workspace_bytes(*d, c_len, split="always")
    assert need > 0
    # whatever is read without having been written shows: NaN bits in the whole workspace
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.full_like(d[0], float("nan"))
    P.block_attn_batch(*[[x] for x in d], c_len, outs=[out], workspace=ws, split="always")
    torch.cuda.synchronize()
    rows = sorted({0, 1, 31, 32, n_q // 2, n_q - 2, n_q - 1})
    ref = oracle.block_attn(q, kc, vc, kb, vb, c_len, rows=rows)
    max_abs, rel = attn_errors(bits_of(out)[rows], ref)
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)
    # all rows: two roundings to bf16 of the same value, of P and of the result, apart
    plain = P.block_attn(*d, c_len).float()
    assert ((out.float() - plain).norm() / plain.norm()).item() <= 2 * BF16_REL_RMS


# AUTO between the key split and key groups inside the workgroup: many keys for few rows are split,
# a nearly full round of workgroups with few keys is not; both ask for the split's workspace.
@pytest.mark.parametrize("H,n_q,c_len,same_as", [(4, 33, 65500, "always"), (16, 1031, 2062, "never")])
def test_auto_takes_the_faster_plan(H, n_q, c_len, same_as):
    import paper_2604_17397_amd as P
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, kb, vb = (torch.randn((n_q, H, 128), generator=gen, device="cuda").bfloat16() for _ in range(3))
    kc, vc = (torch.randn((c_len, H, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    d = (q, kc, vc, kb, vb)
    need = P.block_attn_workspace_bytes(*d, c_len, split="auto")
    assert need == P.block_attn_workspace_bytes(*d, c_len, split="always") > 0
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = {m: P.block_attn_batch(*[[x] for x in d], c_len, workspace=ws, split=m)[0].view(torch.int16)
           for m in ("never", "auto", "always")}
    assert not torch.equal(out["never"], out["always"])
    assert torch.equal(out["auto"], out[same_as])
