"""The key split's cut: on the CPU, every workgroup of some three thousand launches walked with the functions that the
kernel uses (tests/host/attn_split_check.cpp); on the GPU, the cuts that other tests do not reach."""
import os
import subprocess

import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, attn_errors, attn_plan, bits_of, to_dev_bf16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_pair_once_and_every_piece_where_the_merge_looks(tmp_path):
    exe = str(tmp_path / "split")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_split_check.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0 and int(res.stdout.split()[1]) > 3000, res.stdout


# (heads, queries, cached keys, block keys, workgroups on 256 compute units): two columns each and no helper; two columns
# and helpers, the seam and the ragged end among the helpers' tiles; one column of all but a few tiles; equal runs
@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,c_len,n_blk,wgs", [(128, 40, 2100, 40, 256), (95, 70, 3200, 77, 256), (230, 33, 6000, 391, 256), (250, 33, 6000, 391, 256)])
def test_cut_matches_oracle(H, n_q, c_len, n_blk, wgs):
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb = si.attn_inputs(H, max(n_q, n_blk), c_len, seed=900 + H, jitter=True, cache_capacity=c_len)
    q, kb, vb = q[:n_q], kb[:n_blk], vb[:n_blk]
    plan = attn_plan(H, n_q, c_len + n_blk, split=2)
    assert plan.split and (plan.workgroups <= wgs or torch.cuda.get_device_properties(0).multi_processor_count != 256)
    d = [to_dev_bf16(x) for x in (q, kc, vc, kb, vb)]
    ws = torch.full((plan.workspace,), 0xFF, dtype=torch.uint8, device="cuda")  # (NaN wherever it is read unwritten)
    out = torch.full_like(d[0], float("nan"))
    P.block_attn_batch(*[[x] for x in d], c_len, outs=[out], workspace=ws, split="always")
    rows = sorted({0, 1, 31, 32, n_q // 2, n_q - 2, n_q - 1})
    max_abs, rel = attn_errors(bits_of(out)[rows], oracle.block_attn(q, kc, vc, kb, vb, c_len, rows=rows))
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)
    plain = P.block_attn(*d, c_len).float()
    assert ((out.float() - plain).norm() / plain.norm()).item() <= 2 * BF16_REL_RMS
