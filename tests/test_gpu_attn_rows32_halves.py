"""The 32-row attention kernel with two workgroups per 32 rows, each with half of the output dims, which the smallest launches
take: its V tiles on the CPU, its rule, the same bits as the kernel with whole V tiles; and that kernel at the edges of its
tiles, in launches that are too large for halves."""
import os
import subprocess

import pytest
import torch

import sdvg_inputs as si
import test_gpu_attn_groups as by_groups
from gpu_util import MI355X_CUS, attn_plan, to_dev_bf16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_v_tiles_on_the_host(tmp_path):
    exe = str(tmp_path / "halves")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_rows32_halves.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout == "ok\n", res.stdout


# An item alone (halves: 50 and 128 workgroups of 32 rows) and in a batch (150 and 256, whole V tiles)
@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_items", [(5, 300, 3), (8, 512, 2)])
@pytest.mark.parametrize("n_blk,c_len", [(300, 330), (193, 0), (33, 512)])
def test_same_bits_as_whole_v_tiles(H, n_q, n_items, n_blk, c_len):
    import paper_2604_17397_amd as P
    alone, batch = attn_plan(H, n_q, c_len + n_blk, n_cu=MI355X_CUS), attn_plan(H, n_q, c_len + n_blk, n_items, n_cu=MI355X_CUS)
    assert alone.rows == batch.rows == 32 and 2 * alone.workgroups <= MI355X_CUS < 2 * batch.workgroups
    items = []
    for s in range(n_items):
        q, kc, vc, kb, vb = si.attn_inputs(H, max(n_q, n_blk), c_len, seed=40 + s, jitter=True, cache_capacity=max(c_len, 1))
        items.append([to_dev_bf16(a) for a in (q[:n_q], kc, vc, kb[:n_blk], vb[:n_blk])])
    outs = P.block_attn_batch(*([it[i] for it in items] for i in range(5)), c_len)
    for it, out in zip(items, outs):
        assert torch.equal(out, P.block_attn(*it, c_len))


# 172 workgroups: the kernel with whole V tiles
@pytest.mark.gpu
@pytest.mark.parametrize("n_k", [193, 224, 255, 257, 513])
@pytest.mark.parametrize("c_len", [0, 31, 33, 160])
def test_edges_of_the_whole_v_tiles(monkeypatch, n_k, c_len):
    monkeypatch.setitem(by_groups.HEADS, 4, 43)
    n_q = 97 + (n_k + c_len) % 32
    plan = attn_plan(43, n_q, n_k, n_cu=MI355X_CUS)
    assert plan.rows == 32 and 2 * plan.workgroups > MI355X_CUS
    by_groups.run_planned(4, n_q, n_k - c_len, c_len, seed=n_k + c_len, commit=c_len > 0)
