"""Row numbering of the copy kernels (csrc/row_map.h), compiled with g++ and checked against plain
divisions and loops; on the GPU the head-major and padded layouts of commit, commit with rotation
and rollback against the oracle's mirror."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import bits_of, to_dev_bf16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_row_map_on_the_host(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "row_map_check.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("L,T,H", [(1, 1, 1), (3, 5, 3), (2, 17, 12), (4, 31, 7)])
@pytest.mark.parametrize("layout", ["token", "head", "padded"])
@pytest.mark.parametrize("rotate", [False, True])
def test_commit_and_rollback_by_layout(L, T, H, layout, rotate):
    import paper_2604_17397_amd as P
    cap = 3 * T + 2

    def storage():
        if layout == "token":
            return torch.zeros((L, cap, H, 128), dtype=torch.bfloat16, device="cuda")
        if layout == "head":
            return torch.zeros((L, H, cap, 128), dtype=torch.bfloat16, device="cuda").transpose(1, 2)
        return torch.zeros((L, cap, H, 136), dtype=torch.bfloat16, device="cuda")[..., :128]
    k, v = storage(), storage()
    cache = P.KVCache(k, v, T)
    mirror = oracle.KVMirror(L, cap, H, 128, T)
    angle = np.random.default_rng(5).random((T, 64)) * 6.28
    cos, sin = np.cos(angle).astype(np.float32), np.sin(angle).astype(np.float32)
    tables = [torch.from_numpy(t).cuda() for t in (cos, sin)]
    for slot in range(3):
        kb = si.f32_to_bf16_bits(np.random.default_rng(slot).standard_normal((L, T, H, 128)).astype(np.float32))
        vb = si.f32_to_bf16_bits(np.random.default_rng(50 + slot).standard_normal((L, T, H, 128)).astype(np.float32))
        if rotate:
            P.kv_commit_rope(cache, to_dev_bf16(kb), to_dev_bf16(vb), slot, *tables)
            kb = np.stack([oracle.rope(kb[l], cos, sin) for l in range(L)])
        else:
            P.kv_commit(cache, to_dev_bf16(kb), to_dev_bf16(vb), slot)
        assert oracle.kv_commit(mirror, kb, vb, slot) == 0
    P.kv_rollback(cache, T + T // 2)
    oracle.kv_rollback(mirror, T + T // 2)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(k), mirror.k) and np.array_equal(bits_of(v), mirror.v)


@pytest.mark.gpu
def test_more_rows_than_a_grid_dimension_holds():
    """2^28 rows and more are 2^32 threads and more. The rows overlap in memory (token and head stride are
    one row), so that 17 MB hold them: all are written with the same values, and only the last row of
    the last slice reaches the last address."""
    import paper_2604_17397_amd as P
    T, H = (1 << 12) + 1, 1 << 16
    rows = torch.ones((T + H - 1, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.zeros_like(rows)
    c, s = torch.ones((T, 64), device="cuda"), torch.zeros((T, 64), device="cuda")
    P.rope(rows.as_strided((T, H, 128), (128, 128, 1)), c, s, out=out.as_strided((T, H, 128), (128, 128, 1)))
    torch.cuda.synchronize()
    assert torch.equal(out, rows)
