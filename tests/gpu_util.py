"""Helpers for the GPU parity tests: bit-exact host <-> device transfer, error metrics, launch plans."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np
import torch

import sdvg_inputs as si


def to_dev_bf16(bits):
    """uint16 bf16 bit patterns (numpy) -> bfloat16 device tensor holding the same bits."""
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()


def bits_of(t):
    """bfloat16 tensor (any device) -> uint16 bit patterns (numpy)."""
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def attn_errors(gpu_bits, ref):
    """max |err| and relative RMS of a bf16 GPU output against the fp64 oracle output."""
    g = si.bf16_bits_to_f64(gpu_bits)
    err = g - ref
    return float(np.max(np.abs(err))), float(np.sqrt(np.sum(err * err) / np.sum(ref * ref)))


def attn_errors_by_head(gpu_bits, ref):
    """(max |err|, pooled rel-RMS, worst single head's rel-RMS, that head) for outputs shaped
    [rows, heads, dim]. Heads whose reference is all zero are skipped for the per-head figure."""
    g = si.bf16_bits_to_f64(gpu_bits)
    err = g - ref
    num = np.sum(err * err, axis=(0, 2))
    den = np.sum(ref * ref, axis=(0, 2))
    per_head = np.sqrt(np.where(den > 0, num / np.where(den > 0, den, 1.0), 0.0))
    worst = int(np.argmax(per_head))
    return (float(np.max(np.abs(err))), float(np.sqrt(num.sum() / den.sum())), float(per_head[worst]), worst)


# Tolerances of the bf16 attention path: absolute and relative-RMS bounds on the output.
# bf16 P and bf16 output rounding are each ~2^-9 relative; sums over many keys average it down.
BF16_MAX_ABS = 2e-2
BF16_REL_RMS = 1e-2
F32_MAX_ABS = 1e-4


Plan = collections.namedtuple("Plan", "groups rows workgroups query_tiles split workspace")
MI355X_CUS = 256


@functools.lru_cache(maxsize=None)
def _plan_library():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    with tempfile.TemporaryDirectory(prefix="sdvg_plan_") as tmp:
        out = os.path.join(tmp, "attn_plan.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I", os.path.join(root, "include"),
                        "-I", os.path.join(root, "paper_2604_17397_amd", "csrc"),
                        os.path.join(root, "tests", "host", "attn_plan.cpp"), "-o", out], check=True)
        lib = ctypes.CDLL(out)
    lib.attn_plan.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                                                   ctypes.POINTER(ctypes.c_int64)]
    lib.attn_plan.restype = None
    lib.attn_plan_static_workspace.restype = ctypes.c_int64
    return lib


def attn_plan(n_heads, n_q, n_k, n_items=1, split=0, n_cu=None):
    """How a bf16 attention launch is cut into workgroups, from the library's own plan header, compiled
    here: `groups` is 1 for the kernel of 256 rows per workgroup, 2 or 4 for the one with key groups. With 4 groups
    `rows` tells the kernel: 64 that one, 32 the one for the smallest launches."""
    if n_cu is None:
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    out = (ctypes.c_int64 * 6)()
    _plan_library().attn_plan(n_items, n_q, n_heads, n_k, n_cu, split, out)
    return Plan(*out)


def attn_plan_rows(n_heads, n_q, n_k, n_items=1, split=0, n_cu=None, rows32_ok=1):
    """Query rows per workgroup of such a launch (32: the kernel for the smallest launches)."""
    if n_cu is None:
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    return _plan_library().attn_plan_rows(n_items, n_q, n_heads, ctypes.c_int64(n_k), n_cu, split, rows32_ok)


def attn_plan_static_workspace(n_heads, n_q, n_k, n_items=1, split=1, n_cu=MI355X_CUS):
    """Bytes of the library's own array that sdvg_block_attn_batch_static needs for such a launch."""
    return _plan_library().attn_plan_static_workspace(n_items, n_q, n_heads, ctypes.c_int64(n_k), n_cu, split)


def attn_plan_halves(n_k, q, out, n_cu=MI355X_CUS):
    """Whether two workgroups share 32 query rows in a call with these q and out ([tokens, heads, 128], any device)."""
    return bool(_plan_library().attn_plan_halves(q.shape[0], q.shape[1], ctypes.c_int64(n_k), n_cu, *[
        f for t in (q, out) for f in (ctypes.c_void_p(t.data_ptr()), ctypes.c_int64(t.stride(0)), ctypes.c_int64(t.stride(1)))]))


def attn_plan_commit(n_heads, n_q, n_blk, n_k, n_cu=MI355X_CUS):
    """Attention and copying workgroups of one launch with the commit fused in."""
    out = (ctypes.c_int * 2)()
    _plan_library().attn_plan_commit(n_q, n_blk, n_heads, ctypes.c_int64(n_k), n_cu, out)
    return tuple(out)
