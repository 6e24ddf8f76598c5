"""Helpers for the GPU parity tests: bf16 rounding on the host (to feed both
sides identical operand values) and relative Frobenius error."""

import numpy as np
import torch


def bf16_round(x):
    """Round a float array to bfloat16 values (returned as float64)."""
    return torch.as_tensor(np.asarray(x, np.float32)).to(torch.bfloat16).to(torch.float64).numpy()


def to_dev_bf16(x):
    return torch.as_tensor(np.asarray(x, np.float32)).to(torch.bfloat16).cuda()


def to_dev_f32(x):
    return torch.as_tensor(np.asarray(x, np.float32)).cuda()


def rel(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def flush(*msg):
    print(*msg, flush=True)


def gemm_tile(A, B, M, N, K, out, *, lda, ldb, a_layout=0, b_layout=0, epilogue=0, ldo=None, bias=None, bias_col0=0,
              resid=None, ldr=None, out2=None, ldo2=0, gelu_col0=0, aux=None, ldaux=0, gelu_erf=0, splitk_ws=None):
    """(tile, K slices) that ops.gemm would run these arguments on; a negative tile is the
    gather kernel's."""
    import ctypes

    from paper_2309_01226_amd import _lib, ops
    d = ops._gemm_desc(A, B, M, N, K, out, lda, ldb, a_layout, b_layout, epilogue, ldo, bias, bias_col0, resid, ldr,
                       out2, ldo2, gelu_col0, aux, ldaux, gelu_erf, splitk_ws)
    s = ctypes.c_int()
    return _lib.lib().sat_test_gemm_tile(ctypes.byref(d), ctypes.byref(s)), s.value


def gemm_on(tile, *args, **kw):
    """ops.gemm, on the kernel of that tile."""
    from paper_2309_01226_amd import ops
    assert gemm_tile(*args, **kw)[0] == tile, (gemm_tile(*args, **kw), tile)
    return ops.gemm(*args, **kw)
