"""GEMM kernel parity against the float64 matmul of the same bf16 operands,
over all operand layouts and epilogues, at shapes that span several tiles with
ragged edges, and the unaligned (scalar-load) path."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import ops as O
from tests.gpu_util import bf16_round, flush, gemm_on, host, rel, to_dev_bf16, to_dev_f32

pytestmark = pytest.mark.gpu


def _operands(rng, M, N, K, a_layout, b_layout):
    A = bf16_round(rng.normal(size=(M, K)))
    B = bf16_round(rng.normal(size=(N, K)))
    Ad = to_dev_bf16(A if a_layout == 0 else A.T.copy())
    Bd = to_dev_bf16(B if b_layout == 0 else B.T.copy())
    lda = K if a_layout == 0 else M
    ldb = K if b_layout == 0 else N
    return A, B, Ad, Bd, lda, ldb


SHAPES = [(64, 64, 64), (300, 200, 136), (513, 257, 520), (256, 128, 64), (8, 8, 8), (1000, 40, 16)]


@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_f32_layouts(a_layout, b_layout, M, N, K):
    from paper_2309_01226_amd import ops
    flush(f"gemm f32 lay=({a_layout},{b_layout}) M={M} N={N} K={K}")
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, a_layout, b_layout)
    bias = rng.normal(size=N)
    out = torch.empty(M, N, device="cuda", dtype=torch.float32)
    ops.gemm(Ad, Bd, M, N, K, out, lda=lda, ldb=ldb, a_layout=a_layout, b_layout=b_layout,
             bias=to_dev_f32(bias))
    torch.cuda.synchronize()
    ref = O.gemm(A, B) + bias
    assert rel(host(out), ref) < 2e-6


@pytest.mark.parametrize("M,N,K", [(300, 200, 100), (77, 45, 588), (129, 65, 37)])
def test_gemm_unaligned_scalar_path(M, N, K):
    from paper_2309_01226_amd import ops
    flush(f"gemm unaligned M={M} N={N} K={K}")
    rng = np.random.default_rng(5)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, 0, 0)
    out = torch.empty(M, N, device="cuda", dtype=torch.float32)
    ops.gemm(Ad, Bd, M, N, K, out, lda=lda, ldb=ldb)
    torch.cuda.synchronize()
    assert rel(host(out), O.gemm(A, B)) < 2e-6


@pytest.mark.parametrize("erf_form", [0, 1])
def test_gemm_epilogues(erf_form):
    from paper_2309_01226_amd import ops
    M, N, K = 390, 272, 200
    flush(f"gemm epilogues erf={erf_form}")
    rng = np.random.default_rng(11)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, 0, 0)
    C = O.gemm(A, B)
    bias = rng.normal(size=N - 40)
    # residual add into fp32, resid aliasing out
    R = rng.normal(size=(M, N))
    out = to_dev_f32(R)
    ops.gemm(Ad, Bd, M, N, K, out, lda=lda, ldb=ldb, epilogue=1, resid=out,
             bias=to_dev_f32(bias), bias_col0=40)
    torch.cuda.synchronize()
    ref = R + C
    ref[:, 40:] += bias
    assert rel(host(out), ref) < 2e-6
    # bf16 store with bias from column 40 and GELU of columns >= 100 into out2
    o1 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    o2 = torch.empty(M, N - 100, device="cuda", dtype=torch.bfloat16)
    ops.gemm(Ad, Bd, M, N, K, o1, lda=lda, ldb=ldb, epilogue=2, bias=to_dev_f32(bias),
             bias_col0=40, out2=o2, ldo2=N - 100, gelu_col0=100, gelu_erf=erf_form)
    torch.cuda.synchronize()
    pre = C.copy()
    pre[:, 40:] += bias
    assert rel(host(o1), pre) < 4e-3
    assert rel(host(o2), O.gelu(pre[:, 100:], erf_form)) < 4e-3
    # GELU-backward epilogue
    U = bf16_round(rng.normal(size=(M, N)))
    o3 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    ops.gemm(Ad, Bd, M, N, K, o3, lda=lda, ldb=ldb, epilogue=3, aux=to_dev_bf16(U), ldaux=N,
             gelu_erf=erf_form)
    torch.cuda.synchronize()
    assert rel(host(o3), C * O.gelu_grad(U, erf_form)) < 4e-3


@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(4100, 4104, 584), (4104, 7944, 584)])
def test_gemm_large_tiles_sampled(M, N, K, a_layout, b_layout, epi):
    """Shapes of more than 256 tiles of 256 x 256, with ragged M and N edges and a K tail,
    every epilogue: the 256 x 256 kernel, except that the smaller one's fp32 outputs (17 x 17
    tiles, a last round of 33) run on 128 x 128, and its M-contiguous A (4100 is no
    multiple of 8) in the gather kernel; checked on 300 sampled rows (always including
    the last) against float64."""
    flush(f"gemm large M={M} N={N} lay=({a_layout},{b_layout}) epi={epi}")
    tile = 256 if N == 7944 else -128 if a_layout == 1 else 128 if epi < 2 else 256
    rng = np.random.default_rng(17 + a_layout + 2 * b_layout + 4 * epi)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, a_layout, b_layout)
    bias = rng.normal(size=N - 8)
    rows = np.sort(rng.choice(M - 1, size=299, replace=False))
    rows = np.append(rows, M - 1)
    C = O.gemm(A[rows], B)
    pre = C.copy()
    pre[:, 8:] += bias
    kw = dict(lda=lda, ldb=ldb, a_layout=a_layout, b_layout=b_layout, epilogue=epi)
    if epi == 0:
        out = torch.empty(M, N, device="cuda", dtype=torch.float32)
        gemm_on(tile, Ad, Bd, M, N, K, out, bias=to_dev_f32(bias), bias_col0=8, **kw)
        torch.cuda.synchronize()
        assert rel(host(out)[rows], pre) < 2e-6
    elif epi == 1:
        R = rng.normal(size=(M, N)).astype(np.float32)
        out = to_dev_f32(R)
        gemm_on(tile, Ad, Bd, M, N, K, out, resid=out, bias=to_dev_f32(bias), bias_col0=8, **kw)
        torch.cuda.synchronize()
        assert rel(host(out)[rows], R[rows] + pre) < 2e-6
    elif epi == 2:
        o1 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        o2 = torch.empty(M, N - 512, device="cuda", dtype=torch.bfloat16)
        gemm_on(tile, Ad, Bd, M, N, K, o1, bias=to_dev_f32(bias), bias_col0=8, out2=o2, ldo2=N - 512,
                 gelu_col0=512, **kw)
        torch.cuda.synchronize()
        assert rel(host(o1)[rows], pre) < 4e-3
        assert rel(host(o2)[rows], O.gelu(pre[:, 512:], 0)) < 4e-3
    else:
        U = bf16_round(rng.normal(size=(M, N)))
        o3 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        gemm_on(tile, Ad, Bd, M, N, K, o3, aux=to_dev_bf16(U), ldaux=N, gelu_erf=1, **kw)
        torch.cuda.synchronize()
        assert rel(host(o3)[rows], C * O.gelu_grad(U[rows], 1)) < 4e-3


# Split-K: fp32-output products with fewer than 256 tiles of 256 x 256 and
# K >= 1024, given a workspace.  Shapes: one tile, ragged M / N, a K that is
# not a multiple of the slice depth (last slice shorter) and not a multiple of
# 64, and a residual + bias epilogue with the residual aliasing the output.
SPLITK = [(256, 256, 2048, 0), (300, 520, 4160, 0), (768, 768, 8192, 0), (520, 264, 3008, 1),
          (1000, 40, 1032, 1)]


@pytest.mark.parametrize("M,N,K,resid", SPLITK)
def test_gemm_splitk(M, N, K, resid):
    from paper_2309_01226_amd import ops
    flush(f"gemm split-K M={M} N={N} K={K} resid={resid}")
    rng = np.random.default_rng(M + N + K)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, 0, 0)
    bias = rng.normal(size=N)
    R = rng.normal(size=(M, N))
    ws = torch.full((16 * M * N,), float("nan"), device="cuda", dtype=torch.float32)
    out = to_dev_f32(R) if resid else torch.empty(M, N, device="cuda", dtype=torch.float32)
    kw = dict(bias=to_dev_f32(bias), epilogue=ops.EPI_RESID_F32 if resid else ops.EPI_F32)
    if resid:
        kw.update(resid=out, ldr=N)
    ops.gemm(Ad, Bd, M, N, K, out, lda=lda, ldb=ldb, splitk_ws=ws, **kw)
    # the same product without a workspace (no split)
    out1 = to_dev_f32(R) if resid else torch.empty(M, N, device="cuda", dtype=torch.float32)
    if resid:
        kw.update(resid=out1)
    ops.gemm(Ad, Bd, M, N, K, out1, lda=lda, ldb=ldb, **kw)
    torch.cuda.synchronize()
    ref = O.gemm(A, B) + bias + (R if resid else 0.0)
    got = host(out)
    assert np.isfinite(got).all()
    assert rel(got, ref) < 2e-6
    assert rel(got, host(out1)) < 2e-6
    # the split path ran: at least two slices of partial products were written
    n_used = int(torch.isfinite(ws).sum().item())
    assert n_used >= 2 * M * N, n_used


# Tail split: fp32-output products with more than 256 tiles of 256 x 256 whose
# last round would run mostly empty (ViT-H/14's 16448 x 1280 products have 325
# tiles), given a workspace: whole rounds of rows unsplit, the remaining rows
# split-K, then the reduction with bias and residual.  Shapes: the ViT-H
# products, a ragged last row tile, ragged columns, and a second shape family.
TAIL = [(16448, 1280, 5120, 1), (16448, 1280, 1280, 0), (16400, 1280, 3840, 1),
        (16448, 1272, 5120, 0), (9000, 2048, 2048, 1)]


@pytest.mark.parametrize("M,N,K,resid", TAIL)
def test_gemm_tail_split(M, N, K, resid):
    from paper_2309_01226_amd import ops
    flush(f"gemm tail split M={M} N={N} K={K} resid={resid}")
    rng = np.random.default_rng(M + N + K + 1)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, 0, 0)
    bias = rng.normal(size=N)
    R = rng.normal(size=(M, N)).astype(np.float32)
    ws = torch.full((16 * 1024 * 1024,), float("nan"), device="cuda", dtype=torch.float32)
    out = to_dev_f32(R) if resid else torch.empty(M, N, device="cuda", dtype=torch.float32)
    kw = dict(bias=to_dev_f32(bias), epilogue=ops.EPI_RESID_F32 if resid else ops.EPI_F32)
    if resid:
        kw.update(resid=out, ldr=N)
    ops.gemm(Ad, Bd, M, N, K, out, lda=lda, ldb=ldb, splitk_ws=ws, **kw)
    out1 = to_dev_f32(R) if resid else torch.empty(M, N, device="cuda", dtype=torch.float32)
    if resid:
        kw.update(resid=out1)
    ops.gemm(Ad, Bd, M, N, K, out1, lda=lda, ldb=ldb, **kw)
    torch.cuda.synchronize()
    got = host(out)
    assert np.isfinite(got).all()
    # rows from the unsplit head, from the split tail and the last row
    head_rows = rng.choice(M // 2, size=150, replace=False)
    tail_rows = M - 1 - rng.choice(2048, size=150, replace=False)
    rows = np.unique(np.concatenate([head_rows, tail_rows, [M - 1]]))
    ref = O.gemm(A[rows], B) + bias + (R[rows].astype(np.float64) if resid else 0.0)
    assert rel(got[rows], ref) < 2e-6
    assert rel(got, host(out1)) < 2e-6
    # the tail ran split-K: partials of at least two slices were written, but
    # fewer than a split of every row would write
    n_used = int(torch.isfinite(ws).sum().item())
    assert 2 * N * 16 <= n_used < 2 * M * N, n_used


# The 128 x 128 and 64 x 64 tile kernels at grids that fill the chip: ragged last
# tiles in M and N, a K tail, rows whose 4-column vectors are aligned and rows
# where they are not (N odd, so every layout but (0, 0) is gathered), every
# layout and epilogue.
TILES = [(3001, 1288, 712, 64), (1285, 520, 200, 64), (2100, 1301, 328, 64), (3001, 2301, 1096, 128),
         (1285, 5160, 1096, 128)]


@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K,tile", TILES)
def test_gemm_tile_kernels(M, N, K, tile, epi, a_layout, b_layout):
    flush(f"gemm tiles lay=({a_layout},{b_layout}) epi={epi} M={M} N={N} K={K}")
    rng = np.random.default_rng(M + epi + 4 * a_layout + 8 * b_layout)
    A = bf16_round(rng.normal(size=(M, K)))
    B = bf16_round(rng.normal(size=(N, K)))
    up = lambda n: (n + 7) // 8 * 8  # noqa: E731  (row pitches of whole 16-byte pieces)

    def stored(X, layout):
        X = X if layout == 0 else X.T
        pad = np.zeros((X.shape[0], up(X.shape[1])))
        pad[:, :X.shape[1]] = X
        return to_dev_bf16(pad), pad.shape[1]

    Ad, lda = stored(A, a_layout)
    Bd, ldb = stored(B, b_layout)
    kw = dict(lda=lda, ldb=ldb, a_layout=a_layout, b_layout=b_layout, epilogue=epi)
    C = O.gemm(A, B)
    bias = rng.normal(size=N - 8)
    pre = C.copy()
    pre[:, 8:] += bias
    if epi < 2:
        R = rng.normal(size=(M, N)).astype(np.float32)
        out = to_dev_f32(R)
        gemm_on(tile, Ad, Bd, M, N, K, out, resid=out if epi else None, bias=to_dev_f32(bias), bias_col0=8, **kw)
        torch.cuda.synchronize()
        assert rel(host(out), pre + (R if epi else 0.0)) < 2e-6
    elif epi == 2:
        o1 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        o2 = torch.empty(M, N - 72, device="cuda", dtype=torch.bfloat16)
        gemm_on(tile, Ad, Bd, M, N, K, o1, bias=to_dev_f32(bias), bias_col0=8, out2=o2, ldo2=N - 72, gelu_col0=72, **kw)
        torch.cuda.synchronize()
        assert rel(host(o1), pre) < 4e-3
        assert rel(host(o2), O.gelu(pre[:, 72:], 0)) < 4e-3
    else:
        U = bf16_round(rng.normal(size=(M, N)))
        o3 = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        gemm_on(tile, Ad, Bd, M, N, K, o3, aux=to_dev_bf16(U), ldaux=N, gelu_erf=1, **kw)
        torch.cuda.synchronize()
        assert rel(host(o3), C * O.gelu_grad(U, 1)) < 4e-3


@pytest.mark.parametrize("a_layout,b_layout", [(0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K,tile", [(264, 392, 4168, 64), (1000, 1288, 4168, 128)])
def test_gemm_splitk_mn_layouts(M, N, K, tile, a_layout, b_layout):
    """An M/N-contiguous operand with a workspace: K slices, the last one short."""
    flush(f"gemm split-K M={M} N={N} lay=({a_layout},{b_layout})")
    rng = np.random.default_rng(23)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, a_layout, b_layout)
    R = rng.normal(size=(M, N)).astype(np.float32)
    ws = torch.full((16 * M * N,), float("nan"), device="cuda", dtype=torch.float32)
    out = to_dev_f32(R)
    gemm_on(tile, Ad, Bd, M, N, K, out, lda=lda, ldb=ldb, a_layout=a_layout, b_layout=b_layout, epilogue=1, resid=out,
            splitk_ws=ws)
    torch.cuda.synchronize()
    assert rel(host(out), R + O.gemm(A, B)) < 2e-6
    assert int(torch.isfinite(ws).sum().item()) >= 2 * M * N


@pytest.mark.parametrize("a_layout,b_layout", [(0, 1), (1, 1), (1, 0)])
def test_gemm_leaves_workspace_to_layout_0(a_layout, b_layout):
    """sat_op_gemm itself splits only products on layout-0 operands: with a layout-1 operand the
    workspace stays untouched and the result is the one without it (and of sat_op_gemm_noalloc)."""
    from paper_2309_01226_amd import _lib, ops
    M, N, K = 264, 392, 4168
    flush(f"gemm workspace untouched lay=({a_layout},{b_layout})")
    rng = np.random.default_rng(29)
    A, B, Ad, Bd, lda, ldb = _operands(rng, M, N, K, a_layout, b_layout)
    ws = torch.full((16 * M * N,), float("nan"), device="cuda", dtype=torch.float32)
    outs = [torch.empty(M, N, device="cuda") for _ in range(3)]
    for out, w in zip(outs, (ws, None)):
        d = ops._gemm_desc(Ad, Bd, M, N, K, out, lda, ldb, a_layout, b_layout, 0, None, None, 0, None, None, None, 0,
                           0, None, 0, 0, w)
        _lib.call("sat_op_gemm", ctypes.byref(d), ops._stream())
    ops.gemm_noalloc(Ad, Bd, M, N, K, outs[2], lda=lda, ldb=ldb, a_layout=a_layout, b_layout=b_layout)
    torch.cuda.synchronize()
    assert torch.isnan(ws).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert rel(host(outs[0]), O.gemm(A, B)) < 2e-6


# A residual / pre-activation whose rows of one tile span 2 GiB (and 4 GiB) or more: the same
# result as from a compact one, with 128 x 128 tiles and with 64 x 64.
@pytest.mark.parametrize("M,N,K,tile", [(128, 25600, 4096, 128), (64, 64, 64, 64)])
@pytest.mark.parametrize("epi", [1, 3])
@pytest.mark.parametrize("span", [1, 2])
def test_gemm_epilogue_operand_spans_2gib(M, N, K, tile, epi, span):
    flush(f"gemm epilogue operand past 2 GiB M={M} N={N} K={K} epi={epi} span={span}")
    g = torch.Generator("cuda").manual_seed(M + epi)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    B = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    dt = torch.float32 if epi == 1 else torch.bfloat16
    X = torch.randn(M, N, generator=g, device="cuda").to(dt)
    ld = (span * (1 << 31) // ((M - 1) * X.element_size()) + 67) // 4 * 4
    wide = torch.empty(M * ld, device="cuda", dtype=dt).view(M, ld)
    wide[:, :N] = X
    res = []
    for x, l in ((X, N), (wide, ld)):
        out = torch.empty(M, N, device="cuda", dtype=dt)
        kw = dict(resid=x, ldr=l) if epi == 1 else dict(aux=x, ldaux=l)
        gemm_on(tile, A, B, M, N, K, out, lda=K, ldb=K, epilogue=epi, **kw)
        res.append(out)
    torch.cuda.synchronize()
    assert torch.equal(res[0], res[1])


# An operand whose rows (or k-rows) of one tile span 2 GiB or more.
@pytest.mark.parametrize("M,N,K", [(128, 25600, 4096), (64, 64, 64)])
@pytest.mark.parametrize("layout", [0, 1])
def test_gemm_operand_spans_2gib(M, N, K, layout):
    if layout == 1:
        K = 64
    flush(f"gemm operand past 2 GiB M={M} N={N} K={K} layout={layout}")
    g = torch.Generator("cuda").manual_seed(M + layout)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    B = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    S = A if layout == 0 else A.t().contiguous()
    ld = ((1 << 31) // ((S.shape[0] - 1) * 2) + 71) // 8 * 8
    wide = torch.empty(S.shape[0] * ld, device="cuda", dtype=torch.bfloat16).view(S.shape[0], ld)
    wide[:, :S.shape[1]] = S
    res = []
    for x, l in ((S, S.shape[1]), (wide, ld)):
        out = torch.empty(M, N, device="cuda")
        gemm_on(M if x is S else -M, x, B, M, N, K, out, lda=l, ldb=K, a_layout=layout)
        res.append(out)
    torch.cuda.synchronize()
    assert torch.equal(res[0], res[1])


def test_gemm_mn_operand_past_2gib():
    """An M/N-contiguous operand of more than 2 GiB (21504 k-rows of 50264) in the 256 x 256 kernel:
    sampled rows against fp64."""
    M, N, K, lda = 16390, 4096, 21504, 50264
    flush(f"gemm M/N-contiguous operand of {2 * K * lda} bytes")
    g = torch.Generator("cuda").manual_seed(4)
    A = torch.randn(K, lda, generator=g, device="cuda", dtype=torch.bfloat16)
    B = torch.randn(K, N, generator=g, device="cuda", dtype=torch.bfloat16)
    out = torch.empty(M, N, device="cuda")
    gemm_on(256, A, B, M, N, K, out, lda=lda, ldb=N, a_layout=1, b_layout=1)
    rows = torch.tensor([0, 1, 255, 256, 8191, 16383, 16384, 16389], device="cuda")
    ref = A[:, rows].double().t() @ B.double()
    assert rel(host(out[rows]), host(ref)) < 2e-6
