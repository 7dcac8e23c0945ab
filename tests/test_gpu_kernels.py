"""Kernel-level parity on the GPU: the tile contraction (every operand layout, tile shape
and dtype, ragged sizes), the implicit-GEMM convolution passes and the kernels of the ViT-shaped
stages (LayerNorm, GELU, attention core) against the oracle."""
import numpy as np
import pytest

import cdp_workloads as wl
from oracle import layers as L
from paper_2403_08837_amd import binding as b

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _dev(a, dtype):
    torch = _torch()
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16).contiguous() if dtype == wl.BF16 else t.contiguous()


def _rnd(a, dtype):
    return L.round_bf16(a) if dtype == wl.BF16 else np.asarray(a, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("a_k,b_k", [(1, 1), (0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", [(8, 64, 64), (64, 200, 136), (130, 257, 70), (333, 129, 515), (5, 7, 3), (32, 300, 1100),
                                   (32, 1024, 1024), (17, 200, 3072), (32, 96, 136), (1, 40, 8), (9, 33, 2056)])
def test_gemm_all_layouts(dtype, shape, a_k, b_k, M, N, K):
    """Every selector of cdp_k_gemm.  6 is the launch of the engine's Linear stages (32 x 32 tiles at up to 32 rows, one slab and
    several), 7 to 9 the generic kernel, which 0 to 2 are too unless both operands are row-contiguous."""
    torch = _torch()
    if 3 <= shape < 7 and not (a_k and b_k):
        pytest.skip("the weight-streaming kernel takes k-contiguous operands only")
    A = wl.random_normal(1, 10 * M + K, M * K).reshape(M, K)
    Bm = wl.random_normal(2, 10 * N + K, N * K).reshape(N, K)
    ref = _rnd(A, dtype) @ _rnd(Bm, dtype).T
    Ad = _dev(A if a_k else A.T, dtype)
    Bd = _dev(Bm if b_k else Bm.T, dtype)
    Cd = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_gemm(dtype, shape, a_k, b_k, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(), M, N, K,
                 K if a_k else M, K if b_k else N)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy().astype(np.float64)
    tol = 2e-5 * np.sqrt(K) * max(1.0, np.abs(ref).max())
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= tol, np.abs(got - ref).max()


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("M,N,K,lda,ldb", [(512, 1024, 64, 512, 1024),     # smallest matrix that is walked in runs of two column tiles
                                           (520, 1160, 33, 528, 1168),     # the same with a ragged run and padded rows
                                           (512, 1024, 65, 512, 1024),     # one row more than a staged slab: single tiles
                                           (96, 136, 200, 100, 137),       # several slabs, rows that are not whole chunks
                                           (33, 1, 1, 33, 1)])
def test_gemm_weight_gradient_tiles(dtype, M, N, K, lda, ldb):
    """C = A^T B with both operands row-contiguous, at the edges of the weight-gradient tiles."""
    torch = _torch()
    A = wl.random_normal(1, 10 * M + K, K * lda).reshape(K, lda)
    Bm = wl.random_normal(2, 10 * N + K, K * ldb).reshape(K, ldb)
    ref = _rnd(A, dtype)[:, :M].T @ _rnd(Bm, dtype)[:, :N]
    Ad, Bd = _dev(A, dtype), _dev(Bm, dtype)
    Cd = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_gemm(dtype, 0, 0, 0, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(), M, N, K, lda, ldb)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy().astype(np.float64)
    # products of exactly representable inputs, fp32 sums of K terms: K 2^-24 of the largest magnitude bounds the error
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 2e-5 * np.sqrt(K) * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("K", [1, 7, 8, 9, 16, 17, 48, 49, 56, 57, 64, 72])
@pytest.mark.parametrize("M,N", [(64, 64), (33, 130), (72, 200), (2080, 2056)])
def test_gemm_weight_gradient_rows(dtype, K, M, N):
    """C = A^T B over few rows: the last slab is contracted by groups of 8 (fp32) or 16 rows, and elements outside the matrix
    read its edge; 2080 x 2056 has tiles 64 rows high, the others of 32."""
    torch = _torch()
    A = wl.random_normal(1, 10 * M + K, K * M).reshape(K, M)
    Bm = wl.random_normal(2, 10 * N + K, K * N).reshape(K, N)
    ref = _rnd(A, dtype).T @ _rnd(Bm, dtype)
    Ad, Bd = _dev(A, dtype), _dev(Bm, dtype)
    Cd = torch.full((M * N + 256,), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_gemm(dtype, 0, 0, 0, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(), M, N, K, M, N)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy().astype(np.float64)
    assert np.isnan(got[M * N:]).all(), "written past the matrix"
    got = got[:M * N].reshape(M, N)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 2e-5 * np.sqrt(K) * max(1.0, np.abs(ref).max())  # as above


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64, 65, 128, 129])
def test_gemm_few_rows(dtype, M):
    """The kernel for one problem of few rows: edges of its row blocks (129: the tick launch's tiles), ragged columns, and
    reductions of less than one piece per wavefront up to several, whole and not."""
    torch = _torch()
    for N, K in ((1, 8), (40, 264), (17, 1032), (130, 1536), (4096, 24), (4099, 40), (8200, 64)):
        A = wl.random_normal(1, 10 * M + K, M * K).reshape(M, K)
        Bm = wl.random_normal(2, 10 * N + K, N * K).reshape(N, K)
        ref = _rnd(A, dtype) @ _rnd(Bm, dtype).T
        Ad, Bd = _dev(A, dtype), _dev(Bm, dtype)
        Cd = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        b.cdp_k_gemm(dtype, 5, 1, 1, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(), M, N, K, K, K)
        torch.cuda.synchronize()
        got = Cd.cpu().numpy().astype(np.float64)
        # products of exactly representable inputs, fp32 sums of K terms: as in test_gemm_all_layouts
        assert np.isfinite(got).all()
        assert np.abs(got - ref).max() <= 2e-5 * np.sqrt(K) * max(1.0, np.abs(ref).max()), (N, K)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("M,N,K,lda,ldb", [(70, 1024, 72, 72, (1 << 22) + 8),            # rows of the weights past 32-bit byte offsets
                                           (64, 33, 1160, (1 << 23) + 8, 1160),          # rows of x
                                           (3, 20, (1 << 22) + 40, (1 << 22) + 40, (1 << 22) + 40),  # long reduction, its end inside a piece
                                           (17, 5, 8, (1 << 25) + 8, (1 << 26) + 8), (40, 16, 64, 64, 1 << 22)])
def test_gemm_few_far_rows(dtype, M, N, K, lda, ldb):
    """The same kernel where rows are far apart.  Exact: -1, 0 and 1, sums below 2^24."""
    torch = _torch()
    t = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)

    def rows(n, ld):  # the last row ends with the memory, what lies between rows is not read
        mem = torch.empty((n - 1) * ld + K, dtype=t, device="cuda")
        view = mem.as_strided((n, K), (ld, 1))
        view.copy_(torch.randint(-1, 2, (n, K), generator=gen, device="cuda"))
        if ld > K and n > 1:
            mem.as_strided((n - 1, min(8, ld - K)), (ld, 1), K).fill_(float("nan"))
        return mem, view
    a, x = rows(M, lda)
    w, k = rows(N, ldb)
    ref = sum(x[:, i:i + (1 << 18)].float().contiguous() @ k[:, i:i + (1 << 18)].float().contiguous().T for i in range(0, K, 1 << 18))
    got = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_gemm(dtype, 5, 1, 1, a.data_ptr(), w.data_ptr(), got.data_ptr(), M, N, K, lda, ldb)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)


CONV_CASES = [
    # B, H, W, Cin, Cout, ks, stride, pad
    (2, 8, 8, 8, 16, 3, 1, 1),
    (3, 9, 7, 16, 8, 3, 2, 1),
    (2, 12, 12, 3, 8, 7, 2, 3),     # stem-like: Cin = 3 takes the element-wise gather path
    (2, 8, 8, 3, 8, 3, 1, 1),
    (4, 6, 6, 32, 64, 1, 1, 0),
    (4, 6, 6, 32, 64, 1, 2, 0),
    (2, 16, 16, 64, 64, 3, 1, 1),
    (1, 5, 5, 24, 40, 3, 1, 1),     # channel counts that are multiples of 8 but not of the tile
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_passes_match_oracle(dtype, case):
    torch = _torch()
    B, H, W, Cin, Cout, ks, st, pad = case
    x = wl.random_normal(3, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    w = wl.random_normal(3, 2, Cout * ks * ks * Cin).reshape(Cout, ks, ks, Cin) / np.sqrt(ks * ks * Cin)
    xr, wr = _rnd(x, dtype), _rnd(w, dtype)
    y = L.conv2d_fwd(xr, wr, st, pad)
    dy = wl.random_normal(3, 3, y.size).reshape(y.shape)
    dyr = _rnd(dy, dtype)
    dx, dw = L.conv2d_bwd(xr, wr, st, pad, dyr)
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    tol_out = 2.0 ** -7 if dtype == wl.BF16 else 1e-5

    xd, wd, dyd = _dev(x, dtype), _dev(w, dtype), _dev(dy, dtype)
    yd = torch.full(y.shape, float("nan"), dtype=tdt, device="cuda")
    b.cdp_k_conv(dtype, 0, xd.data_ptr(), wd.data_ptr(), yd.data_ptr(), B, H, W, Cin, Cout, ks, st, pad)
    wtd = _dev(np.transpose(w, (3, 1, 2, 0)), dtype)        # [Cin][k][k][Cout]
    dxd = torch.full(x.shape, float("nan"), dtype=tdt, device="cuda")
    b.cdp_k_conv(dtype, 1, dyd.data_ptr(), wtd.data_ptr(), dxd.data_ptr(), B, H, W, Cin, Cout, ks, st, pad)
    dwd = torch.full(w.shape, float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.full((w.size * (y.size // Cout // 1024 + 4),), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_conv(dtype, 2, dyd.data_ptr(), xd.data_ptr(), dwd.data_ptr(), B, H, W, Cin, Cout, ks, st, pad,
                 ws.data_ptr(), ws.numel() * 4)
    dw2 = torch.full(w.shape, float("nan"), dtype=torch.float32, device="cuda")      # single-pass kernel, no workspace
    b.cdp_k_conv(dtype, 2, dyd.data_ptr(), xd.data_ptr(), dw2.data_ptr(), B, H, W, Cin, Cout, ks, st, pad)
    torch.cuda.synchronize()
    for name, got, ref, tol in (("fwd", yd, y, tol_out), ("dgrad", dxd, dx, tol_out), ("wgrad", dwd, dw, 1e-5),
                                ("wgrad-1pass", dw2, dw, 1e-5)):
        g = got.float().cpu().numpy().astype(np.float64)
        assert np.isfinite(g).all(), name
        err = np.abs(g - ref).max() / max(1e-6, np.abs(ref).max())
        assert err <= tol, (name, err)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", [(1, 7, 7, 512, 512, 3, 1, 1),     # 8 tiles of 64 x 64, 72 slabs, eight workgroups a tile
                                  (2, 5, 5, 256, 136, 3, 1, 1),     # ragged in both directions
                                  (1, 1, 130, 2048, 64, 1, 1, 0), (3, 9, 7, 192, 96, 3, 2, 1), (1, 3, 3, 1000, 72, 3, 1, 1),
                                  (4, 8, 8, 32, 40, 3, 1, 1),       # fp32: two slabs of 32 a tap, too short to share
                                  (2, 14, 14, 64, 256, 3, 1, 1)])
def test_conv_launches_of_the_engine(dtype, case):
    """Forward and data gradient as the engine launches them (which = 7, 8): few tiles share their reductions over workgroups in a
    workspace whose counters are zero again afterwards.  Twice with the same bits."""
    torch = _torch()
    B, H, W, Cin, Cout, ks, st, pad = case
    x = wl.random_normal(3, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    w = wl.random_normal(3, 2, Cout * ks * ks * Cin).reshape(Cout, ks, ks, Cin) / np.sqrt(ks * ks * Cin)
    xr, wr = _rnd(x, dtype), _rnd(w, dtype)
    y = L.conv2d_fwd(xr, wr, st, pad)
    dy = wl.random_normal(3, 3, y.size).reshape(y.shape)
    dx, _ = L.conv2d_bwd(xr, wr, st, pad, _rnd(dy, dtype))
    tol = 2.0 ** -7 if dtype == wl.BF16 else 1e-5
    share = (32 << 20) + 8192
    ws = torch.full((share,), 255, dtype=torch.uint8, device="cuda")
    ws[-8192:] = 0
    xd, wd, dyd, wtd = _dev(x, dtype), _dev(w, dtype), _dev(dy, dtype), _dev(np.transpose(w, (3, 1, 2, 0)), dtype)
    for which, a, k, ref in ((7, xd, wd, y), (8, dyd, wtd, dx)):
        got = []
        for _ in range(2):
            got.append(torch.full(ref.shape, float("nan"), dtype=xd.dtype, device="cuda"))
            b.cdp_k_conv(dtype, which, a.data_ptr(), k.data_ptr(), got[-1].data_ptr(), *case, ws_ptr=ws.data_ptr(), ws_bytes=share)
        torch.cuda.synchronize()
        assert torch.equal(got[0], got[1])
        assert int(ws[-8192:].sum()) == 0
        _close(got[0], ref, tol, which)
    with pytest.raises(b.CdpError):
        b.cdp_k_conv(dtype, 7, xd.data_ptr(), wd.data_ptr(), got[0].data_ptr(), *case, ws_ptr=ws.data_ptr(), ws_bytes=share - 1)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", [(2, 8, 8, 32, 64, 3, 1, 1), (8, 28, 28, 24, 40, 3, 1, 1), (1, 1, 200, 512, 4104, 1, 1, 0), (4, 20, 20, 16, 16, 3, 1, 1)])
def test_conv_weight_gradient_added_to_an_accumulator(dtype, case):
    """which = 9: the fold adds to what dw holds, as in a step of several micro-batches; by rows (4104 of them) and by pieces, with one
    range and with many."""
    torch = _torch()
    B, H, W, Cin, Cout, ks, st, pad = case
    Ho, Wo = (H + 2 * pad - ks) // st + 1, (W + 2 * pad - ks) // st + 1
    x = wl.random_normal(6, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    dy = wl.random_normal(6, 2, B * Ho * Wo * Cout).reshape(B, Ho, Wo, Cout)
    _, dw = L.conv2d_bwd(_rnd(x, dtype), np.zeros((Cout, ks, ks, Cin)), st, pad, _rnd(dy, dtype))
    old = wl.random_normal(6, 3, dw.size).reshape(dw.shape) * np.abs(dw).max()
    xd, dyd = _dev(x, dtype), _dev(dy, dtype)
    for sums in (1, B * Ho * Wo // 512 + 4):
        got = _dev(old, wl.F32)
        ws = torch.full((dw.size * sums,), float("nan"), dtype=torch.float32, device="cuda")
        b.cdp_k_conv(dtype, 9, dyd.data_ptr(), xd.data_ptr(), got.data_ptr(), *case, ws_ptr=ws.data_ptr(), ws_bytes=ws.numel() * 4)
        torch.cuda.synchronize()
        # products of exactly representable inputs, fp32 sums
        _close(got, _rnd(old, wl.F32) + dw, 1e-5, sums)
    with pytest.raises(b.CdpError):
        b.cdp_k_conv(dtype, 9, dyd.data_ptr(), xd.data_ptr(), got.data_ptr(), *case)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", [(4, 40, 40, 8, 40, 3, 1, 1), (4, 40, 40, 16, 24, 3, 1, 1)])
def test_conv_weight_gradient_fold_of_many_ranges(dtype, case):
    """Folds at every number of 32-lane groups to a weight row, rows that end inside a chunk of 128 columns; nothing around the
    accumulator is touched."""
    torch = _torch()
    B, H, W, Cin, Cout, ks, st, pad = case
    x = wl.random_normal(8, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    dy = wl.random_normal(8, 2, B * H * W * Cout).reshape(B, H, W, Cout)
    _, dw = L.conv2d_bwd(_rnd(x, dtype), np.zeros((Cout, ks, ks, Cin)), st, pad, _rnd(dy, dtype))
    old = wl.random_normal(8, 3, dw.size).reshape(dw.shape) * np.abs(dw).max()
    xd, dyd = _dev(x, dtype), _dev(dy, dtype)
    for sums in (1, 7, 9, 30, 60):
        for which in (2, 9):
            mem = torch.full((dw.size + 16,), 7.0, dtype=torch.float32, device="cuda")
            mem[8:8 + dw.size] = _dev(old, wl.F32).flatten()
            ws = torch.full((dw.size * sums,), float("nan"), dtype=torch.float32, device="cuda")
            b.cdp_k_conv(dtype, which, dyd.data_ptr(), xd.data_ptr(), mem.data_ptr() + 32, *case, ws_ptr=ws.data_ptr(), ws_bytes=ws.numel() * 4)
            torch.cuda.synchronize()
            got = mem[8:8 + dw.size].reshape(dw.shape)
            # products of exactly representable inputs, fp32 sums
            _close(got, dw if which == 2 else _rnd(old, wl.F32) + dw, 1e-5, (sums, which))
            assert bool((mem[:8] == 7).all()) and bool((mem[8 + dw.size:] == 7).all())


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("sums", [1, 2, 5, 12])
@pytest.mark.parametrize("case", [(1, 1, 1, 8, 8, 1, 1, 0),       # one position
                                  (3, 5, 7, 24, 40, 3, 1, 1),     # 105 positions: a group (or slab) and a part of one
                                  (2, 8, 8, 8, 72, 3, 1, 1),      # 128 positions: whole slabs; a second row of tiles with 8 rows
                                  (3, 8, 8, 16, 64, 5, 1, 2),     # 25 taps, 400 columns
                                  (5, 9, 9, 40, 136, 3, 2, 1),    # stride 2 on an odd map
                                  (4, 11, 13, 48, 24, 1, 2, 0),   # 1x1, stride 2: gathered
                                  (2, 1, 321, 136, 200, 1, 1, 0), # plain rows, 642 positions: every remainder of the three stages
                                  (1, 1, 961, 32, 32, 1, 1, 0)])
def test_conv_weight_gradient_short_of_workgroups(dtype, case, sums):
    """The tiles of launches short of workgroups, from one range to several (some of them empty), operands 16-byte aligned and not,
    against the oracle; nothing is written past the result."""
    torch = _torch()
    B, H, W, Cin, Cout, ks, st, pad = case
    Ho, Wo = (H + 2 * pad - ks) // st + 1, (W + 2 * pad - ks) // st + 1
    x = wl.random_normal(6, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    dy = wl.random_normal(6, 2, B * Ho * Wo * Cout).reshape(B, Ho, Wo, Cout)
    _, dw = L.conv2d_bwd(_rnd(x, dtype), np.zeros((Cout, ks, ks, Cin)), st, pad, _rnd(dy, dtype))
    xd = _dev(x, dtype)
    for shift in (0, 4):
        room = torch.empty(dy.size + 8, dtype=xd.dtype, device="cuda")
        dyd = room[shift:shift + dy.size]
        dyd.copy_(_dev(dy, dtype).reshape(-1))
        got = torch.full((dw.size + 64,), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.full((dw.size * sums + 64,), float("nan"), dtype=torch.float32, device="cuda")
        b.cdp_k_conv(dtype, 2, dyd.data_ptr(), xd.data_ptr(), got.data_ptr(), *case, ws_ptr=ws.data_ptr(), ws_bytes=dw.size * sums * 4)
        torch.cuda.synchronize()
        assert torch.isnan(got[dw.size:]).all() and torch.isnan(ws[dw.size * sums:]).all(), "written past the end"
        # products of exactly representable inputs, fp32 sums
        _close(got[:dw.size].reshape(dw.shape), dw, 1e-5, (sums, shift))


LARGE_TILE_CASES = [
    # pass, B, H, W, Cin, Cout, ks, stride, pad: shapes that fill the chip with 256 x 256 tiles
    ("fwd", 16, 56, 56, 64, 256, 3, 1, 1),
    ("dgrad", 16, 56, 56, 256, 64, 3, 1, 1),
    ("fwd", 64, 56, 56, 64, 256, 3, 2, 1),       # stride 2: padding on one side only
    ("dgrad", 16, 56, 56, 256, 64, 3, 2, 1),     # stride 2: taps on the stride lattice
    ("dgrad", 4, 45, 45, 4040, 128, 1, 1, 0),    # ragged in both directions
    ("fwd", 8, 28, 28, 1024, 2048, 1, 1, 0),     # 16 slabs
    ("fwd", 2, 9, 7, 64, 64, 3, 1, 1),           # a single ragged tile
    ("dgrad", 3, 10, 10, 64, 128, 3, 2, 1),
]


@pytest.mark.parametrize("tile", ["256x256", "256x128"])
@pytest.mark.parametrize("case", LARGE_TILE_CASES)
def test_conv_large_tile_matches_oracle(case, tile):
    """Forward / data gradient on the direct-to-LDS kernel (bf16; swizzled rows), 256 x 256 tiles with two stages and 256 x 128 tiles
    with three, against the oracle's convolution."""
    torch = _torch()
    which, B, H, W, Cin, Cout, ks, st, pad = case
    dtype = wl.BF16
    x = wl.random_normal(7, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    w = wl.random_normal(7, 2, Cout * ks * ks * Cin).reshape(Cout, ks, ks, Cin) / np.sqrt(ks * ks * Cin)
    xr, wr = _rnd(x, dtype), _rnd(w, dtype)
    if which == "fwd":
        ref = L.conv2d_fwd(xr, wr, st, pad)
        xd, wd = _dev(x, dtype), _dev(w, dtype)
        got = torch.full(ref.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        b.cdp_k_conv(dtype, 3 if tile == "256x256" else 5, xd.data_ptr(), wd.data_ptr(), got.data_ptr(), B, H, W, Cin, Cout, ks, st, pad)
    else:
        Ho, Wo = (H + 2 * pad - ks) // st + 1, (W + 2 * pad - ks) // st + 1
        dy = wl.random_normal(7, 3, B * Ho * Wo * Cout).reshape(B, Ho, Wo, Cout)
        ref, _ = L.conv2d_bwd(xr, wr, st, pad, _rnd(dy, dtype))
        dyd, wtd = _dev(dy, dtype), _dev(np.transpose(w, (3, 1, 2, 0)), dtype)
        got = torch.full(x.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        b.cdp_k_conv(dtype, 4 if tile == "256x256" else 6, dyd.data_ptr(), wtd.data_ptr(), got.data_ptr(), B, H, W, Cin, Cout, ks, st, pad)
    torch.cuda.synchronize()
    g = got.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all()
    assert np.abs(g - ref).max() / np.abs(ref).max() <= 2.0 ** -7


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("which", ["fwd", "dgrad"])
def test_conv_gemm_many_tiles(dtype, which):
    """A 1x1 convolution with 8100 positions and 4040 output (forward) or input (data gradient)
    channels: about two thousand of the largest tiles (several rounds over the chip), ragged in
    both directions."""
    torch = _torch()
    B, H, W = 4, 45, 45
    Cin, Cout = (128, 4040) if which == "fwd" else (4040, 128)
    x = wl.random_normal(5, 1, B * H * W * Cin).reshape(B, H, W, Cin)
    w = wl.random_normal(5, 2, Cout * Cin).reshape(Cout, 1, 1, Cin) / np.sqrt(Cin)
    xr, wr = _rnd(x, dtype), _rnd(w, dtype)
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    tol = 2.0 ** -7 if dtype == wl.BF16 else 1e-5
    if which == "fwd":
        ref = L.conv2d_fwd(xr, wr, 1, 0)
        xd, wd = _dev(x, dtype), _dev(w, dtype)
        got = torch.full(ref.shape, float("nan"), dtype=tdt, device="cuda")
        b.cdp_k_conv(dtype, 0, xd.data_ptr(), wd.data_ptr(), got.data_ptr(), B, H, W, Cin, Cout, 1, 1, 0)
    else:
        dy = wl.random_normal(5, 3, B * H * W * Cout).reshape(B, H, W, Cout)
        dyr = _rnd(dy, dtype)
        ref, _ = L.conv2d_bwd(xr, wr, 1, 0, dyr)
        dyd, wtd = _dev(dy, dtype), _dev(np.transpose(w, (3, 1, 2, 0)), dtype)
        got = torch.full(x.shape, float("nan"), dtype=tdt, device="cuda")
        b.cdp_k_conv(dtype, 1, dyd.data_ptr(), wtd.data_ptr(), got.data_ptr(), B, H, W, Cin, Cout, 1, 1, 0)
    torch.cuda.synchronize()
    g = got.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all()
    assert np.abs(g - ref).max() / np.abs(ref).max() <= tol


def _close(got, ref, tol, what):
    g = got.float().cpu().numpy().astype(np.float64).reshape(ref.shape)
    assert np.isfinite(g).all(), what
    err = np.abs(g - ref).max() / max(1e-6, np.abs(ref).max())
    assert err <= tol, (what, err)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,C", [(6272, 768), (100, 20), (37, 1000), (5, 3)])
def test_layernorm_kernels_match_oracle(dtype, rows, C):
    """Forward and backward (with a residual addend and running gamma / beta sums) at the
    ViT-B/16 shape and at ragged ones (rows that are not whole 16-byte chunks take the
    element-wise kernels)."""
    torch = _torch()
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    x = wl.random_normal(7, 1, rows * C).reshape(rows, C) * 1.5 + 0.3
    dy = wl.random_normal(7, 2, rows * C).reshape(rows, C)
    add = wl.random_normal(7, 3, rows * C).reshape(rows, C)
    gamma = 1.0 + 0.2 * wl.random_normal(7, 4, C)
    beta = 0.1 * wl.random_normal(7, 5, C)
    g0, b0 = wl.random_normal(7, 6, C), wl.random_normal(7, 7, C)   # running sums the backward adds to
    xr, dyr, addr = _rnd(x, dtype), _rnd(dy, dtype), _rnd(add, dtype)
    gam, bet = _rnd(gamma, wl.F32), _rnd(beta, wl.F32)
    y = L.layernorm_fwd(xr, gam, bet)
    dx, dg, db = L.layernorm_bwd(xr, gam, dyr)
    xd, dyd, addd = _dev(x, dtype), _dev(dy, dtype), _dev(add, dtype)
    gd, bd = _dev(gamma, wl.F32), _dev(beta, wl.F32)
    yd = torch.full((rows, C), float("nan"), dtype=tdt, device="cuda")
    b.cdp_k_layernorm(dtype, 0, xd.data_ptr(), 0, 0, gd.data_ptr(), bd.data_ptr(), yd.data_ptr(), 0, 0, 0, 0, rows, C)
    dxd = torch.full((rows, C), float("nan"), dtype=tdt, device="cuda")
    dgd, dbd = _dev(g0, wl.F32), _dev(b0, wl.F32)
    ws = torch.full((2 * rows + 2 * C * ((rows + 31) // 32) + 64,), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_layernorm(dtype, 1, xd.data_ptr(), dyd.data_ptr(), addd.data_ptr(), gd.data_ptr(), 0, dxd.data_ptr(),
                      dgd.data_ptr(), dbd.data_ptr(), ws.data_ptr(), ws.numel() * 4, rows, C)
    torch.cuda.synchronize()
    tol = 2.0 ** -7 if dtype == wl.BF16 else 1e-5
    _close(yd, y, tol, "y")
    _close(dxd, dx + addr, tol, "dx")
    _close(dgd, _rnd(g0, wl.F32) + dg, 1e-5, "dgamma")
    _close(dbd, _rnd(b0, wl.F32) + db, 1e-5, "dbeta")


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_gelu_kernels_match_oracle(dtype):
    torch = _torch()
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    n = 1000003   # not a multiple of the vector width: the tail runs element by element
    x = wl.random_normal(8, 1, n) * 2.0
    dy = wl.random_normal(8, 2, n)
    xr, dyr = _rnd(x, dtype), _rnd(dy, dtype)
    xd, dyd = _dev(x, dtype), _dev(dy, dtype)
    yd = torch.full((n,), float("nan"), dtype=tdt, device="cuda")
    dxd = torch.full((n,), float("nan"), dtype=tdt, device="cuda")
    b.cdp_k_gelu(dtype, 0, xd.data_ptr(), 0, yd.data_ptr(), n)
    b.cdp_k_gelu(dtype, 1, xd.data_ptr(), dyd.data_ptr(), dxd.data_ptr(), n)
    torch.cuda.synchronize()
    tol = 2.0 ** -7 if dtype == wl.BF16 else 2e-6
    _close(yd, L.gelu_fwd(xr), tol, "gelu")
    _close(dxd, L.gelu_bwd(xr, dyr), tol, "dgelu")


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("B,T,D,heads", [(2, 196, 768, 12), (3, 9, 20, 4), (1, 324, 16, 2), (2, 16, 32, 4), (2, 50, 64, 2),
                                         (1, 256, 128, 2), (1, 33, 64, 1), (1, 70, 160, 2), (2, 129, 48, 3), (1, 200, 96, 1),
                                         (1, 260, 64, 2)])
def test_attention_kernels_match_oracle(dtype, B, T, D, heads):
    """Probabilities, output and the gradient with respect to q | k | v: the ViT-B/16 shape,
    a shape where nothing is a multiple of four (element-wise staging, ragged tiles), 324
    tokens, the reduced test shape, heads of width 32 / 64 with 50, 256 and 33 tokens; in bf16 head widths 80 and 16 (the
    widest and narrowest of the fused kernels) and 96 (too wide for them), 256 and 260 tokens (scores kept in registers up to 256,
    contracted twice past that), 129 tokens (a second workgroup of one query)."""
    torch = _torch()
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    eb = 2 if dtype == wl.BF16 else 4
    qkv = wl.random_normal(9, 1, B * T * 3 * D).reshape(B, 1, T, 3 * D)
    dout = wl.random_normal(9, 2, B * T * D).reshape(B, 1, T, D)
    qr, dor = _rnd(qkv, dtype), _rnd(dout, dtype)
    # the stored probabilities and the stored score gradient carry the element type's rounding
    P = _rnd(L.attention_probs(qr, heads), dtype)
    out = L.attention_apply(qr, P, heads)
    dqkv = L.attention_input_grad(qr, P, _rnd(L.attention_score_grad(qr, P, heads, dor), dtype), heads, dor)
    qd, dod = _dev(qkv, dtype), _dev(dout, dtype)
    tt = B * heads * T * T
    Pd = torch.full((B, heads, T, T), float("nan"), dtype=tdt, device="cuda")
    outd = torch.full((B, T, D), float("nan"), dtype=tdt, device="cuda")
    dqd = torch.full((B, T, 3 * D), float("nan"), dtype=tdt, device="cuda")
    ws = torch.full((2 * tt + 128,), float("nan"), dtype=torch.float32, device="cuda")
    b.cdp_k_attention(dtype, 0, qd.data_ptr(), Pd.data_ptr(), 0, outd.data_ptr(), ws.data_ptr(), ws.numel() * 4, B, T, D, heads)
    b.cdp_k_attention(dtype, 1, qd.data_ptr(), Pd.data_ptr(), dod.data_ptr(), dqd.data_ptr(), ws.data_ptr(), ws.numel() * 4,
                      B, T, D, heads)
    torch.cuda.synchronize()
    tol = 2.0 ** -6 if dtype == wl.BF16 else 2e-5
    _close(Pd, P, tol, "P")
    _close(outd, out, tol, "out")
    _close(dqd, dqkv, tol, "dqkv")



@pytest.mark.parametrize("B,T,D,heads", [(2, 208, 128, 2), (1, 17, 48, 3), (2, 224, 64, 1), (1, 400, 160, 2), (1, 321, 48, 1),
                                         (1, 624, 64, 1), (1, 640, 64, 1), (1, 577, 128, 2), (1, 255, 80, 1), (1, 262, 96, 2),
                                         (2, 364, 96, 2), (2, 368, 96, 2), (1, 384, 160, 2)])
def test_attention_fused_edges(B, T, D, heads):
    """Edges of the fused kernels: token counts that end on 16 of a block of 32, one token past a step of 16, more than
    256 tokens (scores contracted twice), the last count that fits LDS and one past it (separate kernels); rows of
    probabilities that start at any element, in each of the pieces that move at once; both sides of the line from which heads
    of width 48 and 80 have their backward in separate kernels."""
    test_attention_kernels_match_oracle(wl.BF16, B, T, D, heads)


@pytest.mark.parametrize("B,T,D,heads", [(1, 1, 8, 1), (2, 31, 40, 5), (1, 33, 96, 1), (1, 128, 72, 1), (1, 129, 64, 2), (1, 385, 32, 1),
                                         (1, 1021, 96, 2), (1, 1024, 80, 1), (1, 64, 104, 1),
                                         (26, 129, 32, 4), (29, 257, 16, 2), (76, 260, 32, 4)])
def test_attention_fused_edges_fp32(B, T, D, heads):
    """The fp32 kernels: a single token, one block of 32 short of one and one more, one to four blocks per
    wavefront, rows of probabilities that are not whole pieces, head widths 8 to 96 and one past them; enough workgroups
    for four wavefronts with two and four blocks each, and for the separate kernels backward."""
    test_attention_kernels_match_oracle(wl.F32, B, T, D, heads)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,C", [(1, 8), (17, 1024), (33, 64), (4100, 520), (8200, 16)])
def test_layernorm_whole_chunk_edges(dtype, rows, C):
    """The one-pass backward: one row, the widest row, a wavefront without a row, several rows per wavefront."""
    test_layernorm_kernels_match_oracle(dtype, rows, C)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,C", [(1, 1), (6, 63), (9, 65), (300, 255), (13, 257), (7, 1021), (5, 1023)])
def test_layernorm_ragged_edges(dtype, rows, C):
    """Rows that are not whole 16-byte pieces: around one value per lane, the widths where a lane holds four and sixteen, the widest."""
    test_layernorm_kernels_match_oracle(dtype, rows, C)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,C", [(6272, 768), (4100, 64), (40, 128)])
def test_layernorm_backward_does_not_depend_on_its_launch(dtype, rows, C):
    """A problem's gradients have the same bits whether it is launched alone or with others of its shape, as the engine does."""
    import ctypes
    torch = _torch()
    launch = getattr(b.lib(), "_ZN3cdp26launch_layernorm_bwd_batchERKNS_10LnBwdBatchEiiiP12ihipStream_t")

    class Prob(ctypes.Structure):
        _fields_ = [(n, ctypes.c_void_p) for n in ("x", "dy", "add", "gamma", "dx", "Ggamma", "Gbeta", "workspace")]

    class Batch(ctypes.Structure):
        _fields_ = [("p", Prob * 8), ("n", ctypes.c_int)]      # LnBwdBatch of csrc/kernels.h

    def run(n):
        batch, out = Batch(), []
        batch.n = n
        for q in range(n):
            gen = torch.Generator(device="cuda")
            gen.manual_seed(q)
            r = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
            x, dy = (r(rows, C).to(torch.bfloat16 if dtype == wl.BF16 else torch.float32) for _ in range(2))
            o = dict(x=x, dy=dy, gamma=r(C), dx=torch.empty_like(x), Ggamma=torch.zeros(C, device="cuda"), Gbeta=torch.zeros(C, device="cuda"),
                     workspace=torch.empty(2 * rows + 2 * C * ((rows + 31) // 32) + 64, device="cuda"))
            for k, t in o.items():
                setattr(batch.p[q], k, t.data_ptr())
            out.append(o)
        torch.cuda.synchronize()
        assert launch(ctypes.byref(batch), rows, C, dtype, None) == 0
        torch.cuda.synchronize()
        return out

    alone, shared = run(1)[0], run(5)[0]
    for k in ("dx", "Ggamma", "Gbeta"):
        assert torch.equal(alone[k], shared[k]), k


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_gelu_over_the_whole_range(dtype):
    """Tails, zeros and infinities: Phi of large negative arguments has to vanish, the derivative too."""
    torch = _torch()
    tdt = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    x = np.concatenate([np.linspace(-40.0, 40.0, 8003), [0.0, -0.0, 1e-30, -1e-30, 3e38, -3e38]])
    dy = np.ones_like(x)
    xr = _rnd(x, dtype)
    xd, dyd = _dev(x, dtype), _dev(dy, dtype)
    y, dx = torch.empty_like(xd), torch.empty_like(xd)
    b.cdp_k_gelu(dtype, 0, xd.data_ptr(), 0, y.data_ptr(), x.size)
    b.cdp_k_gelu(dtype, 1, xd.data_ptr(), dyd.data_ptr(), dx.data_ptr(), x.size)
    torch.cuda.synchronize()
    # half a unit in the last place of the stored type plus the fp32 error of Phi (2e-7) times |x|
    ulp = 2.0 ** -8 if dtype == wl.BF16 else 2.0 ** -23
    for got, ref in ((y, L.gelu_fwd(xr)), (dx, L.gelu_bwd(xr, dy))):
        g = got.float().cpu().numpy().astype(np.float64)
        assert (np.abs(g - ref) <= ulp * np.abs(ref) + 4e-7 * np.maximum(1.0, np.minimum(np.abs(xr), 10.0))).all()


def _conv_1x1_bf16(which, rows, cin, cout, seed=3):
    """A 1x1 convolution over `rows` positions through cdp_k_conv against the fp64 product."""
    torch = _torch()
    red, out = (cin, cout) if which == 0 else (cout, cin)
    a = wl.random_normal(seed, 1, rows * red).reshape(rows, red)
    w = wl.random_normal(seed, 2, out * red).reshape(out, red) / np.sqrt(red)
    ref = _rnd(a, wl.BF16) @ _rnd(w, wl.BF16).T
    ad, wd = _dev(a, wl.BF16), _dev(w, wl.BF16)
    got = torch.full((rows, out), float("nan"), dtype=torch.bfloat16, device="cuda")
    b.cdp_k_conv(wl.BF16, which, ad.data_ptr(), wd.data_ptr(), got.data_ptr(), 1, 1, rows, cin, cout, 1, 1, 0)
    torch.cuda.synchronize()
    g = got.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all()
    assert np.abs(g - ref).max() / np.abs(ref).max() <= 2.0 ** -7


@pytest.mark.parametrize("rows,out", [(4100, 1032), (19300, 120), (700, 200), (190, 72), (513, 40)])
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5, 6, 7, 16, 17, 18])
def test_conv_short_of_workgroups(rows, out, slabs):
    """The tiles of the launches that do not fill the chip (192 x 128, 128 x 128, 64 x 64 with slabs of 64 and of 32), ragged
    in both directions, with every number of slabs that the unrolled pipeline can end on; forward and data gradient."""
    for red in ((64 * slabs, 32 * slabs) if slabs <= 7 else (64 * slabs,)):
        _conv_1x1_bf16(0, rows, red, out)
        _conv_1x1_bf16(1, rows, out, red)


@pytest.mark.parametrize("rows,out,slabs", [(13000, 500, 1), (13000, 500, 2), (13000, 500, 5),    # 256 x 128: 272 tiles of 192 x 128
                                            (9310, 1032, 16), (9310, 1032, 17),                    # 192 x 128, 441 tiles in two rounds
                                            (16330, 256, 3),                                       # 128 x 128, a full round (256 tiles)
                                            (16390, 256, 3)])                                      # a tile row more: 192 x 128
def test_conv_rounds_of_tiles(rows, out, slabs):
    """One round of tiles or two, at the lines of the rule."""
    _conv_1x1_bf16(0, rows, 64 * slabs, out)


@pytest.mark.parametrize("which,rows,cin,cout", [(0, 1041000, 64, 1032), (3, 1041000, 64, 1032), (5, 1041000, 64, 1032), (10, 1041000, 64, 1032),
                                                 (4, 1041000, 1032, 64),                                   # results of more than 2 GiB
                                                 (0, 33554430, 64, 72), (3, 33554430, 64, 72)])            # an operand of 4 GiB less two rows
def test_conv_tiles_of_large_tensors(which, rows, cin, cout):
    """Exact: -1, 0 and 1, whole numbers of at most 64 in bf16."""
    torch = _torch()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(which)
    k, n = (cout, cin) if which == 4 else (cin, cout)
    x = torch.randint(-1, 2, (rows, k), generator=gen, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    w = torch.randint(-1, 2, (n, k), generator=gen, device="cuda").to(torch.bfloat16)
    y = torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    act = torch.full((rows, n) if which == 10 else (1, 1), float("nan"), dtype=torch.bfloat16, device="cuda")
    b.cdp_k_conv(wl.BF16, which, x.data_ptr(), w.data_ptr(), y.data_ptr(), rows, 1, 1, cin, cout, 1, 1, 0, ws_ptr=act.data_ptr(), ws_bytes=act.numel() * 2)
    torch.cuda.synchronize()
    wf = w.float().T.contiguous()
    for i in range(0, rows, 1 << 20):
        assert torch.equal(y[i:i + (1 << 20)], (x[i:i + (1 << 20)].float() @ wf).to(torch.bfloat16)), i
    if which == 10:
        ref = torch.empty_like(y)
        b.cdp_k_gelu(wl.BF16, 0, y.data_ptr(), 0, ref.data_ptr(), y.numel())
        torch.cuda.synchronize()
        assert torch.equal(act, ref)


def _launch_tile(rows, out, depth, beside=False):
    """conv_launch_tile for one product, asked of the library as tests/launch_rules/tiles.cpp does."""
    import os
    import subprocess
    here = os.path.dirname(os.path.abspath(b.__file__))
    exe = os.path.join(_launch_tile.folder, "tiles")
    if not os.path.exists(exe):
        subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(here, "csrc"),
                        os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_rules", "tiles.cpp"), "-o", exe, os.path.join(here, "libcdp.so"),
                        "-Wl,-rpath," + here, "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    line = "%d %d %d 0 %d\n" % (rows, out, depth, 2 * beside)
    return int(subprocess.run([exe], input=line, capture_output=True, text=True, check=True, timeout=60).stdout)


@pytest.fixture(scope="module")
def launch_tile(tmp_path_factory):
    _launch_tile.folder = str(tmp_path_factory.mktemp("tiles"))
    return _launch_tile


# rows, columns, slabs of 64, tile
@pytest.mark.parametrize("rows,out,slabs,tile", [(21800, 376, 6, 7), (21800, 376, 7, 7), (33000, 600, 9, 7), (140100, 72, 8, 7), (140100, 72, 7, 7),  # walked: odd
                                                 (8200, 1992, 8, 7),                                  # numbers of slabs and even, columns past a tile
                                                 (21800, 376, 1, 0), (33000, 600, 5, 0), (140100, 72, 1, 0),                       # conv_gemm_kernel
                                                 (65500, 136, 5, 1), (65500, 136, 9, 1), (24000, 2040, 34, 1),                     # 256 x 256
                                                 (21800, 376, 17, 6), (24000, 760, 34, 6)])                                        # 192 x 128
def test_conv_many_tiles(launch_tile, rows, out, slabs, tile):
    """Launches of 512 tiles of 128 x 128 and more."""
    assert launch_tile(rows, out, 64 * slabs) == tile
    _conv_1x1_bf16(0, rows, 64 * slabs, out)


@pytest.fixture(scope="module")
def many(tmp_path_factory):
    """launch_conv_dl of several problems (tests/launch_rules/many.cpp)."""
    import ctypes
    import os
    import subprocess
    here = os.path.dirname(os.path.abspath(b.__file__))
    so = str(tmp_path_factory.mktemp("many") / "many.so")
    b.lib()
    subprocess.run(["g++", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(here, "csrc"),
                    os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_rules", "many.cpp"), "-o", so, os.path.join(here, "libcdp.so"),
                    "-Wl,-rpath," + here, "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    f = ctypes.CDLL(so).many

    def launch(tile, problems):  # (A, B, out)
        mnk = [v for a, w, _ in problems for v in (a.shape[0], w.shape[0], a.shape[1])]
        ptrs = [x.data_ptr() for p in problems for x in p]
        assert f(len(problems), (ctypes.c_int * len(mnk))(*mnk), (ctypes.c_void_p * len(ptrs))(*ptrs), tile, None) == 0
    return launch


WALKED = 7


@pytest.mark.parametrize("n,tiles", [(1, 63), (1, 513), (2, 64), (2, 511), (2, 513), (3, 575), (3, 1025), (5, 640), (5, 1999), (8, 512), (8, 700), (16, 1100), (24, 449), (24, 1600)])
def test_conv_many_tiles_of_several_problems(many, n, tiles):
    """Launches of several problems on the walked tiles: the workgroups' shares are every tile of every problem.  Reductions of 1 to 16 slabs, odd ones
    among them, tile counts around whole rounds, one problem with most of the tiles, columns past a tile.  Exact: -1, 0 and 1, small whole sums."""
    torch = _torch()
    gen = torch.Generator(device="cuda")
    for seed in range(3):
        gen.manual_seed(100 * tiles + 10 * n + seed)
        rng = np.random.default_rng(1000 * n + tiles + seed)
        cuts = np.sort(rng.choice(np.arange(1, tiles), n - 1, replace=False)) if seed else np.arange(1, n)  # seed 0: all but the last have one tile
        problems, refs = [], []
        for count in np.diff(np.concatenate(([0], cuts, [tiles]))):
            cols = max(c for c in (1, 2, 3, 4) if count % c == 0 and (seed or c == 1))
            m, k = 128 * int(count // cols) - int(rng.integers(0, 127)), 64 * int(rng.integers(1, 17 if count < 300 else 6))
            x = torch.randint(-1, 2, (m, k), generator=gen, device="cuda").to(torch.bfloat16)
            w = torch.randint(-1, 2, (128 * cols - 8 * int(rng.integers(0, 15)), k), generator=gen, device="cuda").to(torch.bfloat16)
            problems.append((x, w, torch.full((m, w.shape[0]), float("nan"), dtype=torch.bfloat16, device="cuda")))
            refs.append((x.float() @ w.float().T.contiguous()).to(torch.bfloat16))
        many(WALKED, problems)
        torch.cuda.synchronize()
        for (x, w, got), ref in zip(problems, refs):
            assert torch.equal(got, ref), (seed, tuple(x.shape), tuple(w.shape))


# tile of the forward and of the data gradient (0: also what is ragged)
@pytest.mark.parametrize("case,forward,backward", [((16, 57, 57, 64, 136, 3, 1, 1), 1, 0), ((24, 57, 57, 64, 72, 3, 1, 1), 7, 0), ((24, 57, 57, 72, 64, 3, 1, 1), 0, 7),
                                                   ((24, 57, 57, 136, 64, 3, 2, 1), 0, 7), ((24, 115, 113, 64, 136, 3, 2, 1), 7, 0)])
def test_conv_many_tiles_taps(launch_tile, case, forward, backward):
    """The same with taps, strides and padding."""
    B, H, W, cin, cout, k, st, pad = case
    out = B * ((H + 2 * pad - k) // st + 1) * ((W + 2 * pad - k) // st + 1)
    for rows, n, c, tile in ((out, cout, cin, forward), (B * H * W, cin, cout, backward)):
        assert (launch_tile(rows, n, k * k * c) if c % 64 == 0 else 0) == tile
    test_conv_passes_match_oracle(wl.BF16, case)


# rows, width beside the GELU, reduction: every tile that a contraction before or after a GELU can run on, ragged in both directions
GELU_CASES = [(700, 200, 64, "64 x 64, slabs of 32"), (700, 200, 1088, "64 x 64, slabs of 64"), (700, 200, 96, "64 x 64, odd multiple of 32"),
              (9700, 200, 128, "128 x 128 in one round"), (13000, 264, 192, "192 x 128"), (16500, 376, 128, "256 x 128"),
              (9310, 1032, 1088, "192 x 128, two rounds"), (12540, 1016, 2048, "256 x 256"), (22000, 376, 128, "conv 128 x 128"),
              (22000, 376, 96, "conv 128 x 128, slabs of 32"), (700, 200, 72, "ragged 64 x 64"), (12000, 264, 72, "ragged 64 x 128"),
              (22000, 376, 40, "ragged 128 x 128")]


@pytest.mark.parametrize("rows,width,red,tile", GELU_CASES, ids=[c[3] for c in GELU_CASES])
def test_gelu_in_the_epilogue_has_the_bits_of_its_own_kernels(rows, width, red, tile):
    """Forward: the contraction and the GELU of it; data gradient: times the GELU's derivative.  Bit for bit what the plain contraction
    followed by cdp_k_gelu gives, nothing written past the end, and the contraction itself within rounding of float64."""
    torch = _torch()
    n = rows * width
    x = _dev(wl.random_normal(8, 1, rows * red).reshape(rows, red), wl.BF16)
    w = _dev(wl.random_normal(8, 2, width * red).reshape(width, red) / np.sqrt(red), wl.BF16)
    h = _dev(wl.random_normal(8, 3, n), wl.BF16)
    new = lambda: torch.full((n + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    y, act, y0, act0, dx, dx0, plain = (new() for _ in range(7))
    fwd, bwd = (1, 1, rows, red, width, 1, 1, 0), (1, 1, rows, width, red, 1, 1, 0)
    b.cdp_k_conv(wl.BF16, 10, x.data_ptr(), w.data_ptr(), y.data_ptr(), *fwd, ws_ptr=act.data_ptr(), ws_bytes=2 * n)
    b.cdp_k_conv(wl.BF16, 0, x.data_ptr(), w.data_ptr(), y0.data_ptr(), *fwd)
    b.cdp_k_gelu(wl.BF16, 0, y0.data_ptr(), 0, act0.data_ptr(), n)
    b.cdp_k_conv(wl.BF16, 11, x.data_ptr(), w.data_ptr(), dx.data_ptr(), *bwd, ws_ptr=h.data_ptr(), ws_bytes=2 * n)
    b.cdp_k_conv(wl.BF16, 1, x.data_ptr(), w.data_ptr(), plain.data_ptr(), *bwd)
    b.cdp_k_gelu(wl.BF16, 1, h.data_ptr(), plain.data_ptr(), dx0.data_ptr(), n)
    torch.cuda.synchronize()
    for got, ref in ((y, y0), (act, act0), (dx, dx0)):
        assert torch.isnan(got[n:]).all()
        assert torch.equal(got[:n].view(torch.int16), ref[:n].view(torch.int16))
    exact = x.double() @ w.double().t()
    err = (y[:n].reshape(rows, width).double() - exact).norm() / exact.norm()
    assert err < 2.0 ** -8, float(err)  # one rounding to bf16: at most half a unit of 2^-7


@pytest.mark.parametrize("case", [(4, 56, 56, 64, 320, 3, 1, 1),       # forward on 192 x 128 tiles, data gradient on 64 x 64
                                  (8, 41, 41, 64, 136, 3, 1, 1),       # forward on 128 x 128
                                  (8, 41, 41, 200, 192, 3, 1, 1),      # data gradient on 128 x 128
                                  (9, 57, 57, 64, 200, 3, 2, 1), (5, 33, 31, 128, 64, 5, 2, 2),
                                  (3, 13, 11, 192, 128, 3, 1, 1), (2, 15, 15, 128, 192, 3, 3, 1)])   # 64 x 64, long reductions
def test_conv_short_of_workgroups_taps(case):
    """The tiles of launches that do not fill the chip, with taps, strides and padding."""
    test_conv_passes_match_oracle(wl.BF16, case)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", [(8, 28, 28, 24, 136, 3, 1, 1), (16, 56, 56, 40, 40, 3, 2, 1), (2, 9, 9, 72, 200, 3, 1, 1),
                                  (1, 1, 3000, 120, 88, 1, 1, 0), (3, 7, 7, 8, 8, 5, 1, 2), (2, 11, 13, 40, 24, 3, 3, 1),
                                  (4, 1, 5000, 1000, 520, 1, 1, 0)])
def test_conv_channels_not_whole_slabs(dtype, case):
    """Channel counts that are whole 16-byte chunks but not whole reduction slabs: slabs across taps, a partial last slab,
    strides 1 to 3, every tile shape."""
    test_conv_passes_match_oracle(dtype, case)


@pytest.mark.parametrize("case", [(1, 1, 1, 32, 32, 1, 1, 0), (1, 5, 7, 96, 36, 1, 1, 0), (3, 9, 9, 64, 160, 3, 2, 1), (2, 8, 8, 32, 32, 5, 1, 2),
                                  (1, 1, 33, 160, 96, 1, 1, 0), (2, 11, 13, 32, 64, 3, 3, 1), (16, 1, 48, 64, 1024, 1, 1, 0),
                                  (16, 1, 49, 64, 1024, 1, 1, 0)])
def test_conv_few_tiles_fp32(case):
    """Tiles of 32 x 32 whose wavefronts share the reduction: one element of a tile, rows and columns past it, fewer slabs than
    wavefronts and one more, taps off the stride lattice, the last count of tiles that takes it and the first that does not."""
    test_conv_passes_match_oracle(wl.F32, case)
