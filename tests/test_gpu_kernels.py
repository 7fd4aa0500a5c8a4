"""GPU kernels against plain references: the join GEMM in its four
precisions and the Jacobi eigensolver."""
import numpy as np
import pytest

from tests.gpu_util import announce, need_gpu
from trg_inputs import random_matrix, random_symmetric, gram_like

pytestmark = pytest.mark.gpu


def _pad(x, r, c):
    out = np.zeros((r, c), dtype=x.dtype)
    out[: x.shape[0], : x.shape[1]] = x
    return out


@pytest.mark.parametrize("M,N,K", [(128, 128, 16), (256, 384, 160), (1024, 512, 1040), (128, 1280, 4096)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gemm_fp64(M, N, K, accumulate):
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm
    announce("gemm fp64", M, N, K, accumulate)
    A = random_matrix(M, K, 1)
    B = random_matrix(N, K, 2)
    C0 = random_matrix(M, N, 3)
    dA = torch.from_numpy(A).cuda()
    dB = torch.from_numpy(B).cuda()
    dC = torch.from_numpy(C0).cuda()
    trg_gemm("fp64", dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K, K, K, N, accumulate,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref = A @ B.T + (C0 if accumulate else 0)
    got = dC.cpu().numpy()
    scale = np.abs(A) @ np.abs(B).T
    assert np.max(np.abs(got - ref) / scale) < 1e-14 * K ** 0.5 + 1e-15


@pytest.mark.parametrize("M,N,K", [(128, 128, 32), (384, 256, 1056), (256, 1024, 4096)])
def test_gemm_fp32(M, N, K):
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm
    announce("gemm fp32", M, N, K)
    A = random_matrix(M, K, 4).astype(np.float32)
    B = random_matrix(N, K, 5).astype(np.float32)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    dC = torch.empty((M, N), dtype=torch.float32, device="cuda")
    trg_gemm("fp32", dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K, K, K, N, False,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    scale = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)).T
    assert np.max(np.abs(dC.cpu().numpy() - ref) / scale) < 4 * 2.0 ** -24 * np.sqrt(K) + 1e-7


@pytest.mark.parametrize("M,N,K,accumulate", [(256, 256, 32, False), (512, 768, 1088, False),
                                              (768, 256, 4096, False), (512, 512, 1056, True)])
def test_gemm_bf16x3(M, N, K, accumulate):
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm, trg_gemm_tile
    announce("gemm bf16x3", M, N, K, accumulate)
    tm, tn, tk = trg_gemm_tile("bf16x3")
    assert M % tm == 0 and N % tn == 0 and K % tk == 0
    A = random_matrix(M, K, 6)
    B = random_matrix(N, K, 7)

    def split(X):
        x32 = torch.from_numpy(X).float()
        hi = x32.to(torch.bfloat16)
        lo = (x32 - hi.float()).to(torch.bfloat16)
        return hi, lo

    ah, al = split(A)
    bh, bl = split(B)
    dA = torch.stack([ah, al]).cuda().contiguous()
    dB = torch.stack([bh, bl]).cuda().contiguous()
    C0 = random_matrix(M, N, 8).astype(np.float32)
    dC = torch.from_numpy(C0).cuda()
    trg_gemm("bf16x3", dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K, K, K, N, accumulate,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    f = lambda t: t.double().numpy()
    ref = f(ah) @ f(bh).T + f(ah) @ f(bl).T + f(al) @ f(bh).T
    scale = np.abs(A) @ np.abs(B).T
    exact = A @ B.T
    if accumulate:
        c0 = C0.astype(np.float64)
        ref, exact, scale = ref + c0, exact + c0, scale + np.abs(c0)
    err = np.max(np.abs(dC.cpu().numpy() - ref) / scale)
    assert err < 4 * 2.0 ** -24 * np.sqrt(K) + 1e-7
    # and the split product is within ~2^-16 of the exact one
    assert np.max(np.abs(dC.cpu().numpy() - exact) / scale) < 2.0 ** -14


@pytest.mark.parametrize("precision,M,N,K,lda_pad", [
    ("fp64", 128, 128, 256, 0),       # K split inside the workgroup: one chunk of 16 per wave and a second
    ("fp64", 256, 128, 272, 16),      # a ragged chunk count, padded rows
    ("fp64", 128, 256, 2752, 0),      # many chunks per wave
    ("fp64", 1024, 1024, 16, 0),      # 64 x 64 tiles, one K tile
    ("fp64", 1024, 1024, 32, 0),      # two K tiles
    ("fp64", 1152, 1024, 48, 16),     # three K tiles
    ("fp64", 3200, 3200, 80, 0),      # 64 x 128 tiles
    ("fp64", 4096, 2048, 64, 0),      # 128 x 128 tiles
    ("fp32", 128, 128, 32, 0),        # 64 x 64 tiles, one K tile of the first FP32 group
    ("fp32", 256, 128, 160, 32),      # a group and one tile
    ("fp32", 3072, 2816, 192, 0),     # 64 x 128 tiles, a group and two tiles
    ("fp32", 3072, 2816, 288, 0),     # two groups and one tile
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gemm_tile_variants(precision, M, N, K, lda_pad, accumulate):
    """Every tile shape the dispatch of the FP64 and FP32 products picks, at
    the smallest K loops (pipeline prologue and tail) and with padded rows:
    every element to the rounding of its own sum, K products of 2^-53 (FP64)
    or a group of 128 in FP32 and one FP32 rounding (2^-24)."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm
    announce("gemm tile variants", precision, M, N, K, lda_pad, accumulate)
    dt = torch.float64 if precision == "fp64" else torch.float32
    npdt = np.float64 if precision == "fp64" else np.float32
    ld = K + lda_pad
    A, B, C0 = (random_matrix(r, c, 50 + i).astype(npdt) for i, (r, c) in enumerate([(M, ld), (N, ld), (M, N)]))
    dA, dB, dC = (torch.from_numpy(x).cuda() for x in (A, B, C0))
    trg_gemm(precision, dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K, ld, ld, N, accumulate,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    A64, B64 = A[:, :K].astype(np.float64), B[:, :K].astype(np.float64)
    ref = A64 @ B64.T + (C0.astype(np.float64) if accumulate else 0.0)
    scale = np.abs(A64) @ np.abs(B64).T + (np.abs(C0) if accumulate else 0.0)
    bound = (K + 2) * 2.0 ** -53 if precision == "fp64" else (min(K, 128) + 2) * 2.0 ** -24
    assert np.max(np.abs(dC.cpu().numpy() - ref) / scale) < bound


def _split3(X):
    """fl32(X) = hi + mid + lo exactly (three bfloat16 planes, round to
    nearest even at each stage), as torch tensors."""
    import torch
    x32 = torch.from_numpy(X).float()
    hi = x32.to(torch.bfloat16)
    r1 = x32 - hi.float()
    mid = r1.to(torch.bfloat16)
    lo = (r1 - mid.float()).to(torch.bfloat16)
    return hi, mid, lo


@pytest.mark.parametrize("M,N,K,accumulate", [(128, 128, 32, False), (384, 256, 1056, False),
                                              (256, 640, 4128, False), (256, 384, 1056, True)])
def test_gemm_bf16x6(M, N, K, accumulate):
    """Three-plane split join: the six products reproduce the product of the
    FP32-rounded operands to FP32 accuracy (the dropped mid*lo, lo*mid and
    lo*lo terms are below 2^-24 of each product), with FP64 sums of the
    FP32 groups (K = 4128: 32 groups and a ragged last one)."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm, trg_gemm_tile
    announce("gemm bf16x6", M, N, K, accumulate)
    tm, tn, tk = trg_gemm_tile("bf16x6")
    assert M % tm == 0 and N % tn == 0 and K % tk == 0
    A = random_matrix(M, K, 16)
    B = random_matrix(N, K, 17)
    pa, pb = _split3(A), _split3(B)
    # the split is exact on the host side too
    f = lambda t: t.double().numpy()
    A32, B32 = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
    assert np.array_equal(f(pa[0]) + f(pa[1]) + f(pa[2]), A32)
    dA = torch.stack(list(pa)).cuda().contiguous()
    dB = torch.stack(list(pb)).cuda().contiguous()
    C0 = random_matrix(M, N, 18).astype(np.float32)
    dC = torch.from_numpy(C0).cuda()
    trg_gemm("bf16x6", dA.data_ptr(), dB.data_ptr(), dC.data_ptr(), M, N, K, K, K, N, accumulate,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref = A32 @ B32.T
    scale = np.abs(A) @ np.abs(B).T
    if accumulate:
        c0 = C0.astype(np.float64)
        ref, scale = ref + c0, scale + np.abs(c0)
    err = np.max(np.abs(dC.cpu().numpy() - ref) / scale)
    print(f"[gemm bf16x6] max err / scale {err:.3e}", flush=True)
    # FP32 output rounding (2^-24 of |C|) plus the dropped terms and the
    # FP32 group sums; no sqrt(K) growth beyond the group length
    assert err < 12 * 2.0 ** -24


@pytest.mark.parametrize("precision,M,N", [("bf16x3", 256, 512), ("bf16x3", 4096, 4096), ("bf16x6", 128, 256),
                                           ("bf16x6", 2048, 2304)])
@pytest.mark.parametrize("K", [32, 64, 96, 160, 288])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gemm_split_tile_variants(precision, M, N, K, accumulate):
    """Both tile shapes of each split-BF16 product (the large ones from about
    256 tiles on) at K loops of one to nine tiles, shorter and longer than the
    ring of LDS stages and than the group of four, with rows farther apart
    than K: bounds as above (every dropped or FP32-summed term)."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm
    announce("gemm split tiles", precision, M, N, K, accumulate)
    planes, ld = (2 if precision == "bf16x3" else 3), K + 64
    g = torch.Generator(device="cuda").manual_seed(M + K)

    def operand(rows):
        x = torch.randn((rows, ld), generator=g, device="cuda")
        out = torch.empty((planes, rows, ld), dtype=torch.bfloat16, device="cuda")
        for p in range(planes):
            out[p] = x.to(torch.bfloat16)
            x = x - out[p].float()
        return out

    A, B = operand(M), operand(N)
    C = torch.randn((M, N), generator=g, device="cuda")
    A64, B64 = (x[:, :, :K].double() for x in (A, B))
    if precision == "bf16x6":
        ref = A64.sum(0) @ B64.sum(0).T
    else:
        ref = A64[0] @ B64[0].T + A64[0] @ B64[1].T + A64[1] @ B64[0].T
    scale = A64.sum(0).abs() @ B64.sum(0).abs().T
    if accumulate:
        ref, scale = ref + C.double(), scale + C.double().abs()
    trg_gemm(precision, A.data_ptr(), B.data_ptr(), C.data_ptr(), M, N, K, ld, ld, N, accumulate,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    bound = 12 * 2.0 ** -24 if precision == "bf16x6" else 4 * 2.0 ** -24 * K ** 0.5 + 1e-7
    assert float(((C.double() - ref).abs() / scale).max()) < bound


@pytest.mark.parametrize("precision,M,N", [("bf16x6", 2176, 2688), ("bf16x6", 4224, 1152), ("bf16x6", 384, 33024),
                                           ("bf16x3", 4352, 4352), ("bf16x3", 768, 1280)])
def test_gemm_split_tile_order_ragged(precision, M, N):
    """Tile counts that are no multiple of the 16 rows, 4 columns and 256 tiles
    of the shared order: every tile is written once.  Bounds as above."""
    test_gemm_split_tile_variants(precision, M, N, 64, False)



@pytest.mark.parametrize("n", [1, 2, 4, 7, 16, 33, 100, 144, 161, 200, 333, 576])
def test_jacobi_eigh(n):
    """Orders up to 160 use cyclic Jacobi, larger ones Householder
    tridiagonalisation + implicit QL."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh
    announce("eigh", n)
    mats = [random_symmetric(n, 10 + n), gram_like(n, min(n, 12), 20 + n)]
    A = np.stack(mats)
    dA = torch.from_numpy(A.copy()).cuda()
    dw = torch.empty((2, n), dtype=torch.float64, device="cuda")
    dV = torch.empty((2, n, n), dtype=torch.float64, device="cuda")
    ds = torch.empty(2, dtype=torch.int32, device="cuda")
    trg_eigh(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, 2,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    w, V, sw = dw.cpu().numpy(), dV.cpu().numpy(), ds.cpu().numpy()
    for b in range(2):
        assert sw[b] >= 0
        ref = np.sort(np.linalg.eigvalsh(A[b]))[::-1]
        nrm = np.linalg.norm(A[b])
        assert np.max(np.abs(w[b] - ref)) < 1e-13 * nrm
        assert np.all(np.diff(w[b]) <= 0)
        assert np.allclose(V[b].T @ V[b], np.eye(n), atol=1e-13)
        assert np.allclose(V[b] @ np.diag(w[b]) @ V[b].T, A[b], atol=1e-13 * nrm)


@pytest.mark.parametrize("n,batch", [(20, 300), (21, 2), (55, 3), (56, 3), (57, 260), (65, 40), (128, 2), (129, 2),
                                     (141, 1), (159, 2), (160, 1)])
def test_jacobi_edges(n, batch):
    """Where the Jacobi solver changes form: two waves or all, the square or the
    triangle of the matrix, odd orders (a dummy player), one or two waves of
    rotations, and from one to many workgroups sharing the vectors' rows (few
    matrices; more than the chip has CUs)."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh
    announce("jacobi edges", n, batch)
    A = np.stack([gram_like(n, n, 70 + i) if i % 2 else random_symmetric(n, 80 + i) for i in range(min(batch, 4))])
    A = A[np.arange(batch) % A.shape[0]]
    dA = torch.from_numpy(A).cuda()
    dw = torch.empty((batch, n), dtype=torch.float64, device="cuda")
    dV = torch.empty((batch, n, n), dtype=torch.float64, device="cuda")
    ds = torch.empty(batch, dtype=torch.int32, device="cuda")
    trg_eigh(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, batch,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    w, V = dw.cpu().numpy(), dV.cpu().numpy()
    assert int(ds.min()) >= 0
    for b in range(batch):
        if b >= 4:   # equal matrices of a batch give equal bits
            assert np.array_equal(w[b], w[b % 4]) and np.array_equal(V[b], V[b % 4])
            continue
        nrm = np.linalg.norm(A[b])
        assert np.max(np.abs(w[b] - np.linalg.eigvalsh(A[b])[::-1])) < 1e-13 * nrm
        assert np.allclose(V[b].T @ V[b], np.eye(n), atol=1e-13)
        assert np.allclose(V[b] @ np.diag(w[b]) @ V[b].T, A[b], atol=1e-13 * nrm)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
def test_gemm_empty_products(precision):
    """K = 0: C is zeroed (or left as it was when accumulating); M = 0 or
    N = 0: nothing is written."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm, trg_gemm_tile
    announce("gemm empty", precision)
    tm, tn, _ = trg_gemm_tile(precision)
    ct = torch.float64 if precision == "fp64" else torch.float32
    st = torch.cuda.current_stream().cuda_stream
    dummy = torch.zeros(16, dtype=torch.float64, device="cuda")
    C = torch.full((tm, tn), 3.0, dtype=ct, device="cuda")
    trg_gemm(precision, dummy.data_ptr(), dummy.data_ptr(), C.data_ptr(), tm, tn, 0, 16, 16, tn, True, st)
    torch.cuda.synchronize()
    assert bool((C == 3.0).all())
    trg_gemm(precision, dummy.data_ptr(), dummy.data_ptr(), C.data_ptr(), tm, tn, 0, 16, 16, tn, False, st)
    torch.cuda.synchronize()
    assert bool((C == 0.0).all())
    C.fill_(5.0)
    trg_gemm(precision, dummy.data_ptr(), dummy.data_ptr(), C.data_ptr(), 0, tn, 32, 32, 32, tn, False, st)
    trg_gemm(precision, dummy.data_ptr(), dummy.data_ptr(), C.data_ptr(), tm, 0, 32, 32, 32, tn, False, st)
    torch.cuda.synchronize()
    assert bool((C == 5.0).all())


@pytest.mark.parametrize("n", [16, 200])
def test_eigh_degenerate_and_zero_matrices(n):
    """Exactly repeated eigenvalues (any orthonormal basis of the eigenspace
    is correct: check the eigenvalues, orthonormality and reconstruction)
    and the zero matrix, on both solver paths."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh
    announce("eigh degenerate", n)
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = np.repeat(np.array([3.0, 1.0, -2.0, 0.5]), n // 4)
    A = np.stack([Q @ np.diag(lam) @ Q.T, np.eye(n), np.zeros((n, n))])
    A = 0.5 * (A + A.transpose(0, 2, 1))
    dA = torch.from_numpy(A.copy()).cuda()
    dw = torch.empty((3, n), dtype=torch.float64, device="cuda")
    dV = torch.empty((3, n, n), dtype=torch.float64, device="cuda")
    ds = torch.empty(3, dtype=torch.int32, device="cuda")
    trg_eigh(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, 3,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    w, V = dw.cpu().numpy(), dV.cpu().numpy()
    for b in range(3):
        ref = np.sort(np.linalg.eigvalsh(A[b]))[::-1]
        scale = max(np.linalg.norm(A[b]), 1.0)
        assert np.max(np.abs(w[b] - ref)) < 1e-13 * scale
        assert np.allclose(V[b].T @ V[b], np.eye(n), atol=1e-13)
        assert np.allclose(V[b] @ np.diag(w[b]) @ V[b].T, A[b], atol=1e-13 * scale)


@pytest.mark.parametrize("n", [100, 200, 400])
@pytest.mark.parametrize("tiny", [1e-160, 1e-250])
def test_eigh_block_far_below_the_matrix_scale(n, tiny):
    """Two diagonal blocks (contiguous, as in a parity-sorted Gram), the
    second scaled by `tiny`, so that sums of squares of its columns fall
    below the FP64 normal range (1e-160: into the subnormals, where an
    unscaled Householder reflector's 2 / v^T v overflows): eigenvalues to
    1e-13 of the matrix norm, orthonormal and finite eigenvectors, each lying
    in one block with exact zeros in the other, and the reconstruction.
    Both solver paths (Jacobi to 160, Householder + QL above)."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh
    announce("eigh tiny block", n, tiny)
    n0 = n // 2 + 3
    a = gram_like(n0, min(n0, 12), 5 + n)
    b = random_symmetric(n - n0, 6 + n)
    b = b @ b.T / (n - n0)                  # positive semi-definite, O(1)
    A = np.zeros((n, n))
    A[:n0, :n0] = a
    A[n0:, n0:] = tiny * b
    dA = torch.from_numpy(A.copy()).cuda()
    dw = torch.empty((1, n), dtype=torch.float64, device="cuda")
    dV = torch.empty((1, n, n), dtype=torch.float64, device="cuda")
    ds = torch.empty(1, dtype=torch.int32, device="cuda")
    trg_eigh(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, 1,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    w, V = dw.cpu().numpy()[0], dV.cpu().numpy()[0]
    assert np.all(np.isfinite(w)) and np.all(np.isfinite(V))
    nrm = np.linalg.norm(A)
    assert np.max(np.abs(w - np.sort(np.linalg.eigvalsh(A))[::-1])) < 1e-13 * nrm
    assert np.allclose(V.T @ V, np.eye(n), atol=1e-13)
    assert np.allclose(V @ np.diag(w) @ V.T, A, atol=1e-13 * nrm)
    in_a = np.abs(V[:n0]).sum(0) > 0
    in_b = np.abs(V[n0:]).sum(0) > 0
    assert not np.any(in_a & in_b)
    assert int(in_a.sum()) == n0 and int(in_b.sum()) == n - n0


def _eigh_top(A, k, rel):
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh_top, trg_eigh_top_work_bytes
    batch, n = A.shape[0], A.shape[1]
    dA = torch.from_numpy(A.copy()).cuda()
    dw = torch.empty((batch, n), dtype=torch.float64, device="cuda")
    dV = torch.empty((batch, n, n), dtype=torch.float64, device="cuda")
    ds = torch.empty(batch, dtype=torch.int32, device="cuda")
    nb = trg_eigh_top_work_bytes(n, batch)
    work = torch.empty(max(nb // 8, 1), dtype=torch.float64, device="cuda")
    trg_eigh_top(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, batch, k, rel, work.data_ptr(),
                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return dw.cpu().numpy(), dV.cpu().numpy(), ds.cpu().numpy()


@pytest.mark.parametrize("n", [150, 169, 256, 576])
def test_eigh_top_leading_pairs(n):
    """Every eigenvalue and the leading eigenvectors of Gram-like matrices
    (fast-decaying spectra, as the HOSVD Grams) and of random symmetric ones,
    against LAPACK: eigenvalues to 1e-13 of the norm, each computed vector an
    eigenvector (residual 1e-12 of the norm) orthonormal to the others, the
    columns beyond those needed zero."""
    announce("eigh_top", n)
    k = 24
    A = np.stack([gram_like(n, min(n, 60), 30 + n), random_symmetric(n, 40 + n)])
    w, V, kk = _eigh_top(A, k, 1e-10)
    for b in range(2):
        ref = np.sort(np.linalg.eigvalsh(A[b]))[::-1]
        nrm = np.linalg.norm(A[b])
        assert np.max(np.abs(w[b] - ref)) < 1e-13 * nrm
        q = int(kk[b]) if n > 160 else n     # the Jacobi path returns every vector (and its sweeps)
        assert k <= q <= n
        Vk = V[b][:, :q]
        assert np.all(V[b][:, q:] == 0.0)
        assert np.allclose(Vk.T @ Vk, np.eye(q), atol=1e-12)
        assert np.max(np.abs(A[b] @ Vk - Vk * w[b][:q])) < 1e-12 * nrm


@pytest.mark.parametrize("n,k,rank,batch", [(161, 1, 161, 1), (161, 65, 161, 3), (193, 20, 8, 2), (400, 130, 400, 1),
                                            (577, 24, 577, 1), (1024, 3, 40, 1)])
def test_eigh_top_edges(n, k, rank, batch):
    """The edges of the selection solver: the smallest and the largest order,
    one column and many reduced before the trailing matrix fits LDS, vectors
    in one and in several chunks of 64, and Grams of low rank, whose zero
    eigenvalues (most of the spectrum) form one cluster that the cut splits, so
    that every vector is computed.  Bounds as above."""
    announce("eigh_top edges", n, k, rank, batch)
    rng = np.random.default_rng(n + k)
    mats = []
    for _ in range(batch):
        X = rng.standard_normal((n, rank)) * 0.9 ** np.arange(rank)
        mats.append(X @ X.T)
    A = np.stack(mats)
    w, V, kk = _eigh_top(A, k, 1e-10)
    for b in range(batch):
        nrm = np.linalg.norm(A[b])
        assert np.max(np.abs(w[b] - np.linalg.eigvalsh(A[b])[::-1])) < 1e-13 * nrm
        q = int(kk[b])
        assert k <= q <= n and (q == n if rank < k else True)
        Vk = V[b][:, :q]
        assert np.all(V[b][:, q:] == 0.0)
        assert np.allclose(Vk.T @ Vk, np.eye(q), atol=1e-12)
        assert np.max(np.abs(A[b] @ Vk - Vk * w[b][:q])) < 1e-12 * nrm


def test_eigh_top_extends_over_a_split_cluster():
    """Eigenvalues 5, 4, 3 (x3), 2, ...: with k = 3 the cut splits the triple,
    so kk = 5 vectors come back, spanning the triple's eigenspace."""
    announce("eigh_top cluster")
    n = 200
    rng = np.random.default_rng(7)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = np.concatenate([[5.0, 4.0, 3.0, 3.0, 3.0, 2.0], np.linspace(1.0, 0.0, n - 6)])
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    w, V, kk = _eigh_top(A[None], 3, 1e-10)
    assert int(kk[0]) == 5
    P = V[0][:, 2:5] @ V[0][:, 2:5].T
    Pref = Q[:, 2:5] @ Q[:, 2:5].T
    assert np.max(np.abs(P - Pref)) < 1e-12


def test_eigh_top_parity_blocks_stay_exact():
    """A sector-ordered block-diagonal matrix (second block 1e-160 of the
    first, and exactly degenerate eigenvalues across the blocks): every
    computed vector lies in one block with exact zeros in the other, and the
    degenerate pair across the blocks gives one vector in each."""
    announce("eigh_top parity blocks")
    n, n0 = 300, 170
    a = gram_like(n0, 40, 11)
    b = gram_like(n - n0, 40, 12)
    A = np.zeros((2, n, n))
    A[0, :n0, :n0] = a
    A[0, n0:, n0:] = 1e-160 * b
    A[1, :n0, :n0] = a
    A[1, n0:, n0:] = a[: n - n0, : n - n0] * 0.0 + np.diag(np.linalg.eigvalsh(a)[::-1][: n - n0])
    w, V, kk = _eigh_top(A, 10, 1e-10)
    for bb in range(2):
        q = int(kk[bb])
        Vk = V[bb][:, :q]
        in_a = np.abs(Vk[:n0]).sum(0) > 0
        in_b = np.abs(Vk[n0:]).sum(0) > 0
        assert not np.any(in_a & in_b)
        assert np.all(np.isfinite(Vk))
        nrm = np.linalg.norm(A[bb])
        assert np.max(np.abs(A[bb] @ Vk - Vk * w[bb][:q])) < 1e-12 * nrm
    # the second matrix: block b holds the leading eigenvalues of block a, so
    # every leading eigenvalue is doubly degenerate across the blocks
    q = int(kk[1])
    in_b = np.abs(V[1][n0:, :q]).sum(0) > 0
    assert 0 < int(in_b.sum()) < q


@pytest.mark.parametrize("n,k", [(161, 12), (300, 300), (640, 25)])
@pytest.mark.parametrize("kind", ["zero", "diagonal", "runs of zero columns", "blocks of 8"])
def test_eigh_top_columns_that_are_reduced_already(n, k, kind):
    """Matrices with columns that are zero below the diagonal, which need no
    reflector: all of them, runs of them between full blocks (the first and last
    columns, and the ones on both sides of the order at which the trailing
    matrix moves to LDS, n - 128), and matrices of many blocks, whose vectors
    are orthogonalised within their blocks.  Beside a full matrix; bounds as
    above, and every vector stays within one block."""
    announce("eigh_top reduced columns", n, k, kind)
    rng = np.random.default_rng(n + len(kind))
    A = np.zeros((2, n, n))
    block = np.arange(n)
    if kind == "diagonal":
        A[1] = np.diag(rng.uniform(-1.0, 1.0, n))
    elif kind == "runs of zero columns":
        d = rng.uniform(0.0, 1.0, n)
        d[5:8] = 0.0
        A[1] = np.diag(d)
        for lo, hi in ((10, 24), (n - 131, n - 129), (n - 127, n - 60), (n - 20, n - 2)):
            A[1, lo:hi, lo:hi] = gram_like(hi - lo, hi - lo, lo)
            block[lo:hi] = lo
    elif kind == "blocks of 8":
        for lo in range(0, n, 8):
            hi = min(lo + 8, n)
            A[1, lo:hi, lo:hi] = random_symmetric(hi - lo, lo)
            block[lo:hi] = lo
    A[0] = gram_like(n, 40, 60)
    w, V, kk = _eigh_top(A, k, 1e-10)
    for b in range(2):
        ref = np.linalg.eigvalsh(A[b])[::-1]
        nrm = np.linalg.norm(A[b])
        assert np.max(np.abs(w[b] - ref)) <= 1e-13 * nrm
        q = int(kk[b])
        assert k <= q <= n and (q == n if kind == "zero" and b else True)
        Vk = V[b][:, :q]
        assert np.all(V[b][:, q:] == 0.0)
        assert np.allclose(Vk.T @ Vk, np.eye(q), atol=1e-12)
        assert np.max(np.abs(A[b] @ Vk - Vk * w[b][:q])) <= 1e-12 * nrm
    for v in V[1][:, : int(kk[1])].T:
        assert len(set(block[v != 0.0])) == 1


@pytest.mark.parametrize("n", [161, 300])
@pytest.mark.parametrize("bad", ["all nan", "all inf", "one nan"])
def test_eigh_top_matrix_that_is_not_finite(n, bad):
    """A matrix of NaN or infinite entries between two finite ones of a batch
    (a run that has overflowed steps on until its error flag is read): the
    number of vectors stays within the order, they are not finite either, so
    that the next norm shows it, and the finite matrices are solved to the
    bounds above.  The ranks of NaN eigenvalues must not coincide, or the
    solver would take block bounds from memory that nobody wrote."""
    announce("eigh_top not finite", n, bad)
    k = 20
    A = np.stack([gram_like(n, 40, 50), gram_like(n, 40, 51), gram_like(n, 40, 52)])
    if bad == "one nan":
        A[1, n // 2, n // 2 + 1] = A[1, n // 2 + 1, n // 2] = np.nan
    else:
        A[1] = np.nan if bad == "all nan" else np.inf
    w, V, kk = _eigh_top(A, k, 1e-10)
    assert k <= int(kk[1]) <= n
    assert not np.any(np.isfinite(V[1][:, : int(kk[1])]).all(0))
    if bad != "one nan":
        assert np.all(np.isnan(w[1]))
    for b in (0, 2):
        nrm = np.linalg.norm(A[b])
        q = int(kk[b])
        assert np.max(np.abs(w[b] - np.linalg.eigvalsh(A[b])[::-1])) < 1e-13 * nrm
        Vk = V[b][:, :q]
        assert np.allclose(Vk.T @ Vk, np.eye(q), atol=1e-12)
        assert np.max(np.abs(A[b] @ Vk - Vk * w[b][:q])) < 1e-12 * nrm


@pytest.mark.parametrize("top", [False, True])
@pytest.mark.parametrize("n,batch", [(2, 65535), (2, 65537), (3, 131071)])
def test_eigh_more_matrices_than_one_launch_takes(n, batch, top):
    """Batches at and beyond the largest second grid dimension (65535): every
    matrix, the first and last of each piece among them, against LAPACK."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_eigh
    announce("eigh batch", n, batch, top)
    X = np.random.default_rng(n).standard_normal((batch, n, n))
    A = X + X.transpose(0, 2, 1)
    if top:
        w, V, sweeps = _eigh_top(A, n, 1e-10)
    else:
        dA = torch.from_numpy(A.copy()).cuda()
        dw = torch.full((batch, n), np.nan, dtype=torch.float64, device="cuda")
        dV = torch.full((batch, n, n), np.nan, dtype=torch.float64, device="cuda")
        ds = torch.full((batch,), -7, dtype=torch.int32, device="cuda")
        trg_eigh(dA.data_ptr(), dw.data_ptr(), dV.data_ptr(), ds.data_ptr(), n, batch,
                 torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        w, V, sweeps = dw.cpu().numpy(), dV.cpu().numpy(), ds.cpu().numpy()
    assert np.all(sweeps >= 0)
    nrm = np.linalg.norm(A, axis=(1, 2))
    assert np.max(np.abs(w - np.linalg.eigvalsh(A)[:, ::-1]) / nrm[:, None]) < 1e-13
    assert np.max(np.abs(A @ V - V * w[:, None, :]) / nrm[:, None, None]) < 1e-12


@pytest.mark.parametrize("precision,M,N", [("bf16x3", 256, 512), ("bf16x6", 128, 256), ("bf16x6", 1280, 1152)])
@pytest.mark.parametrize("K", [32, 64, 96, 160, 288])
@pytest.mark.parametrize("off_a,off_b", [(1, 0), (0, 4), (2, 6)])
def test_gemm_split_operands_off_16_bytes(precision, M, N, K, off_a, off_b):
    """Operands that start 2, 4, 8 or 12 bytes past a 16-byte boundary, which a
    16-byte load straight to LDS is not known to take: the bits of the same
    product from aligned operands, from one K tile to past two FP32 groups."""
    torch = need_gpu()
    from paper_1911_12954_amd import trg_gemm
    announce("gemm split off 16 bytes", precision, M, N, K, off_a, off_b)
    planes = 2 if precision == "bf16x3" else 3
    g = torch.Generator(device="cuda").manual_seed(K)

    def operand(rows, off):
        x = torch.randn((rows, K), generator=g, device="cuda")
        out = torch.empty((planes, rows, K), dtype=torch.bfloat16, device="cuda")
        for p in range(planes):
            out[p] = x.to(torch.bfloat16)
            x = x - out[p].float()
        moved = torch.empty(out.numel() + off, dtype=torch.bfloat16, device="cuda")
        moved[off:] = out.flatten()
        assert out.data_ptr() % 16 == 0 and moved.data_ptr() % 16 == 0
        return out, moved[off:]

    A, A2 = operand(M, off_a)
    B, B2 = operand(N, off_b)
    for accumulate in (False, True):
        C = [torch.ones((M, N), dtype=torch.float32, device="cuda") for _ in range(2)]
        for a, b, c in ((A, B, C[0]), (A2, B2, C[1])):
            trg_gemm(precision, a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, K, K, N, accumulate,
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(C[0], C[1])


@pytest.mark.parametrize("n,k,rank", [(640, 130, 640), (600, 20, 8), (1024, 70, 1024)])
def test_eigh_top_several_chunks_at_large_orders(n, k, rank):
    """Above order 576 (the widest back-transformation) with more than one
    chunk of 64 vectors, so that every solve factors its chunk anew: by the
    number of vectors asked for, and by a rank below it, whose zero cluster
    the cut splits so that every vector is computed.  Bounds as above."""
    announce("eigh_top chunks", n, k, rank)
    X = np.random.default_rng(n + k).standard_normal((n, rank)) * 0.95 ** np.arange(rank)
    A = X @ X.T
    w, V, kk = _eigh_top(A[None], k, 1e-10)
    nrm = np.linalg.norm(A)
    q = int(kk[0])
    assert 64 < q <= n and (q == n if rank < k else q >= k)
    assert np.max(np.abs(w[0] - np.linalg.eigvalsh(A)[::-1])) < 1e-13 * nrm
    Vk = V[0][:, :q]
    assert np.all(V[0][:, q:] == 0.0)
    assert np.allclose(Vk.T @ Vk, np.eye(q), atol=1e-12)
    assert np.max(np.abs(A @ Vk - Vk * w[0][:q])) < 1e-12 * nrm


@pytest.mark.parametrize("precision,M,N", [("bf16x3", 256, 256), ("bf16x3", 3072, 2048), ("bf16x3", 2048, 3328),
                                           ("bf16x6", 256, 128)])
@pytest.mark.parametrize("K", [32, 64, 96, 128, 192, 224, 256, 352])
def test_gemm_split_through_registers(precision, M, N, K):
    """Operands off 16 bytes in both tiles of the BF16x3 kernel that takes them
    (the larger from 192 tiles on) and that of BF16x6: every remainder of K
    behind groups of four tiles, bit for bit as aligned operands."""
    test_gemm_split_operands_off_16_bytes(precision, M, N, K, 1, 4)
