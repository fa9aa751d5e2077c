"""The direct decomposition of bf16 pages (tridiagonalization, eigenvalues by
Sturm counts, twisted factorizations) and its way out: pages whose eigenvalues
cannot be told apart are marked in the page table and decomposed by one-sided
Jacobi in the same call, ordinary pages are not."""
import numpy as np
import pytest

import oracle
from helpers import storage_round

pytestmark = pytest.mark.gpu

# Bounds on |X - L R| over the optimum, on L^T L - 1 and on the row norms of R:
# fp32 Gram and eigenvectors give 1e-5 |X| (n eps |G| with n = 64), bf16
# storage rounds every entry by 2^-9, which two sums of r = 24 products of
# unit vectors' entries carry to below 1e-2.
TOL = {"f32": (1e-5, 1e-5, 1e-5), "bf16": (6e-3, 1e-2, 4e-3)}


def _hadamard(n):
    h = np.ones((1, 1))
    while h.shape[0] < n:
        h = np.block([[h, h], [h, -h]])
    return h


def _pages(P, d, rng):
    """Ordinary and degenerate page halves: (name, X)."""
    plain = lambda r0: rng.standard_normal((P, r0)) @ rng.standard_normal((r0, d)) + 0.05 * rng.standard_normal((P, d))
    half = rng.standard_normal((P // 2, d))
    graded = rng.standard_normal((P, d)) * 2.0 ** -rng.integers(0, 8, (P, 1))
    return [("planted rank + noise", plain(min(12, P // 2))),
            ("equal eigenvalues", 3.0 * _hadamard(d)[:P]),             # G = 9 d I exactly
            ("every row twice", np.concatenate([half, half])),        # top P/2 eigenvalues distinct
            ("one row repeated", np.tile(half[:1], (P, 1))),           # rank 1
            ("zero", np.zeros((P, d))),
            ("graded rows", graded),
            ("white noise", rng.standard_normal((P, d)))]


@pytest.mark.parametrize("P,d,r", [(16, 32, 1), (16, 64, 4), (16, 128, 9), (16, 256, 16), (32, 64, 1), (32, 128, 14), (32, 32, 16), (64, 64, 8), (64, 128, 24), (64, 256, 32),
                                   (64, 128, 33), (64, 128, 48), (64, 64, 64)])
@pytest.mark.parametrize("factors", ["bf16", "f32"])
@pytest.mark.parametrize("how", ["prefill", "compress"])
def test_direct_decomposition_and_marked_pages(P, d, r, factors, how):
    import torch
    import paper_2608_23843_amd as pk
    cases = _pages(P, d, np.random.default_rng(P + d + r))
    n = len(cases)
    X = storage_round(np.concatenate([x for _, x in cases]), "bf16").reshape(1, 1, n * P, d)
    Xv = np.ascontiguousarray(X.reshape(n, P, d)[::-1]).reshape(X.shape)   # values: the same pages in reverse
    kt, vt = (torch.from_numpy(a).to("cuda", torch.bfloat16).contiguous() for a in (X, Xv))
    W = 0 if how == "prefill" else n * P
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, 2 * n, r, 0, W, "bf16", factors)
    cache.compress_sweeps()
    if how == "prefill":
        cache.prefill(0, kt, vt, [n * P], default_rank=(r, r))
    else:   # dense pages first, then appended tokens until all of them have left the window
        cache.prefill(0, kt, vt, [n * P], default_rank=(r, r))
        cache.import_pages(0, [0] * n, [0] * n, range(n, 2 * n), [pk.PKV_FACTOR] * n, [r] * n, [r] * n,
                           torch.zeros(2 * n * (P + d) * r, dtype=cache.fdtype, device="cuda"),
                           np.arange(n) * 2 * (P + d) * r)
        cache.compress_pages(0, [0] * n, [0] * n, range(n), [r] * n, [r] * n)
    assert cache.device_status() == 0
    table = cache.page_table(0).cpu().numpy()[0, 0, :n]
    assert np.all(table[:, 4] == oracle.FACTOR) and np.all(table[:, 5] == r) and np.all(table[:, 6] == r)
    assert np.all(table[:, 7] == 0), "the mark must be gone"
    # the degenerate pages went through Jacobi (one vector alone is never degenerate)
    assert (cache.compress_sweeps() > 0) == (r > 1)
    blk = cache.export_pages(0, [0] * n, [0] * n, list(range(n))).cpu().numpy().astype(np.float64)
    rec_tol, orth_tol, sig_tol = TOL[factors]
    for i in range(n):
        o = 0
        for Y, name in ((X.reshape(n, P, d)[i], cases[i][0]), (Xv.reshape(n, P, d)[i], cases[n - 1 - i][0])):
            L, R = blk[i][o:o + P * r].reshape(P, r), blk[i][o + P * r:o + (P + d) * r].reshape(r, d)
            o += (P + d) * r
            Y = Y.astype(np.float64)
            s = np.linalg.svd(Y, compute_uv=False)
            scale = max(np.linalg.norm(Y), 1e-30)
            assert np.abs(L.T @ L - np.eye(r)).max() <= orth_tol, name
            tail = np.sqrt(np.sum(s[r:] ** 2))
            assert np.linalg.norm(Y - L @ R) <= (1 + 1e-3) * tail + rec_tol * scale, name
            s = np.pad(s, (0, max(0, r - len(s))))[:r]
            bound = sig_tol * s + 1e-5 * s[0] ** 2 / np.maximum(s, 1e-3 * s[0] + 1e-30) + 1e-6 * s[0]
            assert np.all(np.abs(np.linalg.norm(R, axis=1) - s) <= bound), name


@pytest.mark.parametrize("P,r", [(16, 9), (32, 16), (64, 24)])
def test_ordinary_pages_are_not_marked(P, r):
    """Pages of a planted rank plus noise, and zero pages, never leave the direct method: no sweeps."""
    import torch
    import paper_2608_23843_amd as pk
    n, d = 64, 128
    rng = np.random.default_rng(3)
    X = rng.standard_normal((2, n, P, 24)) @ rng.standard_normal((2, n, 24, d)) + 0.05 * rng.standard_normal((2, n, P, d))
    X[:, 5] = 0.0
    X[0, 9] = 0.0
    k, v = torch.from_numpy(X).to("cuda", torch.bfloat16).reshape(2, 1, 1, n * P, d)
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, r, 0, 0)
    cache.compress_sweeps()
    cache.prefill(0, k.contiguous(), v.contiguous(), [n * P], default_rank=(r, r))
    assert cache.device_status() == 0
    assert cache.compress_sweeps() == 0
    blk = cache.export_pages(0, [0, 0], [0, 0], [5, 9]).cpu().numpy()
    L, R = blk[:, :P * r].reshape(2, P, r), blk[:, P * r:(P + d) * r]
    assert np.all(R == 0) and np.abs(np.matmul(L.transpose(0, 2, 1), L) - np.eye(r)).max() == 0


def test_16_token_pages_off_16_byte_rows():
    """A prompt whose rows do not start on 16 bytes takes the element-wise
    kernel; its factors agree with those of the aligned prompt in the products."""
    import torch
    import paper_2608_23843_amd as pk
    n, P, d, r = 9, 16, 64, 5
    X = torch.randn(2, n * P * d + 8, generator=torch.Generator().manual_seed(1)).to("cuda", torch.bfloat16)
    out = []
    for shift in (0, 1):
        k, v = (torch.empty(n * P * d + 8, dtype=torch.bfloat16, device="cuda")[shift:shift + n * P * d] for _ in range(2))
        k.copy_(X[0, :n * P * d])
        v.copy_(X[1, :n * P * d])
        cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, r, 0, 0, "bf16", "f32")
        cache.compress_sweeps()
        cache.prefill(0, k.view(1, 1, n * P, d), v.view(1, 1, n * P, d), [n * P], default_rank=(r, r))
        assert (cache.compress_sweeps() > 0) == (shift == 1)
        blk = cache.export_pages(0, [0] * n, [0] * n, list(range(n)))[:, :2 * (P + d) * r].reshape(n, 2, (P + d) * r)
        out.append(torch.matmul(blk[..., :P * r].reshape(n, 2, P, r), blk[..., P * r:].reshape(n, 2, r, d)))
    # rank r of a page's noise spectrum: its gaps are 1% or more, so the fp32
    # Gram's n eps |G| moves the products by 1e-4 at most
    assert (out[0] - out[1]).norm() <= 1e-4 * out[0].norm()


@pytest.mark.parametrize("P,r,n,factors,eps", [(16, 6, 4500, "bf16", 0.0), (32, 12, 3300, "bf16", 0.0), (64, 24, 1700, "bf16", 0.0),
                                               (64, 0, 3200, "bf16", 0.05), (64, 24, 1700, "int4", 0.0)])
@pytest.mark.parametrize("which", ["K", "V", "both", "run"])
def test_many_marked_pages(P, r, n, factors, eps, which):
    """More marked pages than the launch over them has wavefronts, only one half of
    them marked, and a run of them: each is factorized and no mark stays."""
    import torch
    import paper_2608_23843_amd as pk
    d, g = 128, torch.Generator(device="cuda").manual_seed(P + n)
    flat = torch.randn(n, 4, d, generator=g, device="cuda").repeat_interleave(P // 4, 1)   # four rows, repeated: rank 4
    if eps:   # equal eigenvalues: rank 32 of 64 leaves half of the energy
        flat = torch.from_numpy(3.0 * _hadamard(d)[:P]).float().cuda().expand(n, P, d)
    # the other pages' planted singular values are a factor of two apart
    full = torch.randn(n, P, 5, generator=g, device="cuda") @ (torch.randn(n, 5, d, generator=g, device="cuda") *
                                                              2.0 ** torch.arange(5, device="cuda")[:, None])
    full = full + 0.05 * torch.randn(n, P, d, generator=g, device="cuda")
    run = torch.zeros(n, 1, 1, dtype=torch.bool, device="cuda")
    run[n // 3:n // 3 + 130] = True
    K = torch.where(run, flat, full) if which == "run" else flat if which in ("K", "both") else full
    V = flat if which in ("V", "both") else full
    k, v = (x.bfloat16().view(1, 1, n * P, d).contiguous() for x in (K, V))
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, r or 32, 0, 0, "bf16", factors, adaptive_rank_error=eps)
    cache.compress_sweeps()
    cache.prefill(0, k, v, [n * P], default_rank=(r, r))
    assert cache.device_status() == 0
    assert cache.compress_sweeps() > 0
    assert torch.all(cache.page_table(0)[0, 0, :n, 7] == 0)
    R = r or 32
    tol = {"bf16": 8e-3, "int4": 0.12}[factors]   # bf16: two roundings of 2^-9 per entry; INT4: of 1/14 of a run's largest
    for i in range(0, n, 500):
        m = min(500, n - i)
        blk = cache.export_pages(0, [0] * m, [0] * m, list(range(i, i + m)))
        o = 0
        for x in (k, v):
            X = x.view(n, P, d)[i:i + m].float()
            Y = blk[:, o:o + P * R].reshape(m, P, R).contiguous() @ blk[:, o + P * R:o + (P + d) * R].reshape(m, R, d).contiguous()
            o += (P + d) * R
            err = (X - Y).flatten(1).norm(dim=1) / X.flatten(1).norm(dim=1)
            assert float(err.max()) <= tol + (0.7072 if eps else 2e-2), (i, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("factors", ["bf16", "f32"])
@pytest.mark.parametrize("eps", [0.0, 0.01])
def test_ranks_above_32(factors, eps):
    """Pages of 64 tokens whose halves ask for, or with adaptive ranks need, ranks on both sides of 32."""
    import torch
    import paper_2608_23843_amd as pk
    P, d, n = 64, 128, 12
    planted = [(40, 8), (8, 40), (48, 48), (12, 12), (64, 33), (33, 64)] * 2
    rng = np.random.default_rng(17)
    X = np.zeros((2, n, P, d))
    for j, rr in enumerate(planted):
        for w, r in enumerate(rr):   # singular values within a factor of two, then noise below the error asked for
            q1, q2 = (np.linalg.qr(rng.standard_normal((s, r)))[0] for s in (P, d))
            X[w, j] = 50.0 * (q1 * np.linspace(1.0, 0.5, r)) @ q2.T + 1e-3 * rng.standard_normal((P, d))
    X = storage_round(X, "bf16")
    k, v = (torch.from_numpy(x).to("cuda", torch.bfloat16).reshape(1, 1, n * P, d).contiguous() for x in X)
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, 64, 0, 0, "bf16", factors, adaptive_rank_error=eps)
    want = np.asarray(planted, dtype=np.uint8)
    if eps:
        cache.prefill(0, k, v, [n * P], default_rank=(0, 0))
    else:
        rk, rv = (torch.from_numpy(np.ascontiguousarray(want[:, w]).reshape(1, 1, n)).cuda() for w in (0, 1))
        cache.prefill(0, k, v, [n * P], rank_k=rk, rank_v=rv)
    assert cache.device_status() == 0
    table = cache.page_table(0).cpu().numpy()[0, 0]
    assert np.all(table[:, 7] == 0)
    if not eps:
        assert np.array_equal(table[:, 5:7], want)
    blk = cache.export_pages(0, [0] * n, [0] * n, list(range(n))).cpu().numpy().astype(np.float64)
    rec_tol, orth_tol, _ = TOL[factors]
    for j in range(n):
        o = 0
        for w in (0, 1):
            r, Y = int(table[j, 5 + w]), X[w, j].astype(np.float64)
            L, R = blk[j][o:o + P * 64].reshape(P, 64), blk[j][o + P * 64:o + (P + d) * 64].reshape(64, d)
            o += (P + d) * 64
            assert np.all(L[:, r:] == 0) and np.all(R[r:] == 0)
            assert np.abs(L[:, :r].T @ L[:, :r] - np.eye(r)).max() <= orth_tol
            s = np.linalg.svd(Y, compute_uv=False)
            tail, norm = np.sqrt(np.sum(s[r:] ** 2)), np.linalg.norm(Y)
            assert np.linalg.norm(Y - L @ R) <= (1 + 1e-3) * tail + rec_tol * norm
            if eps:   # the smallest rank within the error
                assert tail <= eps * 1.001 * norm and np.sqrt(np.sum(s[r - 1:] ** 2)) >= eps * 0.999 * norm


@pytest.mark.parametrize("P,points", [(16, [((2, 2, 7), 28)]),
                                      (32, [((13, 1, 12), 36), ((4, 2, 12), 36), ((7, 10, 9), 36), ((6, 7, 12), 43),
                                            ((0, 3, 15), 40), ((9, 2, 15), 40), ((5, 1, 12), 50), ((14, 0, 12), 50)])])
def test_projection_holds_all_bits_of_l(P, points):
    """R = L^T X for bf16 factors is the rounding of products with L in 24 bits.
    Rank-1 pages a b^T with n1, n3, n5 tokens of 1, 3, 5: R = |a| b, at b where
    |a| b lies 2e-6 or more off a rounding boundary of bf16 and products with L
    in 16 bits (two bf16 parts) fall on its other side. fp32 gives |a| to a few 1e-7."""
    import torch
    import paper_2608_23843_amd as pk
    d, n = 64, len(points)
    X, want = np.zeros((n, P, d), dtype=np.float32), np.zeros((n, d))
    for i, (cnt, m) in enumerate(points):
        a = np.repeat([1.0, 3.0, 5.0], cnt)
        a = np.concatenate([a, np.zeros(P - len(a))])
        b = m * np.where(np.arange(d) % 3 == 0, -1.0, 1.0)
        X[i] = a[:, None] * b
        assert np.array_equal(storage_round(X[i], "bf16"), X[i])
        want[i] = storage_round(np.linalg.norm(a) * b, "bf16")
    x = torch.from_numpy(X).to("cuda", torch.bfloat16).reshape(1, 1, n * P, d).contiguous()
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, 1, 0, 0, "bf16", "bf16")
    cache.compress_sweeps()
    cache.prefill(0, x, x, [n * P], default_rank=(1, 1))
    assert cache.device_status() == 0 and cache.compress_sweeps() == 0
    blk = cache.export_pages(0, [0] * n, [0] * n, list(range(n)))[:, :2 * (P + d)].cpu().numpy().reshape(n, 2, P + d)
    for w in (0, 1):
        R = blk[:, w, P:] * np.where(blk[:, w, P:P + 1] * want[:, :1] < 0, -1, 1)   # the sign of the vector is free
        assert np.array_equal(R, want), (w, np.argwhere(R != want)[:4])


@pytest.mark.parametrize("P,r,planted,bound", [(16, 9, 16, 6e-7), (16, 12, 6, 1.9e-5), (32, 16, 24, 5e-7), (32, 28, 16, 1.25e-5),
                                               (64, 16, 24, 1.9e-6), (64, 24, 24, 2.95e-7), (64, 32, 24, 1.35e-5)])
def test_fp32_factors_as_near_the_optimum_as_jacobi(P, r, planted, bound):
    """fp32 factors of bf16 pages, at ranks inside the planted spectrum and in the noise
    past it: L R departs from the best rank-r product by no more, on average, than with
    one-sided Jacobi on every page (`bound`, its mean over six other draws of such pages)."""
    import torch
    import paper_2608_23843_amd as pk
    n, d = 256, 128
    rng = np.random.default_rng(100 * P + r)
    X = rng.standard_normal((2, n, P, planted)) @ rng.standard_normal((2, n, planted, d)) + 0.05 * rng.standard_normal((2, n, P, d))
    X = storage_round(X, "bf16")
    k, v = (torch.from_numpy(x).to("cuda", torch.bfloat16).reshape(1, 1, n * P, d).contiguous() for x in X)
    cache = pk.PuzzleKVCache(1, 1, 1, 1, d, P, n, r, 0, 0, "bf16", "f32")
    cache.prefill(0, k, v, [n * P], default_rank=(r, r))
    assert cache.device_status() == 0
    blk = cache.export_pages(0, [0] * n, [0] * n, list(range(n))).cpu().double()[:, :2 * (P + d) * r]
    for w, o in ((0, 0), (1, (P + d) * r)):
        L, R = blk[:, o:o + P * r].reshape(n, P, r), blk[:, o + P * r:o + (P + d) * r].reshape(n, r, d)
        U, s, Vh = torch.linalg.svd(torch.from_numpy(X[w]).double(), full_matrices=False)
        best = (U[:, :, :r] * s[:, None, :r]) @ Vh[:, :r]
        dep = (L @ R - best).flatten(1).norm(dim=1) / best.flatten(1).norm(dim=1)
        assert float(dep.mean()) <= bound, (w, float(dep.mean()))
        assert float((L.transpose(1, 2) @ L - torch.eye(r, dtype=torch.float64)).abs().max()) <= 1e-6
