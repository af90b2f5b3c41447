"""Dense Cholesky and triangular solves at the edges of their blocks: the
64-column inner and 256-column outer blocks, the 128-row tiles of the large
trailing updates (from 32 such tiles on), the 128-row blocks of the solves."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2409_16385_amd as E
from paper_2409_16385_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return E.Context(0)


@pytest.mark.parametrize("n,pad,nrhs", [(1, 0, 1), (2, 3, 2), (63, 0, 1), (64, 1, 1), (65, 0, 3), (127, 0, 1),
                                        (128, 0, 1), (129, 5, 2), (192, 0, 1), (255, 0, 1), (256, 0, 1), (257, 1, 5),
                                        (320, 0, 1), (513, 0, 1), (1000, 7, 1), (4352, 0, 1), (4481, 0, 2)])
def test_factor_and_solve(ctx, n, pad, nrhs):
    """Backward errors of the factor and of the solve: |A - L L^T| and
    |A X - B| of order n eps |A| (|X|), with the constant 8 for the two
    roundings of each of the blocked sums and the reciprocal pivots.  The
    strict upper triangle and the padding stay as they were."""
    rng = np.random.default_rng(n)
    G = torch.as_tensor(rng.normal(size=(n, n)), device="cuda")
    A = G @ G.T / n + torch.eye(n, dtype=torch.float64, device="cuda")
    A = 0.5 * (A + A.T)
    buf = torch.full((n, n + pad), 7.0, dtype=torch.float64, device="cuda")
    buf[:, :n] = A + torch.triu(torch.ones_like(A), 1)  # the upper triangle is not read
    keep = buf.clone()
    info = C.c_int64(-1)
    L = B._load()
    ctx.check(L.eipc_cholesky(ctx.handle, buf.data_ptr(), n, n + pad, C.byref(info), ctx.stream()))
    assert info.value == 0
    up = torch.triu(torch.ones((n, n + pad), dtype=torch.bool, device="cuda"), 1)
    assert torch.equal(buf[up], keep[up])
    F = torch.tril(buf[:, :n])
    tol = 8 * max(n, 8) * 2.2e-16
    assert float(torch.linalg.matrix_norm(F @ F.T - A)) <= tol * float(torch.linalg.matrix_norm(A))
    rhs = torch.as_tensor(rng.normal(size=(n, nrhs)), device="cuda")
    x = rhs.clone()
    ctx.check(L.eipc_cholesky_solve(ctx.handle, buf.data_ptr(), n, n + pad, x.data_ptr(), nrhs, ctx.stream()))
    r = float(torch.linalg.matrix_norm(A @ x - rhs))
    assert r <= 3 * tol * float(torch.linalg.matrix_norm(A)) * float(torch.linalg.matrix_norm(x))


@pytest.mark.parametrize("n,bad", [(64, 63), (300, 0), (300, 64), (300, 200), (700, 256), (700, 699)])
def test_first_bad_minor(ctx, n, bad):
    A = torch.eye(n, dtype=torch.float64, device="cuda")
    A[bad, bad] = -1.0
    if bad + 70 < n:
        A[bad + 70, bad + 70] = float("nan")
    assert E.cholesky(ctx, A) == bad + 1


@pytest.mark.parametrize("n,cond", [(64, 1e13), (200, 1e13), (500, 1e13), (500, 1e6)])
def test_stiff_blocks(ctx, n, cond):
    """Independent 12 x 12 blocks with eigenvalues over 13 decades (stiff
    contacts; the blocks cross the factorization's tiles of 16): entry by
    entry |A - L L^T|_ij <= c u sqrt(A_ii A_jj), the bound of substitution.
    An entry has at most 12 products, c = 2 (12 + 4) with four more roundings
    for the pivots and the solve, doubled; an error that grows with the
    condition of the diagonal tiles is beyond it."""
    rng = np.random.default_rng(0)
    A = np.zeros((n, n))
    for b in range(0, n, 12):
        m = min(12, n - b)
        Q, _ = np.linalg.qr(rng.normal(size=(m, m)))
        A[b:b + m, b:b + m] = (Q * np.geomspace(1, 1 / cond, m)) @ Q.T
    A = 0.5 * (A + A.T)
    F = torch.as_tensor(A, device="cuda")
    assert E.cholesky(ctx, F) == 0
    L = np.tril(F.cpu().numpy()).astype(np.longdouble)
    D = np.sqrt(np.diag(A))
    R = np.abs((L @ L.T - A) / np.outer(D, D)).astype(float)
    assert R.max() <= 2 * (12 + 4) * 1.1e-16


def _spread(n, cond):
    """Dense, eigenvalues over `cond` evenly in the logarithm."""
    G = torch.as_tensor(np.random.default_rng(n).normal(size=(n, n)), device="cuda")
    Q, _ = torch.linalg.qr(G)
    A = (Q * torch.logspace(0, -np.log10(cond), n, dtype=torch.float64, device="cuda")) @ Q.T.contiguous()
    return (0.5 * (A + A.T)).cpu().numpy()


def _backward(L, A):
    """|A - L L^T| / |A| in the Frobenius norm, from four products with
    vectors of signs in extended precision."""
    rng, LD, e = np.random.default_rng(1), np.longdouble, 0.0
    for _ in range(4):
        v = rng.choice([-1.0, 1.0], size=len(A)).astype(LD)
        t, r = np.zeros_like(v), np.zeros_like(v)
        for i in range(0, len(A), 256):
            t += L[i:i + 256].T.astype(LD) @ v[i:i + 256]
        for i in range(0, len(A), 256):
            r[i:i + 256] = L[i:i + 256].astype(LD) @ t - A[i:i + 256].astype(LD) @ v
        e += float((r * r).sum()) / 4
    return np.sqrt(e) / np.linalg.norm(A)


def _by_64(A):
    """The same factorization in numpy, 64 columns at a time: each is
    subtracted before the next 64 are summed."""
    A, L = A.copy(), np.zeros_like(A)
    for k in range(0, len(A), 64):
        e = min(k + 64, len(A))
        L[k:e, k:e] = np.linalg.cholesky(A[k:e, k:e])
        for j in range(k, e):
            L[e:, j] = (A[e:, j] - L[e:, k:j] @ L[j, k:j]) / L[j, j]
        A[e:, e:] -= L[e:, k:e] @ L[e:, k:e].T
    return L


@pytest.mark.parametrize("n,cond", [(500, 1e6), (500, 1e13), (4700, 1e6)])
def test_sums_of_64_columns(ctx, n, cond):
    """The trailing update reads 256 columns at a time but sums no more than
    64 in one go: its error is that of 64-column steps (measured at n = 500;
    it does not depend on n), half again allowed for the other order."""
    small = _spread(500, cond)
    most = 1.5 * _backward(_by_64(small), small)
    A = small if n == 500 else _spread(n, cond)
    F = torch.as_tensor(A, device="cuda")
    assert E.cholesky(ctx, F) == 0
    assert _backward(np.tril(F.cpu().numpy()), A) <= most


@pytest.mark.parametrize("n", [1, 2, 3, 31, 63, 64, 65, 100, 129, 190, 193])
@pytest.mark.parametrize("nrhs", [1, 3, 4, 5, 1030])
def test_solve_sizes(ctx, n, nrhs):
    """Solves of one launch (64 unknowns) and in blocks of 128, the last of
    one half or two, against the backward error of the factor test."""
    rng = np.random.default_rng(1000 * n + nrhs)
    F = np.tril(rng.normal(size=(n, n))) / np.sqrt(n) + 2 * np.eye(n)
    rhs = rng.normal(size=(n, nrhs))
    pad = np.full((n, n + 3), np.nan)  # only the lower triangle is read
    pad[np.tril_indices(n)] = F[np.tril_indices(n)]
    pad = torch.as_tensor(pad, device="cuda")
    x = torch.as_tensor(rhs, device="cuda").clone()
    ctx.check(B._load().eipc_cholesky_solve(ctx.handle, pad.data_ptr(), n, n + 3, x.data_ptr(), nrhs, ctx.stream()))
    x = x.cpu().numpy()
    A = np.abs(F) @ np.abs(F.T) @ np.abs(x) + np.abs(rhs)
    assert (np.abs(F @ (F.T @ x) - rhs) <= 3 * 8 * max(n, 8) * 1.1e-16 * A).all()


def test_small_systems_with_many_right_hand_sides(ctx):
    """The work follows the size: 3 unknowns take less than half of 64."""
    def ms(n):
        F, x = torch.eye(n, dtype=torch.float64, device="cuda"), torch.ones((n, 65536), dtype=torch.float64, device="cuda")
        best = np.inf
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                E.cholesky_solve(ctx, F, x)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        return best

    t3, t64 = ms(3), ms(64)
    print(f"3 unknowns {t3:.4f} ms, 64 {t64:.4f}")
    assert t3 <= 0.5 * t64


@pytest.mark.parametrize("n,at", [(40, 20), (64, 63), (65, 30), (65, 64), (129, 20), (129, 100), (300, 150)])
def test_an_infinite_unknown_stays_in_its_rows(ctx, n, at):
    """An unknown that passes the range in the backward pass reaches the rows
    before it (their products with it, 0 x Inf among them) and none after."""
    L = np.eye(n)
    L[at, at] = 1e-200
    b = np.arange(1.0, n + 1)
    x = torch.as_tensor(b[:, None], device="cuda").clone()
    E.cholesky_solve(ctx, torch.as_tensor(L, device="cuda"), x)
    x = x.cpu().numpy()[:, 0]
    assert np.isinf(x[at]) and np.array_equal(x[at + 1:], b[at + 1:])
