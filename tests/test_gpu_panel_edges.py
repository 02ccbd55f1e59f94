"""Register panels at the edges of their column tiles: widths around every multiple of 16, with a
full panel and a last panel of fewer rows than columns (whose later columns have nothing left
below the pivot row), against the CPU oracle.  The bars are those of the parity tests (FP64 1e-12,
FP32 1e-5): the rounding of n Householder steps on Gaussian columns stays near 1e-14 (1e-6)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

WIDTHS = [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 81, 96, 97, 112, 113, 127, 128]


def _height(n):
    return 384 if n <= 32 else 512 if n <= 64 else 256


def _check(A, Q, R, tol):
    _, Ro = oracle.tsqr(A, block_rows=1000)
    assert np.all(np.tril(R, -1) == 0) and np.all(np.diag(R) > 0)
    assert np.linalg.norm(R - Ro) <= tol * np.linalg.norm(Ro)
    assert oracle.metric_orth(Q) <= tol
    assert oracle.metric_backward(A, Q, R) <= tol


@pytest.mark.parametrize("dtype,tol", [(np.float64, 1e-12), (np.float32, 1e-5)])
@pytest.mark.parametrize("n", WIDTHS)
def test_qr_tile_edges(n, dtype, tol):
    import paper_1301_1071_amd as t
    m = 2 * _height(n) + max(1, n // 3)              # two full panels and a short one
    A = np.random.default_rng(8000 + n).standard_normal((m, n)).astype(dtype)
    print(f"panel edges n={n} m={m} {np.dtype(dtype)}", flush=True)
    Ad = torch.from_numpy(A).cuda()
    Q, R = t.qr(Ad)
    _check(A.astype(np.float64), Q.cpu().numpy().astype(np.float64),
           R.cpu().numpy().astype(np.float64), tol)
    assert torch.equal(t.r(Ad), R)                   # R alone: the same steps


@pytest.mark.parametrize("n", [17, 33, 50, 64, 100])
def test_qr_columns_without_a_reflection(n):
    """Columns that are zero below the diagonal of the panel (upper triangular rows on top, zero
    rows below): tau = 0 in every step, R is the input up to signs."""
    import paper_1301_1071_amd as t
    T = np.triu(np.random.default_rng(n).standard_normal((n, n))) + 3.0 * np.eye(n)
    A = np.vstack([T, np.zeros((200, n))])
    Q, R = (x.cpu().numpy() for x in t.qr(torch.from_numpy(A).cuda()))
    s = np.sign(np.diag(T))
    assert np.array_equal(R, s[:, None] * T)
    assert np.array_equal(Q, np.vstack([np.diag(s), np.zeros((200, n))]))


@pytest.mark.parametrize("n", [8, 33, 64])
def test_batched_tile_edges(n):
    import paper_1301_1071_amd as t
    As = [np.random.default_rng(90 + m + n).standard_normal((m, n)) for m in (n, 3 * n + 1, 1100)]
    for A, (Q, R) in zip(As, t.qr_batched([torch.from_numpy(A).cuda() for A in As])):
        _check(A, Q.cpu().numpy(), R.cpu().numpy(), 1e-11 if A.shape[0] == n else 1e-12)


@pytest.mark.parametrize("m,n,bar", [(60_000, 2, 1.0e-7), (60_000, 5, 1.1e-7), (5000, 8, 1.2e-7)])
def test_fp32_error_of_narrow_panels(m, n, bar):
    """Mean relative error of FP32 Q over 24 inputs: below 1.08e-7, 1.18e-7 and 1.28e-7, the figures of
    column steps with a separately rounded square root (tau, which stands in 1 - tau on Q's diagonal,
    with its three roundings gives 1.15e-7, 1.21e-7 and 1.31e-7)."""
    import paper_1301_1071_amd as t
    err = []
    for s in range(24):
        A = torch.randn(m, n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1000 * s + n))
        B = A.double()
        R = torch.linalg.cholesky((B.t().contiguous() @ B).cpu()).t().contiguous().cuda()
        ref = torch.linalg.solve_triangular(R, B, upper=True, left=False)
        err.append(float(torch.linalg.norm(t.qr(A)[0].double() - ref) / torch.linalg.norm(ref)))
    assert np.mean(err) <= bar, np.mean(err)
