"""The blocked wide panels (128 < n <= 512) at their edges: one panel and several, a last panel
shorter than n, the two block widths (panels up to and above 1024 rows), the last block of one
column, and explicit heights on both sides of the blocked kernels' 2048 rows.  Bars as in the parity
tests of the wide path: FP64 1e-12, FP32 1e-5."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _orth(Q):
    return np.linalg.norm(Q.T @ Q - np.eye(Q.shape[1]), 2)


@pytest.mark.parametrize("m,n,panel_rows,dtype", [
    (129, 129, 0, "f64"), (1100, 161, 0, "f64"), (600, 160, 0, "f32"),
    (1028, 257, 0, "f64"), (2300, 257, 0, "f32"), (1500, 385, 0, "f64"),
    (3000, 140, 512, "f64"), (3000, 140, 513, "f64"), (3000, 140, 1024, "f32"),
    (3000, 140, 1025, "f64"), (4200, 140, 2048, "f64"), (4200, 140, 2049, "f64")])
def test_wide_block_edges(m, n, panel_rows, dtype):
    import paper_1301_1071_amd as t
    tol = 1e-12 if dtype == "f64" else 1e-5
    A = np.random.default_rng(m + n).standard_normal((m, n))
    A = A if dtype == "f64" else A.astype(np.float32)
    print(f"wide blocks m={m} n={n} panel_rows={panel_rows} {dtype}", flush=True)
    Ad = torch.from_numpy(A).cuda()
    Q, R = t.qr(Ad, panel_rows=panel_rows)
    assert torch.equal(t.r(Ad, panel_rows=panel_rows), R)
    A, Q, R = A.astype(np.float64), Q.cpu().numpy().astype(np.float64), R.cpu().numpy().astype(np.float64)
    _, Ro = oracle.tsqr(A, block_rows=1000)
    assert np.all(np.tril(R, -1) == 0) and np.all(np.diag(R) > 0)
    assert np.linalg.norm(R - Ro) <= tol * np.linalg.norm(Ro)
    assert _orth(Q) <= tol
    assert np.linalg.norm(A - Q @ R, 2) <= tol * np.linalg.norm(A, 2)


@pytest.mark.parametrize("m,n,panel_rows,dtype", [
    (300, 130, 0, "f64"), (700, 144, 0, "f32"), (2100, 144, 1024, "f64"), (2100, 145, 1024, "f64"),
    (1500, 130, 700, "f32"), (3000, 65, 0, "f64"), (6000, 80, 0, "f64"), (9000, 81, 0, "f64"),
    (9000, 112, 0, "f64")])
def test_last_block_of_up_to_16_columns(m, n, panel_rows, dtype):
    """The last block's own shape (one column tile), at both row capacities, on both sides of 16
    columns, in scratch panels and in place in the tree; equal on a second run."""
    import paper_1301_1071_amd as t
    tol = 1e-12 if dtype == "f64" else 1e-5
    A = np.random.default_rng(3 * m + n).standard_normal((m, n))
    A = A if dtype == "f64" else A.astype(np.float32)
    print(f"last block m={m} n={n} panel_rows={panel_rows} {dtype}", flush=True)
    Ad = torch.from_numpy(A).cuda()
    Q, R = t.qr(Ad, panel_rows=panel_rows)
    Q2, R2 = t.qr(Ad, panel_rows=panel_rows)
    assert torch.equal(Q, Q2) and torch.equal(R, R2)
    A, Q, R = A.astype(np.float64), Q.cpu().numpy().astype(np.float64), R.cpu().numpy().astype(np.float64)
    _, Ro = oracle.tsqr(A, block_rows=1000)
    assert np.linalg.norm(R - Ro) <= tol * np.linalg.norm(Ro)
    assert _orth(Q) <= tol
    assert np.linalg.norm(A - Q @ R, 2) <= tol * np.linalg.norm(A, 2)


def test_wide_columns_without_a_reflection():
    """Upper triangular on top, zeros below: tau = 0 in every step of every block."""
    import paper_1301_1071_amd as t
    n = 150
    T = np.triu(np.random.default_rng(n).standard_normal((n, n))) + 3.0 * np.eye(n)
    A = np.vstack([T, np.zeros((300, n))])
    Q, R = (x.cpu().numpy() for x in t.qr(torch.from_numpy(A).cuda()))
    s = np.sign(np.diag(T))
    assert np.array_equal(R, s[:, None] * T)
    assert np.array_equal(Q, np.vstack([np.diag(s), np.zeros((300, n))]))
