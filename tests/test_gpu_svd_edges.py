"""The Jacobi SVD of R at the edges of its forms: the LDS kernels' column capacities (32, 64, 96,
100), block sweeps from n = 101 on with an even and an odd number of blocks, a last block of one
column, and both block widths, against the CPU oracle's singular values.  The bars are those of the
parity tests; V = G / |g| is orthogonal to the sweeps' tolerance, 1e-15 n entrywise."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,log_cond", [(1, 0), (2, 1), (31, 3), (32, 0), (33, 12), (64, 2), (65, 0),
                                        (96, 5), (97, 1), (100, 8), (101, 2), (112, 0), (113, 3),
                                        (128, 6), (257, 2), (301, 1)])
def test_svd_forms(n, log_cond):
    import paper_1301_1071_amd as t
    m = 2 * n + 37
    print(f"svd edges n={n} m={m}", flush=True)
    A = workloads.spectrum_matrix(m, n, float(log_cond), seed=60 + n)[0]
    U, S, V, Q, R = (x.cpu().numpy() for x in t.svd(torch.from_numpy(A).cuda(), want_qr=True))
    _, So, _ = oracle.tsqr_svd(A, block_rows=1000)
    eye = np.eye(n)
    assert np.abs(S - So).max() <= 1e-12 * So[0] and np.all(np.diff(S) <= 0)
    assert np.linalg.norm(U.T @ U - eye, 2) <= 1e-12
    assert np.abs(V.T @ V - eye).max() <= max(1e-15 * n, 1e-14)
    assert np.linalg.norm(A - (U * S) @ V.T, 2) <= 1e-12 * So[0]
    assert np.linalg.norm(A - Q @ R, 2) <= 1e-12 * So[0]
    assert np.all(V[np.abs(V).argmax(axis=0), np.arange(n)] > 0)


def test_svd_block_sweeps_in_a_graph():
    """The block sweeps' launches and flags under capture: replays after other work give the eager
    result bit for bit."""
    import paper_1301_1071_amd as t
    m, n = 900, 130
    dev = torch.device("cuda:0")
    A = torch.from_numpy(np.random.default_rng(4).standard_normal((m, n))).to(dev)
    out = tuple(torch.empty(s, dtype=torch.float64, device=dev) for s in ((m, n), (n,), (n, n)))
    ws = torch.empty(t.workspace_bytes("svd", m, n), dtype=torch.uint8, device=dev)
    info = torch.zeros(1, dtype=torch.int32, device=dev)

    def step():
        t.svd(A, ws=ws, out=(*out, None, None), info=info, check_info=False)

    step()
    ref = [o.clone() for o in out]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for k in range(3):
        for o in out:
            o.fill_(float(k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, out)) and int(info.item()) == 0


@pytest.mark.parametrize("n", [3, 40, 100, 160])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_svd_of_non_finite_input(n, bad):
    """info = -1, and singular values of NaN are ordered without reaching past the columns."""
    import paper_1301_1071_amd as t
    m = 3 * n + 5
    print(f"svd non-finite n={n} {bad}", flush=True)
    A = np.random.default_rng(n).standard_normal((m, n))
    A[m // 2, n // 2] = bad
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    U, S, V = t.svd(torch.from_numpy(A).cuda(), info=info, check_info=False)[:3]
    assert info.item() == -1
    assert U.shape == (m, n) and S.shape == (n,) and V.shape == (n, n)
    S = S.cpu().numpy()
    num = S[~np.isnan(S)]
    assert np.all(np.diff(num) <= 0) and not np.isnan(S[:len(num)]).any()


@pytest.mark.parametrize("n", [2, 40, 100, 160])
@pytest.mark.parametrize("e", [400, -400])
def test_svd_scaled_by_a_power_of_two(n, e):
    """Entries near 1e120 and 1e-120: the same factors bit for bit, the singular values scaled."""
    import paper_1301_1071_amd as t
    m = 2 * n + 37
    print(f"svd scaled n={n} 2^{e}", flush=True)
    A = workloads.spectrum_matrix(m, n, 3.0, seed=n)[0]
    U, S, V = t.svd(torch.from_numpy(A).cuda())[:3]
    Us, Ss, Vs = t.svd(torch.from_numpy(np.ldexp(A, e)).cuda())[:3]
    assert torch.isfinite(S).all()
    assert torch.equal(Us, U) and torch.equal(Vs, V)
    assert np.array_equal(Ss.cpu().numpy(), np.ldexp(S.cpu().numpy(), e))


@pytest.mark.parametrize("n", [2, 40, 100, 160])
@pytest.mark.parametrize("hi,lo", [(100, 0), (80, 70), (100, -100)])
def test_svd_of_graded_columns(n, hi, lo):
    """Columns scaled from 1e<hi> down to 1e<lo>: orthogonal factors, and the singular values' product
    is that of R's diagonal (each of the n values is relatively exact to n rounding errors)."""
    import paper_1301_1071_amd as t
    m = 3 * n + 37
    print(f"svd graded n={n} 1e{hi}..1e{lo}", flush=True)
    A = np.random.default_rng(n).standard_normal((m, n)) * np.logspace(hi, lo, n)
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    U, S, V, Q, R = (x.cpu().numpy() for x in t.svd(torch.from_numpy(A).cuda(), want_qr=True, info=info))
    assert info.item() == 0 and np.all(S > 0) and np.all(np.diff(S) <= 0)
    eye = np.eye(n)
    assert np.linalg.norm(U.T @ U - eye, 2) <= 1e-12
    assert np.abs(V.T @ V - eye).max() <= max(1e-15 * n, 1e-14)
    assert np.linalg.norm((A - (U * S) @ V.T) / S[0], 2) <= 1e-12
    assert abs(np.log(S).sum() - np.log(np.diag(R)).sum()) <= 1e-12 * n


def test_svd_of_two_columns_apart():
    """Norms 1e10 apart at 1e80: both values against the closed form of R's in 60 digits."""
    import decimal
    import paper_1301_1071_amd as t
    rng = np.random.default_rng(7)
    A = rng.standard_normal((4000, 2)) * np.array([1e80, 1e70])
    U, S, V, Q, R = (x.cpu().numpy() for x in t.svd(torch.from_numpy(A).cuda(), want_qr=True))
    with decimal.localcontext(decimal.Context(prec=60)):
        a, b, c = (decimal.Decimal(float(x)) for x in (R[0, 0], R[0, 1], R[1, 1]))
        f, d = a * a + b * b + c * c, a * c
        s0 = ((f + (f * f - 4 * d * d).sqrt()) / 2).sqrt()
        ref = [float(s0), float(d / s0)]
    assert np.abs(S / ref - 1).max() <= 1e-14
