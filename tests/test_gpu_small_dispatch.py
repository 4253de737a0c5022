"""Which kernel takes a small-space solve, by the size of the space, its entries, its longest row and the
tolerance: the second-order equation in SciPy on both sides of each line (dense spaces, a row of every column,
few and many rows; tight and loose tolerances), and the iterations of a solve beyond 256 rows, which are those of
the textbook CG at the tolerance given."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2407_08901_amd as P
    P.lib()
    return P


def _matrix(kind, n0, n1, rng, scale=0.3, gap=0.0):
    """Symmetric H whose leading n0 rows form the small space (gap: between three low diagonals and the rest);
    values exact in float32."""
    if kind == "dense":
        M = sp.csr_matrix(np.triu(rng.standard_normal((n0, n0)) / np.sqrt(n0), 1))
    else:
        r = np.repeat(np.arange(n0), 6)
        c = rng.integers(0, n0, r.size)
        M = sp.triu(sp.csr_matrix((scale * rng.standard_normal(r.size), (np.minimum(r, c), np.maximum(r, c))),
                                  shape=(n0, n0)), 1).tolil()
        if kind == "hub":
            M[0, 1:] = rng.standard_normal(n0 - 1) / np.sqrt(n0)
    M = sp.bmat([[M, None], [None, sp.csr_matrix((n1, n1))]]).tocsr()
    r = np.repeat(np.arange(n0), 4)
    C = sp.csr_matrix((0.3 * rng.standard_normal(r.size), (r, n0 + rng.integers(0, n1, r.size))), shape=M.shape)
    dg = np.concatenate([np.sort(rng.uniform(1.0, 4.0, n0)), rng.uniform(8.0, 12.0, n1)])
    dg[3:n0] += gap
    U = (M + C + sp.diags(dg)).tocsr()
    U.data = U.data.astype(np.float32).astype(np.float64)
    U.sort_indices()
    return U, (U + sp.triu(U, 1).T).tocsr()


def _upload(U):
    return (torch.from_numpy(U.indptr.astype(np.int64)).cuda(), torch.from_numpy(U.indices.astype(np.int32)).cuda(),
            torch.from_numpy(U.data).cuda())


@pytest.mark.parametrize("kind,n0", [("sparse", 20), ("sparse", 64), ("sparse", 65), ("sparse", 256), ("sparse", 257),
                                     ("sparse", 1024), ("sparse", 1025), ("dense", 200), ("dense", 250), ("dense", 300),
                                     ("hub", 256), ("hub", 420), ("hub", 900)])
def test_second_order_equation(P, kind, n0):
    rng = np.random.default_rng(n0)
    U, H = _matrix(kind, n0, 700, rng)
    H0, n, k = H[:n0, :n0], H.shape[0], 3
    rp, col, val = _upload(U)
    # the relative residual a solve leaves is its tolerance; 10% and 4e-12 for the recursion's rounding and the
    # right-hand side's (a loose solve ends at the tolerance itself, a tight one at or below it)
    for tol in (1e-12, 1e-9, 1e-4):
        print("case %s n0=%d tol=%g" % (kind, n0, tol), flush=True)
        ctx = P.sppc_setup(rp, col, val, [0, n0, n], 1, k, P.sppc_default_opts(inner_tol=tol, n_deflate=3 * k))
        E0 = np.array(P.sppc_get(ctx, 0, 3 * k))[:k]
        psi = P.sppc_get(ctx, 9, n0 * 3 * k, device=True).view(n0, 3 * k).cpu().numpy()[:, :k]
        Psi = []
        for _ in (1, 2):
            P.sppc_correct(ctx, P.SPPC_CORR_PERTURBATIVE)
            Psi.append(P.sppc_get(ctx, 5, n * k, device=True).view(n, k).cpu().numpy())
            P.sppc_rayleigh_ritz(ctx)
        b = -(H @ Psi[0])[:n0]
        b -= psi * np.sum(psi * b, axis=0)
        x = Psi[1][:n0]
        r = np.linalg.norm(H0 @ x - x * E0 - b, axis=0) / np.linalg.norm(b, axis=0)
        assert np.max(r) < 1.1 * tol + 4e-12, (tol, r)
        assert np.max(np.abs(np.sum(psi * x, axis=0))) < 1e-12 * np.max(np.linalg.norm(x, axis=0))
        P.sppc_destroy(ctx)


@pytest.mark.parametrize("n0", [257, 505, 1100])
def test_tolerance_as_given_beyond_256_rows(P, n0):
    rng = np.random.default_rng(n0)
    U, H = _matrix("sparse", n0, 700, rng, 0.05, 2.0)
    H0, n = H[:n0, :n0], H.shape[0]
    rp, col, val = _upload(U)
    ctx = P.sppc_setup(rp, col, val, [0, n0, n], 1, 1, P.sppc_default_opts(n_deflate=3))
    E0 = np.array(P.sppc_get(ctx, 0, 3))
    Ps = P.sppc_get(ctx, 9, n0 * 3, device=True).view(n0, 3).cpu().numpy()
    P.sppc_correct(ctx, P.SPPC_CORR_PERTURBATIVE)
    Psi1 = P.sppc_get(ctx, 5, n, device=True).cpu().numpy()
    P.sppc_destroy(ctx)
    proj = lambda y: y - Ps @ (Ps.T @ y)
    b = proj(-(H @ Psi1)[:n0])
    r, p, g = b.copy(), np.zeros(n0), [b @ b]
    for j in range(40):
        p = r + (g[j] / g[j - 1] * p if j else 0.0)
        q = H0 @ p - E0[0] * p
        r = proj(r - g[j] / (p @ q) * q)
        g.append(r @ r)
    # a tolerance just above the residual of step j (5% of its square): CG stops there, one with a margin goes on
    j = next(i for i in range(40) if g[i] < (5e-10) ** 2 * g[0])
    assert g[j] < 0.8 * g[j - 1] and g[j] > (2e-11) ** 2 * g[0]
    opts = P.sppc_default_opts(inner_tol=float(np.sqrt(g[j] / g[0] / 0.95)), n_deflate=3, maxiter=2, p_switch=0, tol=1e-300,
                               final_check=0)
    ctx = P.sppc_setup(rp, col, val, [0, n0, n], 1, 1, opts)
    st = P.sppc_solve(ctx, want_vectors=False)[3]
    P.sppc_destroy(ctx)
    assert st["cg_iterations"] == j, (st["cg_iterations"], j)
