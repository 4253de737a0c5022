"""Eigensolver of the projected matrix at every size class: one and two registers per lane (m <= 64, 128),
the global-memory head (m > 128, <= 256 and beyond), odd sizes, one row; against LAPACK on the same T."""
import numpy as np
import pytest
import torch

import levelgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2407_08901_amd as P
    P.lib()
    return P


def _check(P, ctx, n, k):
    m = int(P.sppc_get(ctx, 2, 1)[0])
    T = np.array(P.sppc_get(ctx, 6, m * m)).reshape(m, m)
    theta = np.array(P.sppc_get(ctx, 1, k))
    Q = P.sppc_get(ctx, 3, n * m, device=True).view(n, m).cpu().numpy()
    Z = P.sppc_get(ctx, 10, n * k, device=True).view(n, k).cpu().numpy()
    V = Q.T @ Z
    norm = np.linalg.norm(T, 2)
    # a backward stable solver's errors are about m eps norm (m <= 320: 7e-14 norm); V through Q adds the
    # basis's own departure from orthonormality (1e-12 at most)
    assert np.max(np.abs(theta - np.linalg.eigvalsh(T)[:k])) < 1e-13 * norm, m
    assert np.max(np.abs(T @ V - V * theta)) < 1e-12 * norm, m
    assert np.max(np.abs(V.T @ V - np.eye(k))) < 2e-12, m
    return m


@pytest.mark.parametrize("k,pmax", [(1, 15), (3, 15), (5, 24), (8, 15), (16, 18)])
def test_eigenpairs_of_every_projected_matrix(P, k, pmax):
    A = levelgen.generate((60, 600, 3000), 60, 400 + k)
    rp, col, val = P.upload(A)
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, k, P.sppc_default_opts(p_switch=0, maxiter=pmax))
    seen = [_check(P, ctx, A.n, k)]
    for p in range(1, pmax + 1):
        # beyond the perturbative orders that still add directions: diagonal steps
        P.sppc_correct(ctx, P.SPPC_CORR_PERTURBATIVE if p < 12 else P.SPPC_CORR_JACOBI)
        _, _, added = P.sppc_rayleigh_ritz(ctx)
        if added == 0:
            break
        seen.append(_check(P, ctx, A.n, k))
        print("case k=%d m=%d" % (k, seen[-1]), flush=True)
    assert len(seen) >= 10
    P.sppc_destroy(ctx)


def test_decoupled_blocks_and_equal_eigenvalues(P):
    # a diagonal H: every off-diagonal of T is zero and eigenvalues repeat exactly
    d = np.repeat(np.arange(-8.0, 8.0), 4)
    n = d.size
    rp = torch.arange(n + 1, dtype=torch.int64, device="cuda")
    col = torch.arange(n, dtype=torch.int32, device="cuda")
    ctx = P.sppc_setup(rp, col, torch.from_numpy(d).cuda(), [0, n // 2, n], 1, 6, P.sppc_default_opts())
    theta = np.array(P.sppc_get(ctx, 1, 6))
    E0 = np.array(P.sppc_get(ctx, 0, 18))
    assert np.max(np.abs(theta - d[:6])) < 1e-13 * 8 and np.max(np.abs(E0 - d[:18])) < 1e-13 * 8
    Z = P.sppc_get(ctx, 10, n * 6, device=True).view(n, 6).cpu().numpy()
    assert np.max(np.abs(Z.T @ Z - np.eye(6))) < 1e-13
    assert np.max(np.abs(d[:, None] * Z - Z * theta)) < 1e-12
    P.sppc_destroy(ctx)
