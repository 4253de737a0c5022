"""The learned preconditioner's gradient with fewer samples than its work array was sized for (k pairs, or a
larger evaluation before), at sizes where the smaller count has more partial sums than the larger; against
the float64 CPU reference, with the bounds of the gradient test."""
import numpy as np
import pytest
import torch

import levelgen
import oracle
from oracle import mpnn as ompnn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2407_08901_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n,k,first,S", [(8600, 16, 16, 15), (9000, 16, 16, 14), (17000, 8, 8, 7), (4228, 2, 32, 31)])
def test_gradient_of_fewer_samples(P, n, k, first, S):
    print("case mpnn samples n=%d k=%d first=%d S=%d" % (n, k, first, S), flush=True)
    A = levelgen.generate((40, n - 40), 12, 700 + n)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    Aoff, dg = ompnn.offdiag(H)
    lev = ompnn.level_feature(A.level_offsets, 1)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, first))
    X /= np.linalg.norm(X, axis=0)
    th = np.einsum("ij,ij->j", X, H @ X)
    R = H @ X - X * th
    E = rng.standard_normal((n, first))
    w = (rng.standard_normal(ompnn.NPARAM) * 0.3).astype(np.float32)
    rp, col, val = P.upload(A)
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, k, P.sppc_default_opts())
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ref = [ompnn.loss_and_grad(w.astype(np.float64), Aoff, dg, lev, th[s], R[:, s], X[:, s], E[:, s])
           for s in range(first)]
    for q in (first, S, first):
        _, loss, grad = P.sppc_mpnn_eval(ctx, w, cu(R[:, :q]), cu(X[:, :q]), th[:q], cu(E[:, :q]), f64=True)
        g = sum(r[1] for r in ref[:q]) / q
        assert np.max(np.abs(np.array(grad) - g)) < 1e-10 * np.max(np.abs(g)), q
        assert np.max(np.abs(np.array(loss) - [r[0] for r in ref[:q]])) < 1e-11, q
    P.sppc_destroy(ctx)
