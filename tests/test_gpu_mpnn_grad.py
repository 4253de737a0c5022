"""Gradient of the learned preconditioner at the edges of its kernel's tiles (64-item steps of a block's
share, tiles of 256 items, more than one tile per block) against the float64 CPU reference."""
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


@pytest.mark.parametrize("n,S", [(63, 1), (64, 1), (65, 1), (51, 5), (64, 4), (257, 1), (43, 32), (33000, 16)])
def test_gradient_at_tile_edges(P, n, S):
    print("case mpnn grad n=%d S=%d" % (n, S), flush=True)
    A = levelgen.generate((20, n - 20), 12, 900 + n)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    Aoff, dg = ompnn.offdiag(H)
    lev = ompnn.level_feature(A.level_offsets, 1)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, S))
    X /= np.linalg.norm(X, axis=0)
    th = np.einsum("ij,ij->j", X, H @ X)
    R = H @ X - X * th
    E = rng.standard_normal((n, S))
    w = (rng.standard_normal(ompnn.NPARAM) * 0.3).astype(np.float32)
    rp, col, val = P.upload(A)
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, 2, P.sppc_default_opts())
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for f64 in (True, False):
        wr = w.astype(np.float64) if f64 else torch.from_numpy(w).to(torch.bfloat16).double().numpy()
        _, loss, grad = P.sppc_mpnn_eval(ctx, w, cu(R), cu(X), th, cu(E), f64=f64)
        ref = [ompnn.loss_and_grad(wr, Aoff, dg, lev, th[s], R[:, s], X[:, s], E[:, s]) for s in range(S)]
        g = sum(r[1] for r in ref) / S
        # the bounds of the forward and gradient test: float64 rounding, or float32 arithmetic per item
        assert np.max(np.abs(np.array(grad) - g)) < (1e-10 if f64 else 2e-4) * np.max(np.abs(g))
        if f64:
            assert np.max(np.abs(np.array(loss) - [r[0] for r in ref])) < 1e-11
    P.sppc_destroy(ctx)
