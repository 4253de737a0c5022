"""The small-space solve of the perturbative correction (eq. sm_lin_proj) on both sides of every size limit
of its kernels: one workgroup per system (up to 256, 1024, 2048, 4096, 6144 rows), then one kernel per
iteration; the residual of the second-order equation in SciPy."""
import numpy as np
import pytest
import torch

import levelgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2407_08901_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n0", [40, 256, 257, 1024, 1025, 2048, 2049, 4096, 4097, 6144, 6145])
def test_second_order_equation(P, n0):
    A = levelgen.generate((n0, 2 * n0 + 7), 26, 500 + n0)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    H0 = H[:n0, :n0]
    rng = np.random.default_rng(n0)
    for mixed, val64 in ((False, False), (True, False), (False, True)):
        print("case n0=%d mixed=%d val64=%d" % (n0, mixed, val64), flush=True)
        k = 5
        rp, col, val = P.upload(A)
        if val64:  # values that need the float64 store
            val = val * (1.0 + 1e-9 * torch.from_numpy(rng.standard_normal(val.numel())).cuda())
            H = oracle.symmetric_from_upper(A.row_ptr, A.col, val.cpu().numpy(), A.n)
            H0 = H[:n0, :n0]
        ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, k,
                           P.sppc_default_opts(precision=P.SPPC_PREC_MIXED if mixed else P.SPPC_PREC_FP64))
        D = (2 if mixed else 3) * k
        E0 = np.array(P.sppc_get(ctx, 0, D))[:k]
        psi = P.sppc_get(ctx, 9, n0 * D, device=True).view(n0, D).cpu().numpy()[:, :k]
        Psi = []
        for p in (1, 2):
            P.sppc_correct(ctx, P.SPPC_CORR_PERTURBATIVE)
            Psi.append(P.sppc_get(ctx, 5, A.n * k, device=True).view(A.n, k).cpu().numpy())
            P.sppc_rayleigh_ritz(ctx)
        # (H0 - E0) x = -(I - psi psi^T) (H Psi^(1))_1 with x orthogonal to psi (Psi^(1) vanishes there)
        b = -(H @ Psi[0])[:n0]
        b -= psi * np.sum(psi * b, axis=0)
        x = Psi[1][:n0]
        r = np.linalg.norm(H0 @ x - x * E0 - b, axis=0) / np.linalg.norm(b, axis=0)
        # the tolerance of the solve (1e-12, mixed 1e-6; deflated pairs to 1e-9 there) and the rounding of
        # a right-hand side and solution of this size: eps |H0| |x| / |b| with |x| / |b| below 1e3
        assert np.max(r) < (1.1e-6 if mixed else 5e-12), r
        assert np.max(np.abs(np.sum(psi * x, axis=0))) < 1e-12 * np.max(np.linalg.norm(x, axis=0))
        P.sppc_destroy(ctx)
