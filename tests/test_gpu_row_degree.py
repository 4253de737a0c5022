"""The row-wise product on both sides of the lines in entries per row and bytes of X where its kernels change
(one row per wave, four, the general kernel with and without full windows), against SciPy in float64."""
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


# X of width 8 reaches 1.6 L2 at 104,857 rows, X of width 4 at 209,715, X of width 5 two L2 there
@pytest.mark.parametrize("n,d", [(1500, 14), (1500, 22), (1500, 36), (1500, 44), (1500, 300), (104857, 110), (104858, 96),
                                 (104858, 112), (209713, 112), (209719, 112), (209719, 60)])
def test_row_degree(P, n, d):
    A = levelgen.generate((n // 43, n // 7, n - n // 43 - n // 7), d, n + d)
    rp, col, val = P.upload(A)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    aH = abs(H)
    longest = int(np.diff(H.indptr).max())
    rng = np.random.default_rng(n + d)
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, 4,
                       P.sppc_default_opts(panel_width=0, precision=P.SPPC_PREC_MIXED, maxiter=0, p_switch=0, m_max=8))
    for b in (4, 5, 8, 16) if n > 2000 else (1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 32):
        Xh = rng.standard_normal((n, b)).astype(np.float32).astype(np.float64)
        ref, scale = H @ Xh, aH @ np.abs(Xh)
        # float64: the roundings of a row's sum on either side; float32 X: one rounding of each product and those
        for xt, tol in ((torch.float64, 0.0), (torch.float32, 2.0 ** -24)):
            print("case n=%d d=%d b=%d %s" % (n, d, b, xt), flush=True)
            Y = torch.full((n, b), np.nan, dtype=torch.float64, device="cuda")
            P.sppc_spmm(ctx, torch.from_numpy(Xh).to("cuda", dtype=xt), Y)
            torch.cuda.synchronize()
            assert np.max(np.abs(Y.cpu().numpy() - ref) / scale) < tol + 2 * longest * 2.0 ** -53
    P.sppc_destroy(ctx)
