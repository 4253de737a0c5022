"""The panel product's launch shapes of widths 4 and 8 by the row blocks per compute unit (one or two waves, a
full or a nearly empty last round), with and without sums over runs, and widths above 16 at 26 entries a row (row
by row with float64 X, column blocks with float32), against SciPy in float64."""
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


# row blocks of 256 per CU (256 of them): 1.99, 2.01, 3.1, 4.1
@pytest.mark.parametrize("n", [130300, 131900, 203001, 268700])
def test_panel_shapes(P, n):
    A = levelgen.generate((n // 43, n // 7, n - n // 43 - n // 7), 26, n)
    rp, col, val = P.upload(A)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    aH = abs(H)
    rng = np.random.default_rng(n)
    for pw in (65536, 4096):  # 6 to 13 entries per row and panel, and below one
        ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, 4,
                           P.sppc_default_opts(panel_width=pw, precision=P.SPPC_PREC_MIXED, maxiter=0, p_switch=0, m_max=8))
        for b in (4, 7, 8, 20, 27):
            Xh = rng.standard_normal((n, b)).astype(np.float32).astype(np.float64)
            ref, scale = H @ Xh, aH @ np.abs(Xh)
            # float64: rounding of the sums; float32 X: one rounding of each product
            for xt, tol in ((torch.float64, 1e-14), (torch.float32, 2.0 ** -24 * 1.01)):
                print("case n=%d pw=%d b=%d %s" % (n, pw, b, xt), flush=True)
                Y = torch.full((n, b), np.nan, dtype=torch.float64, device="cuda")
                P.sppc_spmm(ctx, torch.from_numpy(Xh).to("cuda", dtype=xt), Y)
                torch.cuda.synchronize()
                assert np.max(np.abs(Y.cpu().numpy() - ref) / scale) < tol
        P.sppc_destroy(ctx)
