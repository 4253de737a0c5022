"""The product of one column by the kernel that holds a panel of X in LDS, at a size where its rule takes it:
panels that go straight to LDS, panels that are copied, panels whose width only the gathers take, several panels
at a time, a ragged last block and panel, rows of every length, against SciPy in float64."""
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


@pytest.fixture(scope="module")
def A():
    return levelgen.generate((500, 5000, 50000, 249763), 60, 77)


@pytest.mark.parametrize("val64", [False, True])
@pytest.mark.parametrize("pw", [16384, 5000, 5001, 1024])
def test_one_column(P, A, pw, val64):
    vals = A.val.astype(np.float64)
    rng = np.random.default_rng(pw)
    if val64:
        vals = vals * (1.0 + 1e-7 * rng.standard_normal(vals.size))
    rp, col, _ = P.upload(A)
    ctx = P.sppc_setup(rp, col, torch.from_numpy(vals).cuda(), A.level_offsets, 1, 4,
                       P.sppc_default_opts(panel_width=pw, precision=P.SPPC_PREC_MIXED))
    for xt in (torch.float64, torch.float32):
        v = vals if xt == torch.float64 else vals.astype(np.float32).astype(np.float64)
        H = oracle.symmetric_from_upper(A.row_ptr, A.col, v, A.n)
        # float64: rounding of the sums; float32 X: one rounding of each product (values rounded beforehand)
        tol = 1e-14 if xt == torch.float64 else 2.0 ** -24 * 1.01
        for off in (0, 1):  # off = 1: X starts one element past a 16-byte boundary
            print("case n=%d pw=%d %s val64=%d off=%d" % (A.n, pw, xt, val64, off), flush=True)
            buf = torch.from_numpy(rng.standard_normal(A.n + off)).to("cuda", dtype=xt)
            X = buf[off:].view(A.n, 1)
            Xh = X.double().cpu().numpy()
            ref, scale = H @ Xh, abs(H) @ np.abs(Xh)
            for product in (P.sppc_spmm, P.sppc_spmm_noalloc):
                Y = torch.full((A.n, 1), np.nan, dtype=torch.float64, device="cuda")
                product(ctx, X, Y)
                torch.cuda.synchronize()
                assert np.max(np.abs(Y.cpu().numpy() - ref) / scale) < tol, off
    P.sppc_destroy(ctx)
