"""The panel product at the widths where its kernel changes: 1, 2 and 4 lanes per entry, one and several
column blocks, aligned and unaligned X, float32 and float64 values, 12, 2.5 and 0.26 entries per row and
panel (with and without sums over runs), against SciPy in float64."""
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


@pytest.mark.parametrize("val64", [False, True])
@pytest.mark.parametrize("xt", [torch.float64, torch.float32])
@pytest.mark.parametrize("sizes,pw", [((40, 200, 17), 64), ((300, 3000, 20000), 1000), ((300, 3000, 20000), 100)])
def test_panel_widths(P, sizes, pw, xt, val64):
    A = levelgen.generate(sizes, 60, 91)   # n = 257: one row beyond a block of 256
    vals = A.val.astype(np.float64)
    rng = np.random.default_rng(7)
    if val64:
        vals = vals * (1.0 + 1e-7 * rng.standard_normal(vals.size))
    rp, col, _ = P.upload(A)
    val = torch.from_numpy(vals).cuda()
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, 4,
                       P.sppc_default_opts(panel_width=pw, precision=P.SPPC_PREC_MIXED))
    v = vals if xt == torch.float64 else vals.astype(np.float32).astype(np.float64)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, v, A.n)
    # float64: rounding of the sums; float32 X: one rounding of each product (values rounded beforehand)
    tol = 1e-14 if xt == torch.float64 else 2.0 ** -24 * 1.01
    for b in (1, 2, 3, 4, 5, 8, 9, 16, 17, 18, 24, 31, 32):
        for off in (0, 1):  # off = 1: X starts one element past a 16-byte boundary
            print("case n=%d pw=%d %s val64=%d b=%d off=%d" % (A.n, pw, xt, val64, b, off), flush=True)
            buf = torch.from_numpy(rng.standard_normal(A.n * b + off)).to("cuda", dtype=xt)
            X = buf[off:].view(A.n, b)
            Xh = X.double().cpu().numpy()
            ref, scale = H @ Xh, abs(H) @ np.abs(Xh)
            for product in (P.sppc_spmm, P.sppc_spmm_noalloc):
                Y = torch.full((A.n, b), np.nan, dtype=torch.float64, device="cuda")
                product(ctx, X, Y)
                torch.cuda.synchronize()
                assert np.max(np.abs(Y.cpu().numpy() - ref) / scale) < tol, (b, off)
    P.sppc_destroy(ctx)
