"""The panel product of up to 16 columns into its own operand (whole and shifted overlaps): X is copied before any
row of Y is written."""
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


def test_in_place(P):
    A = levelgen.generate((300, 3000, 60000), 40, 5)
    rp, col, val = P.upload(A)
    H = oracle.symmetric_from_upper(A.row_ptr, A.col, A.val, A.n)
    ctx = P.sppc_setup(rp, col, val, A.level_offsets, 1, 4, P.sppc_default_opts(panel_width=4096))
    rng = np.random.default_rng(1)
    for b in (1, 2, 3, 4, 5, 8, 12, 16):
        for shift in (0, 2 * b):  # Y starts at X, or two rows into it
            print("case b=%d shift=%d" % (b, shift), flush=True)
            Xh = rng.standard_normal((A.n, b))
            for product in (P.sppc_spmm, P.sppc_spmm_noalloc):
                buf = torch.zeros(A.n * b + shift, dtype=torch.float64, device="cuda")
                buf[:A.n * b] = torch.from_numpy(Xh.ravel())
                Y = buf[shift:].view(A.n, b)
                product(ctx, buf[:A.n * b].view(A.n, b), Y)
                torch.cuda.synchronize()
                assert np.max(np.abs(Y.cpu().numpy() - H @ Xh) / (abs(H) @ np.abs(Xh))) < 1e-14
    P.sppc_destroy(ctx)
