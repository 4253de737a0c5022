"""The row-wise product at the widths of its 16-byte gathers, on both sides of the row counts where its rows
per wave change and with the row lengths of its edges (a few, one window of 64, one entry more, longer), with aligned and
unaligned X, against SciPy in float64."""
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


@pytest.mark.parametrize("n", [65, 1021, 65536, 65537, 99999, 100001, 200001, 500001])
def test_row_product(P, n):
    rng = np.random.default_rng(n)
    # rows of 64, 65 and 200 entries and their columns; the others hold the diagonal and a few more
    r, c = rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n)
    for i, m in ((3, 64), (17, 65), (n - 1, min(200, n - 1)), (n // 2, 63)):
        c2 = rng.permutation(n)[:m]
        r, c = np.concatenate([r, np.full(m, i)]), np.concatenate([c, c2])
    r, c = np.concatenate([np.minimum(r, c), np.arange(n)]), np.concatenate([np.maximum(r, c), np.arange(n)])
    U = sp.coo_matrix((rng.standard_normal(r.size), (r, c)), shape=(n, n)).tocsr()
    U.sort_indices()
    rp = torch.from_numpy(U.indptr.astype(np.int64)).cuda()
    col = torch.from_numpy(U.indices.astype(np.int32)).cuda()
    for f32 in (False, True):
        vals = U.data.astype(np.float32).astype(np.float64) if f32 else U.data
        V = sp.csr_matrix((vals, U.indices, U.indptr), shape=(n, n))
        H = (V + sp.triu(V, 1).T).tocsr()
        ctx = P.sppc_setup(rp, col, torch.from_numpy(vals).cuda(), np.array([0, 20, n]), 1, 2,
                           P.sppc_default_opts(panel_width=0))
        for b in (4, 6, 8, 16):
            for off in (0, 1):  # off = 1: X 8 bytes past a 16-byte boundary, the general kernel
                print("case n=%d f32=%d b=%d off=%d" % (n, f32, b, off), flush=True)
                buf = torch.from_numpy(rng.standard_normal(n * b + off)).cuda()
                X = buf[off:].view(n, b)
                Y = torch.full((n, b), np.nan, dtype=torch.float64, device="cuda")
                P.sppc_spmm(ctx, X, Y)
                torch.cuda.synchronize()
                Xh = X.cpu().numpy()
                scale = abs(H) @ np.abs(Xh)
                # sums of up to about 210 products in float64 on either side: 2 x 210 roundings of 2^-53 at most
                assert np.max(np.abs(Y.cpu().numpy() - H @ Xh) / scale) < 420 * 2.0 ** -53
        P.sppc_destroy(ctx)
