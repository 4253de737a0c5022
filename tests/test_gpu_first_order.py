"""The first-order correction vanishes on the small space, exactly: its right-hand side there is
H0hat Psi^(0) - (H Psi^(0))_1, whose two products have to add the same terms in the same order.  For every
width with a kernel of its own, short and long rows, float32 and float64 values."""
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


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 11, 12, 16])
def test_small_space_rows_are_zero(P, k):
    for sizes, d in (((60, 400, 1500), 30), ((150, 300, 900), 260)):
        A = levelgen.generate(sizes, d, 31 + k)
        rp, col, val = P.upload(A)
        for mixed, val64 in ((0, False), (1, False), (0, True)):
            print("case k=%d d=%d mixed=%d val64=%d" % (k, d, mixed, val64), flush=True)
            v = val * (1.0 + 1e-9 * torch.rand(val.numel(), dtype=val.dtype, device=val.device)) if val64 else val
            ctx = P.sppc_setup(rp, col, v, A.level_offsets, 2, k, P.sppc_default_opts(precision=mixed))
            P.sppc_correct(ctx, P.SPPC_CORR_PERTURBATIVE)
            Psi = P.sppc_get(ctx, 5, A.n * k, device=True).view(A.n, k).cpu().numpy()
            n0 = A.level_offsets[2]
            assert not np.any(Psi[:n0]) and np.all(np.any(Psi[n0:], axis=0))
            P.sppc_destroy(ctx)
