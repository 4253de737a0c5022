"""The float64 refinement after a failed check of the SPPC + RMM-DIIS hybrid, inside the queried workspace.  Whether
a sweep's residuals, which come from the H x carried through the DIIS combinations, end just below a tolerance that
the checked ones miss depends on the rounding of the whole solve, so the tolerance is scanned over the band where
this matrix's last sweeps end: about every third solve there refines."""
import numpy as np
import pytest

import levelgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2407_08901_amd as P
    P.lib()
    return P


def test_refinement_inside_the_workspace(P):
    A = levelgen.generate((54, 451, 3771), 46, 789128)
    rp, col, val = P.upload(A)
    refined, evs = 0, []
    for tol in np.geomspace(5e-10, 1.4e-9, 24):
        opts = P.sppc_default_opts(precond=P.SPPC_CORR_RMMDIIS, tol=tol, max_cont=200)
        need = P.sppc_workspace_size(rp, col, val, A.level_offsets, 2, 16, opts)
        ctx = P.sppc_setup(rp, col, val, A.level_offsets, 2, 16, opts, workspace=P.workspace_tensor(need))
        ev, _, rrn, st, status = P.sppc_solve(ctx, want_vectors=False)
        P.sppc_destroy(ctx)
        print("case tol=%.3g refine_steps=%d handover=%d" % (tol, st["refine_steps"], st["rmm_handover"]), flush=True)
        assert status == P.SPPC_OK and max(rrn) < tol and 0 < st["workspace_peak"] <= need
        refined += st["refine_steps"] > 0
        evs.append(ev)
    assert refined > 0
    assert np.max(np.ptp(np.array(evs), axis=0) / np.abs(evs[0])) < 1e-10
