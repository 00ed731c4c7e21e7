"""Krylov reductions that take four values per thread, at vector lengths and right-hand
side counts on every side of their rules: a length that is no multiple of four (one
right-hand side), two (values one at a time), four, twelve (a group count that is no
power of two), 16 and 64, in a context whose basis slots are wider than the batch by
an odd count.  Multi-launch FGMRES and PCG solves against the oracle's direct solve at
1e-10 (rtol 1e-12), as for the other solves."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("nb", [1, 2, 4, 12, 16, 63, 64])
@pytest.mark.parametrize("f0", [0.0, 1.0])
def test_solve_widths(nb, f0):
    import torch
    from oracle.hdg import HdgOracle
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(5, 5)   # 75 facets, 150 trace unknowns
    print(f"[case] nb={nb} f0={f0}", flush=True)
    s = HdgSolver(hier, 1, 0.5, 1.0, 1.0, f0, max_rhs=min(64, nb + 1 + nb % 2), rtol=1e-12, persistent=0)
    r = hi.iid_rhs(hier.fine, 1, 40 + nb, nrhs=nb)
    q, lam, info = s.stage_solve(torch.from_numpy(np.ascontiguousarray(r)).cuda())
    assert all(i.status == 0 and i.rel_res <= 1e-12 for i in info)
    o = HdgOracle(hier.fine, 1, 0.5, 1.0, 1.0, f0)
    for k in sorted({0, nb // 2, nb - 1}):
        q_ref, lam_ref = o.solve(r[..., k])
        assert _rel(lam[..., k].cpu().numpy().ravel(), lam_ref) < 1e-10
        assert _rel(q[..., k].cpu().numpy().ravel(), q_ref.ravel()) < 1e-10
    s.close()
