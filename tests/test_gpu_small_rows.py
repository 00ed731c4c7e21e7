"""The persistent solve with its operators in global memory, where a thread takes one
row of a facet (p >= 2): item counts below, at and above the 512 threads of a workgroup
and not a multiple of them, every shape of the V-cycle's first and last phases (one,
two and three pre- and post-sweeps), PCG and flexible GMRES, with the P1 cycle as its
matrix and by levels.  Against the oracle's direct solve at 1e-10 (rtol 1e-12), as for
the other persistent solves, and with solves split from their condensation."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,coarse,p", [
    (6, 3, 3),     # 108 facets, 432 rows: one partial round
    (8, 4, 3),     # 768 rows: one and a half rounds
    (8, 4, 2),     # 576 rows: the odd row length reads entries one by one
    (10, 5, 2),    # 900 rows, P1 cycle by levels
    (12, 3, 2),    # 1296 rows, three P1 levels
])
@pytest.mark.parametrize("f0,sweeps", [(0.0, 2), (1.0, 2), (0.0, 1), (1.0, 3)])
def test_rowwise_solve_matches_oracle(n, coarse, p, f0, sweeps):
    import torch
    from oracle.hdg import HdgOracle
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(n, coarse)
    print(f"[case] torus {n}/{coarse} p={p} f0={f0} sweeps={sweeps}", flush=True)
    s = HdgSolver(hier, p, 4.0 / n, 1.0, 1.0, f0, max_rhs=2, rtol=1e-12, nu_pre=sweeps, nu_post=sweeps)
    assert s.sizes.persistent == 1
    r = hi.iid_rhs(hier.fine, p, 90 + n, nrhs=2)
    rd = torch.from_numpy(np.ascontiguousarray(r)).cuda()
    q, lam, info = s.stage_solve(rd)
    assert all(i.status == 0 and i.rel_res <= 1e-12 for i in info)
    lam2, info2 = s.solve(s.condense(rd))
    o = HdgOracle(hier.fine, p, 4.0 / n, 1.0, 1.0, f0)
    for k in range(2):
        q_ref, lam_ref = o.solve(r[..., k])
        assert _rel(lam[..., k].cpu().numpy().ravel(), lam_ref) < 1e-10
        assert _rel(lam2[..., k].cpu().numpy().ravel(), lam_ref) < 1e-10
        assert _rel(q[..., k].cpu().numpy().ravel(), q_ref.ravel()) < 1e-10
    s.close()
