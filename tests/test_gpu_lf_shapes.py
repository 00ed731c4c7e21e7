"""Lax-Friedrichs kernels split over rows and patch slots: the operator with one row of a
facet per thread (one right-hand side, small meshes) against one thread per (facet, rhs)
(the same column of a two-column call, bit for bit) and the oracle (1e-12), on both
sides of the launch rule's size; and the RT0 V-cycle at (vertex, rhs) counts that leave
ragged blocks of vertex patches, against the oracle's (1e-11)."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,coarse,p", [(3, 3, 2), (5, 5, 3), (20, 5, 2), (20, 5, 3), (72, 9, 3), (76, 19, 3), (88, 11, 2)])
def test_rowwise_operator(n, coarse, p):
    import torch
    from oracle.lf import HdgLfOracle
    from paper_2004_09389_amd.hdg import HDG_FLUX_LF, HDG_MIXED, HdgSolver
    hier = hi.torus_hierarchy(n, coarse)
    print(f"[case] lf torus {n}/{coarse} p={p}", flush=True)
    s = HdgSolver(hier, p, 4.0 / n, 1.0, 1.0, 0.5, 0.0, flux=HDG_FLUX_LF, max_rhs=2)
    x = np.random.default_rng(5).standard_normal((s.n_facet, s.m, 2))
    xd = torch.from_numpy(x).cuda()
    one = xd[..., :1].contiguous()
    for prec in (0, HDG_MIXED):
        assert torch.equal(s.trace_apply(one, prec)[..., 0], s.trace_apply(xd, prec)[..., 0])
    if n <= 20:
        o = HdgLfOracle(hier.fine, p, 4.0 / n, 1.0, 1.0, 0.5, 0.0)
        assert _rel(s.trace_apply(one).cpu().numpy().ravel(), o.apply(x[..., 0].ravel())) < 1e-12
    s.close()


@pytest.mark.parametrize("n,coarse", [(6, 3), (10, 5), (20, 5)])
@pytest.mark.parametrize("nb", [1, 3, 16])
def test_patch_slots(n, coarse, nb):
    import torch
    from oracle.lf import HdgLfOracle, LfTraceMultigrid
    from paper_2004_09389_amd.hdg import HDG_FLUX_LF, HdgSolver
    hier = hi.torus_hierarchy(n, coarse)
    print(f"[case] lf torus {n}/{coarse} nb={nb}", flush=True)
    s = HdgSolver(hier, 1, 4.0 / n, 1.0, 1.0, 0.5, 0.0, flux=HDG_FLUX_LF, max_rhs=nb)
    mg = LfTraceMultigrid(HdgLfOracle(hier.fine, 1, 4.0 / n, 1.0, 1.0, 0.5, 0.0), hier, smoother="jacobi", rt_nu=1)
    x = np.random.default_rng(6).standard_normal((s.n_facet, s.m, nb))
    z = s.mg_vcycle(torch.from_numpy(x).cuda()).cpu().numpy()
    for c in sorted({0, nb // 2, nb - 1}):
        assert _rel(z[..., c].ravel(), mg.vcycle(x[..., c].ravel())) < 1e-11
    s.close()
