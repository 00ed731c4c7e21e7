"""The tuning field cell_cells: hdg_autotune times it only where a kernel depends on it, and
in the kernels that read it no value changes a bit."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu

HMS = 6.371e6


# Every candidate runs the same kernels: Lax-Friedrichs and varying f up to the largest batch
# read per thread, uniform f at any batch.  A choice among them would be noise, and would
# stay on the context for batches where it matters.
@pytest.mark.parametrize("case,p,nb", [("lf", 3, 8), ("lf", 1, 3), ("sphere", 2, 5), ("torus", 2, 32)])
def test_autotune_leaves_the_default_where_nothing_depends_on_it(case, p, nb):
    from paper_2004_09389_amd.hdg import HDG_FLUX_LF, HdgSolver
    print(f"[case] {case} p {p} nb {nb}", flush=True)
    if case == "sphere":
        s = HdgSolver(hi.icosphere_hierarchy(3, HMS), p, 1800.0, 9.81, 5960.0, 0.0, 7.292e-5, max_rhs=32)
    else:
        s = HdgSolver(hi.torus_hierarchy(16, 4), p, 0.5, 1.0, 1.0, 1.0, max_rhs=32,
                      flux=HDG_FLUX_LF if case == "lf" else 0)
    for _ in range(8):
        assert s.autotune(nb)["cell_cells"] == 0
    s.close()


# The staged-row kernels of both passes (Lax-Friedrichs, just above the batches read per
# thread and at 32) and of the condensation with f varying inside the cells.
@pytest.mark.parametrize("case,p", [("lf", 1), ("lf", 2), ("lf", 3), ("sphere", 1), ("sphere", 3)])
@pytest.mark.parametrize("nb", [9, 32])
def test_cells_per_block_change_no_bit(case, p, nb):
    import torch
    from oracle.hdg import HdgOracle
    from oracle.lf import HdgLfOracle
    from paper_2004_09389_amd.hdg import HDG_FLUX_LF, HdgSolver
    print(f"[case] {case} p {p} nb {nb}", flush=True)
    if case == "sphere":
        hier, phys = hi.icosphere_hierarchy(2, HMS), (1800.0, 9.81, 5960.0, 0.0, 7.292e-5)
        s, oracle = HdgSolver(hier, p, *phys, max_rhs=nb), HdgOracle(hier.fine, p, *phys)
    else:
        hier, phys = hi.torus_hierarchy(13, 13), (0.5, 2.0, 0.5, 0.7)   # 338 cells: a ragged last block
        s = HdgSolver(hier, p, *phys, max_rhs=nb, flux=HDG_FLUX_LF)
        oracle = HdgLfOracle(hier.fine, p, *phys)
    r = hi.iid_rhs(hier.fine, p, 90 + nb, nrhs=nb)
    lam = np.random.default_rng(91 + nb).standard_normal((s.n_facet, s.m, nb))
    rd, ld = torch.from_numpy(r).cuda(), torch.from_numpy(lam).cuda()
    ref = None
    for cc in (0, 1, 3, 8, 32):
        s.set_tuning(cell_cells=cc)
        got = s.condense(rd), s.recover(rd, ld)
        ref = ref or got
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), cc
    rhat, q = (t.cpu().numpy() for t in ref)
    for k in (0, nb - 1):
        o = oracle.rhat(r[..., k])
        assert np.linalg.norm(rhat[..., k].ravel() - o) / np.linalg.norm(o) < 1e-12
        o = oracle.recover(r[..., k], lam[..., k].ravel())
        for f in range(3):   # depth and velocity differ by orders of magnitude on the sphere
            assert np.linalg.norm(q[:, f, :, k] - o[:, f]) / np.linalg.norm(o[:, f]) < 1e-12
    s.close()
