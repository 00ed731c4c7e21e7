"""The tuning field cell_cells: hdg_autotune times it only where a kernel depends on it."""
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
