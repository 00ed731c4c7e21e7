"""Dense level products of the P1 cycle (the coarsest inverse, or the small levels'
whole V-cycle collapsed into one matrix) against the oracle's V-cycle, at right-hand
side counts on both sides of every tile edge (one; 16, 32 and 64 per launch shape) and at
level sizes around the 8-column and 16-row tiles.  Tolerance: the operator parity of
the FP64 path, 1e-11."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,coarse,tail", [
    (1, 1, 4096),     # a 1 x 1 map
    (3, 3, 4096),     # 9 rows: one row tile, a ragged second chunk
    (4, 4, 0),        # 16 rows exactly, no level collapsed
    (5, 5, 4096),     # 25 rows
    (12, 3, 4096),    # three levels collapsed into 144 rows
    (12, 3, 50),      # two of them (36 rows) below the finest level's own kernels
    (44, 11, 4096),   # 1936 rows: more chunks than one run per wavefront; 8 rows a block
    (49, 49, 0),      # 2401 rows (odd): 12 rows a block, ragged last one
    (50, 25, 4096),   # 2500 rows, collapsed
])
@pytest.mark.parametrize("nb", [1, 2, 16, 17, 32, 33, 64])
def test_collapsed_levels_match_oracle(n, coarse, tail, nb):
    import torch
    from oracle.hdg import HdgOracle
    from oracle.p1 import TraceMultigrid
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(n, coarse)
    print(f"[case] torus {n}/{coarse} tail {tail} nb {nb}", flush=True)
    s = HdgSolver(hier, 1, 4.0 / n, 1.0, 1.0, 0.5, max_rhs=nb, p1_tail_max=tail)
    mg = TraceMultigrid(HdgOracle(hier.fine, 1, 4.0 / n, 1.0, 1.0, 0.5), hier)
    x = np.random.default_rng(71).standard_normal((s.n_facet, s.m, nb))
    r = torch.from_numpy(x).cuda()
    z = s.mg_vcycle(r)
    again = s.mg_vcycle(r)
    assert torch.equal(z, again)
    z = z.cpu().numpy()
    for c in sorted({0, nb // 2, nb - 1}):
        assert _rel(z[..., c].ravel(), mg.vcycle(x[..., c].ravel())) < 1e-11, c
    s.close()
