"""Dense inverses of coarsest levels above 3072 unknowns (16 rows per block of the product)
in the V-cycle of both fluxes, with a ragged last block and right-hand side counts in each
launch shape (up to 16, 32 and 64 per block) besides one.  Tolerance: the operator parity
of the FP64 path, 1e-11."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("flux,n", [
    ("upwind", 57),   # 3249 vertices: 203 whole blocks and one row
    ("lf", 33),       # 3267 RT0 facets: 204 whole blocks and three rows
])
def test_large_dense_inverse_matches_oracle(flux, n):
    import torch
    from oracle.hdg import HdgOracle
    from oracle.lf import HdgLfOracle, LfTraceMultigrid
    from oracle.p1 import TraceMultigrid
    from paper_2004_09389_amd.hdg import HDG_FLUX_LF, HdgSolver
    hier, phys = hi.torus_hierarchy(n, n), (4.0 / n, 1.0, 1.0, 0.5)
    print(f"[case] {flux} {n} setup", flush=True)
    s = HdgSolver(hier, 1, *phys, max_rhs=64, flux=HDG_FLUX_LF if flux == "lf" else 0)
    print("[case] oracle", flush=True)
    if flux == "lf":
        mg = LfTraceMultigrid(HdgLfOracle(hier.fine, 1, *phys), hier)
    else:
        mg = TraceMultigrid(HdgOracle(hier.fine, 1, *phys), hier)
    x = np.random.default_rng(73).standard_normal((s.n_facet, s.m, 64))
    ref = {c: mg.vcycle(x[..., c].ravel()) for c in (0, 1, 15, 16, 31, 32, 63)}
    for nb in (1, 2, 16, 17, 32, 33, 64):
        print(f"[case] {flux} {n} nb {nb}", flush=True)
        r = torch.from_numpy(np.ascontiguousarray(x[..., :nb])).cuda()
        z = s.mg_vcycle(r)
        assert torch.equal(z, s.mg_vcycle(r))
        z = z.cpu().numpy()
        for c in ref:
            if c < nb:
                assert _rel(z[..., c].ravel(), ref[c]) < 1e-11, (nb, c)
    s.close()
