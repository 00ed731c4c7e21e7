"""The columns of an FGMRES cycle do not depend on when the host looks at their estimates.

Near the end of a cycle the host waits for a column before it queues the next one; before
that it looks one column late.  A loose tolerance brings that wait forward, an unreachable
one with maxit = k never waits: the first k columns, and so the solution, must be the same
bits.  With the learned smoother the estimates also decide the fallback to block-Jacobi
(fallback_ratio = 1e-3 makes every estimate too weak), which must not come earlier for
having been looked at earlier."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("smoother", ["bjacobi", "mlp"])
@pytest.mark.parametrize("precision", [0, 1])
def test_columns_do_not_depend_on_the_wait(smoother, precision):
    import torch
    from paper_2004_09389_amd.hdg import HDG_SMOOTH_BJACOBI, HDG_SMOOTH_MLP, HdgSolver
    hier = hi.torus_hierarchy(12, 3)
    mlp = smoother == "mlp"
    W1, _ = hi.mlp_init(3, 64, 5)
    W2 = np.random.default_rng(6).standard_normal((3, 64)) * 0.05

    def context(rtol, maxit):
        s = HdgSolver(hier, 2, 0.3, 2.0, 0.5, 0.7, precision=precision, rtol=rtol, maxit=maxit, persistent=0,
                      smoother=HDG_SMOOTH_MLP if mlp else HDG_SMOOTH_BJACOBI, fallback_ratio=1e-3)
        if mlp:
            s.mlp_set_weights(W1, W2)
        return s

    rhat = None
    columns = {}
    for rtol in (0.3, 0.2, 0.1, 0.07, 0.05, 0.03, 0.02, 0.01, 5e-3, 2e-3, 1e-3, 1e-4):
        print(f"[case] {smoother} precision {precision} rtol {rtol}", flush=True)
        s = context(rtol, 200)
        if rhat is None:
            rhat = s.condense(torch.from_numpy(hi.iid_rhs(hier.fine, 2, 19)).cuda())
        lam, info = s.solve(rhat)
        k = info[0].iters
        assert info[0].refinements == 1 and k >= 1
        s.close()
        # the reported count may include a column queued behind the last one used
        for n in (k, k - 1):
            if n >= 1 and n not in columns:
                t = context(1e-30, n)
                columns[n] = t.solve(rhat, allow_notconv=True)[0]
                t.close()
        assert any(n in columns and torch.equal(lam, columns[n]) for n in (k, k - 1)), (rtol, k)
    assert max(columns) >= 4
