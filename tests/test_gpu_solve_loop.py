"""The solve loop's start and end: a stage solved from the known zero guess takes the same
steps, bit for bit, as the general solve given zeros; a zero and a non-finite right-hand
side end at once; maxit and the reported iterations hold."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("nb", [1, 4, 5])
def test_stage_from_zero_equals_general_solve(precision, nb):
    import torch
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(16, 4)
    print(f"[case] precision {precision} nb {nb}", flush=True)
    s = HdgSolver(hier, 2, 0.5, 1.0, 1.0, 1.0, precision=precision, max_rhs=nb, rtol=1e-9, persistent=0)
    r = torch.from_numpy(hi.iid_rhs(hier.fine, 2, 91, nrhs=nb)).cuda()
    q, lam, info = s.stage_solve(r)
    lam2, info2 = s.solve(s.condense(r))
    q2 = s.recover(r, lam2)
    assert torch.equal(lam, lam2) and torch.equal(q, q2)
    assert [i.iters for i in info] == [i.iters for i in info2]
    assert all(i.status == 0 and i.rel_res <= 1e-9 for i in info)
    # the iterations reported reach the tolerance and one fewer does not
    t = HdgSolver(hier, 2, 0.5, 1.0, 1.0, 1.0, precision=precision, max_rhs=nb, rtol=1e-9, persistent=0,
                  maxit=info[0].iters - 1)
    _, _, short = t.stage_solve(r, allow_notconv=True)
    assert max(i.rel_res for i in short) > 1e-9 or precision == 2
    assert short[0].iters <= info[0].iters - 1
    s.close()
    t.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_degenerate_right_hand_sides_end_at_once(precision):
    import torch
    from paper_2004_09389_amd.hdg import HdgError, HdgSolver
    hier = hi.torus_hierarchy(16, 4)
    s = HdgSolver(hier, 1, 0.5, 1.0, 1.0, 1.0, precision=precision, max_rhs=2, persistent=0)
    r = s.cell_zeros(2)
    q, lam, info = s.stage_solve(r)
    assert not q.any() and not lam.any() and all(i.iters == 0 and i.status == 0 for i in info)
    r[0, 0, 0, 1] = float("nan")
    with pytest.raises(HdgError) as e:
        s.stage_solve(r)
    assert e.value.code == -4
    r = torch.from_numpy(hi.iid_rhs(hier.fine, 1, 92, nrhs=2)).cuda()   # and the context solves again
    _, _, info = s.stage_solve(r)
    assert all(i.status == 0 for i in info)
    s.close()
