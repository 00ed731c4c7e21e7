"""hdg_solve returns with its work done: the stream is idle (lam, the context's scalars and
PCG's copy of the solution are written), so another stream may use lam and the context at
once, and an error of the launch is this call's own.  The single-launch path instead
publishes every result before it returns (a fence behind its outputs)."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


# f0 = 0: PCG in FP64; f0 = 1: FGMRES; precisions 1 and 2: mixed, refinement
@pytest.mark.parametrize("f0,precision", [(0.0, 0), (1.0, 0), (1.0, 1), (1.0, 2)])
@pytest.mark.parametrize("nb", [1, 4])
def test_stream_is_idle_when_solve_returns(f0, precision, nb):
    import torch
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(32, 4)
    print(f"[case] f0 {f0} precision {precision} nb {nb}", flush=True)
    s = HdgSolver(hier, 2, 0.25, 1.0, 1.0, f0, precision=precision, max_rhs=nb, persistent=0)
    rhat = s.condense(torch.from_numpy(hi.iid_rhs(hier.fine, 2, 17, nrhs=nb)).cuda())
    lam = s.trace_zeros(nb)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    for k in range(20):
        lam.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            s.solve(rhat, lam)
            idle = st.query()
        other = lam.clone()   # on the default stream, not ordered after st but by solve itself
        torch.cuda.synchronize()
        assert idle, k
        assert torch.equal(other, lam), k
    res = rhat - s.trace_apply(lam)
    assert float((res.norm() / rhat.norm()).cpu()) <= 1.01e-8   # every column to rtol
    s.close()


@pytest.mark.parametrize("f0", [0.0, 1.0])
def test_single_launch_solve_is_published_when_it_returns(f0):
    import torch
    from paper_2004_09389_amd.hdg import HdgSolver
    hier = hi.torus_hierarchy(8, 4)
    s = HdgSolver(hier, 1, 0.5, 1.0, 1.0, f0, max_rhs=2)
    assert s.sizes.persistent == 1
    rhat = s.condense(torch.from_numpy(hi.iid_rhs(hier.fine, 1, 18, nrhs=2)).cuda())
    ref, _ = s.solve(rhat)
    torch.cuda.synchronize()
    ref = ref.cpu().numpy()
    st = torch.cuda.Stream()
    lam = s.trace_zeros(2)
    for _ in range(20):
        lam.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            s.solve(rhat, lam)
        other = lam.clone()
        torch.cuda.synchronize()
        assert np.array_equal(other.cpu().numpy(), ref)
    s.close()
