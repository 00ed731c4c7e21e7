"""Facet-row kernels with rows staged in LDS and P1 kernels with four right-hand
sides per thread, on a mesh large enough that every launch rule is reached (25392
facets, a ragged last block; 8464 vertices): right-hand side counts that are odd and
even, on both sides of the 64- and 32-facet blocks and of the largest staged batch.
They add in the order of the one-thread-per-value kernels, so apply and V-cycles are
equal bit for bit; columns against the oracle at the operator parity (apply 1e-12,
V-cycle 1e-11)."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("p", [1, 2, 3])
def test_staged_rows_bitwise(p):
    import torch
    from oracle.hdg import HdgOracle
    from oracle.p1 import TraceMultigrid
    from paper_2004_09389_amd.hdg import HDG_MIXED, HdgSolver
    hier = hi.torus_hierarchy(92, 23)
    phys = (4.0 / 92, 1.0, 1.0, 0.5)
    s = HdgSolver(hier, p, *phys, max_rhs=64)
    oracle = HdgOracle(hier.fine, p, *phys)
    mg = TraceMultigrid(oracle, hier)
    for nb in (3, 4, 6, 8, 15, 17, 31, 32, 33, 34, 64):
        print(f"[rows] p={p} nb={nb}", flush=True)
        x = np.random.default_rng(80 + nb).standard_normal((s.n_facet, s.m, nb))
        xd = torch.from_numpy(x).cuda()
        outs = {}
        for rb in (1, 4):
            s.set_tuning(rhs_block=rb)
            outs[rb] = [s.trace_apply(xd), s.trace_apply(xd, HDG_MIXED), s.mg_vcycle(xd), s.mg_vcycle(xd, HDG_MIXED)]
        for a, b in zip(outs[1], outs[4]):
            assert torch.equal(a, b)
        if nb in (3, 33, 64):
            c = nb - 1
            assert _rel(outs[4][0][..., c].cpu().numpy().ravel(), oracle.apply(x[..., c].ravel())) < 1e-12
            assert _rel(outs[4][2][..., c].cpu().numpy().ravel(), mg.vcycle(x[..., c].ravel())) < 1e-11
    s.close()


def test_operator_on_a_large_mesh_same_bits_for_every_batch():
    """FP32 rows with FP64 vectors at 589824 unknowns: one thread per (facet, right-hand side) up
    to six of them, staged from seven on; each column is the same whatever batch it is in."""
    import torch
    from paper_2004_09389_amd.hdg import HDG_MIXED, HdgSolver
    s = HdgSolver(hi.torus_hierarchy(256, 4), 2, 4.0 / 256, 1.0, 1.0, 0.7, max_rhs=8, restart=2)
    assert s.n_facet * s.m >= 8 * 256 * 4 * 64
    x = torch.from_numpy(np.random.default_rng(5).standard_normal((s.n_facet, s.m, 8))).cuda()
    for mode in ((), (HDG_MIXED,)):
        whole = s.trace_apply(x, *mode)
        for nb in (1, 2, 3, 4, 6, 7):
            print(f"[rows] 256x256 nb={nb} {mode}", flush=True)
            assert torch.equal(s.trace_apply(x[..., :nb].contiguous(), *mode), whole[..., :nb])
    s.close()
