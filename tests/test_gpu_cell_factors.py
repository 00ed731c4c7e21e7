"""Cell passes with the cells' factors in LDS, around the lines where they begin (f varying:
9 right-hand sides, 17 at p = 3; uniform f: the condensation at p = 3 from 33), with batches
that leave threads of a block without a cell and cell counts that leave a block without
cells.  Every form adds in one order, so a column equals the single-column result bit for bit;
one column against the oracle at the operator parity of the FP64 path, 1e-12."""
import numpy as np
import pytest

import hdg_inputs as hi

pytestmark = pytest.mark.gpu

HMS = 6.371e6


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("name", ["torus", "sphere"])
@pytest.mark.parametrize("p", [1, 2, 3])
def test_factor_forms_add_in_one_order(name, p):
    import torch
    from oracle.hdg import HdgOracle
    from paper_2004_09389_amd.hdg import HdgSolver
    if name == "torus":
        hier, phys = hi.torus_hierarchy(7, 7), (0.3, 2.0, 0.5, 0.7, 0.0)
    else:
        hier, phys = hi.icosphere_hierarchy(1, HMS), (1800.0, 9.81, 5960.0, 0.0, 7.292e-5)
    s = HdgSolver(hier, p, *phys, max_rhs=64, persistent=0)
    o = HdgOracle(hier.fine, p, *phys)
    r = hi.iid_rhs(hier.fine, p, 84, nrhs=64)
    lam = np.random.default_rng(85).standard_normal((s.n_facet, s.m, 64))
    rd, ld = torch.from_numpy(r).cuda(), torch.from_numpy(lam).cuda()
    single = {}
    for k in (0, 8, 32, 63):
        a, b = rd[..., k:k + 1].contiguous(), ld[..., k:k + 1].contiguous()
        single[k] = s.condense(a)[..., 0], s.recover(a, b)[..., 0]
    for nb in (9, 15, 16, 17, 31, 32, 33, 43, 48, 63, 64):
        print(f"[case] {name} p {p} nb {nb}", flush=True)
        a, b = rd[..., :nb].contiguous(), ld[..., :nb].contiguous()
        rhat, q = s.condense(a), s.recover(a, b)
        for k in single:
            if k < nb:
                assert torch.equal(q[..., k], single[k][1]), (nb, k)
                if name == "torus":
                    assert torch.equal(rhat[..., k], single[k][0]), (nb, k)
        k = nb - 1
        assert _rel(rhat[..., k].cpu().numpy().ravel(), o.rhat(r[..., k])) < 1e-12
        ref = o.recover(r[..., k], lam[..., k].ravel())
        got = q[..., k].cpu().numpy()
        for f in range(3):
            assert _rel(got[:, f], ref[:, f]) < 1e-12, (nb, f)
    s.close()
