"""The sums for every kind of group that a number of right-hand sides splits into: each right-hand side of one call
against the same density alone.  FP64: the same terms in another order, a few thousand of them (1e-12 relative L2 is
about 1e4 roundings); FP32: the kernels' parity bar."""
import numpy as np
import pytest

import paper_2502_05507_amd as P

from gpu_common import device, rel_l2, small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 7, 15, 16, 17, 18, 21, 23])
@pytest.mark.parametrize("kind,n,sigma", [("ellipsoid", 65, 0.0), ("star", 85, 10.0)])
def test_groups_of_right_hand_sides(kind, n, sigma, nrhs):
    import torch
    with P.Context.from_problem(small_problem(kind, n, sigma), max_rhs=23) as c:
        m, nt = c.sizes["n_gamma_minus"], c.sizes["n_targets"]
        q = torch.from_numpy(np.random.default_rng(9).standard_normal((nrhs, m))).to(device())
        v = torch.full((nrhs + 1, nt), 7.0, dtype=torch.float64, device=device())
        one = torch.empty((1, nt), dtype=torch.float64, device=device())
        for prec, bar in ((P.PREC_FP64, 1e-12), (P.PREC_FP32, 2e-5)):
            c.apply_double_layer(q, v[:nrhs], prec)
            for r in sorted({0, 1, nrhs // 2, nrhs - 1}):
                c.apply_double_layer(q[r:r + 1], one, prec)
                torch.cuda.synchronize()
                assert rel_l2(v[r].cpu().numpy(), one[0].cpu().numpy()) < bar, (prec, r)
            assert bool((v[nrhs] == 7.0).all())
