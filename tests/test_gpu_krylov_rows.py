"""GMRES with several right-hand sides against each of them alone, on both sides of the rule that splits the rows of the
Gram-Schmidt subtraction: blocks of 64 rows while 256-row blocks number at most 256 over all right-hand sides (here 8
to a right-hand side, the last one partly filled), of 256 rows beyond."""
import numpy as np
import pytest

import paper_2502_05507_amd as P

from gpu_common import rel_l2, small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [2, 32, 33, 64])
def test_iterates_equal_one_by_one(nrhs):
    with P.Context.from_problem(small_problem("sphere", 36), max_rhs=64, max_krylov=32) as c:
        n = c.sizes["n_gamma_minus"]
        assert -(-n // 256) == 8 and n % 256 and n % 64, n
        g = np.random.default_rng(3).standard_normal((nrhs, n))
        for steps in (1, 2, 9, 12):
            # an iterate is the same arithmetic in another order of summation: rounding, far below 1e-10 at these steps
            c.set_rhs(g)
            c.solve(P.SOLVE_FP64, tol=1e-14, maxit=steps)
            q = [c.density(r).copy() for r in range(nrhs)]
            hist = [c.history(r).copy() for r in range(nrhs)]
            for r in sorted({0, 1, nrhs // 2, nrhs - 1}):
                c.set_rhs(g[r])
                c.solve(P.SOLVE_FP64, tol=1e-14, maxit=steps)
                assert len(c.history()) == len(hist[r]) == steps
                assert abs(c.history() - hist[r]).max() < 1e-10 and rel_l2(q[r], c.density()) < 1e-10
