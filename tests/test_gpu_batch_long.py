"""Batched GMRES over more steps than its kernels stage at a time: 512 Gram-Schmidt coefficients and 256 Givens
rotations.  Slender bodies converge slowly: at step 512 the longer one is still two decades short of the tolerance, so
its true residual shows whether the steps beyond count."""
import numpy as np
import pytest

import paper_2502_05507_amd as P

pytestmark = pytest.mark.gpu


def _context(length):
    h = 1.0 / 2048
    half = (length + 0.3, 3.4, 2.7)
    n = tuple(2 * int(a) + 11 for a in half)
    c = P.Context(n, h, (0.0, 0.0, 0.0), 0.0, "ellipsoid", tuple(0.5 * h * (m - 1) for m in n),
                  tuple(a * h for a in half), max_rhs=1, max_krylov=700)
    c.set_rhs(np.random.default_rng(0).standard_normal(c.sizes["n_gamma_minus"]))
    return c


@pytest.mark.parametrize("use_graph", [True, False])
def test_more_steps_than_the_kernels_stage(use_graph, tmp_path, monkeypatch):
    monkeypatch.setenv("BAE_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    ctxs = [_context(900), _context(500)]
    with P.Batch(ctxs) as b:
        res = b.solve(P.SOLVE_FP64, tol=1e-11, use_graph=use_graph)
    steps = [len(c.history()) for c in ctxs]
    print(steps, [r["rel_residual_true"] for r in res], flush=True)
    assert steps[0] > 520 and 264 < steps[1] < 512
    assert ctxs[0].history()[511] > 1e-10
    for c, r in zip(ctxs, res):
        # two orthogonalisations keep the estimate and the true residual together (to about 1e-14 here)
        assert c.history()[-1] <= 1e-11 and r["rel_residual_true"] < 2e-11
        c.close()
