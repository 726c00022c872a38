"""Batched GMRES stopped after a given number of steps against the solo solver's iterate: step counts around the
wavefronts of a dot-product block (8) and the vectors a row block reads at a time (8), vectors below one
row block (256) and just beyond one and several dot-product slices (1024)."""
import pytest

import paper_2502_05507_amd as P
import workloads as W
from oracle import geometry

from gpu_common import rel_l2

pytestmark = pytest.mark.gpu


def _contexts():
    out = []
    for nn, a in ((10, 0.3), (16, 0.33), (36, 0.34), (49, 0.36)):
        n, h, o = W.padded_cube(nn)
        p = W.Problem("sphere", n, h, o, 0.0, "sphere", (0.5, 0.5, 0.5), (a,), 
                      boundary=lambda x, y, z: x * y + z)
        assert (geometry.from_problem(p).d_count() > 0).all()
        c = P.Context.from_problem(p, max_rhs=1, max_krylov=64)
        xs, _, _ = c.boundary_points()
        c.set_rhs(p.g(xs))
        out.append(c)
    sizes = [c.sizes["n_gamma_minus"] for c in out]
    assert min(sizes) < 256 and any(1024 < s < 2048 for s in sizes) and max(sizes) > 2048, sizes
    return out


@pytest.mark.parametrize("use_graph", [True, False])
def test_iterates_equal_solo(use_graph, tmp_path, monkeypatch):
    monkeypatch.setenv("BAE_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    ctxs = _contexts()
    # the same arithmetic in another order of summation, at residuals above 1e-10: rounding, far below 1e-10
    for steps in (1, 2, 7, 8, 9, 10):
        ref = []
        for c in ctxs:
            c.solve(P.SOLVE_FP64, tol=1e-14, maxit=steps)
            ref.append((c.density().copy(), c.history().copy()))
        with P.Batch(ctxs) as b:
            b.solve(P.SOLVE_FP64, tol=1e-14, maxit=steps, use_graph=use_graph)
            for c, (q, hist) in zip(ctxs, ref):
                print(steps, c.sizes["n_gamma_minus"], len(hist), rel_l2(c.density(), q), flush=True)
                assert len(c.history()) == len(hist)
                assert abs(c.history() - hist).max() < 1e-10
                assert rel_l2(c.density(), q) < 1e-10
    for c in ctxs:
        c.close()
