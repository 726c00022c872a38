"""The batched sum's work items taken in the fixed order, drawn, and both, in and out of step: tilings that give a
workgroup from less than one item to more than its 64 slots hold, against each problem alone."""
import pytest

import paper_2502_05507_amd as P

from gpu_common import rel_l2, small_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def members():
    out = []
    for kind, n, sigma in (("ellipsoid", 107, 0.0), ("sphere", 81, 10.0), ("torus", 33, 0.0), ("ellipsoid", 65, 40.0)):
        p = small_problem(kind, n, sigma)
        c = P.Context.from_problem(p, max_rhs=1, max_krylov=64)
        xs, _, _ = c.boundary_points()
        c.set_rhs(xs[:, 0] * xs[:, 1] + xs[:, 2])
        c.solve(P.SOLVE_FP64, tol=1e-14, maxit=3)
        q64 = c.density().copy()
        c.solve(P.SOLVE_FP64, tol=1e-10)
        out.append((c, q64, c.gamma_values().copy()))
    yield out
    for c, _, _ in out:
        c.close()


@pytest.mark.parametrize("blocks,grid", [(64, 4), (64, 1), (8, 1), (4, 1), (2, 1), (1, 1)])
def test_every_order_gives_the_same(members, blocks, grid, tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BAE_AUTOTUNE_CACHE", str(cache))
    ctxs = [m[0] for m in members]
    with P.Batch(ctxs) as b:
        b.autotune(P.PREC_FP64)
    cache.write_text(" ".join(cache.read_text().split()[:-2] + [str(blocks), str(grid)]) + "\n")
    items = sum(-(-c.sizes["n_targets"] // 1024) * -(-(-(-c.sizes["n_sources"] // 64)) // blocks) for c in ctxs)
    print("items to a workgroup", items / (256 * grid), flush=True)
    if blocks == 1:
        assert 65 * 256 < items < 78 * 256   # the last 32 turns cross the 64th, where slots are freed
    with P.Batch(ctxs) as b:
        for use_graph in (False, True):
            b.solve(P.SOLVE_FP64, tol=1e-14, maxit=3, use_graph=use_graph)
            for c, q, _ in members:
                assert rel_l2(c.density(), q) < 1e-10    # the same arithmetic in another order of summation
        res = b.solve(P.SOLVE_FP32_REFINED, tol=1e-10)
        for (c, _, u), r in zip(members, res):
            assert r["converged"] and rel_l2(c.gamma_values(), u) < 1e-8
