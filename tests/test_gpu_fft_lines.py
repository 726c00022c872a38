"""The FFT convolution at the sizes where its line kernels change: box lengths whose transforms take two, three and
four register stages, odd and even half spectra, a box that is no cube, sets with few and with many points per row,
and more right-hand sides than one group of grids holds; against the FP64 direct sum and, for the dense sets, the
oracle's grid solution."""
import numpy as np
import pytest

import paper_2502_05507_amd as P
import workloads as W
from oracle import geometry, sparse

from gpu_common import device, rel_l2, small_problem

pytestmark = pytest.mark.gpu


def _both(p, nrhs):
    import torch
    with P.Context.from_problem(p, max_rhs=max(nrhs, 2)) as c:
        q = torch.from_numpy(np.random.default_rng(7).standard_normal((nrhs, c.sizes["n_gamma_minus"]))).to(device())
        v = [torch.empty((nrhs, c.sizes["n_targets"]), dtype=torch.float64, device=device()) for _ in range(2)]
        c.apply_double_layer(q, v[0], P.PREC_FFT)
        c.apply_double_layer(q, v[1], P.PREC_FP64)
        torch.cuda.synchronize()
        z = c.get_sizes()
    return v[0].cpu().numpy(), v[1].cpu().numpy(), z


@pytest.mark.parametrize("kind,n", [("sphere", 8), ("sphere", 13), ("torus", 18), ("ellipsoid", 23), ("star", 31),
                                    ("ellipsoid", 44), ("torus", 53), ("star", 71), ("ellipsoid", 86), ("sphere", 102)])
def test_lengths(kind, n):
    # the direct sum is exact to its far field's 7e-11 (the FFT takes the same kernel values)
    a, b, z = _both(small_problem(kind, n), 2)
    for r in range(2):
        assert rel_l2(a[r], b[r]) < 1e-10, (z["conv_box"], z["conv_fft"])


@pytest.mark.parametrize("axes,n", [((0.45, 0.1, 0.2), (461, 111, 211)), ((0.06, 0.45, 0.08), (71, 461, 91))])
def test_three_and_four_stage_lines(axes, n):
    h = 1.0 / 500
    p = W.Problem("slab", n, h, (0.0, 0.0, 0.0), 0.0, "ellipsoid", tuple(0.5 * h * (m - 1) for m in n), axes)
    a, b, z = _both(p, 1)
    assert max(z["conv_fft"]) > 625
    assert rel_l2(a[0], b[0]) < 1e-10


def test_more_right_hand_sides_than_one_group():
    a, b, _ = _both(small_problem("star", 129, 10.0), 11)   # 22 MB of C each: groups of 6 and 5
    for r in range(11):
        assert rel_l2(a[r], b[r]) < 1e-10


def test_dense_sources_and_targets():
    p = W.poisson_ellipsoid(45)
    g = geometry.from_problem(p)
    u = sparse.solve(g, 0.0, p.g(g.xstar), p.f_grid())
    m = ~np.isnan(u)
    with P.Context.from_problem(p) as c:
        xs, _, _ = c.boundary_points()
        c.set_rhs(np.stack([p.g(xs)] * 2), np.stack([p.f_grid()] * 2))   # the free-space volume potential
        assert all(r["converged"] for r in c.solve(P.SOLVE_FFT, tol=1e-12, compute_grid=True))
        for r in range(2):
            assert rel_l2(c.solution(r)[m], u[m]) < 1e-10
