"""A captured FFT convolution apply stays valid whatever the context computes afterwards: the convolution's memory is
allocated with its plan and stays where it is, so a graph of one density replays correctly after eager applies, a
free-space volume potential and a solve with more densities."""
import numpy as np
import pytest

import paper_2502_05507_amd as P

from gpu_common import device, small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [("star", 41), ("ellipsoid", 23)])
def test_replay_after_more_densities(kind, n):
    import torch
    p = small_problem(kind, n)
    gen = torch.Generator().manual_seed(11)
    with P.Context.from_problem(p, max_rhs=16) as c:
        ngm = c.sizes["n_gamma_minus"]

        def draw(rows):
            return torch.randn(rows, ngm, dtype=torch.float64, generator=gen).to(device())

        q, v, ref = draw(1), draw(1), draw(1)
        q16, v16 = draw(16), draw(16)
        c.apply_operator(q, v, P.PREC_FFT)      # the plan, and a warm-up
        torch.cuda.synchronize()
        held = c.get_sizes()["device_bytes"]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            c.apply_operator(q, v, P.PREC_FFT)
        for step in range(4):
            if step == 1:
                c.apply_operator(q16, v16, P.PREC_FFT)
                torch.cuda.synchronize()
                assert c.get_sizes()["device_bytes"] == held
            elif step == 2:
                xs, _, _ = c.boundary_points()
                f = np.random.default_rng(3).standard_normal((16,) + tuple(p.n))
                c.set_rhs(np.tile(xs[:, 0], (16, 1)), f)   # the free-space volume potential of 16 sources
            elif step == 3:
                c.solve(P.SOLVE_FFT, tol=1e-8, maxit=8)
            q.copy_(draw(1))
            c.apply_operator(q, ref, P.PREC_FFT)
            v.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(v, ref), step
            # the same density among sixteen: its group's place does not change what is computed
            q16[9] = q[0]
            c.apply_operator(q16, v16, P.PREC_FFT)
            torch.cuda.synchronize()
            assert torch.equal(v16[9], ref[0]), step
