"""FFT convolution lines that no smaller box has: transforms of four register stages (2187 and 3645 points), in blocks of
512 threads, along each axis; against the FP64 direct sum, and the dense z passes of such lengths against the
finite-grid particular solution."""
import numpy as np
import pytest

import paper_2502_05507_amd as P
import workloads as W

from gpu_common import device, rel_l2

pytestmark = pytest.mark.gpu


def _slab(axis, nodes):
    """An ellipsoid whose box has 2 nodes + 5 nodes along `axis` and about 30 along the others."""
    h = 1.0 / 2048
    half = [nodes + 0.3, 14.4, 12.7]
    half = half[-axis:] + half[:-axis] if axis else half
    n = tuple(2 * int(a) + 11 for a in half)
    return W.Problem("slab", n, h, (0.0, 0.0, 0.0), 0.0, "ellipsoid", tuple(0.5 * h * (m - 1) for m in n),
                     tuple(a * h for a in half), boundary=lambda x, y, z: x * y + z)


@pytest.mark.parametrize("axis,nodes,length", [(0, 543, 2187), (1, 543, 2187), (2, 543, 2187), (0, 905, 3645),
                                               (1, 905, 3645)])
def test_four_stages(axis, nodes, length):
    import torch
    with P.Context.from_problem(_slab(axis, nodes), max_rhs=2, max_krylov=8) as c:
        q = torch.from_numpy(np.random.default_rng(7).standard_normal((2, c.sizes["n_gamma_minus"]))).to(device())
        a, b = (torch.empty((2, c.sizes["n_targets"]), dtype=torch.float64, device=device()) for _ in range(2))
        c.apply_double_layer(q, a, P.PREC_FFT)
        c.apply_double_layer(q, b, P.PREC_FP64)
        torch.cuda.synchronize()
        assert c.get_sizes()["conv_fft"][axis] == length
    for r in range(2):
        # the direct sum is exact to its far field's 7e-11 (the FFT takes the same kernel values)
        assert rel_l2(a[r].cpu().numpy(), b[r].cpu().numpy()) < 1e-10


@pytest.mark.parametrize("axis", [0, 2])
def test_volume_potential(axis):
    import torch
    p = _slab(axis, 543)
    x, y, z = np.meshgrid(*[np.arange(m) for m in p.n], indexing="ij")
    f = 1.0 + 0.5 * np.sin(0.21 * x + 0.4) * np.cos(0.17 * y) + 0.3 * np.sin(0.11 * z)
    with P.Context.from_problem(p, max_rhs=1, max_krylov=8) as c:
        xs, _, _ = c.boundary_points()
        c.set_rhs(np.zeros(len(xs)), f)
        c.solve(P.SOLVE_FFT, tol=0.5)      # any density q: u on gamma is D q and the volume potential h^2 sum G f
        assert c.get_sizes()["conv_fft"][axis] == 2187
        v = torch.empty(c.sizes["n_targets"], dtype=torch.float64, device=device())
        c.apply_double_layer(torch.from_numpy(c.density()).to(device()), v, P.PREC_FFT)
        torch.cuda.synchronize()
        got = c.gamma_values() - v.cpu().numpy()
        gamma = np.concatenate(c.sets()[:2])
        inner = np.argwhere(sum(((p.h * a - b) / d) ** 2 for a, b, d in zip((x, y, z), p.center, p.params)) < 1.0)
        rows = np.linspace(0, len(gamma) - 1, 40).astype(int)
        G = torch.empty(len(inner), dtype=torch.float64, device=device())
        want = []
        for r in rows:                      # the kernel's own values, summed row by row
            c.lgf_eval(torch.from_numpy((gamma[r] - inner).astype(np.int32)).to(device()).contiguous(), G, P.PREC_FP64)
            torch.cuda.synchronize()
            want.append(p.h ** 2 * float(G.cpu().numpy() @ f[tuple(inner.T)]))
    # positive terms: the transforms' rounding, some 1e-15 of the largest value on the box, which is a few times these
    assert rel_l2(got[rows], np.array(want)) < 1e-12


def test_x_pass_beyond_4_gb():
    """Two balls in opposite corners of a box whose x pass takes 64-bit offsets: its smallest radix, 3 of 2187, spans
    more than 4 GB of the grid."""
    import torch
    n, r = (1095, 243, 771), 2.6
    phi = np.full(n, 1.0)
    for at in ([6, 6, 6], [m - 7 for m in n]):
        near = np.ogrid[tuple(slice(a - 4, a + 5) for a in at)]
        phi[tuple(slice(a - 4, a + 5) for a in at)] = np.sqrt(sum((x - a) ** 2 for x, a in zip(near, at))) - r
    with P.Context(n, 1.0 / 64, (0.0, 0.0, 0.0), 0.0, "sampled", phi=phi, max_rhs=2, max_krylov=8) as c:
        del phi
        q = torch.from_numpy(np.random.default_rng(5).standard_normal((2, c.sizes["n_gamma_minus"]))).to(device())
        a, b = (torch.empty((2, c.sizes["n_targets"]), dtype=torch.float64, device=device()) for _ in range(2))
        c.apply_double_layer(q, a, P.PREC_FFT)
        c.apply_double_layer(q, b, P.PREC_FP64)
        torch.cuda.synchronize()
        M = c.get_sizes()["conv_fft"]
        assert M[0] == 2187 and (M[0] // 3 + 1) * M[1] * (M[2] // 2 + 1) * 16 > 2 ** 32
    for r in range(2):
        # the direct sum is exact to its far field's 7e-11 (the FFT takes the same kernel values)
        assert rel_l2(a[r].cpu().numpy(), b[r].cpu().numpy()) < 1e-10
