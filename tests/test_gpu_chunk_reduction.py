"""The reduction of the sum's source chunks at the numbers of chunks where its loads in flight change: a small sum has one
chunk for each of its source blocks (4 and 5, 16 and 17), and the FFT convolution, the reference here, one."""
import numpy as np
import pytest

import paper_2502_05507_amd as P
import workloads as W

from gpu_common import device, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,n,radius", [(2, 10, 0.2), (4, 12, 0.2), (5, 13, 0.25), (8, 15, 0.3), (9, 16, 0.29),
                                             (16, 19, 0.34), (17, 20, 0.34), (21, 21, 0.36)])
def test_numbers_of_chunks(blocks, n, radius):
    import torch
    p = W.Problem("sphere", (n,) * 3, 1.0 / (n - 1), (0.0,) * 3, 0.0, "sphere", (0.5,) * 3, (radius,))
    with P.Context.from_problem(p, max_rhs=2) as c:
        assert -(-c.sizes["n_sources"] // 64) == blocks
        q = torch.from_numpy(np.random.default_rng(1).standard_normal((2, c.sizes["n_gamma_minus"]))).to(device())
        a, b = (torch.empty((2, c.sizes["n_targets"]), dtype=torch.float64, device=device()) for _ in range(2))
        c.apply_double_layer(q, a, P.PREC_FP64)
        c.apply_double_layer(q, b, P.PREC_FFT)
        torch.cuda.synchronize()
    for r in range(2):
        # the same kernel values (all from the table at these sizes), some thousand terms and transforms of 60 points
        assert rel_l2(a[r].cpu().numpy(), b[r].cpu().numpy()) < 1e-12
