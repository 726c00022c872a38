"""The LGF table at the radii where its kernels' tiles and branches change: one 16-wide tile, its edges, and
the radius from which a wavefront takes four values of c; s small, ordinary and large (entries down to
1e-100, whose quadrature nodes take every branch of the Bessel recurrences)."""
import numpy as np
import pytest

import paper_2502_05507_amd as P
from oracle import lgf

from gpu_common import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [0, 1, 15, 16, 17, 127, 128, 131])
@pytest.mark.parametrize("s", [0.0, 0.05, 1.0])
def test_table_at_tile_edges(s, R):
    import torch
    out = torch.full((P.lgf_table_size(R),), float("nan"), dtype=torch.float64, device=device())
    P.lgf_table(s, R, out)
    torch.cuda.synchronize()
    ref = lgf.LGFTable(R, s).values
    err = np.abs(out.cpu().numpy() - ref)
    assert np.all(err <= 1e-13 * np.abs(ref) + 1e-17 * ref[0]), err.max()   # the table's parity bar
