"""The autotuner's cache: a line that bae_batch_autotune writes for several problems is the one bae_batch_create finds
for them.  The tiling decides in which order partial sums are added, so it shows in the last bits of a solve."""
import numpy as np
import pytest

import paper_2502_05507_amd as P

from gpu_common import small_problem

pytestmark = pytest.mark.gpu


def test_a_stored_line_is_found_for_several_problems(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BAE_AUTOTUNE_CACHE", str(cache))
    ctxs = []
    for n in (35, 37, 41):
        p = small_problem("sphere", n)
        c = P.Context.from_problem(p, max_rhs=1, max_krylov=64)
        assert c.sizes["n_sources"] > 16 * 64   # more source blocks than the smallest chunk and the default one hold
        xs, _, _ = c.boundary_points()
        c.set_rhs(xs[:, 0] * xs[:, 1] + xs[:, 2])
        ctxs.append(c)

    def solve():
        with P.Batch(ctxs) as b:
            b.solve(P.SOLVE_FP64, tol=1e-14, maxit=20)
            return np.concatenate([c.density() for c in ctxs])

    default = solve()                        # nothing stored: 8 blocks per chunk, one workgroup per compute unit
    with P.Batch(ctxs) as b:
        b.autotune(P.PREC_FP64)
    key = cache.read_text().split()[:-2]     # the line as written: key, blocks per chunk, grid
    assert len(cache.read_text().splitlines()) == 1 and key[-1] == "2"   # three problems: round(log2 3)
    found = {}
    for blocks in (8, 2):
        cache.write_text(" ".join(key + [str(blocks), "1"]) + "\n")
        found[blocks] = solve()
    assert np.array_equal(found[8], default)
    # lines that are not read: one problem's, and one tuned for items in a fixed order
    for line in (key[:-1] + ["0"], [key[0].removesuffix("/drawn")] + key[1:]):
        assert line != key
        cache.write_text(" ".join(line + ["2", "1"]) + "\n")
        assert np.array_equal(solve(), default)
    assert not np.array_equal(found[2], default)
    assert np.linalg.norm(found[2] - default) < 1e-11 * np.linalg.norm(default)   # rounding only
    for c in ctxs:
        c.close()
