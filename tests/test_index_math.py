"""The library's own index functions, compiled from its headers and run on the CPU over the ranges the kernels use: the
bricks of the FP64 global table and the modulo of the convolution's z sums."""
import pytest

from host_program import run

BRICKS = r"""
#include <cstdio>
#include <vector>
#include "internal.hpp"
using namespace bae;
int main() {
    const int R = %d;
    std::vector<char> used(brick_entries(R), 0);
    int64_t bricks = 0;   // in the planes before H = hi / 2
    for (int hi = 0; hi <= R; ++hi) {
        if (hi %% 2 == 0 && hi > 0)
            for (int M = 0; M < hi / 2; ++M) bricks += M / 2 + 1;
        int64_t rows = 0;   // bricks of this plane before M = mid / 2
        for (int mid = 0; mid <= hi; ++mid) {
            if (mid %% 2 == 0 && mid > 0) rows += (mid / 2 - 1) / 2 + 1;
            for (int lo = 0; lo <= mid; ++lo) {
                const uint32_t at = brick_hi(hi) + brick_mid(mid) + brick_lo(lo);
                const int64_t want = 128 * (bricks + rows + lo / 4) + 64 * (hi %% 2) + 32 * (mid %% 2) + 8 * (lo %% 4);
                if (at != want || brick_lo(lo) != brick_lo_quantised(kQuant * lo)) {
                    std::printf("(%%d, %%d, %%d) at %%u, not %%lld\n", hi, mid, lo, at, (long long)want);
                    return 1;
                }
                if (at / 8 >= used.size() || used[at / 8]++) {
                    std::printf("(%%d, %%d, %%d) has no place of its own\n", hi, mid, lo);
                    return 1;
                }
            }
        }
        if (hi %% 2 == 1 || hi == R) {
            const int H = hi / 2;
            if (brick_count(H) != bricks) { std::printf("brick_count(%%d)\n", H); return 1; }
        }
    }
    std::printf("ok\n");
}
"""

MODULO = r"""
#include <cstdio>
#include "conv.hpp"
using namespace bae;
int main() {
    long count = 0;
    for (int M = 2; M <= kFftMaxLen; M = fft_smooth_length(M + 1)) {
        const uint32_t magic = mod_magic(M);
        // k z with k <= M / 2 + 1, and 64 z, for z of a box of at most (M + 1) / 2 nodes
        const uint32_t zmax = (M + 1) / 2 - 1, top = (M / 2 + 1) * zmax > 64 * zmax ? (M / 2 + 1) * zmax : 64 * zmax;
        if (top >= 1u << 23) return 1;
        for (uint32_t a = 0, r = 0; a <= top; ++a, r = r + 1 == (uint32_t)M ? 0 : r + 1)
            if (mod_by(a, M, magic) != r) { std::printf("%u mod %d\n", a, M); return 1; }
        ++count;
    }
    std::printf("%ld\n", count);
}
"""


@pytest.mark.parametrize("R", [47, 48, 61, 238])
def test_table_bricks(tmp_path, R):
    assert run(tmp_path, BRICKS % R) == ["ok"]


def test_offsets_fit_32_bits_at_the_largest_radius(tmp_path):
    out = run(tmp_path, r"""
#include <cstdio>
#include "internal.hpp"
int main() { std::printf("%lld\n", 8ll * (long long)bae::brick_entries(bae::kMaxTableRadius)); }
""")
    assert int(out[0]) < 2 ** 32


def test_modulo_is_exact_over_every_length(tmp_path):
    assert int(run(tmp_path, MODULO)[0]) > 100
