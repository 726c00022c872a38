"""Reads of the convolution's kernel transform, checked on the CPU: the x pass reads its rows of K2 values at columns
k0 + live_column(pl, live) for all P lines of a block, those past the last of the H2 columns too.  Over every pair of
transform lengths along x (they set P) and z (they set H2), with the library's own plans, the largest index
read must lie within H0 H1 K2 for any H0 and H1: the largest column within its row."""
from host_program import run

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "conv.hpp"
int main() {
    using namespace bae;
    std::vector<int> lengths;
    for (int e = 5; 2 * e - 1 <= kFftMaxLen; ++e) {
        const int m = fft_smooth_length(2 * e - 1);
        if (m <= kFftMaxLen && (lengths.empty() || lengths.back() != m)) lengths.push_back(m);
    }
    long bad = 0, past = 0;
    for (int m0 : lengths) {
        FftDev p;
        p.M = m0;
        std::vector<int> c = fft_radices(m0);
        if (c.size() < 2) { std::printf("no radices %d\n", m0); return 1; }
        std::sort(c.begin(), c.end(), std::greater<int>());   // as the x pass orders them
        p.nc = (int)c.size();
        std::copy(c.begin(), c.end(), p.c);
        const int P = lines_for(p);
        for (int m2 : lengths) {
            const int H2 = m2 / 2 + 1, K2 = (H2 + 7) / 8 * 8;
            for (int k0 = 0; k0 < H2; k0 += P) {
                const int live = std::min(P, H2 - k0);
                if (k0 + P > K2) ++past;
                for (int pl = 0; pl < P; ++pl) {
                    const int col = k0 + live_column(pl, live);
                    if (col < 0 || col >= H2 || (pl < live && col != k0 + pl)) ++bad;
                }
            }
        }
    }
    std::printf("%zu %ld %ld\n", lengths.size(), bad, past);
}
"""


def test_columns_stay_within_the_rows(tmp_path):
    lengths, bad, past = map(int, run(tmp_path, PROGRAM)[-1].split())
    assert lengths > 100 and past > 0   # blocks that reach past the rows' pitch do occur
    assert bad == 0
