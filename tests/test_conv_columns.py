"""Reads of the convolution's kernel transform, checked on the CPU: the x pass reads its rows of K2 values for all P
lines of a block, those past the last of the H2 columns too.  Over every pair of transform lengths along x (they
set P) and z (they set H2), with the library's own plans, the last block's reads of the last row must lie
within the allocation."""
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
            const int64_t end = (int64_t)((H2 + P - 1) / P) * P;   // one past the last column read
            if (end > K2) ++past;
            for (int H0 : {5, m0 / 2 + 1})
                for (int H1 : {5, 2305})
                    if (((int64_t)H0 * H1 - 1) * K2 + end > octant_entries(H0, H1, K2)) ++bad;
        }
    }
    std::printf("%zu %ld %ld\n", lengths.size(), bad, past);
}
"""


def test_reads_stay_within_the_allocation(tmp_path):
    lengths, bad, past = map(int, run(tmp_path, PROGRAM)[-1].split())
    assert lengths > 100 and past > 0   # blocks that reach past a row's pitch do occur
    assert bad == 0
