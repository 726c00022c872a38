// The LGF sum as an FFT convolution on the grid box (conv.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "fft.hpp"
#include "internal.hpp"

namespace bae {

struct ConvPlan;

// The points of one set (sources or targets) on the convolution's box, in the set's own order.  A set with few
// points per row (i, j) of the box (a surface) also carries them by row: its z transforms are then sums over
// those points instead of FFTs of mostly empty rows.
struct ConvPoints {
    int64_t n = 0;
    bool sparse = false;
    void* mem = nullptr;          // holds the arrays below
    int32_t* at = nullptr;        // box index of every point (not sparse)
    int2* pts = nullptr;          // (z, point) sorted by row (sparse)
    int4* rows = nullptr;         // (i, j, first point, one past the last) of the rows of every plane's range (sparse)
    int64_t nrows = 0;
    int2* range = nullptr;        // per plane i, the first and last row j that holds points (sparse)
    ConvPoints() = default;
    ConvPoints(const ConvPoints&) = delete;
    ConvPoints& operator=(const ConvPoints&) = delete;
    ~ConvPoints();
    void build(const ConvPlan& cp, const PointSet& ps, hipStream_t st);
};

// v(t) = sum_s w(s) G_s(t - s) for lattice points t, s of one box, by zero-padded FFTs:
// the box of extents e (lo its first node) is embedded in a periodic grid of M_d >= 2 e_d - 1
// nodes, on which the kernel sampled at the wrapped offsets is a circulant (Hockney's
// method), so the cyclic convolution equals the free-space sum at every node of the box.
struct ConvPlan {
    int lo[3] = {0, 0, 0}, e[3] = {0, 0, 0}, M[3] = {0, 0, 0}, H[3] = {0, 0, 0};
    int K2 = 0;                   // pitch of the half spectra along z: H2 rounded up to 128 bytes of C
    int64_t plane = 0;            // pitch of the planes of C
    FftDev fx, fy, fz;            // transforms along the three axes (lengths M0, M1, M2)
    double* ghat = nullptr;       // [H0][H1][K2] real (octant_entries): the kernel's transform on one octant
    double* R = nullptr;          // [e0][e1][e2] real: a dense set's weights in, potentials out (lazy)
    double2* C = nullptr;         // [nc][e0][M1][K2] complex: the partly transformed grids of nc right-hand sides
    int nc = 0;                   // right-hand sides of a group
    int64_t bytes = 0;
    ~ConvPlan();
    // Plans, the kernel's transform (G exactly as the FP64 sum evaluates it: the table within
    // tab_r64, the far-field expansion beyond it when the sum has one, else the full table), and C for as many of
    // max_rhs right-hand sides as stay in the memory-side cache together (one where memory is short).  C stays where
    // it is until the plan ends: a graph captured from an apply holds its address.
    void build(const int lo_[3], const int hi_[3], const SumTables& tabs, int max_rhs, hipStream_t st);
    // Allocates R once, before a set that is not sparse is first used.
    void dense_rows();
    // out[r ldo + t] = scale sum_s w[r ldw + s] G(T_t - S_s) for any nrhs (r < nrhs), in groups of nc; skipped while
    // *skip is set (when given).  Launches only.
    void apply(const double* w, int64_t ldw, const ConvPoints& src, const ConvPoints& tgt, double* out, int64_t ldo,
               int nrhs, double scale, const int32_t* skip, hipStream_t st);
};

// Lines of a transform per block of the line passes (the LDS holds their root table beside them).
int lines_for(const FftDev& p);

constexpr int kMaxLinesPerBlock = 32;   // lines_for's cap (packed real rows included)
// Values of the kernel's transform on the octant [H0][H1][H2], rows K2 apart: a block of the x pass takes P lines
// wherever it starts and reads the values of them all, up to P - 1 past the end of its row.
__host__ __device__ constexpr int64_t octant_entries(int H0, int H1, int K2) {
    return (int64_t)H0 * H1 * K2 + kMaxLinesPerBlock;
}

// a mod M for a < 2^23, 2 <= M <= kFftMaxLen, with mod_magic(M) = floor(2^32 / M) + 1: the quotient by the high product
// is exact or one too large, and the unsigned minimum takes back the step where it is.
inline uint32_t mod_magic(int M) { return (uint32_t)((1ull << 32) / (uint64_t)M) + 1u; }
__host__ __device__ inline uint32_t mod_by(uint32_t a, uint32_t M, uint32_t magic) {
    const uint32_t t = a - (uint32_t)(((uint64_t)a * magic) >> 32) * M;
    return t < t + M ? t : t + M;
}

// Smallest length >= n whose prime factors are 2, 3 and 5 (the LDS FFT's register radices).
int fft_smooth_length(int n);

}  // namespace bae
