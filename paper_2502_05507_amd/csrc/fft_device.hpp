// Device side of the LDS FFT (shared by the sine transforms and the LGF convolution).
//
// Stockham autosort stages in LDS: stage s with radix R and stride Ns maps input j + r M/R
// (r < R), twiddled by w^(r (j mod Ns) M/(Ns R)), to output (j div Ns) Ns R + (j mod Ns) + k Ns
// after an R-point DFT (w = e^(-2 pi i / M)); all inputs of a stage are read into registers
// before any output is written, so one LDS buffer serves.  Radices 2, 3, 4 and 5 have their butterflies
// written out, in registers; any other prime evaluates each output as an R-term sum straight
// from LDS.  The root table is staged in LDS by the caller.  The direction is a template
// parameter, so conjugated roots and the rotations by -i or +i fold into sign modifiers.
// Index divisions by stage constants go through a float reciprocal rounded up (below).
#pragma once

#include <type_traits>

#include "fft.hpp"

namespace bae {
namespace fftdev {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(s * a.x, s * a.y); }
// the root w^t, conjugated for the inverse transform
template <bool INV>
__device__ __forceinline__ double2 root(const double2* tw, int t) {
    const double2 w = tw[t];
    return INV ? make_double2(w.x, -w.y) : w;
}
// multiplication by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ double2 rot(double2 a) {
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}
// 1/d rounded up: the hardware reciprocal (within one ulp) times 1 + 2^-16.  For 1 <= d <= 8192
// and 0 <= e < 2^14 the product e rcp_up(d), rounded to float, lies in [e/d, floor(e/d) + 1),
// so its truncation is e div d with no correction step: the excess over e/d, below
// (e/d) 2^-15, is less than 1/d, the least distance from e/d up to the next integer.  Checked
// exhaustively over that range with reciprocals up to two ulps either side of 1/d.
__device__ __forceinline__ float rcp_up(int d) { return __builtin_amdgcn_rcpf((float)d) * (1.0f + 0x1p-16f); }
__device__ __forceinline__ int fdiv_up(int e, float rd) { return (int)((float)e * rd); }

// The R-point DFT in registers; the inputs from NZ on are zero and not read.
template <int R, bool INV, int NZ = R>
__device__ __forceinline__ void butterfly(double2 (&v)[R]) {
    if constexpr (NZ == 1) {
#pragma unroll
        for (int k = 1; k < R; ++k) v[k] = v[0];
    } else if constexpr (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 4) {
        const double2 a = NZ > 2 ? cadd(v[0], v[2]) : v[0], b = NZ > 2 ? csub(v[0], v[2]) : v[0];
        const double2 c = NZ > 3 ? cadd(v[1], v[3]) : v[1], d = rot<INV>(NZ > 3 ? csub(v[1], v[3]) : v[1]);
        v[0] = cadd(a, c);
        v[1] = cadd(b, d);
        v[2] = csub(a, c);
        v[3] = csub(b, d);
    } else if constexpr (R == 3) {
        constexpr double s3 = 0.86602540378443864676;   // sin(2 pi / 3)
        const double2 a = NZ > 2 ? cadd(v[1], v[2]) : v[1];
        const double2 t = make_double2(v[0].x - 0.5 * a.x, v[0].y - 0.5 * a.y);
        const double2 d = rot<INV>(cscale(NZ > 2 ? csub(v[1], v[2]) : v[1], s3));
        v[0] = cadd(v[0], a);
        v[1] = cadd(t, d);
        v[2] = csub(t, d);
    } else if constexpr (R == 5) {
        constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;   // cos(2pi/5), cos(4pi/5)
        constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;    // sin(2pi/5), sin(4pi/5)
        const double2 x0 = v[0];
        const double2 a1 = NZ > 4 ? cadd(v[1], v[4]) : v[1], b1 = NZ > 4 ? csub(v[1], v[4]) : v[1];
        double2 p1 = make_double2(x0.x + c1 * a1.x, x0.y + c1 * a1.y), p2 = make_double2(x0.x + c2 * a1.x, x0.y + c2 * a1.y);
        double2 q1 = cscale(b1, s1), q2 = cscale(b1, s2), sum = a1;
        if constexpr (NZ > 2) {
            const double2 a2 = NZ > 3 ? cadd(v[2], v[3]) : v[2], b2 = NZ > 3 ? csub(v[2], v[3]) : v[2];
            p1 = make_double2(p1.x + c2 * a2.x, p1.y + c2 * a2.y);
            p2 = make_double2(p2.x + c1 * a2.x, p2.y + c1 * a2.y);
            q1 = make_double2(q1.x + s2 * b2.x, q1.y + s2 * b2.y);
            q2 = make_double2(q2.x - s1 * b2.x, q2.y - s1 * b2.y);
            sum = cadd(a1, a2);
        }
        q1 = rot<INV>(q1);
        q2 = rot<INV>(q2);
        v[0] = cadd(x0, sum);
        v[1] = cadd(p1, q1);
        v[4] = csub(p1, q1);
        v[2] = cadd(p2, q2);
        v[3] = csub(p2, q2);
    }
}

// In-place stages: a block of kFftThreads threads holds `count` lines of length M (count M <=
// kFftPoints) in one LDS buffer; every thread reads its butterflies' inputs into registers,
// the block synchronises, and the outputs overwrite the buffer.
constexpr int kFftThreads = 1024;
constexpr int kFftPoints = 8192;                         // count * M per block at most

// THREADS: the block size; a block holds at most kFftPointsPerThread * THREADS points.
constexpr int kFftPointsPerThread = kFftPoints / kFftThreads;

// tstep = M / (Ns R), passed by the caller, which forms it without a division.
template <int R, int THREADS, bool INV>
__device__ __forceinline__ void stage(double2* __restrict__ buf, int count, int M, int Ns, int tstep,
                                      const double2* __restrict__ tw) {
    const int m = M / R, total = count * m;
    const float rm = rcp_up(m), rns = rcp_up(Ns);
    constexpr int I = (kFftPointsPerThread * THREADS / R + THREADS - 1) / THREADS;
    double2 v[I][R];
    int o[I];
#pragma unroll
    for (int it = 0; it < I; ++it) {
        int e = threadIdx.x + it * THREADS;
        // opaque, so that its quotients are formed here and not kept live across every stage
        // of the transform (they are invariant per radix; held, they spill)
        asm volatile("" : "+v"(e));
        o[it] = -1;
        if (e >= total) continue;
        const int c = fdiv_up(e, rm), j = e - c * m;
        const int jq = fdiv_up(j, rns), jm = j - jq * Ns;
        const double2* in = buf + c * M;
#pragma unroll
        for (int r = 0; r < R; ++r) v[it][r] = in[j + r * m];
        if (jm > 0) {
            const int t1 = jm * tstep;   // the roots w^(r t1), r t1 < M
            int t = 0;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                t += t1;
                v[it][r] = cmul(v[it][r], root<INV>(tw, t));
            }
        }
        butterfly<R, INV>(v[it]);
        o[it] = c * M + jq * Ns * R + jm;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < I; ++it) {
        if (o[it] < 0) continue;
#pragma unroll
        for (int k = 0; k < R; ++k) buf[o[it] + k * Ns] = v[it][k];
    }
}

// any radix R: every output an R-term sum, X = sum_r in[j + r m] w^(r base)
template <int THREADS, bool INV>
__device__ __forceinline__ void stage_any(double2* __restrict__ buf, int count, int M, int Ns, int R, int tstep,
                                          const double2* __restrict__ tw) {
    const int m = M / R, total = count * M;
    const float rM = rcp_up(M), rm = rcp_up(m), rns = rcp_up(Ns);
    constexpr int I = kFftPointsPerThread;
    double2 acc[I];
    int o[I];
#pragma unroll
    for (int it = 0; it < I; ++it) {
        const int e = threadIdx.x + it * THREADS;
        o[it] = -1;
        if (e >= total) continue;
        const int c = fdiv_up(e, rM), q = e - c * M;
        const int k = fdiv_up(q, rm), j = q - k * m;
        const int jq = fdiv_up(j, rns), jm = j - jq * Ns;
        const double2* in = buf + c * M;
        const int base = jm * tstep + k * m;   // < M
        double2 a = in[j];
        int t = 0;
        for (int r = 1; r < R; ++r) {
            t += base;
            if (t >= M) t -= M;
            a = cadd(a, cmul(in[j + r * m], root<INV>(tw, t)));
        }
        acc[it] = a;
        o[it] = c * M + jq * Ns * R + jm + k * Ns;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < I; ++it)
        if (o[it] >= 0) buf[o[it]] = acc[it];
}

// Workgroups are dispatched to the 8 XCDs of an MI355X round-robin (workgroup b to XCD b mod 8).
// The group of lines a workgroup takes is chosen so that each XCD walks a contiguous range of
// groups: neighbouring groups share cache lines at their edges, which that XCD's L2 then fetches
// once.  A bijection of [0, n).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_group(int b, int n) {
    const int x = b % kXcds, k = b / kXcds, q = n / kXcds, r = n % kXcds;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// Copies the root table (M entries) into LDS; the caller synchronises before fft_lds.
__device__ __forceinline__ void load_roots(const FftDev& p, double2* tw) {
    for (int t = threadIdx.x; t < p.M; t += blockDim.x) tw[t] = p.tw[t];
}

// `count` FFTs of length p.M (count p.M <= kFftPointsPerThread THREADS <= 8192) stored one
// after another in buf (LDS), in place, by a block of THREADS threads; tw: the root table in
// LDS; INV: the inverse (unnormalised) transform.  Every thread of the block must call it; the
// result is in buf when it returns.
template <int THREADS, bool INV>
__device__ __forceinline__ void fft_lds(double2* buf, int count, const FftDev& p, const double2* tw) {
    const int M = p.M;
    int Ns = 1, rest = M;   // rest = M / Ns: the product of the radices still to apply
    for (int s = 0; s < p.nf; ++s) {
        const int R = p.f[s];
        switch (R) {
            case 2: rest /= 2; stage<2, THREADS, INV>(buf, count, M, Ns, rest, tw); break;
            case 3: rest /= 3; stage<3, THREADS, INV>(buf, count, M, Ns, rest, tw); break;
            case 4: rest /= 4; stage<4, THREADS, INV>(buf, count, M, Ns, rest, tw); break;
            case 5: rest /= 5; stage<5, THREADS, INV>(buf, count, M, Ns, rest, tw); break;
            default: rest /= R; stage_any<THREADS, INV>(buf, count, M, Ns, R, rest, tw); break;
        }
        __syncthreads();
        Ns *= R;
    }
}

// ------------------------------------------------------------------ register stages
// The convolution's passes (lengths with register radices, FftDev::c).  Radices up to 25 are built from the
// butterflies above in registers, so a length up to 625 takes two stages where radices up to 5 take five; the
// first stage takes its inputs from memory and the last one gives its outputs to memory, so a line passes through
// LDS once instead of six times.  A thread holds up to 25 points (of 168 VGPRs: three wavefronts per SIMD), and
// their loads are in flight together.

// cos and sin of 2 pi k / R
template <int R>
struct Unit;
template <>
struct Unit<6> {
    static constexpr double c[6] = {1.0, 0.5, -0.5, -1.0, -0.5, 0.5};
    static constexpr double s[6] = {0.0, 0.8660254037844386, 0.8660254037844386, 0.0, -0.8660254037844386,
        -0.8660254037844386};
};
template <>
struct Unit<8> {
    static constexpr double c[8] = {1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0,
        -0.7071067811865476, 0.0, 0.7071067811865476};
    static constexpr double s[8] = {0.0, 0.7071067811865476, 1.0, 0.7071067811865476, 0.0, -0.7071067811865476,
        -1.0, -0.7071067811865476};
};
template <>
struct Unit<9> {
    static constexpr double c[9] = {1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084,
        -0.9396926207859084, -0.5, 0.17364817766693036, 0.766044443118978};
    static constexpr double s[9] = {0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386,
        0.3420201433256687, -0.3420201433256687, -0.8660254037844386, -0.984807753012208, -0.6427876096865394};
};
template <>
struct Unit<10> {
    static constexpr double c[10] = {1.0, 0.8090169943749475, 0.30901699437494745, -0.30901699437494745,
        -0.8090169943749475, -1.0, -0.8090169943749475, -0.30901699437494745, 0.30901699437494745,
        0.8090169943749475};
    static constexpr double s[10] = {0.0, 0.5877852522924731, 0.9510565162951535, 0.9510565162951535,
        0.5877852522924731, 0.0, -0.5877852522924731, -0.9510565162951535, -0.9510565162951535,
        -0.5877852522924731};
};
template <>
struct Unit<12> {
    static constexpr double c[12] = {1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0,
        -0.8660254037844386, -0.5, 0.0, 0.5, 0.8660254037844386};
    static constexpr double s[12] = {0.0, 0.5, 0.8660254037844386, 1.0, 0.8660254037844386, 0.5, 0.0, -0.5,
        -0.8660254037844386, -1.0, -0.8660254037844386, -0.5};
};
template <>
struct Unit<15> {
    static constexpr double c[15] = {1.0, 0.9135454576426009, 0.6691306063588582, 0.30901699437494745,
        -0.10452846326765347, -0.5, -0.8090169943749475, -0.9781476007338057, -0.9781476007338057,
        -0.8090169943749475, -0.5, -0.10452846326765347, 0.30901699437494745, 0.6691306063588582,
        0.9135454576426009};
    static constexpr double s[15] = {0.0, 0.4067366430758002, 0.7431448254773942, 0.9510565162951535,
        0.9945218953682733, 0.8660254037844386, 0.5877852522924731, 0.20791169081775934, -0.20791169081775934,
        -0.5877852522924731, -0.8660254037844386, -0.9945218953682733, -0.9510565162951535,
        -0.7431448254773942, -0.4067366430758002};
};
template <>
struct Unit<16> {
    static constexpr double c[16] = {1.0, 0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0,
        -0.3826834323650898, -0.7071067811865476, -0.9238795325112867, -1.0, -0.9238795325112867,
        -0.7071067811865476, -0.3826834323650898, 0.0, 0.3826834323650898, 0.7071067811865476,
        0.9238795325112867};
    static constexpr double s[16] = {0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867, 1.0,
        0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898,
        -0.7071067811865476, -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476,
        -0.3826834323650898};
};
template <>
struct Unit<18> {
    static constexpr double c[18] = {1.0, 0.9396926207859084, 0.766044443118978, 0.5, 0.17364817766693036,
        -0.17364817766693036, -0.5, -0.766044443118978, -0.9396926207859084, -1.0, -0.9396926207859084,
        -0.766044443118978, -0.5, -0.17364817766693036, 0.17364817766693036, 0.5, 0.766044443118978,
        0.9396926207859084};
    static constexpr double s[18] = {0.0, 0.3420201433256687, 0.6427876096865394, 0.8660254037844386,
        0.984807753012208, 0.984807753012208, 0.8660254037844386, 0.6427876096865394, 0.3420201433256687, 0.0,
        -0.3420201433256687, -0.6427876096865394, -0.8660254037844386, -0.984807753012208, -0.984807753012208,
        -0.8660254037844386, -0.6427876096865394, -0.3420201433256687};
};
template <>
struct Unit<20> {
    static constexpr double c[20] = {1.0, 0.9510565162951535, 0.8090169943749475, 0.5877852522924731,
        0.30901699437494745, 0.0, -0.30901699437494745, -0.5877852522924731, -0.8090169943749475,
        -0.9510565162951535, -1.0, -0.9510565162951535, -0.8090169943749475, -0.5877852522924731,
        -0.30901699437494745, 0.0, 0.30901699437494745, 0.5877852522924731, 0.8090169943749475,
        0.9510565162951535};
    static constexpr double s[20] = {0.0, 0.30901699437494745, 0.5877852522924731, 0.8090169943749475,
        0.9510565162951535, 1.0, 0.9510565162951535, 0.8090169943749475, 0.5877852522924731,
        0.30901699437494745, 0.0, -0.30901699437494745, -0.5877852522924731, -0.8090169943749475,
        -0.9510565162951535, -1.0, -0.9510565162951535, -0.8090169943749475, -0.5877852522924731,
        -0.30901699437494745};
};
template <>
struct Unit<24> {
    static constexpr double c[24] = {1.0, 0.9659258262890683, 0.8660254037844386, 0.7071067811865476, 0.5,
        0.25881904510252074, 0.0, -0.25881904510252074, -0.5, -0.7071067811865476, -0.8660254037844386,
        -0.9659258262890683, -1.0, -0.9659258262890683, -0.8660254037844386, -0.7071067811865476, -0.5,
        -0.25881904510252074, 0.0, 0.25881904510252074, 0.5, 0.7071067811865476, 0.8660254037844386,
        0.9659258262890683};
    static constexpr double s[24] = {0.0, 0.25881904510252074, 0.5, 0.7071067811865476, 0.8660254037844386,
        0.9659258262890683, 1.0, 0.9659258262890683, 0.8660254037844386, 0.7071067811865476, 0.5,
        0.25881904510252074, 0.0, -0.25881904510252074, -0.5, -0.7071067811865476, -0.8660254037844386,
        -0.9659258262890683, -1.0, -0.9659258262890683, -0.8660254037844386, -0.7071067811865476, -0.5,
        -0.25881904510252074};
};
template <>
struct Unit<25> {
    static constexpr double c[25] = {1.0, 0.9685831611286311, 0.8763066800438636, 0.7289686274214116,
        0.5358267949789967, 0.30901699437494745, 0.06279051952931337, -0.18738131458572463,
        -0.42577929156507266, -0.6374239897486897, -0.8090169943749475, -0.9297764858882515,
        -0.9921147013144779, -0.9921147013144779, -0.9297764858882515, -0.8090169943749475,
        -0.6374239897486897, -0.42577929156507266, -0.18738131458572463, 0.06279051952931337,
        0.30901699437494745, 0.5358267949789967, 0.7289686274214116, 0.8763066800438636, 0.9685831611286311};
    static constexpr double s[25] = {0.0, 0.2486898871648548, 0.48175367410171527, 0.6845471059286887,
        0.8443279255020151, 0.9510565162951535, 0.9980267284282716, 0.9822872507286887, 0.9048270524660196,
        0.7705132427757893, 0.5877852522924731, 0.368124552684678, 0.12533323356430426, -0.12533323356430426,
        -0.368124552684678, -0.5877852522924731, -0.7705132427757893, -0.9048270524660196, -0.9822872507286887,
        -0.9980267284282716, -0.9510565162951535, -0.8443279255020151, -0.6845471059286887,
        -0.48175367410171527, -0.2486898871648548};
};

// a w_R^k for a constant k (w the root of the direction)
template <int R, bool INV>
__device__ __forceinline__ double2 cunit(double2 a, int k) {
    if (k == 0) return a;
    if (4 * k == R) return rot<INV>(a);
    if (2 * k == R) return make_double2(-a.x, -a.y);
    if (4 * k == 3 * R) return rot<!INV>(a);
    const double c = Unit<R>::c[k], s = INV ? Unit<R>::s[k] : -Unit<R>::s[k];
    return make_double2(fma(a.x, c, -a.y * s), fma(a.x, s, a.y * c));
}

template <int R, bool INV, int NZ = R>
__device__ __forceinline__ void dft(double2 (&v)[R]);

// An A B-point DFT in registers: B of A points, the twiddles, A of B points.
template <int A, int B, bool INV, int NZ, int Q = 0>
__device__ __forceinline__ void dft2_columns(const double2 (&v)[A * B], double2 (&t)[B][A]) {
    if constexpr (Q < B) {
        constexpr int nz = (NZ - Q + B - 1) / B;   // the column's nonzero inputs (NZ >= B)
        double2 u[A];
#pragma unroll
        for (int p = 0; p < nz; ++p) u[p] = v[B * p + Q];
        dft<A, INV, nz>(u);
#pragma unroll
        for (int p = 0; p < A; ++p) t[Q][p] = cunit<A * B, INV>(u[p], p * Q);
        dft2_columns<A, B, INV, NZ, Q + 1>(v, t);
    }
}
template <int A, int B, bool INV, int NZ>
__device__ __forceinline__ void dft2(double2 (&v)[A * B]) {
    double2 t[B][A];
    dft2_columns<A, B, INV, NZ>(v, t);
#pragma unroll
    for (int p = 0; p < A; ++p) {
        double2 u[B];
#pragma unroll
        for (int q = 0; q < B; ++q) u[q] = t[q][p];
        dft<B, INV>(u);
#pragma unroll
        for (int q = 0; q < B; ++q) v[p + A * q] = u[q];
    }
}

template <int R, bool INV, int NZ>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
    if constexpr (R <= 5) butterfly<R, INV, NZ>(v);
    else if constexpr (R == 6) dft2<2, 3, INV, NZ>(v);
    else if constexpr (R == 8) dft2<2, 4, INV, NZ>(v);
    else if constexpr (R == 9) dft2<3, 3, INV, NZ>(v);
    else if constexpr (R == 10) dft2<2, 5, INV, NZ>(v);
    else if constexpr (R == 12) dft2<3, 4, INV, NZ>(v);
    else if constexpr (R == 15) dft2<3, 5, INV, NZ>(v);
    else if constexpr (R == 16) dft2<4, 4, INV, NZ>(v);
    else if constexpr (R == 18) dft2<3, 6, INV, NZ>(v);
    else if constexpr (R == 20) dft2<4, 5, INV, NZ>(v);
    else if constexpr (R == 24) dft2<4, 6, INV, NZ>(v);
    else dft2<5, 5, INV, NZ>(v);
}

// fn(integral constant R) for a register radix known at run time
template <typename F>
__device__ __forceinline__ void with_radix(int R, F&& fn) {
    switch (R) {
        case 3: fn(std::integral_constant<int, 3>{}); break;
        case 4: fn(std::integral_constant<int, 4>{}); break;
        case 5: fn(std::integral_constant<int, 5>{}); break;
        case 6: fn(std::integral_constant<int, 6>{}); break;
        case 8: fn(std::integral_constant<int, 8>{}); break;
        case 9: fn(std::integral_constant<int, 9>{}); break;
        case 10: fn(std::integral_constant<int, 10>{}); break;
        case 12: fn(std::integral_constant<int, 12>{}); break;
        case 15: fn(std::integral_constant<int, 15>{}); break;
        case 16: fn(std::integral_constant<int, 16>{}); break;
        case 18: fn(std::integral_constant<int, 18>{}); break;
        case 20: fn(std::integral_constant<int, 20>{}); break;
        case 24: fn(std::integral_constant<int, 24>{}); break;
        default: fn(std::integral_constant<int, 25>{}); break;
    }
}

// The lines of a block: P of length M, line pl at A + pl LS.  LS is odd, so that lines start in different LDS
// banks.  Items (butterflies) take the line index fastest: neighbouring lines are neighbours in memory.
struct Lines {
    double2* A;
    const double2* tw;   // root table in LDS
    int P, M, LS;
    float rP;
};

// One stage of radix R and stride Ns (the product of the radices before it), tstep = M / (Ns R): the butterflies of
// this thread, their inputs n = j + r M/R and outputs n = o + k Ns of line pl.  HALF: the inputs n >= (M + 1) / 2
// are zero, so those of r >= (R + 1) / 2 are not read (the first stage of a padded line).
template <int R, int THREADS, bool INV, bool HALF = false>
struct Stage {
    static constexpr int NZ = HALF ? (R + 1) / 2 : R;
    static constexpr int I = fft_items(R, THREADS);
    double2 v[I][R];
    int o[I], pl[I], jm[I];   // o: -1 where this thread has no butterfly

    // ld(pl, j, r M/R)
    template <typename Ld>
    __device__ __forceinline__ void load(const Lines& L, int Ns, Ld&& ld) {
        const int m = L.M / R, total = L.P * m;
        const float rns = rcp_up(Ns);
#pragma unroll
        for (int it = 0; it < I; ++it) {
            int e = threadIdx.x + it * THREADS;
            asm volatile("" : "+v"(e));   // its quotients are formed here, not kept live across the stages
            o[it] = -1;
            if (e >= total) continue;
            const int j = fdiv_up(e, L.rP);
            pl[it] = e - j * L.P;
            const int jq = fdiv_up(j, rns);
            jm[it] = j - jq * Ns;
            o[it] = jq * Ns * R + jm[it];
#pragma unroll
            for (int r = 0; r < NZ; ++r) v[it][r] = ld(pl[it], j, r * m);
        }
    }
    __device__ __forceinline__ void transform(const Lines& L, int Ns, int tstep) {
#pragma unroll
        for (int it = 0; it < I; ++it) {
            if (o[it] < 0) continue;
            if (Ns > 1) {
                // the roots' LDS addresses by one addition each
                const double2* w = L.tw;
                const int t1 = jm[it] * tstep;
#pragma unroll
                for (int r = 1; r < NZ; ++r) {
                    w += t1;
                    v[it][r] = cmul(v[it][r], root<INV>(w, 0));
                }
            }
            dft<R, INV, NZ>(v[it]);
        }
    }
    // st(pl, o, k Ns, value) for k < K
    template <int K = R, typename St>
    __device__ __forceinline__ void store(int Ns, St&& st) const {
#pragma unroll
        for (int it = 0; it < I; ++it) {
            if (o[it] < 0) continue;
#pragma unroll
            for (int k = 0; k < K; ++k) st(pl[it], o[it], k * Ns, v[it][k]);
        }
    }
};

// A stage in LDS, in place: the outputs overwrite the lines that the inputs came from.
template <int R, int THREADS, bool INV, typename Ld, typename St>
__device__ __forceinline__ void stage_in_place(const Lines& L, int Ns, int tstep, Ld&& ld, St&& st) {
    Stage<R, THREADS, INV> s;
    s.load(L, Ns, ld);
    s.transform(L, Ns, tstep);
    __syncthreads();
    s.store(Ns, st);
}

// The first stage of lines from memory (HALF: elements from (M + 1) / 2 on are zero), outputs by st.
template <int R, int THREADS, bool INV, bool HALF, typename Ld, typename St>
__device__ __forceinline__ void first_stage(const Lines& L, Ld&& ld, St&& st) {
    Stage<R, THREADS, INV, HALF> s;
    s.load(L, 1, ld);
    s.transform(L, 1, 0);
    s.store(1, st);
}

// The last stage of lines to memory (HALF: elements from (M + 1) / 2 on are not wanted), inputs by ld.
template <int R, int THREADS, bool INV, bool HALF, typename Ld, typename St>
__device__ __forceinline__ void last_stage(const Lines& L, Ld&& ld, St&& st) {
    Stage<R, THREADS, INV> s;
    s.load(L, L.M / R, ld);
    s.transform(L, L.M / R, 1);
    s.template store<HALF ? (R + 1) / 2 : R>(L.M / R, st);
}

// The stages between the first and the last, in LDS: radices c[from], c[from + dir], ... (count of them),
// Ns the product of the radices applied before.  Synchronised at both ends.
template <int THREADS, bool INV>
__device__ __forceinline__ void middle_stages(const Lines& L, const FftDev& p, int from, int dir, int count, int& Ns) {
    auto ld = [&](int pl, int j, int rm) { return L.A[pl * L.LS + j + rm]; };
    auto st = [&](int pl, int o, int kn, double2 x) { L.A[pl * L.LS + o + kn] = x; };
    __syncthreads();
    for (int s = 0; s < count; ++s) {
        const int R = p.c[from + dir * s];
        with_radix(R, [&](auto rc) {
            constexpr int RC = decltype(rc)::value;
            stage_in_place<RC, THREADS, INV>(L, Ns, L.M / (Ns * RC), ld, st);
        });
        __syncthreads();
        Ns *= R;
    }
}

}  // namespace fftdev
}  // namespace bae
