// FP64 generation of the free-space lattice Green's function table on the GPU.
//
// Paper Sec. 2.2: with L = (6+s) I - sum of the 6 shifts (s = sigma h^2), the LGF is
//   G_s(a,b,c) = int_0^inf exp(-(6+s) t) I_a(2t) I_b(2t) I_c(2t) dt
//              = int_0^inf exp(-s t) It_a(2t) It_b(2t) It_c(2t) dt,  It_n(x) = exp(-x) I_n(x),
// (Watson's transformation of eq. "lgf"; the sigma factor enters as exp(-s t)).  As in the
// paper the integral is split at T*: a quadrature rule on [0, T*] and the large-argument
// series of I_n (Abramowitz-Stegun 9.7.1) integrated term by term beyond T*.
//
// Design for the GPU (not from the paper):
//   * quadrature in u = ln t, composite 20-point Gauss-Legendre (width-4 panels on
//     [-40,-8], width-1.5 panels on [-8, ln T*]), T* = 8 R^2 + 64 so that every factor's
//     asymptotic series has ratio <= 1/32 beyond T*;
//   * B[n][q] = It_n(2 t_q), n = 0..R (nodes fastest, padded to whole steps of kStep with
//     zeros), by one of three forms without a division chain (bessel_kernel);
//   * the separable sum sum_q W_q B_a B_b B_c as FP64 matrix products, one per c (table_kernel),
//     with the tail series as its last steps.
// Table layout: sorted triple a <= b <= c at index c(c+1)(c+2)/6 + b(b+1)/2 + a (the
// 1/48 symmetry of Sec. 4).
#include <algorithm>
#include <array>
#include <cmath>
#include <mutex>

#include "internal.hpp"

namespace bae {

namespace {

constexpr int kGL = 20;          // Gauss-Legendre points per panel
constexpr int kTail = 10;        // asymptotic terms per Bessel factor
constexpr int kStep = 8;         // quadrature nodes of one unrolled step of the table's products
constexpr double kULo = -40.0;

// Gauss-Legendre nodes/weights on [-1, 1] by Newton iteration on P_n.
void gauss_legendre(int n, double* x, double* w) {
    for (int i = 0; i < n; ++i) {
        double z = std::cos(M_PI * (i + 0.75) / (n + 0.5));
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            const double dp = n * (z * p1 - p0) / (z * z - 1.0);
            const double dz = p1 / dp;
            z -= dz;
            if (std::fabs(dz) < 1e-16) {
                // final derivative at the converged node
                p0 = 1.0;
                p1 = z;
                for (int k = 2; k <= n; ++k) {
                    const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                    p0 = p1;
                    p1 = p2;
                }
                const double d = n * (z * p1 - p0) / (z * z - 1.0);
                x[i] = z;
                w[i] = 2.0 / ((1.0 - z * z) * d * d);
                break;
            }
        }
    }
}

struct TailParams {
    double J[3 * kTail + 1];   // (4 pi)^-3/2 2^-k int_T^inf e^{-st} t^{-3/2-k} dt
};

// The composite rule in u = ln t: kGL-point panels of width 4 on [kULo, -8] (n_lo of them),
// then of width 1.5 from -8, the last one ending at u_hi = ln T* (n_hi of them).
struct Rule {
    double gx[kGL], gw[kGL];   // Gauss-Legendre on [-1, 1]
    double s, u_hi;
    int n_lo, n_hi;
};

// Node q of the rule: t_q = e^u and the weight of dt = t du with the factor e^{-s t}.
__device__ inline void node(const Rule& rule, int q, double* t, double* w) {
    const int p = q / kGL, i = q % kGL;
    double lo, hi;
    if (p < rule.n_lo) {
        lo = kULo + 4.0 * p;
        hi = p + 1 < rule.n_lo ? lo + 4.0 : -8.0;
    } else {
        const int k = p - rule.n_lo;
        lo = -8.0 + 1.5 * k;
        hi = k + 1 < rule.n_hi ? lo + 1.5 : rule.u_hi;
    }
    const double u = 0.5 * (hi - lo) * rule.gx[i] + 0.5 * (hi + lo);
    const double tq = exp(u);
    *t = tq;
    *w = 0.5 * (hi - lo) * rule.gw[i] * tq * exp(-rule.s * tq);
}

// int_T^inf exp(-s t) t^{-3/2-k} dt for k = 0..kmax (host).
void tail_moments(double s, double T, int kmax, double* J) {
    if (s == 0.0) {
        for (int k = 0; k <= kmax; ++k) J[k] = std::pow(T, -(k + 0.5)) / (k + 0.5);
        return;
    }
    // s^{k+1/2} Gamma(-k-1/2, sT); Gamma(a-1,x) = (Gamma(a,x) - x^{a-1} e^{-x})/(a-1)
    const double x = s * T;
    double g = std::sqrt(M_PI) * std::erfc(std::sqrt(x));  // Gamma(1/2, x)
    double a = 0.5;
    for (int k = 0; k <= kmax; ++k) {
        g = (g - std::pow(x, a - 1.0) * std::exp(-x)) / (a - 1.0);
        a -= 1.0;
        J[k] = std::pow(s, k + 0.5) * g;
    }
}

// It_n(x) at the nodes x = 2 t_q, by the size of x:
//   x < 2^-20       the ratio I_n / I_{n-1} = (x / 2n) (1 - x^2 / (4n (n + 1))) to FP64 rounding, multiplied up;
//   x < hankel_x    Miller's recurrence I_{n-1} = I_{n+1} + (2n/x) I_n downward: one fused multiply-add
//                   per step on the chain.  For x >= 100 it starts from the ratio
//                   I_{N+1} / I_N = x / (N + 1/2 + sqrt((N + 3/2)^2 + x^2)) (to about 1e-4) at
//                   (N - 60)^2 = R^2 + 28 x, which the recurrence contracts by at least e^{-28} on the
//                   way to R, and is normalised by the series of It_0; below, from zero at
//                   (N - 60)^2 = R^2 + 81 x, normalised by It_0 + 2 sum It_{2k} = (1 + e^{-2x}) / 2.
//                   The values are scaled down by 2^-600 whenever they pass 2^300 (they grow by at most
//                   2^272 per 8 steps for x >= 2^-20); a stored row knows by its index how many
//                   scalings it has missed.  The node is in effect 2 / fl(2 / x): its weight follows,
//                   so that the integrand's stationary point hides the difference;
//   else            (x >= R^2 + 100) the large-argument series, whose terms fall at least like 1 / (2^k k!).
// What bounds it: the chain of the largest recurrence, N = 5.4 R + 60 dependent steps on one wavefront per
// 64 nodes: 46 us at R = 238.  In ratio form, each step an FP64 division, and with N = R + 60 + 10 sqrt(x) up
// to x = 16 R^2, it took 857 us (227 us at R = 60).
constexpr int kBesselThreads = 64;
constexpr int kHankelTerms = 16;

__device__ inline double bessel_large(int n, double x) {
    const double mu = 4.0 * n * (double)n, r = 1.0 / (8.0 * x);
    double term = 1.0, sum = 1.0;
#pragma unroll
    for (int k = 1; k <= kHankelTerms; ++k) {
        term *= ((2.0 * k - 1.0) * (2.0 * k - 1.0) - mu) * r * (1.0 / k);
        sum += term;
    }
    return sum / sqrt(2.0 * M_PI * x);
}

// Blocks [0, chain_blocks): one thread per node of [0, Qp); the rest: one thread per (row, node) of the
// nodes [large_q0, Q) (those of them with x >= hankel_x).
__global__ __launch_bounds__(kBesselThreads) void bessel_kernel(const Rule rule, int Q, int Qp, int R,
                                                                int chain_blocks, int large_q0, double hankel_x,
                                                                double* __restrict__ w, double* __restrict__ B) {
    constexpr double kBig = 0x1p300, kDown = 0x1p-600;
    double t, wq;
    if ((int)blockIdx.x >= chain_blocks) {
        const int64_t i = (int64_t)(blockIdx.x - chain_blocks) * kBesselThreads + threadIdx.x;
        const int nq = Q - large_q0;
        const int n = (int)(i / nq), q = large_q0 + (int)(i % nq);
        if (n > R) return;
        node(rule, q, &t, &wq);
        if (2.0 * t >= hankel_x) B[(int64_t)n * Qp + q] = bessel_large(n, 2.0 * t);
        return;
    }
    const int q = blockIdx.x * kBesselThreads + threadIdx.x;
    if (q >= Qp) return;
    double* col = B + q;
    if (q >= Q) {   // padding of the last step
        w[q] = 0.0;
        for (int n = 0; n <= R; ++n) col[(int64_t)n * Qp] = 0.0;
        return;
    }
    node(rule, q, &t, &wq);
    w[q] = wq;
    const double x = 2.0 * t;
    if (x >= hankel_x) return;
    if (x < 0x1p-20) {
        const double x2 = x * x;
        double In = exp(-x) * fma(0.25 * x2, fma(0.0625, x2, 1.0), 1.0);
        col[0] = In;
        double rn = 1.0;   // 1 / n
        for (int n = 1; n <= R; ++n) {
            const double rn1 = 1.0 / (n + 1.0);
            In *= (0.5 * x * rn) * fma(-0.25 * x2, rn * rn1, 1.0);
            rn = rn1;
            col[(int64_t)n * Qp] = In;
        }
        return;
    }
    const double c = 2.0 / x;
    w[q] = wq * fma(-rule.s * t, 0.5 * fma(-c, x, 2.0), 1.0);   // e^{-s t} at the node 2 / c
    const bool large = x >= 100.0;
    int n = 2 * ((int)(0.5 * sqrt(fma((double)R, (double)R, (large ? 28.0 : 81.0) * x))) + 30);   // even
    double f = 0x1p-300, up = 0.0, even = 0.0;   // f_n, f_{n+1}, sum of f_{2k}, 2k > n
    if (large) up = f * x / (n + 0.5 + sqrt(fma(n + 1.5, n + 1.5, x * x)));
    // f_n -> f_{n-2}, f_{n-1} (n even)
    auto pair = [&] {
        const double nd = (double)n;
        even += f;
        up = fma(nd * c, f, up);
        f = fma(fma(nd, c, -c), up, f);
        n -= 2;
    };
    // rows past e1, e2, e3 have missed one, two, three scalings, and past e4 they are below 2^-1000
    int e1 = 1 << 30, e2 = 1 << 30, e3 = 1 << 30, e4 = 1 << 30;
    auto scale_down = [&] {
        if (f > kBig) {
            f *= kDown;
            up *= kDown;
            even *= kDown;
            e4 = e3;
            e3 = e2;
            e2 = e1;
            e1 = n;
        }
    };
    while (n - 8 > R) {   // rows above R
#pragma unroll
        for (int k = 0; k < 4; ++k) pair();
        scale_down();
    }
    while (n > 0 && (n > R || n % 8 != 0)) {   // down to a multiple of 8 in the table's range
        if (n <= R) col[(int64_t)n * Qp] = f;
        pair();
        if (n + 1 <= R) col[(int64_t)(n + 1) * Qp] = up;
        scale_down();
    }
    while (n > 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            col[(int64_t)n * Qp] = f;
            pair();
            col[(int64_t)(n + 1) * Qp] = up;
        }
        scale_down();
    }
    const double norm = large ? bessel_large(0, x) / f : 0.5 * (1.0 + exp(-2.0 * x)) / (f + 2.0 * even);
    col[0] = f * norm;
    constexpr int K = 24;   // loads in flight
    for (int m0 = 1; m0 <= R; m0 += K) {
        double v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = col[(int64_t)min(m0 + k, R) * Qp];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int m = m0 + k;
            double y = v[k] * norm;
            if (m > e1) y *= kDown;
            if (m > e2) y *= kDown;
            if (m > e3) y *= kDown;
            if (m <= R) col[(int64_t)m * Qp] = m > e4 ? 0.0 : y;
        }
    }
}

__device__ inline int64_t tetra(int64_t c) { return c * (c + 1) * (c + 2) / 6; }

// alpha_k(n): It_n(x) ~ (2 pi x)^{-1/2} sum_k alpha_k x^{-k}; evaluated at x = 2t the
// factor 2^-k is folded into J.
__device__ inline void hankel(int n, double* a) {
    const double mu = 4.0 * n * (double)n;
    a[0] = 1.0;
    for (int k = 1; k <= kTail; ++k) a[k] = a[k - 1] * (-(mu - (2.0 * k - 1.0) * (2.0 * k - 1.0))) / (8.0 * k);
}

// Entries (a, b, c), a <= b <= c, of 16 x 16 tiles of (b, a) and CN values of c per wavefront:
//   G(a, b, c) = sum_q (W_q B_b B_c)(q) B_a(q) + sum_i V_bc(i) alpha_i(a),
//   V_bc(i) = sum_j alpha_j(b) U_c(i + j),  U_c(m) = sum_l alpha_l(c) J[m + l],
// both sums contracted by v_mfma_f64_16x16x4 (A: the row's b, B: the column's a, so that a store is a run
// of 16 consecutive entries).  A lane loads two nodes at a time: the order of the contraction is free.
// What bounds it: the FP64 matrix cores (one product of 64 cycles per 64 triples and 4 nodes) and, at small
// R, one wavefront's chain of products: 76 us at R = 238, where the products alone need 31.  One thread per
// entry, with three loads per node and the 11^3 terms of the tail, took 1425 us (105 us at R = 60).
constexpr int kTableWaves = 4;
constexpr int kTile = 16;

template <int CN>
__global__ __launch_bounds__(kTableWaves * 64) void table_kernel(const double* __restrict__ B,
                                                                 const double* __restrict__ W, int Qp, int R,
                                                                 const TailParams tp, double* __restrict__ out) {
    using V4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int kU = 2 * kTail + 2;   // U_c(m), m <= 2 kTail, and a zero
    __shared__ double sJ[3 * kTail + 1], sU[kTableWaves][CN][kU], sA[kTableWaves][kTile][kTail + 2];
    // the pair of tiles: y = tb (tb + 1) / 2 + ta, ta <= tb
    const int y = blockIdx.y;
    int tb = (int)((sqrtf(8.0f * (float)y + 1.0f) - 1.0f) * 0.5f);
    while (tb * (tb + 1) / 2 > y) --tb;
    while ((tb + 1) * (tb + 2) / 2 <= y) ++tb;
    const int b0 = tb * kTile, a0 = (y - tb * (tb + 1) / 2) * kTile;
    if (((int)blockIdx.x + 1) * CN * kTableWaves - 1 < b0) return;   // the block's every c is below b
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 15, kq = lane >> 4;
    const int c0 = ((int)blockIdx.x * kTableWaves + wave) * CN;
    if (threadIdx.x <= 3 * kTail) sJ[threadIdx.x] = tp.J[threadIdx.x];
    const int a = min(a0 + row, R), b = min(b0 + row, R);
    double h[kTail + 1];
    hankel(a, h);
    if (kq == 0) {
        for (int i = 0; i <= kTail; ++i) sA[wave][row][i] = h[i];
        sA[wave][row][kTail + 1] = 0.0;
    }
    __syncthreads();
    for (int cn = 0; cn < CN; ++cn) {
        hankel(min(c0 + cn, R), h);
        if (lane < kU) {
            double u = 0.0;
            if (lane <= 2 * kTail)
                for (int l = 0; l <= kTail; ++l) u = fma(h[l], sJ[lane + l], u);
            sU[wave][cn][lane] = u;
        }
    }
    __syncthreads();
    if (c0 > R || c0 + CN - 1 < b0) return;   // (no barrier below)
    typedef double d2 __attribute__((ext_vector_type(2)));
    const double *pa = B + (int64_t)a * Qp + 2 * kq, *pb = B + (int64_t)b * Qp + 2 * kq, *pw = W + 2 * kq;
    const double* pc[CN];
    V4 acc[CN];
#pragma unroll
    for (int cn = 0; cn < CN; ++cn) {
        pc[cn] = B + (int64_t)min(c0 + cn, R) * Qp + 2 * kq;
        acc[cn] = V4{0.0, 0.0, 0.0, 0.0};
    }
    // the next step's loads in flight while this one is contracted
    d2 va = *(const d2*)pa, vb = *(const d2*)pb, vw = *(const d2*)pw, vc[CN];
#pragma unroll
    for (int cn = 0; cn < CN; ++cn) vc[cn] = *(const d2*)pc[cn];
    for (int q = 0; q < Qp; q += kStep) {
        const int nq = q + kStep < Qp ? q + kStep : q;
        const d2 na = *(const d2*)(pa + nq), nb = *(const d2*)(pb + nq), nw = *(const d2*)(pw + nq);
        d2 nc[CN];
#pragma unroll
        for (int cn = 0; cn < CN; ++cn) nc[cn] = *(const d2*)(pc[cn] + nq);
        const double bx = vb.x * vw.x, by = vb.y * vw.y;
#pragma unroll
        for (int cn = 0; cn < CN; ++cn) acc[cn] = __builtin_amdgcn_mfma_f64_16x16x4f64(bx * vc[cn].x, va.x, acc[cn], 0, 0, 0);
#pragma unroll
        for (int cn = 0; cn < CN; ++cn) acc[cn] = __builtin_amdgcn_mfma_f64_16x16x4f64(by * vc[cn].y, va.y, acc[cn], 0, 0, 0);
        va = na;
        vb = nb;
        vw = nw;
#pragma unroll
        for (int cn = 0; cn < CN; ++cn) vc[cn] = nc[cn];
    }
    hankel(b, h);
#pragma unroll
    for (int s = 0; s < 3; ++s) {   // the tail: i = 4 s + kq <= kTail (i = kTail + 1 has alpha = 0)
        const int i = 4 * s + kq;
        const double ha = sA[wave][row][i];
#pragma unroll
        for (int cn = 0; cn < CN; ++cn) {
            double v = 0.0;
            for (int j = 0; j <= kTail; ++j) v = fma(h[j], sU[wave][cn][i + j], v);
            acc[cn] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, ha, acc[cn], 0, 0, 0);
        }
    }
    const int ao = a0 + row;
#pragma unroll
    for (int cn = 0; cn < CN; ++cn) {
        const int c = c0 + cn;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int bo = b0 + kq + 4 * v;   // the f64 result's row
            if (c <= R && bo <= c && ao <= bo) out[tetra(c) + (int64_t)bo * (bo + 1) / 2 + ao] = acc[cn][v];
        }
    }
}

}  // namespace

int64_t table_size(int R) { return (int64_t)(R + 1) * (R + 2) * (R + 3) / 6; }

// Host part of the rule for radius R (no heap allocation): T* = 8 R^2 + 64.
static void make_rule(double s, int R, Rule& rule, TailParams& tp, int& Q) {
    static const struct Nodes {
        double x[kGL], w[kGL];
        Nodes() { gauss_legendre(kGL, x, w); }
    } gl;
    const double T = 8.0 * R * (double)R + 64.0;
    rule.s = s;
    rule.u_hi = std::log(T);
    for (int i = 0; i < kGL; ++i) {
        rule.gx[i] = gl.x[i];
        rule.gw[i] = gl.w[i];
    }
    rule.n_lo = 0;
    for (double u = kULo; u < -8.0 - 1e-12; u += 4.0) rule.n_lo++;
    rule.n_hi = 0;
    for (double u = -8.0; u < rule.u_hi - 1e-9; u += 1.5) rule.n_hi++;
    Q = (rule.n_lo + rule.n_hi) * kGL;
    double J[3 * kTail + 1];
    tail_moments(s, T, 3 * kTail, J);
    const double c0 = std::pow(4.0 * M_PI, -1.5);
    for (int k = 0; k <= 3 * kTail; ++k) tp.J[k] = c0 * std::ldexp(J[k], -k);
}

static int padded_nodes(int Q) { return (Q + kStep - 1) / kStep * kStep; }

// The two launches on `stream`; scratch: Qp (R + 2) doubles, Qp = padded_nodes(Q), 16-byte aligned (weights,
// then the scaled Bessel values B[n][q]).
static void launch_table(const Rule& rule, const TailParams& tp, int Q, int R, double* scratch, double* out,
                         hipStream_t stream) {
    const int Qp = padded_nodes(Q);
    double* dw = scratch;
    double* dB = scratch + Qp;
    const double hankel_x = (double)R * R + 100.0;
    // nodes from the panel that holds x = hankel_x on
    const int panel = std::max(0, std::min(rule.n_hi, (int)((std::log(0.5 * hankel_x) + 8.0) / 1.5)));
    const int large_q0 = (rule.n_lo + panel) * kGL;
    const int chain = (Qp + kBesselThreads - 1) / kBesselThreads;
    const int64_t large = ((int64_t)(Q - large_q0) * (R + 1) + kBesselThreads - 1) / kBesselThreads;
    bessel_kernel<<<(unsigned)(chain + large), kBesselThreads, 0, stream>>>(rule, Q, Qp, R, chain, large_q0, hankel_x,
                                                                            dw, dB);
    BAE_HIP_CHECK(hipGetLastError());
    const int tiles = R / kTile + 1;
    const unsigned pairs = (unsigned)(tiles * (tiles + 1) / 2);
    // four values of c share a wavefront's loads of the tile rows (76 us at R = 238; 115 with two); below
    // R = 128 that leaves too few wavefronts (80 at R = 60, for 1024 SIMDs) and each takes one
    auto grid = [&](int cn) { return dim3((unsigned)((R + kTableWaves * cn) / (kTableWaves * cn)), pairs); };
    if (R < 128) table_kernel<1><<<grid(1), kTableWaves * 64, 0, stream>>>(dB, dw, Qp, R, tp, out);
    else table_kernel<4><<<grid(4), kTableWaves * 64, 0, stream>>>(dB, dw, Qp, R, tp, out);
    BAE_HIP_CHECK(hipGetLastError());
}

void lgf_table_generate(double s, int R, double* out, hipStream_t stream) {
    Rule rule;
    TailParams tp;
    int Q = 0;
    make_rule(s, R, rule, tp, Q);
    double* scratch = nullptr;
    if (hipMalloc((void**)&scratch, sizeof(double) * (int64_t)padded_nodes(Q) * (R + 2)) != hipSuccess)
        throw Error{BAE_ERR_OOM, "LGF table scratch allocation failed"};
    try {
        launch_table(rule, tp, Q, R, scratch, out, stream);
    } catch (...) {
        (void)hipStreamSynchronize(stream);
        (void)hipFree(scratch);
        throw;
    }
    BAE_HIP_CHECK(hipStreamSynchronize(stream));   // the scratch must outlive the kernels
    BAE_HIP_CHECK(hipFree(scratch));
}

// ------------------------------------------------------------------ allocation-free form
// For callers that cannot allocate (graph capture, serving loops): the same kernels with
// their scratch in a file-scope device array that each GPU holds until the process ends.
// Host code reaches it only through the address hipGetSymbolAddress returns on that
// device; the array's own name is a host-side stand-in there.
constexpr int kNoAllocQMax = 540;   // nodes of the rule for any R <= 4096 (at most 520)
constexpr int64_t kNoAllocDoubles = (int64_t)kNoAllocQMax * (kNoAllocMaxR + 2);
static __device__ __align__(256) double scratch[kNoAllocDoubles];   // 8.9 MB

static std::mutex g_scratch_mu;
static std::array<double*, 64> g_scratch_ptr{};   // per device ordinal

static double* scratch_on(int device) {
    if (device < 0 || device >= (int)g_scratch_ptr.size()) throw Error{BAE_ERR_ARG, "device ordinal out of range"};
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // this device's copy
        if (e != hipSuccess || !p)
            throw Error{BAE_ERR_HIP, std::string("scratch address: ") + hipGetErrorString(e)};
        g_scratch_ptr[device] = (double*)p;
    }
    return g_scratch_ptr[device];
}

void lgf_table_generate_noalloc(double s, int R, double* out, hipStream_t stream) {
    if (R > kNoAllocMaxR)
        throw Error{BAE_ERR_ARG, "bae_lgf_table_noalloc: R = " + std::to_string(R) + " exceeds its scratch (R <= " +
                                     std::to_string(kNoAllocMaxR) + ")"};
    Rule rule;
    TailParams tp;
    int Q = 0;
    make_rule(s, R, rule, tp, Q);
    if (padded_nodes(Q) > kNoAllocQMax) throw Error{BAE_ERR_ARG, "bae_lgf_table_noalloc: quadrature rule exceeds its scratch"};
    int device = 0;
    BAE_HIP_CHECK(hipGetDevice(&device));
    launch_table(rule, tp, Q, R, scratch_on(device), out, stream);
}

}  // namespace bae
