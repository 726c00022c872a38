// Fast summation of the LGF sum by FFT convolution (the paper's stated future work, Sec. 3.5
// and Sec. 5): every source and target of one context lies in the box of N+ u E, so the sum
// v(t) = sum_s w(s) G(t - s) is a convolution on that box.  Zero padding to M_d >= 2 e_d - 1
// per axis makes the cyclic convolution on the padded grid exact on the box (Hockney), with
// the kernel sampled at the wrapped offsets: g(i) = G(i) for i < e, G(M - i) for i > M - e.
// G is even in every coordinate, so its transform is real and even: one octant is stored.
//
// Per right-hand side the transform is pruned to where data are, on half spectra k <= M2/2 along z (real data):
//   y pass    the z spectra of the e0 x e1 rows, formed from the few points of each row (conv_y_fwd), and the
//             forward y transforms of e0 x (M2/2 + 1) lines
//   x pass    forward x transforms of all M1 x (M2/2 + 1) lines, the product by the kernel's transform and the
//             inverse x transforms, which keep only the e0 planes of the box (conv_x)
//   y inverse back to the box's rows that hold targets (conv_y_inv)
//   z         the inverse z transform at the targets of each row, a sum over its half spectrum (conv_z_targets)
// A set with many points per row (the volume potential's M+) goes through dense rows instead: two real rows per
// complex z FFT (conv_z_fwd, conv_z_inv).  All passes are FP64; lines transform in LDS.
#include <algorithm>
#include <cmath>
#include <functional>
#include <mutex>

#include "conv.hpp"
#include "fft_device.hpp"
#include "lgf_device.hpp"

namespace bae {

namespace {

using namespace fftdev;

constexpr int kConvThreads = kFftThreads;
constexpr int kIt = kFftPoints / kConvThreads;   // elements per thread of a block's lines, at most

__device__ __forceinline__ int64_t idx3(int i, int j, int k, int n1, int n2) { return ((int64_t)i * n1 + j) * n2 + k; }

// Pass 1: forward z transforms of the real rows (i < e0, j < e1) of R [e0][e1][e2], zero-padded
// to M2, two rows per complex FFT (Z = F(a + i b): F a = (Z_k + conj Z_{-k}) / 2,
// F b = (Z_k - conj Z_{-k}) / 2i); the half spectrum k < H2 = M2/2 + 1 into C [e0][M1][H2].
template <int THREADS>
__global__ __launch_bounds__(THREADS, 4) void conv_z_fwd(const double* __restrict__ R, int e0, int e1, int e2,
                                                          int64_t plane, int K2, double2* __restrict__ C, const FftDev p, int P,
                                                          const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    __shared__ int64_t cbase[kMaxLinesPerBlock];   // start of row l0 + pl's half spectrum in C (-1: none)
    if (skip && *skip) return;
    const int M = p.M, nfft = P / 2;
    double2* A = lds;
    double2* tw = A + (int64_t)nfft * M;
    load_roots(p, tw);
    double* Ad = (double*)A;
    const int64_t l0 = (int64_t)xcd_group(blockIdx.x, gridDim.x) * P, nl = (int64_t)e0 * e1;
    const int H = M / 2 + 1;
    if ((int)threadIdx.x < P) {
        const int64_t l = l0 + threadIdx.x;
        cbase[threadIdx.x] = l < nl ? (l / e1) * plane + (l % e1) * K2 : -1;
    }
    for (int e = threadIdx.x; e < nfft * M; e += blockDim.x) A[e] = make_double2(0.0, 0.0);
    __syncthreads();
    const float re2 = rcp_up(e2), rH = rcp_up(H);
    // every load of the thread issued before the first LDS write (one memory latency, not eight)
    {
        double v[kIt];
        int at[kIt];
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int e = threadIdx.x + it * THREADS;
            at[it] = -1;
            if (e >= P * e2) continue;
            const int pl = fdiv_up(e, re2), k = e - pl * e2;
            if (cbase[pl] < 0) continue;
            v[it] = R[(l0 + pl) * e2 + k];
            at[it] = 2 * ((pl >> 1) * M + k) + (pl & 1);
        }
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            if (at[it] >= 0) Ad[at[it]] = v[it];
        // P e2 can pass kFftPoints by up to P / 2 (e2 <= (M + 1) / 2)
        for (int e = threadIdx.x + kIt * THREADS; e < P * e2; e += THREADS) {
            const int pl = fdiv_up(e, re2), k = e - pl * e2;
            if (cbase[pl] >= 0) Ad[2 * ((pl >> 1) * M + k) + (pl & 1)] = R[(l0 + pl) * e2 + k];
        }
    }
    __syncthreads();
    fft_lds<THREADS, false>(A, nfft, p, tw);
    const double2* Z = A;
    for (int e = threadIdx.x; e < P * H; e += blockDim.x) {
        const int pl = fdiv_up(e, rH), k = e - pl * H;
        const int64_t cb = cbase[pl];
        if (cb < 0) continue;
        const double2* z = Z + (int64_t)(pl >> 1) * M;
        const double2 a = z[k], b = z[k == 0 ? 0 : M - k];
        // b is conjugated: conj(b) = (b.x, -b.y)
        const double2 X = (pl & 1) ? make_double2(0.5 * (a.y + b.y), -0.5 * (a.x - b.x))
                                   : make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
        C[cb + k] = X;
    }
}

// The lines of a block in LDS: buffer, then the root table.
__device__ __forceinline__ Lines block_lines(double2* lds, int M, int P) {
    Lines L;
    L.A = lds;
    L.P = P;
    L.M = M;
    L.LS = M | 1;
    L.tw = lds + (int64_t)P * L.LS;
    L.rP = rcp_up(P);
    return L;
}

// base[off bytes] with a wavefront-uniform base and a per-lane offset
template <typename T, typename Off>
__device__ __forceinline__ T& at_bytes(T* base, Off off) {
    return *(T*)((char*)base + off);
}

// Forward transforms along y: the lines k of plane i (element n at n K2 + k) hold the z spectra at k of the plane's
// rows n of range[i] (all n < e1 without it), zero beyond.  A block takes P lines k of one plane.
// What bounds it: writing C (318 MB per right-hand side at 257^3): 95 us, 4.8 TB/s (143 us before the register stages).
template <int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == kLineThreads ? 3 : 2) void conv_y_fwd(double2* __restrict__ C, int64_t cstride, int kblocks, int e1,
                                                          int H2, int K2, int64_t plane, const FftDev p, int P, const int2* __restrict__ range,
                                                          const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    if (skip && *skip) return;
    const int M = p.M;
    const Lines L = block_lines(lds, M, P);
    const int group = xcd_group(blockIdx.x, gridDim.x);
    const int i = group / kblocks, k0 = (group - i * kblocks) * P;
    const int2 held = range ? range[i] : make_int2(0, e1 - 1);
    double2* base = C + (blockIdx.y * cstride + i * plane + k0);
    const int live = min(P, H2 - k0);
    load_roots(p, const_cast<double2*>(L.tw));
    auto st_lds = [&](int pl, int o, int kn, double2 x) { L.A[pl * L.LS + o + kn] = x; };
    auto ld_lds = [&](int pl, int j, int rm) { return L.A[pl * L.LS + j + rm]; };
    int Ns = 1;
    with_radix(p.c[0], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        first_stage<R, THREADS, false, true>(
            L,
            [&](int pl, int j, int rm) {
                const int n = j + rm;
                return n >= held.x && n <= held.y && pl < live
                           ? at_bytes(base + (int64_t)rm * K2, 16u * (uint32_t)(j * K2 + pl))
                           : make_double2(0.0, 0.0);
            },
            st_lds);
        Ns = R;
    });
    middle_stages<THREADS, false>(L, p, 1, 1, p.nc - 2, Ns);
    with_radix(p.c[p.nc - 1], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        last_stage<R, THREADS, false, false>(L, ld_lds, [&](int pl, int o, int kn, double2 x) {
            if (pl < live) at_bytes(base + (int64_t)kn * K2, 16u * (uint32_t)(o * K2 + pl)) = x;
        });
    });
}

// Inverse transforms along y of the same lines; of each, the rows n of range[i] are kept (all n < e1 without it).
// What bounds it: reading C: 110 us at 257^3 (139 before the register stages).
template <int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == kLineThreads ? 3 : 2) void conv_y_inv(double2* __restrict__ C, int64_t cstride, int kblocks, int e1,
                                                          int H2, int K2, int64_t plane, const FftDev p, int P, const int2* __restrict__ range,
                                                          const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    if (skip && *skip) return;
    const int M = p.M;
    const Lines L = block_lines(lds, M, P);
    const int group = xcd_group(blockIdx.x, gridDim.x);
    const int i = group / kblocks, k0 = (group - i * kblocks) * P;
    const int2 keep = range ? range[i] : make_int2(0, e1 - 1);
    if (keep.y < keep.x) return;   // no target in the plane
    double2* base = C + (blockIdx.y * cstride + i * plane + k0);
    const int live = min(P, H2 - k0);
    load_roots(p, const_cast<double2*>(L.tw));
    auto st_lds = [&](int pl, int o, int kn, double2 x) { L.A[pl * L.LS + o + kn] = x; };
    auto ld_lds = [&](int pl, int j, int rm) { return L.A[pl * L.LS + j + rm]; };
    int Ns = 1;
    with_radix(p.c[0], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        first_stage<R, THREADS, true, false>(
            L,
            [&](int pl, int j, int rm) {
                return pl < live ? at_bytes(base + (int64_t)rm * K2, 16u * (uint32_t)(j * K2 + pl)) : make_double2(0.0, 0.0);
            },
            st_lds);
        Ns = R;
    });
    middle_stages<THREADS, true>(L, p, 1, 1, p.nc - 2, Ns);
    with_radix(p.c[p.nc - 1], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        last_stage<R, THREADS, true, true>(L, ld_lds, [&](int pl, int o, int kn, double2 x) {
            const int n = o + kn;
            if (n >= keep.x && n <= keep.y && pl < live) at_bytes(base + (int64_t)kn * K2, 16u * (uint32_t)(o * K2 + pl)) = x;
        });
    });
}

// Forward x transforms (elements n < e0 loaded, zero beyond) of the lines (j, k), P values of k to a block, the
// product by the kernel's transform (even in every index: one octant), the inverse x transforms (n < e0 stored).
// The last forward stage leaves in a thread's registers exactly the inputs of the inverse's first stage (the same
// radix, n = j + k M / R), so the product and the two stages are one step.
// Off: the type of a lane's byte offset (64 bits where a stage's part of C, or the kernel's transform, passes 4 GB).
// What bounds it: reading and writing C (e0 of the M0 planes) and reading the kernel's transform, 146 us at 257^3 for
// memory alone, and about 141 us of vector issue, which three blocks per compute unit overlap little: 287 us per
// right-hand side (408 with stages of radix at most 5 that passed through LDS six times).  Leaving out the zero half of
// the first stage and the unwanted half of the last (HALF) costs registers here and made it 295 us.
template <int THREADS, typename Off>
__global__ __launch_bounds__(THREADS, THREADS == kLineThreads ? 3 : 2) void conv_x(
    double2* __restrict__ C, int64_t cstride, int kblocks, int e0, int M1, int H1, int H2, int K2, int64_t plane,
    const FftDev p, int P, const double* __restrict__ ghat, const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    if (skip && *skip) return;
    const int M = p.M;
    const Lines L = block_lines(lds, M, P);
    const int group = xcd_group(blockIdx.x, gridDim.x);
    const int row = group / kblocks, k0 = (group - row * kblocks) * P;
    double2* base = C + (blockIdx.y * cstride + (int64_t)row * K2 + k0);
    const double* gbase = ghat + ((int64_t)min(row, M1 - row) * K2 + k0);   // its row of the kernel's transform
    const int live = min(P, H2 - k0);
    load_roots(p, const_cast<double2*>(L.tw));
    auto st_lds = [&](int pl, int o, int kn, double2 x) { L.A[pl * L.LS + o + kn] = x; };
    auto ld_lds = [&](int pl, int j, int rm) { return L.A[pl * L.LS + j + rm]; };
    int Ns = 1;
    with_radix(p.c[0], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        first_stage<R, THREADS, false, false>(
            L,
            [&](int pl, int j, int rm) {
                return rm < (pl < live ? e0 - j : 0) ? at_bytes(base + rm * plane, 16 * ((Off)j * (Off)plane + (Off)pl))
                                                     : make_double2(0.0, 0.0);
            },
            st_lds);
        Ns = R;
    });
    middle_stages<THREADS, false>(L, p, 1, 1, p.nc - 2, Ns);
    with_radix(p.c[p.nc - 1], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        Stage<R, THREADS, false> s;
        constexpr int I = Stage<R, THREADS, false>::I;
        const Off gplane = (Off)H1 * (Off)K2;
        // (of lines past the row's columns too: octant_entries has room for them, and they are not stored.  Clamped to
        // the last column, whose registers this pass lacks, 16 right-hand sides at 257^3 took 10.2 ms, 9.6 so)
        auto kernel_value = [&](int pl, int n) {
            return at_bytes(gbase, 8 * ((Off)min(n, M - n) * gplane + (Off)pl));
        };
        // the values of the kernel's transform are in flight while the forward stage runs, where the registers
        // (168 of them) hold them beside its points
        constexpr bool ahead = R <= 16;
        double g[ahead ? I : 1][R];
        if constexpr (ahead) {
#pragma unroll
            for (int it = 0; it < I; ++it) {
                const int e = threadIdx.x + it * THREADS;
                if (e >= P * Ns) continue;
                const int j = fdiv_up(e, L.rP), pl = e - j * P;
#pragma unroll
                for (int k = 0; k < R; ++k) g[it][k] = kernel_value(pl, j + k * Ns);
            }
        }
        s.load(L, Ns, ld_lds);
        s.transform(L, Ns, 1);
#pragma unroll
        for (int it = 0; it < I; ++it) {
            if (s.o[it] < 0) continue;
#pragma unroll
            for (int k = 0; k < R; ++k)
                s.v[it][k] = cscale(s.v[it][k], ahead ? g[it][k] : kernel_value(s.pl[it], s.o[it] + k * Ns));
            dft<R, true>(s.v[it]);
            s.o[it] *= R;   // the inverse's first stage: outputs j R + k
        }
        __syncthreads();
        s.store(1, st_lds);
        Ns = R;
    });
    middle_stages<THREADS, true>(L, p, p.nc - 2, -1, p.nc - 2, Ns);
    with_radix(p.c[0], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        last_stage<R, THREADS, true, false>(L, ld_lds, [&](int pl, int o, int kn, double2 x) {
            if (kn < (pl < live ? e0 - o : 0)) at_bytes(base + kn * plane, 16 * ((Off)o * (Off)plane + (Off)pl)) = x;
        });
    });
}

// Complex transforms of all M elements of the lines (l / lin) sout + (l % lin) + n sline of g, in place (the
// set-up's transforms of the kernel).
template <int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == kLineThreads ? 3 : 2) void conv_lines(double2* __restrict__ g, int64_t nlines, int64_t lin,
                                                          int64_t sout, int64_t sline, const FftDev p, int P) {
    extern __shared__ double2 lds[];
    __shared__ int64_t lbase[kMaxLinesPerBlock];
    const Lines L = block_lines(lds, p.M, P);
    const int64_t l0 = (int64_t)xcd_group(blockIdx.x, gridDim.x) * P;
    load_roots(p, const_cast<double2*>(L.tw));
    if ((int)threadIdx.x < P) {
        const int64_t l = l0 + threadIdx.x;
        lbase[threadIdx.x] = l < nlines ? (l / lin) * sout + (l % lin) : -1;
    }
    __syncthreads();
    auto st_lds = [&](int pl, int o, int kn, double2 x) { L.A[pl * L.LS + o + kn] = x; };
    auto ld_lds = [&](int pl, int j, int rm) { return L.A[pl * L.LS + j + rm]; };
    int Ns = 1;
    with_radix(p.c[0], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        first_stage<R, THREADS, false, false>(L, [&](int pl, int j, int rm) {
            return lbase[pl] >= 0 ? g[lbase[pl] + (j + rm) * sline] : make_double2(0.0, 0.0);
        }, st_lds);
        Ns = R;
    });
    middle_stages<THREADS, false>(L, p, 1, 1, p.nc - 2, Ns);
    with_radix(p.c[p.nc - 1], [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        last_stage<R, THREADS, false, false>(L, ld_lds, [&](int pl, int o, int kn, double2 x) {
            if (lbase[pl] >= 0) g[lbase[pl] + (o + kn) * sline] = x;
        });
    });
}

// The half spectra along z of the rows that hold sources (and of the rows between them): X_k = sum w e^{-2 pi i k z / M2}
// over the row's sources (z, w).  One wavefront per row, its lanes along k.
// What bounds it: writing the rows (125 MB per right-hand side at 257^3): 50 us.  Clearing the box, scattering the
// weights and transforming its dense rows took 95 us.
constexpr int kZThreads = 256;
constexpr int kZRows = 4;   // spectral values of a lane in flight

__global__ __launch_bounds__(kZThreads) void conv_z_sources(double2* __restrict__ C, int64_t cstride, int64_t plane, int H2,
                                                            int K2, const FftDev pz, uint32_t zmagic,
                                                            const int4* __restrict__ rows, int nrows,
                                                            const int2* __restrict__ pts, const double* __restrict__ w,
                                                            int64_t ldw, const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    if (skip && *skip) return;
    load_roots(pz, lds);
    __syncthreads();
    C += blockIdx.y * cstride;
    w += blockIdx.y * ldw;
    const uint32_t M = (uint32_t)pz.M;
    const int lane = threadIdx.x & 63, waves = gridDim.x * (kZThreads / 64);
    for (int r = blockIdx.x * (kZThreads / 64) + (threadIdx.x >> 6); r < nrows; r += waves) {
        const int4 row = rows[r];
        const int q0 = __builtin_amdgcn_readfirstlane(row.z), q1 = __builtin_amdgcn_readfirstlane(row.w);
        double2* X = C + (row.x * plane + (int64_t)row.y * K2);
        for (int k0 = 0; k0 < H2; k0 += 64 * kZRows) {
            double2 acc[kZRows];
#pragma unroll
            for (int u = 0; u < kZRows; ++u) acc[u] = make_double2(0.0, 0.0);
            for (int q = q0; q < q1; q += 64) {   // (a surface has few sources in a row: one turn)
                const int nq = min(64, q1 - q);
                const int2 mine = pts[q + min(lane, nq - 1)];
                const double wm = w[mine.y];
                for (int t = 0; t < nq; ++t) {
                    const uint32_t z = (uint32_t)__builtin_amdgcn_readlane(mine.x, t);
                    const double x = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(wm), t),
                                                      __builtin_amdgcn_readlane(__double2loint(wm), t));
                    const uint32_t step = mod_by(64u * z, M, zmagic);
                    uint32_t a = mod_by((uint32_t)min(k0 + lane, H2) * z, M, zmagic);
#pragma unroll
                    for (int u = 0; u < kZRows; ++u) {
                        const double2 c = lds[a];
                        acc[u].x = fma(x, c.x, acc[u].x);
                        acc[u].y = fma(x, c.y, acc[u].y);
                        a += step;
                        a = min(a, a - M);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kZRows; ++u) {
                const int k = k0 + 64 * u + lane;
                if (k < H2) X[k] = acc[u];
            }
        }
    }
}

// The inverse z transform at the targets of each row (i, j) that holds some: out = scale (X_0 + 2 sum_{0 < k <
// M2/2} Re X_k e^{2 pi i k z / M2} (+ X_{M2/2} (-1)^z for even M2)).  One wavefront per row, its lanes along k;
// four targets at a time, whose sums are folded together (each fold halves the lanes and the sums).
// What bounds it: reading the rows of C that hold targets (125 MB at 257^3): 60 us.  The dense inverse and a gather
// took 81 us.
__global__ __launch_bounds__(kZThreads) void conv_z_targets(const double2* __restrict__ C, int64_t cstride, int64_t plane,
                                                            int H2, int K2, const FftDev pz, uint32_t zmagic,
                                                            const int4* __restrict__ rows, int nrows,
                                                            const int2* __restrict__ pts, double* __restrict__ out,
                                                            int64_t ldo, double scale, const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    if (skip && *skip) return;
    load_roots(pz, lds);
    __syncthreads();
    C += blockIdx.y * cstride;
    out += blockIdx.y * ldo;
    const uint32_t M = (uint32_t)pz.M;
    const int lane = threadIdx.x & 63, waves = gridDim.x * (kZThreads / 64);
    for (int r = blockIdx.x * (kZThreads / 64) + (threadIdx.x >> 6); r < nrows; r += waves) {
        const int4 row = rows[r];
        const int q0 = __builtin_amdgcn_readfirstlane(row.z), q1 = __builtin_amdgcn_readfirstlane(row.w);
        const double2* X = C + (row.x * plane + (int64_t)row.y * K2);
        for (int q = q0; q < q1; q += 64) {   // (a surface has few targets in a row: one turn)
            const int nq = min(64, q1 - q);
            const int2 mine = pts[q + min(lane, nq - 1)];
            double sum = 0.0;   // of target q + lane
            for (int k0 = 0; k0 < H2; k0 += 64 * kZRows) {
                double2 x[kZRows];
#pragma unroll
                for (int u = 0; u < kZRows; ++u) {
                    const int k = k0 + 64 * u + lane;
                    x[u] = k < H2 ? X[k] : make_double2(0.0, 0.0);
                    if (k > 0 && 2 * k < (int)M) x[u] = cscale(x[u], 2.0);
                }
                for (int t0 = 0; t0 < nq; t0 += 4) {
                    double v[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const uint32_t z = (uint32_t)__builtin_amdgcn_readlane(mine.x, min(t0 + t, nq - 1));
                        const uint32_t step = mod_by(64u * z, M, zmagic);
                        uint32_t a = mod_by((uint32_t)min(k0 + lane, H2) * z, M, zmagic);
                        double s = 0.0;
#pragma unroll
                        for (int u = 0; u < kZRows; ++u) {
                            const double2 c = lds[a];   // (cos, -sin)
                            s = fma(x[u].x, c.x, s);
                            s = fma(x[u].y, c.y, s);
                            a += step;
                            a = min(a, a - M);
                        }
                        v[t] = s;
                    }
                    // lanes 16 t .. 16 t + 15 end with the sum of target t0 + t
                    const bool up = lane & 32, odd = lane & 16;
                    const double p0 = (up ? v[2] : v[0]) + __shfl_xor(up ? v[0] : v[2], 32, 64);
                    const double p1 = (up ? v[3] : v[1]) + __shfl_xor(up ? v[1] : v[3], 32, 64);
                    double s = (odd ? p1 : p0) + __shfl_xor(odd ? p0 : p1, 16, 64);
#pragma unroll
                    for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                    const double got = __shfl(s, ((lane - t0) & 3) * 16, 64);
                    if ((unsigned)(lane - t0) < 4u) sum += got;
                }
            }
            if (lane < nq) out[mine.y] = scale * sum;
        }
    }
}

// Last pass: inverse z transforms of the rows (i < e0, j < e1) of C (half spectra, the rest the
// conjugate mirror X_k = conj X_{M-k}), two rows per complex FFT (the results are real:
// F^-1(X_a + i X_b) = a + i b), n < e2 kept, times scale, into R.
template <int THREADS>
__global__ __launch_bounds__(THREADS, 4) void conv_z_inv(const double2* __restrict__ C, int e0, int e1, int e2,
                                                          int64_t plane, int K2, double* __restrict__ R, const FftDev p, int P,
                                                          double scale, const int32_t* __restrict__ skip) {
    extern __shared__ double2 lds[];
    __shared__ int64_t cbase[kMaxLinesPerBlock];   // start of row l0 + pl's half spectrum in C (-1: none)
    if (skip && *skip) return;
    const int M = p.M, nfft = P / 2;
    double2* A = lds;
    double2* tw = A + (int64_t)nfft * M;
    load_roots(p, tw);
    const int64_t l0 = (int64_t)xcd_group(blockIdx.x, gridDim.x) * P, nl = (int64_t)e0 * e1;
    const int H = M / 2 + 1;
    if ((int)threadIdx.x < P) {
        const int64_t l = l0 + threadIdx.x;
        cbase[threadIdx.x] = l < nl ? (l / e1) * plane + (l % e1) * K2 : -1;
    }
    __syncthreads();
    const float rM = rcp_up(M), re2 = rcp_up(e2);
    // every load of the thread issued before the first LDS write (one memory latency, not four)
    {
        double2 xa[kIt], xb[kIt];   // nfft M <= kFftPoints
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int e = threadIdx.x + it * THREADS;
            xa[it] = xb[it] = make_double2(0.0, 0.0);
            if (e >= nfft * M) continue;
            const int c = fdiv_up(e, rM), k = e - c * M;
            const int kk = k >= H ? M - k : k;
            const int64_t ba = cbase[2 * c], bb = cbase[2 * c + 1];
            if (ba >= 0) xa[it] = C[ba + kk];
            if (bb >= 0) xb[it] = C[bb + kk];
        }
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int e = threadIdx.x + it * THREADS;
            if (e >= nfft * M) continue;
            const int c = fdiv_up(e, rM), k = e - c * M;
            double2 a = xa[it], b = xb[it];
            if (k >= H) {   // the conjugate mirror
                a.y = -a.y;
                b.y = -b.y;
            }
            A[e] = make_double2(a.x - b.y, a.y + b.x);
        }
    }
    __syncthreads();
    fft_lds<THREADS, true>(A, nfft, p, tw);
    const double2* Z = A;
    for (int e = threadIdx.x; e < P * e2; e += blockDim.x) {
        const int pl = fdiv_up(e, re2), k = e - pl * e2;
        if (cbase[pl] < 0) continue;
        const double2 z = Z[(int64_t)(pl >> 1) * M + k];
        R[(l0 + pl) * e2 + k] = scale * ((pl & 1) ? z.y : z.x);
    }
}

// The kernel sampled at the wrapped offsets of the padded grid (full M0 x M1 x M2, complex with
// zero imaginary part), G exactly as the FP64 sum evaluates it.
__global__ void conv_kernel_grid(double2* __restrict__ g, int M0, int M1, int M2, int e0, int e1, int e2,
                                 const double* __restrict__ tab, int bricked, int tab_r, int full_r,
                                 int far_ok) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)M0 * M1 * M2) return;
    const int i = (int)(q / ((int64_t)M1 * M2)), j = (int)((q / M2) % M1), k = (int)(q % M2);
    auto wrap = [](int x, int M, int e) { return x < e ? x : (x > M - e ? M - x : -1); };
    const int a = wrap(i, M0, e0), b = wrap(j, M1, e1), c = wrap(k, M2, e2);
    double v = 0.0;
    if (a >= 0 && b >= 0 && c >= 0) {
        const int hi = max(a, max(b, c)), lo = min(a, min(b, c)), mid = a + b + c - hi - lo;
        if (hi > tab_r && far_ok) {
            const double X = (double)(kQuant * a), Y = (double)(kQuant * b), Z = (double)(kQuant * c);
            v = lgfdev::far_field<double>(X, Y, Z);
        } else if (hi <= full_r) {
            v = lgfdev::full_entry(tab, bricked != 0, hi, mid, lo);
        } else {
            v = __builtin_nan("");
        }
    }
    g[q] = make_double2(v, 0.0);
}

// The real part of the transformed kernel on the octant [H0][H1][H2] (rows K2 apart), zeros elsewhere.
__global__ void conv_octant(const double2* __restrict__ g, int M1, int M2, int H0, int H1, int H2, int K2,
                            double* __restrict__ out) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= octant_entries(H0, H1, K2)) return;
    const int a = (int)(q / ((int64_t)H1 * K2)), b = (int)((q / K2) % H1), c = (int)(q % K2);
    out[q] = a < H0 && c < H2 ? g[idx3(a, b, c, M1, M2)].x : 0.0;
}

__global__ void conv_scatter(const double* __restrict__ w, const int32_t* __restrict__ sidx, int64_t ns,
                             double* __restrict__ R) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < ns) R[sidx[s]] = w[s];
}

__global__ void conv_gather(const double* __restrict__ R, const int32_t* __restrict__ tidx, int64_t nt,
                            double* __restrict__ out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nt) out[t] = R[tidx[t]];
}

__global__ void conv_fill(double* __restrict__ x, int64_t n, const int32_t* __restrict__ skip) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (skip && *skip) return;
    if (i < n) x[i] = 0.0;
}

// Lines per block of the dense z passes: two packed real rows to a complex line.
int rows_for(int M) {
    const int P = 2 * fft_lines_per_block(M, 16);
    if (P > kMaxLinesPerBlock) throw Error{BAE_ERR_ARG, "LGF convolution: too many lines per block"};
    return P;
}

// The passes run 256-thread blocks of a quarter of the points and LDS, four to a compute unit,
// so that some blocks' loads and stores overlap the others' LDS stages (a 1024-thread block at
// 128 VGPRs holds a compute unit alone and runs its phases in series);
// lines longer than such a block holds (2048) take 1024-thread blocks.
constexpr int kSplit = 4;
constexpr int kSplitThreads = kConvThreads / kSplit;
constexpr size_t kSplitLdsBytes = kFftLdsBytes / kSplit;
bool split_blocks(int M) { return M <= kFftPointsPerThread * kSplitThreads; }   // one line fits a block
int split_rows(int M) {
    const int by_points = kFftPointsPerThread * kSplitThreads / M;
    const int by_lds = (int)(kSplitLdsBytes / (16 * (size_t)M)) - 1;
    return 2 * std::max(1, std::min(kMaxLinesPerBlock / 2, std::min(by_points, by_lds)));
}
// The register-stage passes: kLineBlocks blocks to a compute unit, of four wavefronts at up to 168 VGPRs.
constexpr int kLineBlocks = 3;
bool short_lines(int M) { return M <= 8 * kLineThreads; }
size_t lines_lds(int M, int P, int roots) { return sizeof(double2) * ((size_t)P * (M | 1) + roots); }

void set_lds_attr() {
    static std::once_flag once;   // (per process: the attribute holds for every device of one architecture)
    std::call_once(once, [] {
        for (const void* f :
             {(const void*)conv_z_fwd<kConvThreads>, (const void*)conv_z_fwd<kSplitThreads>,
              (const void*)conv_z_inv<kConvThreads>, (const void*)conv_z_inv<kSplitThreads>,
              (const void*)conv_y_fwd<kLongThreads>, (const void*)conv_y_fwd<kLineThreads>,
              (const void*)conv_y_inv<kLongThreads>, (const void*)conv_y_inv<kLineThreads>,
              (const void*)conv_x<kLongThreads, uint64_t>, (const void*)conv_x<kLineThreads, uint64_t>,
              (const void*)conv_x<kLongThreads, uint32_t>, (const void*)conv_x<kLineThreads, uint32_t>,
              (const void*)conv_lines<kLongThreads>, (const void*)conv_lines<kLineThreads>,
              (const void*)conv_z_sources, (const void*)conv_z_targets})
            BAE_HIP_CHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFftLdsBytes));
    });
}

// Blocks of P lines each
unsigned groups_of(int64_t nlines, int P) { return (unsigned)((nlines + P - 1) / P); }

// A transform pass of the set-up over every line of the kernel's grid.
void kernel_pass(double2* g, int64_t nlines, int64_t lin, int64_t sout, int64_t sline, const FftDev& p, hipStream_t st) {
    const int P = lines_for(p);
    const size_t lds = lines_lds(p.M, P, p.M);
    if (short_lines(p.M))
        conv_lines<kLineThreads><<<groups_of(nlines, P), kLineThreads, lds, st>>>(g, nlines, lin, sout, sline, p, P);
    else
        conv_lines<kLongThreads><<<groups_of(nlines, P), kLongThreads, lds, st>>>(g, nlines, lin, sout, sline, p, P);
    BAE_HIP_CHECK(hipGetLastError());
}

// A set's z transforms as sums over its points: a spectral value costs an LDS read and two fused multiply-adds per
// point of its row there, and a whole set of LDS stages by FFT.  Surfaces have 5 to 6 points per row, a volume's
// rows tens.
constexpr int64_t kSparseRow = 16;

// Right-hand sides whose grids C stay in the 256 MB memory-side cache together (at least one).
constexpr int64_t kCacheBytes = 128ll << 20;

void device_alloc(void** p, size_t n) {
    if (hipMalloc(p, n) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        throw Error{BAE_ERR_OOM, "LGF convolution: device allocation failed"};
    }
}

}  // namespace

// Lines per block (the LDS holds their root table beside them): those for which the wavefronts' turns through the
// stages, at about 9 + 14 R instructions each, are fewest per line.  A wavefront pays for a whole turn however
// few of its lanes hold a butterfly: at M = 375 = 25 15, eight lines are 120 and 200 butterflies (2 and 4 wavefronts).
int lines_for(const FftDev& p) {
    const int threads = short_lines(p.M) ? kLineThreads : kLongThreads;
    const size_t budget = short_lines(p.M) ? kFftLdsBytes / kLineBlocks : kFftLdsBytes;
    const int most = std::min(kMaxLinesPerBlock, (int)((budget / sizeof(double2) - p.M) / (p.M | 1)));
    int best = 1;
    double best_cost = 1e300;
    for (int P = 1; P <= most; ++P) {
        double cost = 0.0;
        for (int s = 0; s < p.nc; ++s) {
            const int waves = (P * (p.M / p.c[s]) + 63) / 64;
            if (P * (p.M / p.c[s]) > threads * fft_items(p.c[s], threads)) cost = 1e300;
            cost += (double)waves * (9.0 + 14.0 * p.c[s]);
        }
        if (cost / P <= best_cost) {
            best_cost = cost / P;
            best = P;
        }
    }
    return best;
}

int fft_smooth_length(int n) {
    for (int m = std::max(1, n);; ++m) {
        int r = m;
        for (int q : {2, 3, 5})
            while (r % q == 0) r /= q;
        if (r == 1) return m;
    }
}

ConvPoints::~ConvPoints() { (void)hipFree(mem); }

void ConvPoints::build(const ConvPlan& cp, const PointSet& ps, hipStream_t st) {
    const int e0 = cp.e[0], e1 = cp.e[1], e2 = cp.e[2];
    const int64_t nr = (int64_t)e0 * e1;
    n = ps.count;
    sparse = n > 0 && n <= kSparseRow * nr;
    auto coord = [&](int64_t i, int a) { return ps.hq[3 * i + a] / kQuant - cp.lo[a]; };
    std::vector<int32_t> row_of(n);
    for (int64_t i = 0; i < n; ++i) row_of[i] = coord(i, 0) * e1 + coord(i, 1);
    if (!sparse) {
        std::vector<int32_t> at_host(n);
        for (int64_t i = 0; i < n; ++i) at_host[i] = row_of[i] * e2 + coord(i, 2);
        device_alloc(&mem, sizeof(int32_t) * std::max<int64_t>(n, 1));
        at = (int32_t*)mem;
        if (n > 0) BAE_HIP_CHECK(hipMemcpyAsync(mem, at_host.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, st));
        BAE_HIP_CHECK(hipStreamSynchronize(st));
        return;
    }
    std::vector<int32_t> ptr(nr + 1, 0);
    std::vector<int2> range_host(e0, make_int2(e1, -1));
    for (int32_t r : row_of) ptr[r + 1]++;
    nrows = 0;
    for (int i = 0; i < e0; ++i) {
        int2& g = range_host[i];
        for (int j = 0; j < e1; ++j) {
            int32_t* p = &ptr[(int64_t)i * e1 + j];
            if (p[1]) {
                g.x = std::min(g.x, j);
                g.y = j;
            }
            p[1] += p[0];
        }
        if (g.y >= g.x) nrows += g.y - g.x + 1;
    }
    // one allocation and one copy: rows, points, ranges
    const size_t rows_bytes = sizeof(int4) * nrows, pts_bytes = sizeof(int2) * n, range_bytes = sizeof(int2) * e0;
    std::vector<char> host(rows_bytes + pts_bytes + range_bytes);
    int4* rows_host = (int4*)host.data();
    int2* pts_host = (int2*)(host.data() + rows_bytes);
    for (int i = 0; i < e0; ++i)
        for (int j = range_host[i].x; j <= range_host[i].y; ++j) {
            const int64_t r = (int64_t)i * e1 + j;
            *rows_host++ = make_int4(i, j, ptr[r], ptr[r + 1]);
        }
    for (int64_t i = 0; i < n; ++i) pts_host[ptr[row_of[i]]++] = make_int2(coord(i, 2), (int)i);
    std::copy(range_host.begin(), range_host.end(), (int2*)(host.data() + rows_bytes + pts_bytes));
    device_alloc(&mem, host.size());
    rows = (int4*)mem;
    pts = (int2*)((char*)mem + rows_bytes);
    range = (int2*)((char*)mem + rows_bytes + pts_bytes);
    BAE_HIP_CHECK(hipMemcpyAsync(mem, host.data(), host.size(), hipMemcpyHostToDevice, st));
    BAE_HIP_CHECK(hipStreamSynchronize(st));   // the host vectors are released here
}

ConvPlan::~ConvPlan() {
    (void)hipFree(ghat);
    (void)hipFree(R);
    (void)hipFree(C);
}

void ConvPlan::build(const int lo_[3], const int hi_[3], const SumTables& tabs, int max_rhs, hipStream_t st) {
    for (int a = 0; a < 3; ++a) {
        lo[a] = lo_[a];
        e[a] = hi_[a] - lo_[a] + 1;
        M[a] = fft_smooth_length(2 * e[a] - 1);
        if (M[a] > kFftMaxLen) throw Error{BAE_ERR_ARG, "LGF convolution: box too long for the LDS FFT"};
        H[a] = M[a] / 2 + 1;
    }
    K2 = (H[2] + 7) / 8 * 8;
    set_lds_attr();
    fx = fft_plan(M[0], st);
    // the x pass holds the kernel's transform beside the points of its last radix: the smallest
    std::sort(fx.c, fx.c + fx.nc, std::greater<int>());
    fy = fft_plan(M[1], st);
    fz = fft_plan(M[2], st);
    if (!fx.nc || !fy.nc || !fz.nc) throw Error{BAE_ERR_ARG, "LGF convolution: a length without register radices"};
    const int64_t full = (int64_t)M[0] * M[1] * M[2], oct = octant_entries(H[0], H[1], K2);
    plane = (int64_t)M[1] * K2;
    const int64_t one = (int64_t)sizeof(double2) * e[0] * plane;
    device_alloc((void**)&ghat, sizeof(double) * oct);
    nc = (int)std::max<int64_t>(1, std::min<int64_t>(max_rhs, kCacheBytes / one));
    // the kernel's transform: sample, three full passes (z, y, x), keep one octant.  Its grid takes C's memory where
    // that is no larger than a group's may be: an allocation and its release are 0.3 ms each, the kernels 0.06 at
    // 65^3 and 0.15 at 129^3 (a first apply there 0.9 and 1.1 ms with a grid of its own, 0.24 and 0.6 so).
    const int64_t grid = (int64_t)sizeof(double2) * full;
    int64_t held = 0;   // bytes of C
    double2* g = nullptr;
    if (grid <= kCacheBytes) {
        try {
            device_alloc((void**)&C, std::max(one * nc, grid));
            held = std::max(one * nc, grid);
            g = C;
        } catch (const Error&) {   // short of memory: in turn, below
        }
    }
    if (!C) device_alloc((void**)&g, grid);
    try {
        conv_kernel_grid<<<(unsigned)((full + 255) / 256), 256, 0, st>>>(g, M[0], M[1], M[2], e[0], e[1], e[2],
                                                                          tabs.full64, tabs.bricked ? 1 : 0, tabs.tab_r64,
                                                                          tabs.full_r, tabs.far64() ? 1 : 0);
        BAE_HIP_CHECK(hipGetLastError());
        kernel_pass(g, (int64_t)M[0] * M[1], 1, M[2], 1, fz, st);                              // rows
        kernel_pass(g, (int64_t)M[0] * M[2], M[2], (int64_t)M[1] * M[2], M[2], fy, st);        // columns of every plane
        kernel_pass(g, (int64_t)M[1] * M[2], (int64_t)M[1] * M[2], 0, (int64_t)M[1] * M[2], fx, st);
        conv_octant<<<(unsigned)((oct + 255) / 256), 256, 0, st>>>(g, M[1], M[2], H[0], H[1], H[2], K2, ghat);
        BAE_HIP_CHECK(hipGetLastError());
        BAE_HIP_CHECK(hipStreamSynchronize(st));
    } catch (...) {
        (void)hipStreamSynchronize(st);
        if (!C) (void)hipFree(g);
        throw;
    }
    if (!C) {
        (void)hipFree(g);
        try {
            device_alloc((void**)&C, one * nc);
        } catch (const Error&) {   // short of memory
            if (nc == 1) throw;
            nc = 1;
            device_alloc((void**)&C, one);
        }
        held = one * nc;
    }
    bytes = (int64_t)sizeof(double) * oct + held;
}

void ConvPlan::dense_rows() {
    if (R) return;
    const int64_t box = (int64_t)e[0] * e[1] * e[2];
    device_alloc((void**)&R, sizeof(double) * box);
    bytes += sizeof(double) * box;
}

void ConvPlan::apply(const double* w, int64_t ldw, const ConvPoints& src, const ConvPoints& tgt, double* out, int64_t ldo,
                     int nrhs, double scale, const int32_t* skip, hipStream_t st) {
    if (!R && !(src.sparse && tgt.sparse)) throw Error{BAE_ERR_STATE, "LGF convolution: no dense rows"};
    const int64_t box = (int64_t)e[0] * e[1] * e[2], one = (int64_t)e[0] * plane;
    const int64_t nrow = (int64_t)e[0] * e[1];
    const double norm = scale / ((double)M[0] * M[1] * M[2]);
    const uint32_t zmagic = mod_magic(M[2]);
    const bool splitz = split_blocks(M[2]);
    const int Pz = splitz ? split_rows(M[2]) : rows_for(M[2]);
    const size_t ldsz = sizeof(double2) * (size_t)(Pz / 2 + 1) * M[2];   // Pz / 2 complex lines, the roots
    const unsigned gz = groups_of(nrow, Pz);
    // with(block size of a line pass)
    auto lines = [&](int len, auto&& with) {
        if (short_lines(len)) with(std::integral_constant<int, kLineThreads>{});
        else with(std::integral_constant<int, kLongThreads>{});
        BAE_HIP_CHECK(hipGetLastError());
    };
    auto rows = [&](auto&& with) {
        if (splitz) with(std::integral_constant<int, kSplitThreads>{});
        else with(std::integral_constant<int, kConvThreads>{});
        BAE_HIP_CHECK(hipGetLastError());
    };
    for (int r0 = 0; r0 < nrhs; r0 += nc) {
        const int nr = std::min(nc, nrhs - r0);
        const double* wr = w + r0 * ldw;
        double* outr = out + r0 * ldo;
        // eight blocks per compute unit, each of whose wavefronts walks rows (one row to a wavefront, with 1024-thread
        // blocks, took 72 and 87 us for the two z kernels at 257^3, against 50 and 62)
        auto zgrid = [&](const ConvPoints& p) { return dim3(std::min(groups_of(p.nrows, kZThreads / 64), 8u * 256u), nr); };
        if (src.sparse) {
            conv_z_sources<<<zgrid(src), kZThreads, sizeof(double2) * M[2], st>>>(
                C, one, plane, H[2], K2, fz, zmagic, src.rows, (int)src.nrows, src.pts, wr, ldw, skip);
            BAE_HIP_CHECK(hipGetLastError());
        } else {
            for (int r = 0; r < nr; ++r) {
                conv_fill<<<(unsigned)((box + 255) / 256), 256, 0, st>>>(R, box, skip);
                if (src.n > 0) conv_scatter<<<(unsigned)((src.n + 255) / 256), 256, 0, st>>>(wr + r * ldw, src.at, src.n, R);
                rows([&](auto t) {
                    conv_z_fwd<decltype(t)::value><<<gz, decltype(t)::value, ldsz, st>>>(R, e[0], e[1], e[2], plane, K2,
                                                                                         C + r * one, fz, Pz, skip);
                });
            }
        }
        // the blocks of a pass take lines of one plane (y) or row (x): kblocks blocks of P lines for each
        const int P = lines_for(fy), kblocks = (H[2] + P - 1) / P;
        const dim3 ygrid((unsigned)(e[0] * kblocks), nr);
        const size_t ylds = lines_lds(M[1], P, M[1]);
        lines(M[1], [&](auto t) {
            constexpr int T = decltype(t)::value;
            conv_y_fwd<T><<<ygrid, T, ylds, st>>>(C, one, kblocks, e[1], H[2], K2, plane, fy, P, src.sparse ? src.range : nullptr, skip);
        });
        const int Px = lines_for(fx), xblocks = (H[2] + Px - 1) / Px;
        lines(M[0], [&](auto t) {
            constexpr int T = decltype(t)::value;
            const dim3 grid((unsigned)(M[1] * xblocks), nr);
            const size_t bytes_lds = lines_lds(M[0], Px, M[0]);
            // a lane's offset: within the largest M / R planes of C, or the kernel's transform
            const int rmin = *std::min_element(fx.c, fx.c + fx.nc);
            const int64_t reach = std::max((int64_t)(M[0] / rmin + 1) * plane * (int64_t)sizeof(double2),
                                           (int64_t)sizeof(double) * H[0] * H[1] * K2);
            if (reach < (1ll << 32))
                conv_x<T, uint32_t><<<grid, T, bytes_lds, st>>>(C, one, xblocks, e[0], M[1], H[1], H[2], K2, plane, fx, Px, ghat, skip);
            else
                conv_x<T, uint64_t><<<grid, T, bytes_lds, st>>>(C, one, xblocks, e[0], M[1], H[1], H[2], K2, plane, fx, Px, ghat, skip);
        });
        lines(M[1], [&](auto t) {
            constexpr int T = decltype(t)::value;
            conv_y_inv<T><<<ygrid, T, ylds, st>>>(C, one, kblocks, e[1], H[2], K2, plane, fy, P, tgt.sparse ? tgt.range : nullptr, skip);
        });
        if (tgt.sparse) {
            conv_z_targets<<<zgrid(tgt), kZThreads, sizeof(double2) * M[2], st>>>(
                C, one, plane, H[2], K2, fz, zmagic, tgt.rows, (int)tgt.nrows, tgt.pts, outr, ldo, norm, skip);
            BAE_HIP_CHECK(hipGetLastError());
        } else {
            for (int r = 0; r < nr; ++r) {
                rows([&](auto t) {
                    conv_z_inv<decltype(t)::value><<<gz, decltype(t)::value, ldsz, st>>>(C + r * one, e[0], e[1], e[2],
                                                                                         plane, K2, R, fz, Pz, norm, skip);
                });
                if (tgt.n > 0)
                    conv_gather<<<(unsigned)((tgt.n + 255) / 256), 256, 0, st>>>(R, tgt.at, tgt.n, outr + r * ldo);
                BAE_HIP_CHECK(hipGetLastError());
            }
        }
    }
}

}  // namespace bae
