// mix_lines.h -- the five passes for axes of n = R0*R1(*R2) cells with freely
// mixed radices (Budiardja & Cardall, arXiv:1106.0557, Sec. 2.1 and 2.2.2).
//
// Half-length lines.  A doubled line of 2n points whose upper half is zero is
// two transforms of n points:
//   Y[2j + s] = sum_{y < n} x[y] exp(-2 pi i y (j + s/2) / n),   s = 0, 1,
// and the inverse of a doubled line of which only the first half is kept is
// the sum of their adjoints.  s = 1 shifts the frequency by one half: in a
// decimation-in-time transform that only replaces k by k + s/2 in the stage
// twiddles exp(-2 pi i r (k + s/2) / (Ns R)), so the first stage (k = 0) is a
// shifted DFT (dft_half) and the others read a table of their own.  One half
// of the line is in LDS at a time, half of what the doubled line takes, so a
// compute unit holds two or more workgroups (one's memory traffic runs under
// another's transforms) with whole 64- or 128-byte row segments.
//
// A line has NB threads; stage R gives thread t the butterflies t, t + NB, ...
// of its N/R.  The inverse is the adjoint of the forward flow graph: it visits
// the stages backwards with the same twiddles and the same LDS positions, so
//  * a z line's spectrum values meet the product in the registers of the last
//    stage, and the inverse starts from those registers;
//  * each transform starts by writing the LDS positions that the same thread
//    read last in the transform before it: no barrier between them.
//
// x rows (length n, the packed real form) take the s = 0 transform.
#pragma once

#include "pass_kernels.h"

namespace pspfft {

// Lengths N = R0*R1*R2 (R2 = 1: two stages) with the threads per line NB and the z lines per
// workgroup: X(N, R0, R1, R2, NB, TILE), by precision.  Measured choices among the splits whose
// stages keep most threads busy (all five passes of one n^3 solve): what counts is that two or
// more workgroups share a CU (their registers, up to about 24 values per thread in FP32 and 16 in
// FP64, and their LDS), then few stages, then whole 128-byte row segments, then an N/R0 with a
// power of two in it, which the workspace's z tiles divide.  For example, one FP32 solve, ms: 480
// as 5*6*16 with 32 threads 2.73, 8*10*6 with 80 threads 3.9; 432 as 24*18 2.00, 9*16*3 2.3; 1024 as
// 8*8*16 35.2, 16*16*4 38; FP64 512 as 8*8*8 6.81, 4*8*16 6.83, 16*8*4 6.9.
template <typename T, int N>
struct MixRadices;
#define PSPFFT_MIX_F32_A(X)                                                                                   \
    X(25, 5, 5, 1, 5, 16) X(27, 9, 3, 1, 9, 16) X(30, 5, 6, 1, 6, 16) X(45, 9, 5, 1, 9, 16)                   \
    X(50, 5, 10, 1, 10, 16) X(54, 9, 6, 1, 9, 16) X(60, 10, 6, 1, 10, 16) X(75, 15, 5, 1, 15, 16)             \
    X(80, 10, 8, 1, 10, 16) X(81, 9, 9, 1, 9, 16) X(90, 9, 10, 1, 10, 16) X(96, 12, 8, 1, 12, 16)             \
    X(100, 10, 10, 1, 10, 16) X(108, 9, 12, 1, 12, 16) X(120, 12, 10, 1, 12, 16) X(125, 5, 5, 5, 25, 16)      \
    X(135, 9, 15, 1, 15, 16) X(144, 12, 12, 1, 12, 16)
#define PSPFFT_MIX_F32_B(X)                                                                                   \
    X(150, 5, 5, 6, 30, 16) X(160, 10, 16, 1, 16, 16) X(162, 18, 9, 1, 9, 16) X(180, 15, 12, 1, 15, 16)       \
    X(192, 16, 12, 1, 16, 16) X(200, 10, 20, 1, 10, 16) X(216, 12, 18, 1, 12, 16) X(225, 15, 15, 1, 15, 16)   \
    X(240, 15, 16, 1, 16, 16) X(243, 3, 9, 9, 27, 16) X(250, 5, 10, 5, 25, 16) X(256, 16, 16, 1, 16, 16)
#define PSPFFT_MIX_F32_C(X)                                                                                   \
    X(270, 9, 6, 5, 32, 16) X(288, 4, 6, 12, 24, 8) X(300, 5, 10, 6, 32, 16) X(320, 20, 4, 4, 16, 16)         \
    X(324, 9, 12, 3, 32, 16) X(360, 20, 18, 1, 20, 8) X(375, 15, 5, 5, 32, 16) X(384, 24, 16, 1, 24, 8)       \
    X(400, 5, 16, 5, 32, 16) X(405, 15, 9, 3, 32, 16) X(432, 24, 18, 1, 24, 8) X(450, 15, 6, 5, 32, 16)       \
    X(480, 5, 6, 16, 32, 8) X(486, 9, 18, 3, 32, 8)
#define PSPFFT_MIX_F32_D(X)                                                                                   \
    X(500, 5, 10, 10, 32, 8) X(512, 8, 8, 8, 32, 8) X(540, 9, 10, 6, 32, 8) X(576, 9, 16, 4, 64, 8)           \
    X(600, 6, 10, 10, 60, 8) X(625, 25, 25, 1, 25, 8) X(640, 20, 8, 4, 32, 8) X(648, 6, 9, 12, 54, 8)         \
    X(675, 15, 9, 5, 64, 8) X(720, 12, 5, 12, 60, 8) X(729, 27, 27, 1, 27, 8) X(750, 25, 30, 1, 30, 8)
#define PSPFFT_MIX_F32_E(X)                                                                                   \
    X(768, 12, 8, 8, 64, 8) X(800, 5, 8, 20, 64, 8) X(810, 15, 9, 6, 64, 8) X(864, 6, 8, 18, 64, 8)           \
    X(900, 15, 15, 4, 64, 8) X(960, 4, 15, 16, 64, 8) X(972, 6, 18, 9, 54, 8) X(1000, 10, 10, 10, 64, 8)      \
    X(1024, 8, 8, 16, 64, 8) X(1080, 12, 9, 10, 90, 8) X(1125, 15, 15, 5, 75, 8) X(1152, 8, 12, 12, 96, 8)
#define PSPFFT_MIX_F64_A(X)                                                                                   \
    X(25, 5, 5, 1, 5, 8) X(27, 9, 3, 1, 9, 8) X(30, 5, 6, 1, 6, 8) X(45, 9, 5, 1, 9, 8)                       \
    X(50, 5, 10, 1, 10, 8) X(54, 9, 6, 1, 9, 8) X(60, 10, 6, 1, 10, 8) X(75, 15, 5, 1, 15, 8)                 \
    X(80, 10, 8, 1, 10, 8) X(81, 9, 9, 1, 9, 8) X(90, 9, 10, 1, 10, 8) X(96, 12, 8, 1, 12, 8)                 \
    X(100, 10, 10, 1, 10, 8) X(108, 9, 12, 1, 12, 8) X(120, 15, 8, 1, 8, 8) X(125, 5, 5, 5, 25, 8)            \
    X(128, 16, 8, 1, 16, 8) X(135, 15, 9, 1, 15, 8) X(144, 12, 12, 1, 12, 8)
#define PSPFFT_MIX_F64_B(X)                                                                                   \
    X(150, 5, 5, 6, 30, 4) X(160, 10, 16, 1, 16, 8) X(162, 9, 6, 3, 27, 8) X(180, 15, 12, 1, 15, 8)           \
    X(192, 16, 12, 1, 16, 8) X(200, 5, 5, 8, 25, 8) X(216, 3, 8, 9, 27, 8) X(225, 5, 5, 9, 25, 8)             \
    X(240, 16, 15, 1, 16, 8) X(243, 3, 9, 9, 27, 8) X(250, 5, 10, 5, 25, 8) X(256, 8, 8, 4, 32, 8)
#define PSPFFT_MIX_F64_C(X)                                                                                   \
    X(270, 3, 10, 9, 30, 8) X(288, 18, 16, 1, 18, 8) X(300, 5, 10, 6, 32, 8) X(320, 20, 16, 1, 20, 8)         \
    X(324, 9, 12, 3, 32, 8) X(360, 5, 6, 12, 30, 8) X(375, 15, 5, 5, 32, 8) X(384, 12, 8, 4, 32, 8)           \
    X(400, 5, 16, 5, 32, 8) X(405, 3, 9, 15, 32, 8) X(432, 9, 16, 3, 32, 8) X(450, 15, 6, 5, 30, 8)           \
    X(480, 15, 16, 2, 32, 8) X(486, 9, 6, 9, 54, 4)
#define PSPFFT_MIX_F64_D(X)                                                                                   \
    X(500, 5, 10, 10, 50, 4) X(512, 8, 8, 8, 32, 8) X(540, 9, 6, 10, 60, 4) X(576, 12, 4, 12, 48, 4)          \
    X(600, 5, 12, 10, 60, 4) X(640, 4, 16, 10, 64, 4) X(648, 6, 9, 12, 54, 4) X(675, 15, 15, 3, 45, 4)        \
    X(720, 15, 12, 4, 64, 4) X(729, 9, 9, 9, 81, 4) X(750, 15, 10, 5, 64, 4)
#define PSPFFT_MIX_F64_E(X)                                                                                   \
    X(768, 8, 8, 12, 64, 4) X(800, 5, 16, 10, 64, 4) X(810, 15, 9, 6, 64, 4) X(864, 12, 8, 9, 96, 4)          \
    X(900, 15, 15, 4, 64, 4) X(960, 12, 10, 8, 96, 4) X(972, 9, 12, 9, 108, 4) X(1000, 10, 10, 10, 100, 4)    \
    X(1024, 8, 16, 8, 128, 4) X(1080, 12, 10, 9, 108, 4) X(1125, 15, 15, 5, 75, 4)                            \
    X(1152, 12, 8, 12, 96, 4)
#define PSPFFT_MIX_ALL(X, P) P##_A(X) P##_B(X) P##_C(X) P##_D(X) P##_E(X)
#define PSPFFT_MIX_RADICES(T, N, A, B, C, THREADS, LINES)                        \
    template <>                                                                  \
    struct MixRadices<T, N> {                                                    \
        static constexpr int R0 = A, R1 = B, R2 = C, NB = THREADS, TILE = LINES; \
    };
#define PSPFFT_MIX_RADICES_F32(N, A, B, C, D, E) PSPFFT_MIX_RADICES(float, N, A, B, C, D, E)
#define PSPFFT_MIX_RADICES_F64(N, A, B, C, D, E) PSPFFT_MIX_RADICES(double, N, A, B, C, D, E)
PSPFFT_MIX_ALL(PSPFFT_MIX_RADICES_F32, PSPFFT_MIX_F32)
PSPFFT_MIX_ALL(PSPFFT_MIX_RADICES_F64, PSPFFT_MIX_F64)

constexpr int mix_max(int a, int b) { return a > b ? a : b; }
constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Stage geometry of a length: butterflies n0, n1, nL and rounds d0, d1, dL of
// the first, second and last stage, values per thread V (any stage).
template <int N_, int R0_, int R1_, int R2_, int NB_>
struct MixGeo {
    static constexpr int N = N_, R0 = R0_, R1 = R1_, R2 = R2_, NB = NB_;
    static_assert(R0 * R1 * R2 == N, "radices of the length");
    static constexpr int ST = R2 > 1 ? 3 : 2;
    static constexpr int RL = ST == 3 ? R2 : R1;
    static constexpr int n0 = N / R0, n1 = N / R1, nL = N / RL;
    static constexpr int d0 = ceil_div(n0, NB), d1 = ceil_div(n1, NB), dL = ceil_div(nL, NB);
    static constexpr int V0 = d0 * R0, VL = dL * RL;
    static constexpr int V = mix_max(mix_max(V0, VL), d1 * R1);
    static constexpr int NTW = N - R0;  // stage twiddles of one s
    static constexpr int off_last = ST == 3 ? R0 * (R1 - 1) : 0;
};
template <typename T, int N>
using MixLen = MixGeo<N, MixRadices<T, N>::R0, MixRadices<T, N>::R1, MixRadices<T, N>::R2, MixRadices<T, N>::NB>;

// Column tiles (lines per workgroup).  z: the table's.  y (fewer values per thread): 128-byte row
// segments (16 lines in FP32, 8 in FP64) where two workgroups share a CU and stay at 512 threads,
// else 64-byte ones.
template <typename T, int N, bool Z>
struct MixTile {
    using G = MixLen<T, N>;
    static constexpr int CSZ = static_cast<int>(sizeof(cx<T>));
    static constexpr int lds(int tile) { return (N * tile + 2 * G::NTW) * CSZ; }
    static constexpr int full = 128 / CSZ;
    static constexpr int TILE =
        Z ? MixRadices<T, N>::TILE : (2 * lds(full) <= 160 * 1024 && full * G::NB <= 512 ? full : full / 2);
    static constexpr int BLOCK = TILE * G::NB;
    static constexpr size_t LDS = static_cast<size_t>(lds(TILE));
    static_assert(BLOCK <= 1024 && LDS <= 160 * 1024, "one workgroup fits");
    static_assert(kSlab % TILE == 0, "no tile has lines of two slabs");
    // wavefronts per SIMD the z kernel is compiled for: two workgroups of 384 to 512 threads per
    // CU, three of 128 to 320; FP64 and the longest registers, what they leave
    static constexpr int WPS = !Z ? 1
                               : sizeof(T) == 8 || G::V > 24
                                   ? 2
                                   : (BLOCK > 512 ? 1 : (BLOCK >= 384 ? 4 : (BLOCK >= 128 ? 3 : 1)));
};

// x rows per workgroup: about 256 threads.  In launches of many tiles a workgroup takes `rounds` of
// them one after the other (mix_rounds), as each begins with the tables: at 1152 points 18 KB beside
// two rows of 9 KB.  LDS row stride: positions P at
// P + P/R0 for even R0 (consecutive butterflies then start on different banks).
template <typename T, int N>
struct MixRow {
    using G = MixLen<T, N>;
    static constexpr int CSZ = static_cast<int>(sizeof(cx<T>));
    static constexpr int PAD = G::R0 % 2 == 0 ? 1 : 0;
    static constexpr int RP = G::R0 + PAD;
    static constexpr int S = (N / G::R0 * RP) | 1;
    static constexpr int ROWS = mix_max(1, 256 / G::NB);
    static constexpr int BLOCK = ROWS * G::NB;
    // rows, stage twiddles (s = 0), split factors
    static constexpr size_t LDS = static_cast<size_t>(ROWS * S + G::NTW + N) * CSZ;
    static_assert(LDS <= 160 * 1024, "one workgroup fits");
};

// The transforms of one line, N = R0*R1(*R2).  LDS position P of the line is at
// pos(P)*LW from `col`; PAD as in MixRow (0: columns).
template <typename T, typename G, int LW, int PAD>
struct MixFFT {
    static constexpr int N = G::N, NB = G::NB;
    static constexpr int RP = G::R0 + PAD;

    // butterflies t, t + NB, ... of a stage of radix R: f(round, butterfly)
    template <int R, typename F>
    static __device__ __forceinline__ void each(int t, F &&f) {
        constexpr int nb = N / R, D = ceil_div(nb, NB);
        sfor<0, D>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int b = t + NB * i;
            if constexpr ((i + 1) * NB <= nb) f(ic, b);
            else if (b < nb) f(ic, b);
        });
    }
    // positions b*R0 + r (after the first stage)
    static __device__ __forceinline__ int out0(int b) { return b * RP * LW; }
    // positions b + r*(N/R): base and step (N/R is a multiple of R0 past the first stage)
    static __device__ __forceinline__ int in(int b) { return (PAD ? b + b / G::R0 : b) * LW; }
    template <int R>
    static constexpr int in_step() { return N / R / G::R0 * RP * LW; }
    // positions q*R0*R1 + k + r*R0 with b = q*R0 + k (after the second of three stages)
    static __device__ __forceinline__ int out1(int b) {
        const int q = b / G::R0, k = b - q * G::R0;
        return (q * G::R1 * RP + k) * LW;
    }

    // Forward transform s of x (first-stage positions b + r*n0 in x[i*R0 + r]);
    // the result is left in v at the last stage's positions b + r*nL.  tw: the
    // table of s, twiddle r of k at [(r - 1)*Ns + k].
    template <int SH, typename TP>
    static __device__ __forceinline__ void fwd(const cx<T> *x, cx<T> *v, cx<T> *col, TP tw, int t) {
        each<G::R0>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> u[G::R0];
            sfor<0, G::R0>([&](auto rc) { constexpr int r = decltype(rc)::value; u[r] = x[i * G::R0 + r]; });
            if constexpr (SH) {
                // (values of their own: the sums that this has in common with the s = 0 transform would
                // otherwise be kept beside x from there on, 6 to 10 registers more and spills in z passes)
                sfor<0, G::R0>([&](auto rc) {
                    cx<T> &q = u[decltype(rc)::value];
                    asm volatile("" : "+v"(q.x), "+v"(q.y));
                });
                dft_half<G::R0>(u);
            } else {
                dft<G::R0, -1>(u);
            }
            cx<T> *p = col + out0(b);
            sfor<0, G::R0>([&](auto rc) { constexpr int r = decltype(rc)::value; p[r * LW] = u[r]; });
        });
        __syncthreads();
        if constexpr (G::ST == 3) {
            each<G::R1>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                const cx<T> *p = col + in(b);
                sfor<0, G::R1>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    v[i * G::R1 + r] = p[r * in_step<G::R1>()];
                });
            });
            __syncthreads();
            each<G::R1>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                const int k = b % G::R0;
                cx<T> u[G::R1];
                u[0] = v[i * G::R1];
                sfor<1, G::R1>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    u[r] = cmul(v[i * G::R1 + r], tw_at(tw, (r - 1) * G::R0 + k));
                });
                dft<G::R1, -1>(u);
                cx<T> *p = col + out1(b);
                sfor<0, G::R1>([&](auto rc) { constexpr int r = decltype(rc)::value; p[r * RP * LW] = u[r]; });
            });
            __syncthreads();
        }
        each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            const cx<T> *p = col + in(b);
            cx<T> u[G::RL];
            u[0] = p[0];
            sfor<1, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                u[r] = cmul(p[r * in_step<G::RL>()], tw_at(tw, G::off_last + (r - 1) * G::nL + b));
            });
            dft<G::RL, -1>(u);
            sfor<0, G::RL>([&](auto rc) { constexpr int r = decltype(rc)::value; v[i * G::RL + r] = u[r]; });
        });
    }

    // Adjoint of fwd: v (last-stage positions, overwritten) to first-stage positions in o,
    // added to what is there if ADD.
    template <int SH, bool ADD, typename TP>
    static __device__ __forceinline__ void inv(cx<T> *v, cx<T> *o, cx<T> *col, TP tw, int t) {
        each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> u[G::RL];
            sfor<0, G::RL>([&](auto rc) { constexpr int r = decltype(rc)::value; u[r] = v[i * G::RL + r]; });
            dft<G::RL, 1>(u);
            cx<T> *p = col + in(b);
            p[0] = u[0];
            sfor<1, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                p[r * in_step<G::RL>()] = cmulc(u[r], tw_at(tw, G::off_last + (r - 1) * G::nL + b));
            });
        });
        __syncthreads();
        if constexpr (G::ST == 3) {
            each<G::R1>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                const cx<T> *p = col + out1(b);
                sfor<0, G::R1>([&](auto rc) { constexpr int r = decltype(rc)::value; v[i * G::R1 + r] = p[r * RP * LW]; });
            });
            __syncthreads();
            each<G::R1>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                const int k = b % G::R0;
                cx<T> u[G::R1];
                sfor<0, G::R1>([&](auto rc) { constexpr int r = decltype(rc)::value; u[r] = v[i * G::R1 + r]; });
                dft<G::R1, 1>(u);
                cx<T> *p = col + in(b);
                p[0] = u[0];
                sfor<1, G::R1>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    p[r * in_step<G::R1>()] = cmulc(u[r], tw_at(tw, (r - 1) * G::R0 + k));
                });
            });
            __syncthreads();
        }
        each<G::R0>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> u[G::R0];
            const cx<T> *p = col + out0(b);
            sfor<0, G::R0>([&](auto rc) { constexpr int r = decltype(rc)::value; u[r] = p[r * LW]; });
            auto put = [&](auto rc, cx<T> w) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                if constexpr (ADD) o[i * G::R0 + r] = o[i * G::R0 + r] + w;
                else o[i * G::R0 + r] = w;
            };
            if constexpr (SH) {
                dft_half_adj<G::R0>(u, put);
            } else {
                dft<G::R0, 1>(u);
                sfor<0, G::R0>([&](auto rc) { put(rc, u[decltype(rc)::value]); });
            }
        });
    }
};

// A value that is the same for the whole workgroup, kept in a scalar register (divisions leave
// theirs in a vector register, and addresses built on it would follow).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Copy of a table of COUNT values into LDS by a workgroup of BLOCK threads in two steps: its loads go
// out ahead of the line's own, and are written when those are on their way, so a workgroup starts
// with one wait for memory instead of two.
template <typename T, int COUNT, int BLOCK>
struct MixTable {
    static constexpr int D = ceil_div(COUNT, BLOCK);
    T re[D], im[D];
    __device__ __forceinline__ void load(const void *src, int tid) {
        const auto *p = as_global(static_cast<const cx<T> *>(src));
        sfor<0, D>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int j = (i + 1) * BLOCK <= COUNT ? tid + i * BLOCK : min(tid + i * BLOCK, COUNT - 1);
            re[i] = p[j].x;
            im[i] = p[j].y;
        });
    }
    __device__ __forceinline__ void store(cx<T> *dst, int tid) const {
        sfor<0, D>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if ((i + 1) * BLOCK <= COUNT || tid + i * BLOCK < COUNT) dst[tid + i * BLOCK] = cx<T>{re[i], im[i]};
        });
    }
};

// Problem and tile of a workgroup.  A segment's problems share a plan: z passes number its tiles
// tile-major, so that the problems read one spectrum slice together; x and y passes, which have nothing
// to share, problem by problem, so that a chunk of the tile order (tile_walk) is adjacent tiles of one problem
// whatever their count.  Measured, tile-major and problem by problem, whole solves in ms: eight FP64 128^3 0.773 and
// 0.742, sixteen 1.475 and 1.396, eight 192^3 2.67 and 2.45; FP32 eight 288^3 4.84 and 4.63 (y passes -10 to -15 %),
// sixteen 192^3 2.48 and 2.41.
struct MixJob {
    const ProbArg *pa;
    int local;
    bool nyq;
};
template <bool TILE_MAJOR>
__device__ __forceinline__ MixJob mix_job(const LaunchArgs &args, int bid) {
    int sgi = 0;
    while (sgi + 1 < args.nseg && bid >= args.seg[sgi + 1].wg_begin) ++sgi;
    const Segment &sg = args.seg[sgi];
    int local = bid - sg.wg_begin, member = 0;
    if constexpr (TILE_MAJOR) {
        member = uniform(local % sg.group);
        local = uniform(local / sg.group);
    } else if (sg.group > 1) {
        const int end = sgi + 1 < args.nseg ? args.seg[sgi + 1].wg_begin : args.nwg;
        const int tiles = uniform((end - sg.wg_begin) / sg.group);  // of each problem
        member = uniform(local / tiles);
        local = uniform(local % tiles);
    }
    const bool nyq = local >= sg.wg_main;
    return MixJob{&args.p[sg.first + member], nyq ? local - sg.wg_main : local, nyq};
}

// First tile (x rows: run of tiles) of an x or y workgroup: one contiguous eighth of the launch for each
// XCD, or the chunked order.
__device__ __forceinline__ int mix_tile(const LaunchArgs &args) {
    const int b = static_cast<int>(blockIdx.x);
    return args.xcd_remap ? (b & 7) * (static_cast<int>(gridDim.x) >> 3) + (b >> 3) : tile_walk<true>().tile();
}

// A lane's line: position p at base + p*step + lane bytes, base and step the same for the
// whole workgroup; the lane's own share (its line and its thread's first position t) in 32 bits.
template <typename T>
struct MixLine {
    char *base;
    size_t step;     // bytes between positions
    uint32_t lane;   // bytes: line within the workgroup's base, and position t
    bool active;
    __device__ __forceinline__ cx<T> &at(int p) const {
        return *reinterpret_cast<cx<T> *>(base + static_cast<size_t>(p) * step + lane);
    }
};

// z lines.  Rows ky and 2ny - ky read the same spectrum values, so the lines are numbered row 0,
// then pair by pair of such rows (within a pair by runs of TILE adjacent kx of the one, then of the
// other), then row ny: tiles that share spectrum values are neighbours, and the octant rows of a
// tile's lines follow one another.
// Spectrum values: for one parity of kz, unit `u` bytes apart; addresses are a base that is the same
// for the whole workgroup plus 32 bits per lane, at its first position t (up) and at NB - t (dn).
template <typename T>
struct MixZ {
    MixLine<T> ln;
    uint64_t g;
    size_t u, odd;  // bytes between kz of one parity; the first odd kz
    uint32_t up, dn;
};

struct MixRowKx {
    int ky, kx;
};
template <int TILE>
__device__ __forceinline__ MixRowKx mix_z_row(int g, int nx, int ny) {
    const int gg = g - nx, pr = gg / (2 * nx), l = gg - pr * 2 * nx;
    const int j = l / (2 * TILE), rem = l - j * 2 * TILE, w = min(TILE, nx - j * TILE);
    const bool second = rem >= w;
    if (g < nx) return MixRowKx{0, g};
    if (g >= (2 * ny - 1) * nx) return MixRowKx{ny, g - (2 * ny - 1) * nx};
    return MixRowKx{second ? 2 * ny - 1 - pr : 1 + pr, j * TILE + rem - (second ? w : 0)};
}

// Slab of a tile that starts at line g0, with `lines` lines per kx (a whole number of tiles fills each
// slab but the last, so that no tile has lines of two).
template <typename P>
__device__ __forceinline__ Slab mix_slab(P &pl, int g0, int lines) {
    return w_slab(pl.ks < 30 ? uniform(g0 / (lines << pl.ks)) : 0, pl.ks, pl.nx, pl.ny, pl.nz);
}

template <typename T, int N, int TILE, int GL>
__device__ __forceinline__ MixZ<T> mix_z_line(const LaunchArgs &args, int bid, int c, int t) {
    using cplan = const __attribute__((address_space(4))) DevPlan;
    constexpr size_t CSZ = sizeof(cx<T>);
    constexpr int NB = MixLen<T, N>::NB;
    const MixJob job = mix_job<true>(args, bid);
    const auto &pl = *(cplan *)job.pa->plan;
    const int nx = pl.nx, ny = pl.ny;
    const int g0 = job.local * TILE, g = g0 + c;
    MixZ<T> z;
    size_t base = 0, line;  // values of the octant: before the tile's first row, and the lane's own
    if (!job.nyq) {
        z.ln.active = g < 2 * ny * nx;
        const Slab sl = mix_slab(pl, g0, 2 * ny);
        const int l0 = g0 - sl.kx0 * 2 * ny, l = z.ln.active ? l0 + c : l0;
        const MixRowKx f = mix_z_row<TILE>(l0, sl.w, ny);
        MixRowKx q = mix_z_row<TILE>(l, sl.w, ny);
        const int zb = pl.zb, sh = __builtin_ctz(static_cast<unsigned>(zb));
        const size_t plane = static_cast<size_t>(2) * ny * sl.w;
        z.ln.base = static_cast<char *>(job.pa->W) + sl.start * CSZ;
        z.ln.step = plane * CSZ;  // zb divides NB and n0: whole tiles from one first-stage register to the next
        z.ln.lane = static_cast<uint32_t>(
            ((static_cast<size_t>(t >> sh) << sh) * plane + (static_cast<size_t>(q.ky) * zb + (t & (zb - 1))) * sl.w + q.kx) * CSZ);
        q.kx += sl.kx0;
        const int k0 = uniform(f.ky <= ny ? f.ky : 2 * ny - f.ky), kyo = q.ky <= ny ? q.ky : 2 * ny - q.ky;
        if constexpr (GL == 2) {
            const int row = (nx + kGroup - 1) / kGroup * kGroup * (N + 1);
            base = static_cast<size_t>(k0) * row;
            line = static_cast<uint32_t>((kyo - k0) * row + q.kx / kGroup * (kGroup * (N + 1)) + q.kx % kGroup);
            z.u = kGroup * sizeof(T);
            z.odd = (N / 2 + 1) * z.u;
        } else {
            base = static_cast<size_t>(k0) * nx;
            line = static_cast<uint32_t>((kyo - k0) * nx + q.kx);
            z.odd = static_cast<size_t>(ny + 1) * nx * sizeof(T);
            z.u = 2 * z.odd;
        }
    } else {
        z.ln.active = g < 2 * ny;
        const int ky = z.ln.active ? g : g0;
        z.ln.base = static_cast<char *>(job.pa->Wn);
        z.ln.step = static_cast<size_t>(2) * ny * CSZ;
        z.ln.lane = static_cast<uint32_t>((static_cast<size_t>(t) * 2 * ny + ky) * CSZ);
        line = static_cast<uint32_t>((ky <= ny ? ky : 2 * ny - ky) * (GL == 2 ? N + 1 : 1));
        z.u = (GL == 2 ? 1 : 2 * (ny + 1)) * sizeof(T);
        z.odd = (GL == 2 ? N / 2 + 1 : ny + 1) * sizeof(T);
    }
    z.g = uniform(reinterpret_cast<uint64_t>(job.nyq ? pl.Gn : pl.G) + base * sizeof(T));
    z.u = uniform(static_cast<uint64_t>(z.u));
    z.odd = uniform(static_cast<uint64_t>(z.odd));
    z.up = static_cast<uint32_t>(line * sizeof(T) + t * z.u);
    z.dn = static_cast<uint32_t>(line * sizeof(T) + (NB - t) * z.u);
    return z;
}

// Load at a workgroup-uniform address plus 32 bits per lane.  The empty asm keeps the uniform part
// whole in scalar registers: where it is a constant distance from another one, the compiler would
// otherwise form 64-bit vector addresses (two registers and an add per load).
template <typename T>
__device__ __forceinline__ T load_from(uint64_t base, uint32_t lane) {
    asm("" : "+s"(base));
    return *reinterpret_cast<const gbl<T> *>(reinterpret_cast<const gbl<char> *>(base) + lane);
}

// Spectrum values of transform s at the last stage's positions p = b + r*nL: kz = 2p + s, even about n.
template <typename T, int N, int SH>
__device__ __forceinline__ void mix_load_g(const MixZ<T> &z, T *gv, int t) {
    using G = MixLen<T, N>;
    using F = MixFFT<T, G, 1, 0>;
    F::template each<G::RL>(t, [&](auto ic, int) {
        constexpr int i = decltype(ic)::value;
        sfor<0, G::RL>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            constexpr int p0 = G::NB * i + r * G::nL;                                   // position for t = 0
            constexpr int p1 = p0 + (G::NB < G::nL - G::NB * i ? G::NB : G::nL - G::NB * i) - 1;  // and the last t
            const uint64_t a = z.g + (SH ? z.odd : 0);
            // (at kz = n both sides name the same value)
            const uint64_t up = a + p0 * z.u;
            const uint64_t dn = a + static_cast<uint64_t>(static_cast<int64_t>(N - p0 - SH - G::NB)) * z.u;
            T &o = gv[i * G::RL + r];
            if constexpr (2 * p1 + SH <= N) o = load_from<T>(up, z.up);
            else if constexpr (2 * p0 + SH >= N) o = load_from<T>(dn, z.dn);
            else o = *reinterpret_cast<const gbl<T> *>(2 * (p0 + t) + SH <= N ? up + z.up : dn + z.dn);
        });
    });
}

// Column passes.  MODE Z_CONV: PERSIST lets one workgroup per CU walk its tiles (lines too long
// for two): the next tile's line is loaded into the registers of this one's as soon as its second
// transform has read them, ahead of the stores (loads and stores retire in order, so no wait for
// the line covers them; lanes without a line store past the buffer's range).
template <typename T, int N, int MODE, int GL, bool PERSIST>
__global__ void __launch_bounds__((MixTile<T, N, MODE == Z_CONV>::BLOCK), (MixTile<T, N, MODE == Z_CONV>::WPS))
mix_col_kernel(const LaunchArgs args) {
    using G = MixLen<T, N>;
    constexpr int TILE = MixTile<T, N, MODE == Z_CONV>::TILE, NB = G::NB;
    using F = MixFFT<T, G, TILE, 0>;
    extern __shared__ __align__(16) unsigned char smem[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem);
    TileWalk walk = tile_walk<true>();
    int bid = MODE == Z_CONV ? walk.tile() : mix_tile(args);
    if (bid >= args.nwg) return;
    const int tid = static_cast<int>(threadIdx.x);
    int c = tid % TILE, t = tid / TILE;  // adjacent lanes on adjacent lines
    const AxisPlan &ax = args.p[0].plan->ax[MODE == Z_CONV ? 2 : 1];
    cx<T> *twl = lds + N * TILE;
    // (y passes with a CU to themselves: measured, 7 % of the inverse pass of 1152 points for the plain copy)
    constexpr bool EARLY = MODE == Z_CONV || 2 * MixTile<T, N, false>::LDS <= 160 * 1024;
    MixTable<T, 2 * G::NTW, MixTile<T, N, MODE == Z_CONV>::BLOCK> table;
    if constexpr (EARLY) table.load(ax.mtw, tid);
    else copy_to_lds<T>(twl, ax.mtw, 2 * G::NTW);
    const cx<T> *tw0 = twl, *tw1 = twl + G::NTW;

    if constexpr (MODE == Z_CONV) {
        cx<T> x[G::V0], v[G::V], e[G::V0];
        T gv[G::VL];
        auto load = [&](const MixZ<T> &z) __attribute__((always_inline)) {
            F::template each<G::R0>(t, [&](auto ic, int) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::R0>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    x[i * G::R0 + r] = z.ln.at(i * NB + r * G::n0);
                });
            });
        };
        auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < G::VL; ++m) v[m] = scale(v[m], gv[m]);
        };
        auto cur = mix_z_line<T, N, TILE, GL>(args, bid, c, t);
        load(cur);
        mix_load_g<T, N, 0>(cur, gv, t);
        table.store(twl, tid);
        if constexpr (PERSIST) __builtin_amdgcn_s_waitcnt(0x0f70);  // nothing outstanding on entry (vmcnt 0)
        __syncthreads();  // twiddles visible
        for (;;) {
            if constexpr (PERSIST) asm volatile("" : "+v"(t), "+v"(c));  // addresses are derived again per tile
            F::template fwd<0>(x, v, lds + c, tw0, t);
            multiply();
            mix_load_g<T, N, 1>(cur, gv, t);
            F::template inv<0, false>(v, e, lds + c, tw0, t);
            F::template fwd<1>(x, v, lds + c, tw1, t);
            multiply();
            auto nxt = cur;
            bool more = false;
            if constexpr (PERSIST) {
                walk.i += walk.step;
                const int nb = walk.tile();
                more = nb < args.nwg;
                bid = more ? nb : bid;
                nxt = mix_z_line<T, N, TILE, GL>(args, bid, c, t);
                load(nxt);
                mix_load_g<T, N, 0>(nxt, gv, t);
            }
            F::template inv<1, true>(v, e, lds + c, tw1, t);
            if constexpr (PERSIST) {
                const uint32_t bytes = static_cast<uint32_t>(NB * cur.ln.step);
                F::template each<G::R0>(t, [&](auto ic, int) {
                    constexpr int i = decltype(ic)::value;
                    sfor<0, G::R0>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        buffer_store<T>(e[i * G::R0 + r], cur.ln.base + static_cast<size_t>(i * NB + r * G::n0) * cur.ln.step,
                                        bytes, cur.ln.active ? cur.ln.lane : 0xfffffff0u);
                    });
                });
                if (!more) break;
                cur = nxt;
            } else {
                if (cur.ln.active)
                    F::template each<G::R0>(t, [&](auto ic, int) {
                        constexpr int i = decltype(ic)::value;
                        sfor<0, G::R0>([&](auto rc) {
                            constexpr int r = decltype(rc)::value;
                            cur.ln.at(i * NB + r * G::n0) = e[i * G::R0 + r];
                        });
                    });
                break;
            }
        }
    } else {
        // y lines: line (z, kx) has position y at w_row(z, y) + kx; the Nyquist line of plane z is
        // contiguous in Wn.  Two lanes' worth of addresses: positions t + ... and 2t + ... (the
        // doubled side of the transform)
        using cplan = const __attribute__((address_space(4))) DevPlan;
        constexpr size_t CSZ = sizeof(cx<T>);
        const MixJob job = mix_job<false>(args, bid);
        const auto &pl = *(cplan *)job.pa->plan;
        const int nx = pl.nx, ny = pl.ny, nz = pl.nz, zb = pl.zb;
        const int g0 = job.local * TILE, g = g0 + c;
        MixLine<T> one, two;
        uint32_t lane;
        if (!job.nyq) {
            one.active = g < nz * nx;
            const Slab sl = mix_slab(pl, g0, nz);
            const int l0 = g0 - sl.kx0 * nz, l = one.active ? l0 + c : l0;
            const int z0 = uniform(l0 / sl.w), z = l / sl.w, kx = l - z * sl.w;
            const size_t row0 = w_row(z0, 0, ny, sl.w, zb);
            one.base = static_cast<char *>(job.pa->W) + (sl.start + row0) * CSZ;
            one.step = static_cast<size_t>(zb) * sl.w * CSZ;
            lane = static_cast<uint32_t>((w_row(z, 0, ny, sl.w, zb) - row0 + kx) * CSZ);
        } else {
            one.active = g < nz;
            one.base = static_cast<char *>(job.pa->Wn);
            one.step = CSZ;
            lane = static_cast<uint32_t>(static_cast<size_t>(one.active ? g : g0) * 2 * ny * CSZ);
        }
        two = one;
        one.lane = lane + static_cast<uint32_t>(t * one.step);
        two.lane = lane + static_cast<uint32_t>(2 * t * one.step);
        cx<T> x[G::V0], v[G::V];
        auto load2 = [&](cx<T> *q, auto sc) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
            F::template each<G::RL>(t, [&](auto ic, int) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::RL>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    q[i * G::RL + r] = two.at(2 * (i * NB + r * G::nL) + s);
                });
            });
        };
        auto store2 = [&](auto sc) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
            if (one.active)
                F::template each<G::RL>(t, [&](auto ic, int) {
                    constexpr int i = decltype(ic)::value;
                    sfor<0, G::RL>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        two.at(2 * (i * NB + r * G::nL) + s) = v[i * G::RL + r];
                    });
                });
        };
        constexpr std::integral_constant<int, 0> even{};
        constexpr std::integral_constant<int, 1> odd{};
        if constexpr (MODE == Y_FWD) {
            F::template each<G::R0>(t, [&](auto ic, int) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::R0>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    x[i * G::R0 + r] = one.at(i * NB + r * G::n0);
                });
            });
            if constexpr (EARLY) table.store(twl, tid);
            __syncthreads();  // twiddles visible
            F::template fwd<0>(x, v, lds + c, tw0, t);
            store2(even);  // every row of the line is in registers since the transform's first barrier
            __syncthreads();
            F::template fwd<1>(x, v, lds + c, tw1, t);
            store2(odd);
        } else {
            cx<T> w[G::V];
            load2(v, even);
            load2(w, odd);
            if constexpr (EARLY) table.store(twl, tid);
            __syncthreads();
            F::template inv<0, false>(v, x, lds + c, tw0, t);
            __syncthreads();
            F::template inv<1, true>(w, x, lds + c, tw1, t);
            if (one.active)
                F::template each<G::R0>(t, [&](auto ic, int) {
                    constexpr int i = decltype(ic)::value;
                    sfor<0, G::R0>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        one.at(i * NB + r * G::n0) = x[i * G::R0 + r];
                    });
                });
        }
    }
}

// Packed value j of a source row s of N reals (zero padding past the row): P0 <= j < P0 + COUNT.
// Odd rows are read as single reals, the last one without a partner.
template <typename T, int N, int P0, int COUNT>
__device__ __forceinline__ cx<T> mix_source(const T *s, int j) {
    constexpr int J = (N + 1) / 2;
    cx<T> u = {T(0), T(0)};
    if constexpr (P0 < J) {
        if (P0 + COUNT <= J || j < J) {
            if constexpr (N % 2 == 0) {
                u = reinterpret_cast<const cx<T> *>(s)[j];
            } else {
                u.x = s[2 * j];
                if (2 * j + 1 < N) u.y = s[2 * j + 1];
            }
        }
    }
    return u;
}
// The same for the potential row f.
template <typename T, int N, int P0, int COUNT>
__device__ __forceinline__ void mix_potential(T *f, int j, cx<T> u) {
    constexpr int J = (N + 1) / 2;
    if constexpr (P0 < J) {
        if (P0 + COUNT <= J || j < J) {
            if constexpr (N % 2 == 0) {
                reinterpret_cast<cx<T> *>(f)[j] = u;
            } else {
                f[2 * j] = u.x;
                if (2 * j + 1 < N) f[2 * j + 1] = u.y;
            }
        }
    }
}
// Split step of the packed real transform, X[k] from u = U[k], w = U[n-k] and e = exp(-i pi k/n):
// (u + w*)/2 - (i/2) e (u - w*); and the inverse one, U[k] from a = X[k], m = X[n-k]:
// (a + m*) + i conj(e) (a - m*).
template <typename T>
__device__ __forceinline__ cx<T> mix_split(cx<T> u, cx<T> w, cx<T> e) {
    const cx<T> a = {static_cast<T>(0.5) * (u.x + w.x), static_cast<T>(0.5) * (u.y - w.y)};
    const cx<T> d = {static_cast<T>(0.5) * (u.x - w.x), static_cast<T>(0.5) * (u.y + w.y)};
    const cx<T> ed = cmul(e, d);
    return cx<T>{a.x + ed.y, a.y - ed.x};
}
template <typename T>
__device__ __forceinline__ cx<T> mix_unsplit(cx<T> a, cx<T> m, cx<T> e) {
    const cx<T> sm = {a.x + m.x, a.y - m.y}, df = {a.x - m.x, a.y + m.y};
    const cx<T> ed = cmulc(df, e);
    return cx<T>{sm.x - ed.y, sm.y + ed.x};
}

// Workspace row (z, y): at<r>(b) is its value k = b + r*nL.  In slabs, rows are kSlab values (fewer in
// the last one) and k moves on to the next slab after each; where kSlab divides nL that takes one
// address per butterfly.
template <typename T, int N, bool SLABS>
struct MixRowAt {
    static constexpr int nL = MixLen<T, N>::nL;
    static constexpr int whole = N / kSlab * kSlab, rest = N - whole;  // kx in slabs of full width
    cx<T> *p, *last;
    size_t size;
    __device__ __forceinline__ MixRowAt(cx<T> *W, const DevPlan &pl, int z, int y) {
        if constexpr (SLABS) {
            const size_t zrow = w_row(z, y, pl.ny, 1, pl.zb);
            size = static_cast<size_t>(2) * pl.ny * pl.nz;
            p = W + zrow * kSlab;
            last = W + whole * size + zrow * rest;
        } else {
            p = W + w_row(z, y, pl.ny, N, pl.zb);
        }
    }
    template <int r>
    __device__ __forceinline__ cx<T> &at(int b) const {
        const int k = b + r * nL;
        if constexpr (!SLABS) {
            return p[k];
        } else if constexpr (rest == 0 && nL % kSlab == 0) {
            return *(p + b / kSlab * kSlab * size + b % kSlab + r * nL * size);
        } else {
            cx<T> *q = p + k / kSlab * kSlab * size + k % kSlab;
            return rest > 0 && k >= whole ? last[k - whole] : *q;
        }
    }
};

// Row passes: rows r = z*ny + y of S / Phi, packed u[j] = s[2j] + i s[2j+1] (zero for 2j >= nx),
// a transform of N = nx points and the split step with exp(-i pi k / n), as in the other row
// kernels.  Consecutive lanes walk along a row.  SLABS: the workspace is in slabs of kx.
// publish(): the tables' writes to LDS, after the loads of the rows.
template <typename T, int N, int MODE, bool SLABS, typename Publish>
__device__ __forceinline__ void mix_row_body(const MixJob &job, cx<T> *lds, int tid, Publish &&publish) {
    using G = MixLen<T, N>;
    using C = MixRow<T, N>;
    constexpr int NB = G::NB, ROWS = C::ROWS, S = C::S;
    using F = MixFFT<T, G, 1, C::PAD>;
    const int c = tid / NB, t = tid % NB;
    const cx<T> *twl = lds + ROWS * S, *post = twl + G::NTW;
    const DevPlan &pl = *job.pa->plan;
    const int ny = pl.ny, nz = pl.nz;
    const int g = job.local * ROWS + c;
    const bool active = g < ny * nz;
    const int z = active ? g / ny : 0, y = active ? g - z * ny : 0;
    const MixRowAt<T, N, SLABS> w(static_cast<cx<T> *>(job.pa->W), pl, z, y);
    cx<T> *wnyq = static_cast<cx<T> *>(job.pa->Wn) + static_cast<size_t>(z) * 2 * ny + y;
    cx<T> *row = lds + c * S;
    const size_t f0 = static_cast<size_t>(active ? g : 0) * N;
    // LDS slot of position P (MixFFT's layout)
    auto slot = [](int P) { return C::PAD ? P + P / G::R0 : P; };
    cx<T> x[G::V0], v[G::V];
    if constexpr (MODE == X_FWD) {
        const T *s = static_cast<const T *>(job.pa->S) + f0;
        F::template each<G::R0>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::R0>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                x[i * G::R0 + r] = mix_source<T, N, r * G::n0, G::n0>(s, b + r * G::n0);
            });
        });
        publish();
        __syncthreads();  // tables visible
        F::template fwd<0>(x, v, row, twl, t);
        // split: X[k] = (U[k] + U*[n-k])/2 - (i/2) exp(-i pi k/n) (U[k] - U*[n-k])
        F::template each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> *p = row + F::in(b);
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                p[r * F::template in_step<G::RL>()] = v[i * G::RL + r];
            });
        });
        __syncthreads();
        if (active)
            F::template each<G::RL>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::RL>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    const int k = b + r * G::nL;
                    const cx<T> u = v[i * G::RL + r], m = row[slot(k == 0 ? 0 : N - k)];
                    w.template at<r>(b) = mix_split(u, m, post[k]);
                    if (k == 0) *wnyq = cx<T>{u.x - u.y, T(0)};
                });
            });
    } else {
        cx<T> xn = {T(0), T(0)};
        F::template each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::RL>([&](auto rc) { constexpr int r = decltype(rc)::value; v[i * G::RL + r] = w.template at<r>(b); });
        });
        if (t == 0) xn = *wnyq;
        publish();
        F::template each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> *p = row + F::in(b);
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                p[r * F::template in_step<G::RL>()] = v[i * G::RL + r];
            });
        });
        __syncthreads();  // row values and tables visible
        // U[k] = (X[k] + X*[n-k]) + i exp(+i pi k/n) (X[k] - X*[n-k]), k < n; X[n] for k = 0
        F::template each<G::RL>(t, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                const int k = b + r * G::nL;
                cx<T> m = row[slot(k == 0 ? 0 : N - k)];
                if (k == 0) m = xn;  // (a choice of values: one of addresses would put xn in memory)
                v[i * G::RL + r] = mix_unsplit(v[i * G::RL + r], m, post[k]);
            });
        });
        __syncthreads();  // partners read
        F::template inv<0, false>(v, x, row, twl, t);
        if (active) {
            T *f = static_cast<T *>(job.pa->Phi) + f0;
            F::template each<G::R0>(t, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::R0>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    mix_potential<T, N, r * G::n0, G::n0>(f, b + r * G::n0, x[i * G::R0 + r]);
                });
            });
        }
    }
}

// MANY: args.rounds row tiles per workgroup, and plans with slabs (a kernel of its own: the loop and
// the second layout cost registers, 10 to 16 % of the inverse passes of 144 points).
template <typename T, int N, int MODE, bool MANY>
__global__ void __launch_bounds__((MixRow<T, N>::BLOCK)) mix_row_kernel(const LaunchArgs args) {
    using C = MixRow<T, N>;
    extern __shared__ __align__(16) unsigned char smem[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem);
    const int rounds = MANY ? args.rounds : 1, first = mix_tile(args) * rounds;
    if (first >= args.nwg) return;
    const AxisPlan &ax = args.p[0].plan->ax[0];
    cx<T> *twl = lds + C::ROWS * C::S, *post = twl + C::G::NTW;
    int tid = static_cast<int>(threadIdx.x);
    if constexpr (!MANY) {
        MixTable<T, C::G::NTW, C::BLOCK> tw;
        MixTable<T, N, C::BLOCK> split;
        tw.load(ax.mtw, tid);
        split.load(ax.post, tid);
        mix_row_body<T, N, MODE, false>(mix_job<false>(args, first), lds, tid, [&]() __attribute__((always_inline)) {
            tw.store(twl, tid);
            split.store(post, tid);
        });
    } else {
        copy_to_lds<T>(twl, ax.mtw, C::G::NTW);
        copy_to_lds<T>(post, ax.post, N);
        for (int i = 0; i < rounds && first + i < args.nwg; ++i) {
            asm volatile("" : "+v"(tid));  // addresses are derived again per tile
            if (MODE == X_INV && i > 0) __syncthreads();  // the rows before are read (X_FWD: its first barrier)
            const MixJob job = mix_job<false>(args, first + i);
            if (job.pa->plan->ks == kSlabShift) mix_row_body<T, N, MODE, true>(job, lds, tid, []() {});
            else mix_row_body<T, N, MODE, false>(job, lds, tid, []() {});
        }
    }
}

// z passes that run persistently: FP32 lines whose workgroup of 8 lines exceeds 512 threads, so that
// one fills a CU.  Measured, z pass of 576 x 576 lines of 1152 points: 7.2 ms with two one-tile
// workgroups of 4 lines per CU, 6.1 ms with 8 lines and one tile, 5.7 ms persistently.
template <typename T, int N>
constexpr bool mix_z_persist() { return sizeof(T) == 4 && MixTile<T, N, true>::BLOCK > 512; }

template <typename T, int N>
hipError_t launch_mix(int mode, const LaunchArgs &args, hipStream_t stream) {
    constexpr int kMaxDevices = 64;
    static int cus[kMaxDevices] = {0};
    constexpr bool PZ = mix_z_persist<T, N>();
    constexpr int GL = mix_spectrum(sizeof(T) == 4 ? 0 : 1, N);
    void (*const fn[7])(LaunchArgs) = {mix_row_kernel<T, N, X_FWD, false>,       mix_col_kernel<T, N, Y_FWD, GL, false>,
                                       mix_col_kernel<T, N, Z_CONV, GL, PZ>,     mix_col_kernel<T, N, Y_INV, GL, false>,
                                       mix_row_kernel<T, N, X_INV, false>,       mix_row_kernel<T, N, X_FWD, true>,
                                       mix_row_kernel<T, N, X_INV, true>};
    if (mode < 0 || mode > 4) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (cus[dev] == 0) {
        for (auto f : fn) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024);
            if (e != hipSuccess) return e;
        }
        int n = 0;
        e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        cus[dev] = n > 0 ? n : 1;
    }
    const bool row = mode == X_FWD || mode == X_INV;
    using CZ = MixTile<T, N, true>;
    using CY = MixTile<T, N, false>;
    const int block = row ? MixRow<T, N>::BLOCK : (mode == Z_CONV ? CZ::BLOCK : CY::BLOCK);
    const size_t lds = row ? MixRow<T, N>::LDS : (mode == Z_CONV ? CZ::LDS : CY::LDS);
    // whole rounds of the tile order, or one persistent workgroup per CU
    const int nwg = args.rounds > 0 ? (args.nwg + args.rounds - 1) / args.rounds : args.nwg;
    const int whole = args.xcd_remap ? 8 : 8 * kTileChunk;
    int grid = (nwg + whole - 1) / whole * whole;
    if (mode == Z_CONV && PZ && grid > cus[dev]) grid = cus[dev];
    const int many = args.rounds > 0 ? (mode == X_FWD ? 5 : 6) : mode;
    hipLaunchKernelGGL(fn[row ? many : mode], dim3(grid), dim3(block), lds, stream, args);
    return hipGetLastError();
}

}  // namespace pspfft

// One translation unit per precision and list of lengths keeps compiles parallel.
#define PSPFFT_MIX_LAUNCH(N, A, B, C, D, E) case N: return launch_mix<MixReal, N>(mode, args, stream);
#define PSPFFT_MIX_UNIT(T, NAME, LIST)                                                   \
    namespace pspfft {                                                                   \
    hipError_t NAME(int n, int mode, const LaunchArgs &args, hipStream_t stream) {       \
        using MixReal = T;                                                               \
        switch (n) {                                                                     \
            LIST(PSPFFT_MIX_LAUNCH)                                                      \
            default: return hipErrorInvalidValue;                                        \
        }                                                                                \
    }                                                                                    \
    }
