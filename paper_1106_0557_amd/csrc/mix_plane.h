// mix_plane.h -- the x and y transforms of one z plane in one workgroup (as in
// plane_kernels.h: Sec. 2.1 and 2.2.2, without the round trip of the
// intermediate through HBM) for nx == ny = n = R0*R1(*R2), on the line
// transforms of mix_lines.h.
//
// Forward: the x step transforms the n rows of a source plane (packed real form
// and split step) into an LDS plane X[y][kx], the real values X[y][0] and
// X[y][n] sharing the slot of kx = 0 as X0 + i Xn; the y step transforms every
// column twice (s = 0: rows 2j of W, s = 1: rows 2j + 1) from a copy of it in
// registers, with the exchanges in the column's own n slots.  Column 0 carries
// C = A + i B, A and B the transforms of the real columns kx = 0 and kx = n:
// its results go through LDS and n threads separate them,
// A[k] = (C[k] + conj C[-k])/2, B[k] = (C[k] - conj C[-k])/(2i).
// Inverse: the same backwards (columns kx = 0 and kx = n travel together as
// Y0 + i Yn and come out as x0 + i xn).
//
// One plane per workgroup.  What bounds a small mesh is latency: few planes, a
// chain of dependent loads, LDS exchanges and arithmetic.  The threads per line
// are therefore as many as keep each at 4 to 10 values where the plane is small.
// Large batches of the longer ones are bounded by one plane per CU, whose stores
// wait for its transforms.  Measured: eight FP32 120^3, whole solves, 383 us in
// five passes and 326 us here (forward planes 3.0 TB/s, inverse 3.2); FP64 32^3,
// sequential solves, 22.2 us with the family planes and 15.3 us here.
#pragma once

#include "mix_lines.h"
#include "plane_kernels.h"

namespace pspfft {

// Lengths with a plane kernel, X(N, R0, R1, R2, NB): the plane of x spectra, the tables and a
// column fit the LDS, and n*NB threads a workgroup.
template <typename T, int N>
struct MixPlaneRadices;
#define PSPFFT_PLANE_F32(X)                                                                                   \
    X(16, 4, 4, 1, 4) X(18, 6, 3, 1, 3) X(20, 5, 4, 1, 4) X(24, 6, 4, 1, 4) X(25, 5, 5, 1, 5) X(27, 9, 3, 1, 3) \
    X(30, 6, 5, 1, 5) X(32, 8, 4, 1, 4) X(36, 6, 6, 1, 6) X(40, 8, 5, 1, 5) X(45, 9, 5, 1, 5) X(48, 8, 6, 1, 6) \
    X(50, 10, 5, 1, 5) X(54, 9, 6, 1, 6) X(60, 10, 6, 1, 6) X(64, 8, 8, 1, 8) X(75, 15, 5, 1, 5)              \
    X(81, 9, 9, 1, 9) X(90, 10, 9, 1, 9) X(100, 10, 10, 1, 10) X(108, 12, 9, 1, 9) X(120, 15, 8, 1, 8)
#define PSPFFT_PLANE_F64(X)                                                                                   \
    X(16, 4, 4, 1, 4) X(18, 6, 3, 1, 3) X(20, 5, 4, 1, 4) X(24, 6, 4, 1, 4) X(25, 5, 5, 1, 5) X(27, 9, 3, 1, 3) \
    X(30, 6, 5, 1, 5) X(32, 8, 4, 1, 4) X(36, 6, 6, 1, 6) X(40, 8, 5, 1, 5) X(45, 9, 5, 1, 5) X(48, 8, 6, 1, 6) \
    X(50, 10, 5, 1, 5) X(54, 9, 6, 1, 6) X(60, 10, 6, 1, 6) X(64, 8, 8, 1, 8) X(75, 15, 5, 1, 5)              \
    X(81, 9, 9, 1, 9)
#define PSPFFT_PLANE_RADICES(T, N, A, B, C, THREADS)              \
    template <>                                                   \
    struct MixPlaneRadices<T, N> {                                \
        using G = MixGeo<N, A, B, C, THREADS>;                    \
    };
#define PSPFFT_PLANE_RADICES_F32(N, A, B, C, D) PSPFFT_PLANE_RADICES(float, N, A, B, C, D)
#define PSPFFT_PLANE_RADICES_F64(N, A, B, C, D) PSPFFT_PLANE_RADICES(double, N, A, B, C, D)
PSPFFT_PLANE_F32(PSPFFT_PLANE_RADICES_F32)
PSPFFT_PLANE_F64(PSPFFT_PLANE_RADICES_F64)

template <typename T, int N>
struct MixPlane {
    using G = typename MixPlaneRadices<T, N>::G;
    static constexpr int CSZ = static_cast<int>(sizeof(cx<T>));
    static constexpr int PAD = G::R0 % 2 == 0 ? 1 : 0;
    static constexpr int S = (N / G::R0 * (G::R0 + PAD)) | 1;
    static constexpr int BLOCK = N * G::NB;
    // the plane, the stage twiddles of both transforms, the split factors, column 0
    static constexpr size_t LDS = static_cast<size_t>(N * S + 2 * G::NTW + N + N) * CSZ;
    static_assert(BLOCK <= 1024 && LDS <= 160 * 1024, "one workgroup fits");
};

template <typename T, int N, bool FWD, typename Args>
__global__ void __launch_bounds__((MixPlane<T, N>::BLOCK)) mix_plane_kernel(const Args args) {
    using C = MixPlane<T, N>;
    using G = typename C::G;
    constexpr int NB = G::NB, S = C::S;
    using Row = MixFFT<T, G, 1, C::PAD>;
    using Col = MixFFT<T, G, S, 0>;
    extern __shared__ __align__(16) unsigned char smem[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem);
    const int tid = static_cast<int>(threadIdx.x);
    const int xc = tid / NB, xt = tid % NB;  // x step: row, thread of the row
    const int yc = tid % N, yt = tid / N;    // y step: column, thread of the column
    const PlaneRef ref = plane_ref(args, static_cast<int>(blockIdx.x));
    cx<T> *W = static_cast<cx<T> *>(ref.pa->W) + static_cast<size_t>(ref.z) * 2 * N * N;
    cx<T> *Wn = static_cast<cx<T> *>(ref.pa->Wn) + static_cast<size_t>(ref.z) * 2 * N;
    const AxisPlan &ax = args.p[0].plan->ax[0];  // the tables depend on n only
    cx<T> *twl = lds + N * S, *post = twl + 2 * G::NTW, *c0 = post + N;
    MixTable<T, 2 * G::NTW, C::BLOCK> table;
    MixTable<T, N, C::BLOCK> split;
    table.load(ax.mtw, tid);
    split.load(ax.post, tid);
    const cx<T> *tw0 = twl, *tw1 = twl + G::NTW;
    auto slot = [](int P) { return C::PAD ? P + P / G::R0 : P; };
    cx<T> *row = lds + xc * S, *col = lds + slot(yc);
    cx<T> x[G::V0], v[G::V];

    if constexpr (FWD) {
        const T *s = static_cast<const T *>(ref.pa->S) + (static_cast<size_t>(ref.z) * N + xc) * N;
        Row::template each<G::R0>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::R0>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                x[i * G::R0 + r] = mix_source<T, N, r * G::n0, G::n0>(s, b + r * G::n0);
            });
        });
        table.store(twl, tid);
        split.store(post, tid);
        __syncthreads();  // tables visible
        Row::template fwd<0>(x, v, row, tw0, xt);
        // split: X[k] = (U[k] + U*[n-k])/2 - (i/2) exp(-i pi k/n) (U[k] - U*[n-k])
        Row::template each<G::RL>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> *p = row + Row::in(b);
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                p[r * Row::template in_step<G::RL>()] = v[i * G::RL + r];
            });
        });
        __syncthreads();
        Row::template each<G::RL>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                const int k = b + r * G::nL;
                const cx<T> u = v[i * G::RL + r], w = row[slot(k == 0 ? 0 : N - k)];
                cx<T> q = mix_split(u, w, post[k]);
                if (k == 0) q.y = u.x - u.y;  // X[0] is real: its imaginary slot takes X[n]
                v[i * G::RL + r] = q;
            });
        });
        __syncthreads();  // partners read
        Row::template each<G::RL>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            cx<T> *p = row + Row::in(b);
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                p[r * Row::template in_step<G::RL>()] = v[i * G::RL + r];
            });
        });
        __syncthreads();
        Col::template each<G::R0>(yt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::R0>([&](auto rc) { constexpr int r = decltype(rc)::value; x[i * G::R0 + r] = col[(b + r * G::n0) * S]; });
        });
        __syncthreads();  // the columns are in registers
        auto emit = [&](auto sc) __attribute__((always_inline)) {
            constexpr int sh = decltype(sc)::value;
            Col::template each<G::RL>(yt, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::RL>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    const int j = b + r * G::nL;
                    if (yc == 0) c0[j] = v[i * G::RL + r];
                    else W[static_cast<uint32_t>((2 * j + sh) * N + yc)] = v[i * G::RL + r];
                });
            });
            __syncthreads();
            if (tid < N) {
                const int j = tid, m = sh ? N - 1 - j : (j == 0 ? 0 : N - j);
                const cx<T> a = c0[j], p = c0[m];
                W[static_cast<uint32_t>((2 * j + sh) * N)] =
                    cx<T>{static_cast<T>(0.5) * (a.x + p.x), static_cast<T>(0.5) * (a.y - p.y)};
                Wn[2 * j + sh] = cx<T>{static_cast<T>(0.5) * (a.y + p.y), static_cast<T>(-0.5) * (a.x - p.x)};
            }
        };
        Col::template fwd<0>(x, v, col, tw0, yt);
        emit(std::integral_constant<int, 0>{});
        Col::template fwd<1>(x, v, col, tw1, yt);
        emit(std::integral_constant<int, 1>{});
    } else {
        cx<T> w[G::VL];
        auto load = [&](cx<T> *q, auto sc) __attribute__((always_inline)) {
            constexpr int sh = decltype(sc)::value;
            Col::template each<G::RL>(yt, [&](auto ic, int b) {
                constexpr int i = decltype(ic)::value;
                sfor<0, G::RL>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    q[i * G::RL + r] = W[static_cast<uint32_t>((2 * (b + r * G::nL) + sh) * N + yc)];
                });
            });
            if (yc == 0)
                Col::template each<G::RL>(yt, [&](auto ic, int b) {
                    constexpr int i = decltype(ic)::value;
                    sfor<0, G::RL>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        const cx<T> a = Wn[2 * (b + r * G::nL) + sh];
                        q[i * G::RL + r] = cx<T>{q[i * G::RL + r].x - a.y, q[i * G::RL + r].y + a.x};
                    });
                });
        };
        load(v, std::integral_constant<int, 0>{});
        load(w, std::integral_constant<int, 1>{});
        table.store(twl, tid);
        split.store(post, tid);
        __syncthreads();  // tables visible
        Col::template inv<0, false>(v, x, col, tw0, yt);
        __syncthreads();
        Col::template inv<1, true>(w, x, col, tw1, yt);
        __syncthreads();
        Col::template each<G::R0>(yt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::R0>([&](auto rc) { constexpr int r = decltype(rc)::value; col[(b + r * G::n0) * S] = x[i * G::R0 + r]; });
        });
        __syncthreads();
        // U[k] = (X[k] + X*[n-k]) + i exp(+i pi k/n) (X[k] - X*[n-k]), k < n
        const cx<T> p0 = row[0];  // X[y][0] + i X[y][n], both real
        Row::template each<G::RL>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::RL>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                const int k = b + r * G::nL;
                const cx<T> a = k == 0 ? cx<T>{p0.x, T(0)} : row[slot(k)];
                const cx<T> m = k == 0 ? cx<T>{p0.y, T(0)} : row[slot(N - k)];
                v[i * G::RL + r] = mix_unsplit(a, m, post[k]);
            });
        });
        __syncthreads();  // partners read
        Row::template inv<0, false>(v, x, row, tw0, xt);
        T *f = static_cast<T *>(ref.pa->Phi) + (static_cast<size_t>(ref.z) * N + xc) * N;
        Row::template each<G::R0>(xt, [&](auto ic, int b) {
            constexpr int i = decltype(ic)::value;
            sfor<0, G::R0>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                mix_potential<T, N, r * G::n0, G::n0>(f, b + r * G::n0, x[i * G::R0 + r]);
            });
        });
    }
}

template <typename T, int N>
hipError_t launch_mix_plane_n(bool fwd, const LaunchArgs &args, hipStream_t stream) {
    constexpr int kMaxDevices = 64;
    static bool ready[kMaxDevices] = {false};
    constexpr bool SOLO = N <= 64;  // up to there the host is slower than the card
    void (*const fn[2])(LaunchArgs) = {mix_plane_kernel<T, N, false, LaunchArgs>, mix_plane_kernel<T, N, true, LaunchArgs>};
    using Solo = std::conditional_t<SOLO, SoloArgs, LaunchArgs>;
    void (*const solo[2])(Solo) = {mix_plane_kernel<T, N, false, Solo>, mix_plane_kernel<T, N, true, Solo>};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!ready[dev]) {
        for (const void *f : {reinterpret_cast<const void *>(fn[0]), reinterpret_cast<const void *>(fn[1]),
                              reinterpret_cast<const void *>(solo[0]), reinterpret_cast<const void *>(solo[1])}) {
            e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        ready[dev] = true;
    }
    const dim3 grid(args.nwg), block(MixPlane<T, N>::BLOCK);
    if constexpr (SOLO) {
        if (args.count == 1) {
            const SoloArgs one = {args.nwg, {args.p[0]}};
            hipLaunchKernelGGL(solo[fwd ? 1 : 0], grid, block, (MixPlane<T, N>::LDS), stream, one);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(fn[fwd ? 1 : 0], grid, block, (MixPlane<T, N>::LDS), stream, args);
    return hipGetLastError();
}

}  // namespace pspfft

#define PSPFFT_PLANE_LAUNCH(N, A, B, C, D) case N: return launch_mix_plane_n<MixReal, N>(fwd, args, stream);
#define PSPFFT_PLANE_UNIT(T, NAME, LIST)                                                    \
    namespace pspfft {                                                                      \
    hipError_t NAME(int n, bool fwd, const LaunchArgs &args, hipStream_t stream) {          \
        using MixReal = T;                                                                  \
        switch (n) {                                                                        \
            LIST(PSPFFT_PLANE_LAUNCH)                                                       \
            default: return hipErrorInvalidValue;                                           \
        }                                                                                   \
    }                                                                                       \
    }
