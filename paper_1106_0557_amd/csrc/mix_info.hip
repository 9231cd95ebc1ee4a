// Lengths of the half-length line kernels and the dispatch to their translation units.
#include "mix_plane.h"

namespace pspfft {

namespace {
template <typename T, int N>
MixInfo info_of() {
    using G = MixLen<T, N>;
    return MixInfo{{G::R0, G::R1, G::R2}, G::NB, MixTile<T, N, true>::TILE, MixTile<T, N, false>::TILE,
                   MixRow<T, N>::ROWS};
}
}  // namespace

bool mix_info(int prec, int n, MixInfo &info) {
    switch (n + (prec << 16)) {
#define PSPFFT_MIX_CASE_F32(N, A, B, C, D, E) case N: info = info_of<float, N>(); return true;
#define PSPFFT_MIX_CASE_F64(N, A, B, C, D, E) case N + (1 << 16): info = info_of<double, N>(); return true;
        PSPFFT_MIX_ALL(PSPFFT_MIX_CASE_F32, PSPFFT_MIX_F32)
        PSPFFT_MIX_ALL(PSPFFT_MIX_CASE_F64, PSPFFT_MIX_F64)
        default: return false;
    }
}

bool mix_plane_info(int prec, int n, MixInfo &info) {
    switch (n + (prec << 16)) {
#define PSPFFT_PLANE_CASE_F32(N, A, B, C, D) case N: info = MixInfo{{A, B, C}, D, 0, 0, N}; return true;
#define PSPFFT_PLANE_CASE_F64(N, A, B, C, D) case N + (1 << 16): info = MixInfo{{A, B, C}, D, 0, 0, N}; return true;
        PSPFFT_PLANE_F32(PSPFFT_PLANE_CASE_F32)
        PSPFFT_PLANE_F64(PSPFFT_PLANE_CASE_F64)
        default: return false;
    }
}

hipError_t mix_plane_f32(int n, bool fwd, const LaunchArgs &args, hipStream_t stream);
hipError_t mix_plane_f64(int n, bool fwd, const LaunchArgs &args, hipStream_t stream);

hipError_t launch_mix_plane(bool fwd, int prec, int n, const LaunchArgs &args, hipStream_t stream) {
    if (args.nwg <= 0) return hipSuccess;
    return prec == 0 ? mix_plane_f32(n, fwd, args, stream) : mix_plane_f64(n, fwd, args, stream);
}

using MixUnit = hipError_t(int n, int mode, const LaunchArgs &args, hipStream_t stream);
MixUnit mix_f32_a, mix_f32_b, mix_f32_c, mix_f32_d, mix_f32_e;
MixUnit mix_f64_a, mix_f64_b, mix_f64_c, mix_f64_d, mix_f64_e;

hipError_t launch_mix_lines(int mode, int prec, int n, const LaunchArgs &args, hipStream_t stream) {
    if (args.nwg <= 0) return hipSuccess;
    MixInfo info;
    if (prec < 0 || prec > 1 || !mix_info(prec, n, info)) return hipErrorInvalidValue;
    // the lists hold ascending lengths
    static constexpr MixUnit *units[2][5] = {{mix_f32_a, mix_f32_b, mix_f32_c, mix_f32_d, mix_f32_e},
                                             {mix_f64_a, mix_f64_b, mix_f64_c, mix_f64_d, mix_f64_e}};
    const int list = n <= 144 ? 0 : n <= 256 ? 1 : n <= 486 ? 2 : n <= 750 ? 3 : 4;
    return units[prec][list](n, mode, args, stream);
}

}  // namespace pspfft
