// Lengths of the half-length line kernels and the dispatch to their translation units.
#include "mix_lines.h"

namespace pspfft {

bool mix_info(int n, MixInfo &info) {
    switch (n) {
#define PSPFFT_MIX_CASE(N, A, B, C)                                                                     \
    case N:                                                                                             \
        info = MixInfo{{A, B, C}, MixLen<N>::NB, {MixTile<float, N>::TILE, MixTile<double, N>::TILE}, \
                       MixRow<float, N>::ROWS};                                                         \
        return true;
        PSPFFT_MIX_ALL(PSPFFT_MIX_CASE)
#undef PSPFFT_MIX_CASE
        default: return false;
    }
}

#undef PSPFFT_MIX_UNIT
#define PSPFFT_MIX_UNIT(NAME) hipError_t NAME(int n, int mode, const LaunchArgs &args, hipStream_t stream);
PSPFFT_MIX_UNIT(mix_f32_a)
PSPFFT_MIX_UNIT(mix_f32_b)
PSPFFT_MIX_UNIT(mix_f32_c)
PSPFFT_MIX_UNIT(mix_f32_d)
PSPFFT_MIX_UNIT(mix_f32_e)
PSPFFT_MIX_UNIT(mix_f64_a)
PSPFFT_MIX_UNIT(mix_f64_b)
PSPFFT_MIX_UNIT(mix_f64_c)
PSPFFT_MIX_UNIT(mix_f64_d)
PSPFFT_MIX_UNIT(mix_f64_e)
#undef PSPFFT_MIX_UNIT

hipError_t launch_mix_lines(int mode, int prec, int n, const LaunchArgs &args, hipStream_t stream) {
    if (args.nwg <= 0) return hipSuccess;
    using Unit = hipError_t (*)(int, int, const LaunchArgs &, hipStream_t);
    static constexpr Unit units[2][5] = {{mix_f32_a, mix_f32_b, mix_f32_c, mix_f32_d, mix_f32_e},
                                         {mix_f64_a, mix_f64_b, mix_f64_c, mix_f64_d, mix_f64_e}};
    switch (n) {
#define PSPFFT_MIX_CASE_0(N, A, B, C) case N: return units[prec][0](n, mode, args, stream);
#define PSPFFT_MIX_CASE_1(N, A, B, C) case N: return units[prec][1](n, mode, args, stream);
#define PSPFFT_MIX_CASE_2(N, A, B, C) case N: return units[prec][2](n, mode, args, stream);
#define PSPFFT_MIX_CASE_3(N, A, B, C) case N: return units[prec][3](n, mode, args, stream);
#define PSPFFT_MIX_CASE_4(N, A, B, C) case N: return units[prec][4](n, mode, args, stream);
        PSPFFT_MIX_A(PSPFFT_MIX_CASE_0)
        PSPFFT_MIX_B(PSPFFT_MIX_CASE_1)
        PSPFFT_MIX_C(PSPFFT_MIX_CASE_2)
        PSPFFT_MIX_D(PSPFFT_MIX_CASE_3)
        PSPFFT_MIX_E(PSPFFT_MIX_CASE_4)
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pspfft
