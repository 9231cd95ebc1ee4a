// Half-length line kernels, float: the lengths of PSPFFT_MIX_F32_A.
#include "mix_lines.h"

PSPFFT_MIX_UNIT(float, mix_f32_a, PSPFFT_MIX_F32_A)
