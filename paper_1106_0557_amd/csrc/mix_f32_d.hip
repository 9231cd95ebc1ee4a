// Half-length line kernels, float: the lengths of PSPFFT_MIX_F32_D.
#include "mix_lines.h"

PSPFFT_MIX_UNIT(float, mix_f32_d, PSPFFT_MIX_F32_D)
