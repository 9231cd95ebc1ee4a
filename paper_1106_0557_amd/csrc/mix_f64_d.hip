// Half-length line kernels, double: the lengths of PSPFFT_MIX_F64_D.
#include "mix_lines.h"

PSPFFT_MIX_UNIT(double, mix_f64_d, PSPFFT_MIX_F64_D)
