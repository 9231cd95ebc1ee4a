// Half-length line kernels, double: the lengths of PSPFFT_MIX_F64_C.
#include "mix_lines.h"

PSPFFT_MIX_UNIT(double, mix_f64_c, PSPFFT_MIX_F64_C)
