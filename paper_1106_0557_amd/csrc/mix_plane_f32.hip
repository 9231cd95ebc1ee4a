// Plane kernels on half-length lines, float.
#include "mix_plane.h"

PSPFFT_PLANE_UNIT(float, mix_plane_f32, PSPFFT_PLANE_F32)
