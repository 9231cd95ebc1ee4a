// Plane kernels on half-length lines, double.
#include "mix_plane.h"

PSPFFT_PLANE_UNIT(double, mix_plane_f64, PSPFFT_PLANE_F64)
