// gfx950 wave-per-site hop kernels of libdwa, F64 storage.
#include "kwave.h"

DWA_INSTANTIATE_WAVE(F64)
