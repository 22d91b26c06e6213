// gfx950 wave-per-site hop kernels of libdwa, F32 storage.
#include "kwave.h"

DWA_INSTANTIATE_WAVE(F32)
DWA_INSTANTIATE_WAVE_LOW(F32)
DWA_INSTANTIATE_WAVE_FOLD(F32)
