// gfx950 wave-per-site hop kernels of libdwa, BF16 storage.
#include "kwave.h"

DWA_INSTANTIATE_WAVE(BF16)
DWA_INSTANTIATE_WAVE_LOW(BF16)
