// The preconditioner's FP32 slice passes (see fft_kernels.h).
#define HMC_FFT_SOURCE
#include "fft_kernels.h"

HMC_PC_KERNELS(, float, GeoOne)
HMC_PC_KERNELS(, float, GeoBatch)
