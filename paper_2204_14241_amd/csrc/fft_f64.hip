// The preconditioner's FP64 slice passes (see fft_kernels.h).
#define HMC_FFT_SOURCE
#include "fft_kernels.h"

HMC_PC_KERNELS(, double, GeoOne)
HMC_PC_KERNELS(, double, GeoBatch)
