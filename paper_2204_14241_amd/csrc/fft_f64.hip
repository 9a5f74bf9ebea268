// The preconditioner's FP64 slice passes and fused steps (see fft_kernels.h).
#define HMC_FFT_SOURCE
#include "fft_kernels.h"

HMC_PC_KERNELS(, double, GeoOne)
HMC_PC_KERNELS(, double, GeoBatch)
HMC_PC_STEPS(, double)
