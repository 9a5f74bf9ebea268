// The preconditioner's FP32 slice passes and fused steps (see fft_kernels.h).
#define HMC_FFT_SOURCE
#include "fft_kernels.h"

HMC_PC_KERNELS(, float, GeoOne)
HMC_PC_KERNELS(, float, GeoBatch)
HMC_PC_STEPS(, float)
