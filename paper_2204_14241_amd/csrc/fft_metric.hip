// The metric's passes (see fft_kernels.h).
#define HMC_FFT_SOURCE
#include "fft_kernels.h"

HMC_MT_KERNELS(, hmc::kFftNarrow)
HMC_MT_KERNELS(, hmc::kFftMaxRadix)
