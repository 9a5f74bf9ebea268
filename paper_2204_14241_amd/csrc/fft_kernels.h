// Where the kernels with an FFT are compiled.  Each holds a register-resident butterfly per radix,
// so they take most of the library's compile time; they are instantiated in sources of their own
// (fft_f32.hip, fft_f64.hip, fft_metric.hip), which the build compiles side by side, and declared
// here for the host code that launches them.
#pragma once

#include "metric.h"
#include "pcstep.h"
#include "precond.h"

#define HMC_PC_KERNELS(PRE, R, GEO)                                                                             \
    PRE template __global__ void hmc::k_pc_xy<R, false, hmc::GEO, hmc::kFftNarrow>(                             \
        hmc::CgCtl, hmc::GEO, const hmc::C2<R>*, hmc::C2<R>*, const double*);                                   \
    PRE template __global__ void hmc::k_pc_xy<R, true, hmc::GEO, hmc::kFftNarrow>(                              \
        hmc::CgCtl, hmc::GEO, const hmc::C2<R>*, hmc::C2<R>*, const double*);                                   \
    PRE template __global__ void hmc::k_pc_xy<R, false, hmc::GEO, hmc::kFftMaxRadix>(                           \
        hmc::CgCtl, hmc::GEO, const hmc::C2<R>*, hmc::C2<R>*, const double*);                                   \
    PRE template __global__ void hmc::k_pc_xy<R, true, hmc::GEO, hmc::kFftMaxRadix>(                            \
        hmc::CgCtl, hmc::GEO, const hmc::C2<R>*, hmc::C2<R>*, const double*);

#define HMC_PC_STEPS_R(PRE, R, NN2, MAXR)                                                                       \
    PRE template __global__ void hmc::k_pc_a<R, NN2, hmc::MAXR>(hmc::CgCtl, hmc::GeoOne, hmc::CgVecs<R>,        \
                                                                const R*, hmc::Coef<R>, const double*);         \
    PRE template __global__ void hmc::k_pc_b<R, NN2, hmc::MAXR>(hmc::CgCtl, hmc::GeoOne, hmc::CgVecs<R>,        \
                                                                const R*, hmc::Coef<R>, const double*);
#define HMC_PC_STEPS(PRE, R)                                                                                    \
    HMC_PC_STEPS_R(PRE, R, false, kFftNarrow)                                                                   \
    HMC_PC_STEPS_R(PRE, R, false, kFftMaxRadix)                                                                 \
    HMC_PC_STEPS_R(PRE, R, true, kFftNarrow)                                                                    \
    HMC_PC_STEPS_R(PRE, R, true, kFftMaxRadix)

#define HMC_MT_KERNELS(PRE, MAXR)                                                                               \
    PRE template __global__ void hmc::k_mt_xy<false, MAXR>(hmc::MetricGeo, const double*, double2*, double*,    \
                                                           int, double, const double*);                        \
    PRE template __global__ void hmc::k_mt_xy<true, MAXR>(hmc::MetricGeo, const double*, double2*, double*,     \
                                                          int, double, const double*);                         \
    PRE template __global__ void hmc::k_mt_t<MAXR>(hmc::MetricGeo, double2*, const double*, int, int, double,   \
                                                   double*, int, double*, const double*);

#ifndef HMC_FFT_SOURCE
HMC_PC_KERNELS(extern, float, GeoOne)
HMC_PC_KERNELS(extern, float, GeoBatch)
HMC_PC_KERNELS(extern, double, GeoOne)
HMC_PC_KERNELS(extern, double, GeoBatch)
HMC_PC_STEPS(extern, float)
HMC_PC_STEPS(extern, double)
HMC_MT_KERNELS(extern, hmc::kFftNarrow)
HMC_MT_KERNELS(extern, hmc::kFftMaxRadix)
#endif
