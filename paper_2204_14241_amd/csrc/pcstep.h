// pcstep.h -- the preconditioned conjugate gradient on small lattices in three launches per
// iteration instead of five: step A with the inverse slice transforms before it, step B with the
// forward ones after it, and the tau pass between them (precond.h).
//
// What bounds a small preconditioned solve is not what its kernels move but that there are five of
// them, each waiting for the one before: 16 x 16 x 80 with four FP32 vectors spends 33 us an
// iteration on 2 us of traffic.  A slice of all four components fits a workgroup's LDS there, so
// that the transforms need not go through memory to the stencils: 26 us with both steps joined (the
// launch code has the rule and more figures).  The rest of the time is each kernel's chain of
// record, loads, four or more transform stages and stores; loading the sites' other operands before
// the transforms made it longer (27 us there, FP64 28 x 28 x 75 with two vectors 48.8 against 47.5).
#pragma once

#include "precond.h"

namespace hmc {

// Dynamic LDS of the two kernels: k_pc_a transforms the slices tau and tau + 1 of four components;
// k_pc_b holds t(tau) beside the working copy of the new residual.
template <typename R>
__host__ __device__ inline size_t pc_step_lds(int L, int P, bool step_b) {
    return (size_t(step_b ? 4 : 8) * L * P + (step_b ? size_t(4) * L * L : 0) + L) * sizeof(C2<R>);
}

__device__ __forceinline__ int wrap_site(int x, int L) { return x < 0 ? x + L : (x >= L ? x - L : x); }

// Step A (see k_cg_a) of one right-hand side's slice tau per workgroup, on z(tau) and z(tau + 1) that
// it transforms back from the tau pass's z (which stays as it is): consumes <r, z>, leaves one |t|^2
// partial per slice.  z(tau + 1), for the time link, is formed again by the next slice's workgroup,
// by the same operations.
template <typename R, bool NN2, int MAXR>
__global__ __launch_bounds__(kPcBlock) void k_pc_a(CgCtl ctl, GeoOne geo, CgVecs<R> v, const R* __restrict__ phi,
                                                 Coef<R> cf, const double* __restrict__ blob) {
    extern __shared__ __align__(16) unsigned char pc_smem[];
    const UPos pos = geo.at(xcd_remap(blockIdx.x, gridDim.x));
    const Lat& lat = pos.lat;
    const int L = lat.L, LL = lat.LL, Lt = lat.Lt, vol = lat.vol, P = pos.sc.pitch, sp = L * P;
    const int tau = pos.blk, tn = tau + 1 == Lt ? 0 : tau + 1;
    C2<R>* buf = reinterpret_cast<C2<R>*>(pc_smem);
    C2<R>* tw = buf + 8 * sp;
    const PcBlob bl = pc_blob_layout(L, Lt);
    for (int i = threadIdx.x; i < L; i += blockDim.x) tw[i] = mk<R>(R(blob[bl.twl + 2 * i]), R(blob[bl.twl + 2 * i + 1]));
    CgState S;
    const int got = cg_finalize(ctl, pos, 4 * pc_groups(LL, kPcCols), S);
    if (S.mode != CG_ACTIVE || got != PEND_RZ) {
        cg_publish(ctl, pos, S);
        return;
    }
    const R alpha = R(S.alpha), alpha_old = R(S.alpha_old), beta = R(S.beta);
    const bool fold = S.alpha_old != 0.0;   // x += both pending steps this iteration (see k_cg_a)
    const int pb = S.pbuf;
    cg_publish_a(ctl, pos, S);
    const C2<R>* z = v.z + pos.voff;
    const C2<R>* pin = (pb ? v.p1 : v.p0) + pos.voff;
    C2<R>* pout = (pb ? v.p0 : v.p1) + pos.voff;
    C2<R>* x = v.x + pos.voff;
    C2<R>* t = v.t + pos.voff;
    const FftPlan& pl = blob_plan(blob, bl.planL);
    __syncthreads();
    fft_slices_in<R, MAXR>(
        ExDevice(), [&](int set, int i) HMC_FLAT { return z[size_t(set & 3) * vol + size_t(set < 4 ? tau : tn) * LL + i]; },
        buf, 8, P, pl, tw, 0);
    // p_new(tau) in place of z(tau)
    for (int i = threadIdx.x; i < LL; i += blockDim.x) {
        const int xr = int(pl.dn.div(uint32_t(i))), y = i - xr * L;
        C2<R> po[4], pq[4], xv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) po[c] = pin[size_t(c) * vol + size_t(tau) * LL + i];
        if (fold) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const size_t g = size_t(c) * vol + size_t(tau) * LL + i;
                xv[c] = x[g];
                pq[c] = pout[g];
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const size_t g = size_t(c) * vol + size_t(tau) * LL + i;
            C2<R>& w = buf[c * sp + xr * P + y];
            const C2<R> pn = axpy<R>(beta, po[c], w);
            w = pn;
            pout[g] = pn;
            if (fold) x[g] = axpy<R>(alpha, po[c], axpy<R>(alpha_old, pq[c], xv[c]));
        }
    }
    __syncthreads();
    double part = 0.0;
    for (int i = threadIdx.x; i < LL; i += blockDim.x) {
        const int xr = int(pl.dn.div(uint32_t(i))), y = i - xr * L;
        const size_t s = size_t(tau) * LL + i;
        C2<R> tt[4], o[4], cen[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            tt[c] = axpy<R>(beta, pin[size_t(c) * vol + size_t(tn) * LL + i], buf[(4 + c) * sp + xr * P + y]);
        stencil_site_at<R, NN2>([&](int d, int c, int yy) HMC_FLAT { return buf[c * sp + wrap_site(xr + d, L) * P + yy]; },
                                xr, y, L, phi[s], phi[vol + s], phi[2 * vol + s], cf, tau == Lt - 1 ? R(-1) : R(1), tt, o,
                                cen);
        R acc = R(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            t[size_t(c) * vol + s] = o[c];
            acc += norm2<R>(o[c]);
        }
        part += double(acc);
    }
    store_partial(ctl, PEND_TT, pos, part);
}

// Step B (see k_cg_b) of one right-hand side's slice tau per workgroup, and the forward transform of
// the new residual's slice into z: consumes |t|^2, leaves one |r|^2 partial per slice for the tau
// pass, which sees whether the solve has converged (the transform is then not used).
template <typename R, bool NN2, int MAXR>
__global__ __launch_bounds__(kPcBlock) void k_pc_b(CgCtl ctl, GeoOne geo, CgVecs<R> v, const R* __restrict__ phi,
                                                 Coef<R> cf, const double* __restrict__ blob) {
    extern __shared__ __align__(16) unsigned char pc_smem[];
    const UPos pos = geo.at(xcd_remap(blockIdx.x, gridDim.x));
    const Lat& lat = pos.lat;
    const int L = lat.L, LL = lat.LL, Lt = lat.Lt, vol = lat.vol, P = pos.sc.pitch, sp = L * P;
    const int tau = pos.blk, tp = tau == 0 ? Lt - 1 : tau - 1;
    C2<R>* buf = reinterpret_cast<C2<R>*>(pc_smem);
    C2<R>* ts = buf + 4 * sp;        // t(tau), component-major
    C2<R>* tw = ts + 4 * LL;
    const PcBlob bl = pc_blob_layout(L, Lt);
    const C2<R>* tin = v.t + pos.voff;
    C2<R>* r = v.r + pos.voff;
    C2<R>* z = v.z + pos.voff;
    // t(tau) does not depend on the record: in flight while it is reduced
    for (int i = threadIdx.x; i < LL; i += blockDim.x) {
#pragma unroll
        for (int c = 0; c < 4; ++c) ts[c * LL + i] = tin[size_t(c) * vol + size_t(tau) * LL + i];
    }
    for (int i = threadIdx.x; i < L; i += blockDim.x) tw[i] = mk<R>(R(blob[bl.twl + 2 * i]), R(blob[bl.twl + 2 * i + 1]));
    CgState S;
    cg_finalize(ctl, pos, Lt, S);
    if (S.mode != CG_ACTIVE) {
        cg_publish(ctl, pos, S);
        return;
    }
    const R alpha = R(S.alpha_cur);
    S.pending = PEND_RR;
    S.zstage = 1;
    cg_publish(ctl, pos, S);
    const FftPlan& pl = blob_plan(blob, bl.planL);
    __syncthreads();
    double part = 0.0;
    for (int i = threadIdx.x; i < LL; i += blockDim.x) {
        const int xr = int(pl.dn.div(uint32_t(i))), y = i - xr * L;
        const size_t s = size_t(tau) * LL + i;
        C2<R> tt[4], rv[4], o[4], cen[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            tt[c] = tin[size_t(c) * vol + size_t(tp) * LL + i];
            rv[c] = r[size_t(c) * vol + s];
        }
        stencil_site_at<R, NN2>([&](int d, int c, int yy) HMC_FLAT { return ts[c * LL + wrap_site(xr + d, L) * L + yy]; }, xr,
                                y, L, phi[s], phi[vol + s], phi[2 * vol + s], cf, tau == 0 ? R(-1) : R(1), tt, o, cen);
        R acc = R(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const C2<R> rn = axpy<R>(-alpha, o[c], rv[c]);
            r[size_t(c) * vol + s] = rn;
            buf[c * sp + xr * P + y] = rn;
            acc += norm2<R>(rn);
        }
        part += double(acc);
    }
    __syncthreads();
    fft_slices_out<R, MAXR>(
        ExDevice(), buf, [&](int set, int i, C2<R> w) HMC_FLAT { z[size_t(set) * vol + size_t(tau) * LL + i] = w; }, 4, P, pl,
        tw, 0);
    store_partial(ctl, PEND_RR, pos, part);
}

}  // namespace hmc
