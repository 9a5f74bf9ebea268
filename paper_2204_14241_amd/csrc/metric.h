// Kernels of the Fourier-diagonal HMC metric ("Scale-invariant sampling": Eq. 30 and the
// momentum draw and kinetic energy stated with it).  They reuse the FFT of the Fourier
// preconditioner (fft.h) and the staging and reduction helpers of kernels.h.
//
// On a real boson-shaped field v (3 components of
// N_tau x L x L) the passes compute, per component, the unitary transform F v and from it
// per-frequency work against a caller table sigma of the same shape in natural frequency
// order: y = Re F(s . F^* v) with s = sigma or sigma^(-1/2), the sums sum_k w(k) |(F v)(k)|^2
// with w = sigma, 1/sigma or 1, and acc(k) += |(F v)(k)|^2 (one term of Eq. 30).  A null
// sigma reads as sigma = 1.  FP64, three passes shaped like the preconditioner's: the slice FFT
// into a complex scratch field, the tau pass, the inverse slice FFT that writes or adds the
// field.
//
// v is real, so that F v at -k is the conjugate of F v at k, and every pass does half the work of a
// complex field's: the slice passes transform two slices as the real and imaginary part of one, and
// the scratch field and the tau pass have only the frequencies 0 <= k_y <= L / 2 of a slice, stored
// (position of k_x, k_y).  The transforms are bound by the vector units and the latency of their
// stages rather than by memory (60 x 60 x 160: 14 us a slice pass, now on half as many workgroups, one per
// CU; the tau pass 13 us, and 21 with a table and the way back, against 25 over all frequencies).
#pragma once

#include "precond.h"

namespace hmc {

// Stage n complex elements between global memory and LDS: element i of the set lives at g(i)
// in global memory and at lds[i].  Up to 64 bytes of loads are in flight per thread before
// their LDS writes (a plain loop would wait out the memory latency once per element).  The
// components are kept in separate arrays so that they stay in registers.
template <typename R, class G>
__device__ __forceinline__ void stage_in(C2<R>* __restrict__ lds, int n, G g) {
    constexpr int U = sizeof(R) == 4 ? 8 : 4;
    const int nt = blockDim.x;
    for (int i0 = threadIdx.x; i0 < n; i0 += nt * U) {
        R vx[U], vy[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (i < n) {
                const C2<R> v = *g(i);
                vx[u] = v.x;
                vy[u] = v.y;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (i < n) lds[i] = mk<R>(vx[u], vy[u]);
        }
    }
}
template <typename R, class G>
__device__ __forceinline__ void stage_out(const C2<R>* __restrict__ lds, int n, G g) {
    constexpr int U = sizeof(R) == 4 ? 8 : 4;
    const int nt = blockDim.x;
    for (int i0 = threadIdx.x; i0 < n; i0 += nt * U) {
        R vx[U], vy[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (i < n) {
                const C2<R> v = lds[i];
                vx[u] = v.x;
                vy[u] = v.y;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (i < n) *g(i) = mk<R>(vx[u], vy[u]);
        }
    }
}

enum MetricMul : int { MUL_SIGMA = 1, MUL_RSQRT = 2 };
enum MetricRed : int { RED_NONE = 0, RED_SIGMA = 1, RED_INV = 2, RED_PLAIN = 3 };

struct MetricGeo {
    int L, Lt, LL, vol, pitch;
    int hw, hl;      // L / 2 + 1 frequencies k_y, and L hw columns of the scratch field
    int ncol;        // columns of a tau-pass workgroup
};

// Dynamic LDS of the slice passes: the working copy, its twiddles and two tables of positions.
__host__ __device__ inline size_t mt_xy_lds(int L, int pitch) {
    return (size_t(L) * pitch + L) * sizeof(double2) + size_t(2 * L) * sizeof(int);
}

// One workgroup per (component, pair of slices tau, tau + 1).  Forward: scr = FFT2(in).  Inverse:
// out = the inverse FFT2 of scr (add == 0) or out += h times it (add == 1).  With
// W = FFT2(v(tau) + i v(tau + 1)): FFT2(v(tau))(k) = (W(k) + W(-k)^*) / 2 and FFT2(v(tau + 1))(k) =
// (W(k) - W(-k)^*) / 2i, so the last stage stays in LDS and W(k) and W(-k) are taken from there.
template <bool INV, int MAXR>
__global__ __launch_bounds__(kPcBlock) void k_mt_xy(MetricGeo g, const double* __restrict__ in,
                                                  double2* __restrict__ scr, double* __restrict__ out, int add,
                                                  double h, const double* __restrict__ blob) {
    extern __shared__ __align__(16) unsigned char pc_smem[];
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int L = g.L, LL = g.LL, P = g.pitch, hw = g.hw, hl = g.hl, half = (g.Lt + 1) / 2;
    const int l = b / half, tau = 2 * (b - l * half);
    const bool two = tau + 1 < g.Lt;         // the last slice of an odd count stands alone
    double2* buf = reinterpret_cast<double2*>(pc_smem);
    double2* tw = buf + L * P;
    int* at_k = reinterpret_cast<int*>(tw + L);   // position of a frequency
    int* k_at = at_k + L;                         // frequency at a position
    const PcBlob bl = pc_blob_layout(L, g.Lt);
    const FftPlan& pl = blob_plan(blob, bl.planL);
    for (int i = threadIdx.x; i < L; i += blockDim.x) {
        tw[i] = make_double2(blob[bl.twl + 2 * i], blob[bl.twl + 2 * i + 1]);
        const int k = fft_freq(pl, i);
        at_k[k] = i;
        k_at[i] = k;
    }
    auto neg = [&](int k) HMC_FLAT { return k == 0 ? 0 : L - k; };
    __syncthreads();
    Div32 dh;
    dh.init(uint32_t(hw));
    const Lines col{L, P, 1, L * P, 1, pl.dn}, row{L, 1, P, L * P, 1, pl.dn};
    auto ld = [&](int, int, int c, int, int pos) HMC_FLAT { return buf[c + pos * P]; };
    const size_t field = (size_t(l) * g.Lt + tau) * LL;
    double2* w = scr + (size_t(l) * g.Lt + tau) * hl;
    if constexpr (!INV) {
        const double *v0 = in + field, *v1 = v0 + (two ? LL : 0);
        const double on = two ? 1.0 : 0.0;
        fft_one_stage<double, false, MAXR>(
            ExDevice(), pl, 0, col, tw,
            [&](int, int, int c, int, int pos) HMC_FLAT { return make_double2(v0[pos * L + c], on * v1[pos * L + c]); },
            [&](int, int, int c, int, int pos, double2 v) HMC_FLAT { buf[c + pos * P] = v; });
        __syncthreads();
        fft_lines<double, false, MAXR>(ExDevice(), buf, col, pl, tw, 1, pl.nst);
        fft_lines<double, false, MAXR>(ExDevice(), buf, row, pl, tw, 0, pl.nst);
        for (int i = threadIdx.x; i < hl; i += blockDim.x) {
            const int px = int(dh.div(uint32_t(i))), ky = i - px * hw;
            const double2 p = buf[px * P + at_k[ky]], m = buf[at_k[neg(k_at[px])] * P + at_k[neg(ky)]];
            w[i] = make_double2(0.5 * (p.x + m.x), 0.5 * (p.y - m.y));
            if (two) w[hl + i] = make_double2(0.5 * (p.y + m.y), 0.5 * (m.x - p.x));
        }
    } else {
        const double2* w1 = w + (two ? hl : 0);
        const double on = two ? 1.0 : 0.0;
        constexpr int U = 4;     // elements whose loads are in flight together
        const int nt = blockDim.x;
        for (int i0 = threadIdx.x; i0 < hl; i0 += nt * U) {
            double2 a[U], c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * nt, hl - 1);
                a[u] = w[i];
                c[u] = w1[i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * nt;
                if (i < hl) {
                    const int px = int(dh.div(uint32_t(i))), ky = i - px * hw;
                    const double2 y = make_double2(on * c[u].x, on * c[u].y);
                    buf[px * P + at_k[ky]] = make_double2(a[u].x - y.y, a[u].y + y.x);
                    // k_y = 0 and L / 2 hold -k themselves
                    if (ky != 0 && 2 * ky != L) buf[at_k[neg(k_at[px])] * P + at_k[L - ky]] = make_double2(a[u].x + y.y, y.x - a[u].y);
                }
            }
        }
        __syncthreads();
        fft_lines<double, true, MAXR>(ExDevice(), buf, row, pl, tw, 0, pl.nst);
        fft_lines<double, true, MAXR>(ExDevice(), buf, col, pl, tw, 1, pl.nst);
        double *y0 = out + field, *y1 = y0 + LL;
        fft_one_stage<double, true, MAXR>(ExDevice(), pl, 0, col, tw, ld,
                                          [&](int, int, int c, int, int pos, double2 v) HMC_FLAT {
                                              const int i = pos * L + c;
                                              y0[i] = add ? y0[i] + h * v.x : v.x;
                                              if (two) y1[i] = add ? y1[i] + h * v.y : v.y;
                                          });
    }
}

// Columns of a tau-pass workgroup (128 bytes of each row) and the LDS it takes; its threads are
// kMtThreads where the launch has two workgroups per CU or more, else kPcBlock, for the latency of
// one.  80 x 80 x 200: 33.8 us, with 16 columns and 512 threads 41.8; 24 x 24 x 80 10.4 against 11.7.
constexpr int kMtCols = 8, kMtThreads = 256;
__host__ __device__ inline size_t mt_t_lds(int L, int Lt, int ncol) {
    return size_t(Lt) * (ncol + 1) * sizeof(double2) + size_t(Lt + L) * sizeof(int);
}

// One workgroup per (component, group of g.ncol consecutive columns of the scratch field): the tau
// FFT of the group's columns, the per-frequency work (positions are in digit-reversed order; each
// knows its frequency), and with `mul` != 0 the scaling by s / V and the inverse tau FFT back into
// scr.  A column with 0 < k_y < L / 2 stands for -k too, whose value is the conjugate: it counts
// with both table entries, and y, being real, takes the even part of the scaling.
// part[workgroup] receives rs times the workgroup's share of the sum; acc(k) receives
// |(F v)(k)|^2, added (acc_add) or stored.
template <int MAXR>
__global__ __launch_bounds__(kPcBlock) void k_mt_t(MetricGeo g, double2* __restrict__ scr,
                                                 const double* __restrict__ sigma, int mul, int red, double rs,
                                                 double* __restrict__ acc, int acc_add, double* __restrict__ part,
                                                 const double* __restrict__ blob) {
    extern __shared__ __align__(16) unsigned char pc_smem[];
    const int L = g.L, Lt = g.Lt, hw = g.hw, hl = g.hl, NC = g.ncol;
    const int ng = pc_groups(hl, NC);
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int l = b / ng, grp = b - l * ng;
    const int col0 = grp * NC, ncol = min(NC, hl - col0);
    double2* buf = reinterpret_cast<double2*>(pc_smem);
    double2* twT = buf + Lt * NC;
    int* fT = reinterpret_cast<int*>(twT + Lt);
    int* fL = fT + Lt;
    const PcBlob bl = pc_blob_layout(L, Lt);
    for (int i = threadIdx.x; i < Lt; i += blockDim.x) twT[i] = make_double2(blob[bl.twT + 2 * i], blob[bl.twT + 2 * i + 1]);
    const FftPlan &pt = blob_plan(blob, bl.planT), &pl = blob_plan(blob, bl.planL);
    for (int i = threadIdx.x; i < Lt; i += blockDim.x) fT[i] = fft_freq(pt, i);
    for (int i = threadIdx.x; i < L; i += blockDim.x) fL[i] = fft_freq(pl, i);
    Div32 dc, dh;
    dc.init(uint32_t(ncol));
    dh.init(uint32_t(hw));
    const Lines lines{ncol, ncol, 1, 0, 1, dc};
    const size_t o = size_t(l) * Lt * hl + size_t(col0);
    auto at = [&](int i) {
        const int tau = int(dc.div(uint32_t(i)));
        return scr + o + size_t(tau) * hl + (i - tau * ncol);
    };
    stage_in<double>(buf, Lt * ncol, at);
    __syncthreads();
    fft_lines<double, false, MAXR>(ExDevice(), buf, lines, pt, twT, 0, pt.nst);
    const double inv_v = 1.0 / double(g.vol);
    const double* sg = sigma ? sigma + size_t(l) * g.vol : nullptr;
    double* ac = acc ? acc + size_t(l) * g.vol : nullptr;
    double sum[1] = {0.0};
    for (int i = threadIdx.x; i < Lt * ncol; i += blockDim.x) {
        const int p = int(dc.div(uint32_t(i))), c = col0 + i - p * ncol;
        const int px = int(dh.div(uint32_t(c))), ky = c - px * hw;
        const int n = fT[p], kx = fL[px];
        const size_t k = (size_t(n) * L + kx) * L + ky;
        const size_t km = (size_t(n == 0 ? 0 : Lt - n) * L + (kx == 0 ? 0 : L - kx)) * L + (ky == 0 ? 0 : L - ky);   // -k
        const bool pair = ky != 0 && 2 * ky != L;
        const double sv = sg ? sg[k] : 1.0, sm = sg ? sg[km] : 1.0;
        const double2 y = buf[i];
        const double n2 = (y.x * y.x + y.y * y.y) * inv_v;
        if (red == RED_SIGMA) sum[0] += (pair ? sv + sm : sv) * n2;
        else if (red == RED_INV) sum[0] += pair ? n2 / sv + n2 / sm : n2 / sv;
        else if (red == RED_PLAIN) sum[0] += pair ? 2.0 * n2 : n2;
        if (ac) {
            ac[k] = acc_add ? ac[k] + n2 : n2;
            if (pair) ac[km] = acc_add ? ac[km] + n2 : n2;
        }
        if (mul) {
            double m;
            if (mul == MUL_SIGMA) {
                m = 0.5 * (sv + sm);
            } else {
                m = 1.0 / sqrt(sv);
                if (sm != sv) m = 0.5 * (m + 1.0 / sqrt(sm));     // an even table pays for one root
            }
            m *= inv_v;
            buf[i] = make_double2(m * y.x, m * y.y);
        }
    }
    block_reduce<1>(sum);   // ends with a barrier
    if (part != nullptr && threadIdx.x == 0) part[b] = rs * sum[0];
    if (mul) {
        fft_lines<double, true, MAXR>(ExDevice(), buf, lines, pt, twT, 0, pt.nst);
        stage_out<double>(buf, Lt * ncol, at);
    }
}

#ifndef HMC_FFT_SOURCE
// chi(k) += scale ((t0(k) + t1(k)) + t2(k)) for the three component planes of t (each vol
// long): one term of the SDW susceptibility of Eq. (34) from the per-component spectra.
__global__ __launch_bounds__(kBlock) void k_mt_sum3(const double* __restrict__ t, double* __restrict__ chi,
                                                    double scale, int vol) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < vol) chi[i] = chi[i] + scale * ((t[i] + t[vol + i]) + t[2 * vol + i]);
}

// Per-workgroup partial sums of each component of a boson-shaped field: part[l * nb + b] for
// component l and workgroup b of nb (the order parameter Phi = sum over sites of phi).
__global__ __launch_bounds__(kBlock) void k_mt_csum(const double* __restrict__ phi, double* __restrict__ part,
                                                    int vol, int nb) {
    const int l = blockIdx.x / nb, b = blockIdx.x - l * nb;
    double v[1] = {0.0};
    for (int i = b * kBlock + threadIdx.x; i < vol; i += nb * kBlock) v[0] += phi[size_t(l) * vol + i];
    block_reduce<1>(v);
    if (threadIdx.x == 0) part[size_t(l) * nb + b] = v[0];
}
#endif

}  // namespace hmc
