// small.h -- the whole conjugate-gradient solve of a small lattice in one kernel: one workgroup per
// right-hand side, one thread per site, the direction and M p in LDS, the residual, direction and
// solution in registers.
//
// What bounds a small lattice is the two launches an iteration takes otherwise (5 us each, whatever the
// lattice), not its arithmetic or memory: an iteration here is two LDS stencils and four
// barriers.  The work of a right-hand side is on one CU, so the time grows with the sites: kSmallSites is
// where a workgroup is full (see small_lattice in hmc.hip for both sides).
#pragma once

#include "kernels.h"

namespace hmc {

constexpr int kSmallSites = 512;

// LDS of a workgroup: one spinor, the components of a site side by side (one address and constant
// offsets) and kSmallPitch entries between sites, an odd count, which spreads the sites of a wavefront
// over the banks.
constexpr int kSmallPitch = 5;
__host__ __device__ inline size_t small_lds(int vol) { return size_t(vol) * kSmallPitch * sizeof(double2); }

// The stencil of dslash_site on a spinor in LDS, with phi times the coupling and the staggered sign in
// registers (q).
template <bool DAG, bool NN2>
__device__ __forceinline__ void small_stencil(const double2* buf, const Lat& lat, const Coef<double>& cf, const Nbr& nb,
                                              int s, const double (&q)[3], double2 (&o)[4]) {
    const int st = DAG ? nb.tm : nb.tp;
    auto at = [&](int c, int i) __attribute__((always_inline)) { return buf[i * kSmallPitch + c]; };
    const double ts = double(DAG ? nb.sbwd : nb.sfwd);
    double2 cen[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) cen[c] = at(c, s);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int a = c >> 1;
        double2 w = scl<double>(cf.diag[a], cen[c]);
        w = axpy<double>(cf.hop[a][0], add<double>(at(c, nb.xp), at(c, nb.xm)), w);
        w = axpy<double>(cf.hop[a][1], add<double>(at(c, nb.yp), at(c, nb.ym)), w);
        w = axpy<double>(ts, at(c, st), w);
        if constexpr (NN2) {
            const Nbr2 n2 = neighbours2(lat, nb, s);
            w = axpy<double>(cf.hop2[a][0], add<double>(at(c, n2.xpp), at(c, n2.xmm)), w);
            w = axpy<double>(cf.hop2[a][1], add<double>(at(c, n2.ypp), at(c, n2.ymm)), w);
        }
        o[c] = w;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const double2 u = cen[2 * (1 - a)], w = cen[2 * (1 - a) + 1];
        o[2 * a].x += q[2] * u.x + q[0] * w.x + q[1] * w.y;
        o[2 * a].y += q[2] * u.y + q[0] * w.y - q[1] * w.x;
        o[2 * a + 1].x += q[0] * u.x - q[1] * u.y - q[2] * w.x;
        o[2 * a + 1].y += q[0] * u.y + q[1] * u.x - q[2] * w.y;
    }
}

// Where a solve goes after its true residual rt: done, stopped, or on (CG_ACTIVE).  capped: the update
// is the one at the iteration cap.  A solve whose iterated residual passes and whose true one does
// not may go on past the cap, as the chunked solver lets it; with a tolerance below FP64's reach it
// could do so for ever, so it is stopped kSmallPast iterations past it, where the chunked solver's host
// loop gives up.
constexpr int kSmallPast = 128;
__host__ __device__ inline int small_next(double rt, double stop_rr, bool capped, int iters, int maxit) {
    if (!(rt - rt == 0.0)) return CG_FAILED;
    if (rt <= stop_rr) return CG_DONE;
    return capped || iters - kSmallPast >= maxit ? CG_STOPPED : CG_ACTIVE;
}

// Solve (M^dagger M) x_k = b_k, k = blockIdx.x, in FP64 from x = 0 (the algebra and the stopping rules
// of the chunked solver: k_cg_a, k_cg_b and the state machine of cg_finalize).  st[k] receives the
// final record.
template <bool NN2>
__global__ __launch_bounds__(kSmallSites) void k_cg_small(Lat lat, const double2* __restrict__ b_base,
                                                   double2* __restrict__ x_base, const double* __restrict__ phi_base,
                                                   Coef<double> cf, CgState* __restrict__ st, double tol2, int maxit) {
    extern __shared__ __align__(16) unsigned char small_smem[];
    __shared__ double red[2][kSmallSites / 64];
    const int vol = lat.vol, tid = threadIdx.x, nw = blockDim.x >> 6;
    double2* buf = reinterpret_cast<double2*>(small_smem);       // [site][component]
    const bool own = tid < vol;
    const int s = own ? tid : vol - 1;      // a thread past the lattice repeats the last site
    const size_t off = size_t(blockIdx.x) * 4 * vol;
    const double2* b = b_base + off;
    const Nbr nb = neighbours(lat, s);
    double q[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) q[l] = cf.cpl * double(nb.stag) * phi_base[l * vol + s];
    // The sum of v over the lattice's own threads, in every thread; a barrier.  Two sets of
    // wavefront sums alternate, so one barrier separates a set's reads from its next writes.
    int par = 0;
    auto total = [&](double v) __attribute__((always_inline)) {
        v = wave_sum(own ? v : 0.0);
        if ((tid & 63) == 0) red[par][tid >> 6] = v;
        __syncthreads();
        double a = 0.0;
        for (int i = 0; i < nw; ++i) a += red[par][i];
        par ^= 1;
        return a;
    };
    auto put = [&](const double2 (&v)[4]) __attribute__((always_inline)) {
        if (own) {
#pragma unroll
            for (int c = 0; c < 4; ++c) buf[s * kSmallPitch + c] = v[c];
        }
        __syncthreads();
    };
    auto norm4 = [&](const double2 (&v)[4]) __attribute__((always_inline)) {
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) a += norm2<double>(v[c]);
        return a;
    };
    double2* x = x_base + off;
    double2 r[4], p[4], o[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        r[c] = b[c * vol + s];
        p[c] = make_double2(0.0, 0.0);
    }
    if (own) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c * vol + s] = make_double2(0.0, 0.0);
    }
    const double bb = total(norm4(r)), stop_rr = tol2 * bb;
    double rz = bb, rz_prev = bb, rr = bb, rr_true = bb, beta = 0.0;
    int mode = !finite(bb) ? CG_FAILED : (bb > 0.0 ? CG_ACTIVE : CG_DONE), iters = 0, n_ru = 0;
    while (mode == CG_ACTIVE) {
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = axpy<double>(beta, p[c], r[c]);
        put(p);
        small_stencil<false, NN2>(buf, lat, cf, nb, s, q, o);
        const double tt = total(norm4(o));
        if (!(tt > 0.0) || !finite(tt)) {
            mode = CG_FAILED;
            break;
        }
        const double alpha = rz / tt;
        put(o);
        if (own) {
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c * vol + s] = axpy<double>(alpha, p[c], x[c * vol + s]);
        }
        small_stencil<true, NN2>(buf, lat, cf, nb, s, q, o);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = axpy<double>(-alpha, o[c], r[c]);
        rr = total(norm4(r));
        if (!finite(rr)) {
            mode = CG_FAILED;
            break;
        }
        rz_prev = rz;
        beta = rr / rz;
        rz = rr;
        iters += 1;
        const bool conv = rr <= stop_rr, last = !conv && iters >= maxit;
        if (!conv && !last) continue;
        // the true residual b - M^dagger M x: done, stopped at the cap, or on from there
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = x[c * vol + s];
        put(o);
        small_stencil<false, NN2>(buf, lat, cf, nb, s, q, o);
        __syncthreads();
        put(o);
        small_stencil<true, NN2>(buf, lat, cf, nb, s, q, o);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = sub<double>(b[c * vol + s], o[c]);
        const double rt = total(norm4(r));
        rr_true = rt;
        n_ru += 1;
        mode = small_next(rt, stop_rr, last, iters, maxit);
        if (mode == CG_ACTIVE) {
            beta = rt / rz_prev;
            rz = rr = rt;
        }
    }
    if (tid == 0) {
        CgState& S = st[blockIdx.x];
        S.bb = bb;
        S.stop_rr = stop_rr;
        S.rr = rr;
        S.rr_true = rr_true;
        S.rz = rz;
        S.rz_prev = rz_prev;
        S.mode = mode;
        S.iters = iters;
        S.n_ru = n_ru;
        S.maxit = maxit;
        S.pending = PEND_NONE;
    }
}

}  // namespace hmc
