// fft.h -- the twisted Fourier preconditioner P = (K K^dagger)^{-1} of Methods C (Eq. 23-26)
// and the in-place mixed-radix FFT it runs on.
//
// K, the phi-independent part of the fermion matrix, is diagonal on twisted plane waves
// exp(i w_n tau + 2 pi i (kx x + ky y) / L) with w_n = pi (2 n + 1) / N_tau (the twist
// exp(i pi tau / N_tau) turns periodic functions of tau into antiperiodic ones).  Its eigenvalue
// is exp(i w_n) - b with b = 1 + dtau (mu_band + 2 t[band][0] cos k_x + 2 t[band][1] cos k_y
// + 2 tn[band][0] cos 2k_x + 2 tn[band][1] cos 2k_y), the tn terms being the hops by two
// sites of the production model, so P multiplies each Fourier coefficient of the untwisted
// field by 1 / |exp(i w_n) - b|^2 = 1 / ((1 - b)^2 + 4 b sin^2(w_n / 2)).
//
// The preconditioner runs in three passes over a spinor: (1) the 2-D (x, y) transform of
// every (component, tau) slice, held in LDS; (2) per (x, y) frequency column, the exact
// inverse of K K^dagger along tau as two first-order recurrences in registers (precond.h),
// which is what the twisted tau transform and the symbol compute; (3) the inverse 2-D
// transform of every slice.  This header holds the transforms and the tables.
//
// FFT: forward is a decimation-in-frequency sequence of radix stages done in place, so its
// output sits in mixed-radix digit-reversed order (position p holds frequency fft_freq(p));
// the inverse applies the conjugate transposes of the same stages in reverse order, which
// takes that order back to natural order.  No permutation pass is ever needed: the symbol is
// applied at permuted positions, and every position knows its frequency.  Radices up to 16
// without prime factors above 7, each a small DFT in one thread's registers; lengths with a
// larger prime factor are rejected.  The functions are __host__ __device__: the host build
// serves the CPU tests of this code.
//
// What bounds the slice passes is the number of instructions per element and of barriers, not HBM
// (64 B per site in FP32): with radices 4, 2, 3 and 5 only, six stages for an 80 x 80 slice, each an
// LDS round trip and a barrier, with 64-bit index divisions and the plan made by the kernel, one
// slice per 512-thread workgroup.  A plan now has as few stages as possible (two per dimension
// up to L = 140), comes from the host and divides by 32-bit reciprocals; twiddles are read from the
// table, and small slices share a workgroup (slice_cut in hmc.hip).  Per pass, before -> after:
// FP32 80 x 80 x 200 33.4 -> 25.5 us; FP32 16 x 16 x 80, four vectors, 14.0 -> 6.2 us; FP64 28 x 28 x 75, two
// vectors, 28.2 -> 9.7 us; FP64 60 x 60 x 160 41.9 -> 24.4 us; FP32, twelve chains of 12 to 48, four
// vectors each, all running, 171 -> 58 us.  Loading the first butterfly's inputs before the record is
// reduced gained nothing (28.3 us at 80 x 80 x 200: the registers cost a workgroup per CU), nor did 256-
// and 384-thread workgroups (33 and 30 us).
#pragma once

#include <hip/hip_runtime.h>

#include <initializer_list>
#include <type_traits>

#include "lattice.h"

namespace hmc {

constexpr int kFftMaxStages = 12;   // 4^12 > any lattice extent accepted
constexpr int kFftMaxRadix = 16;
// Largest radix of the kernels' narrower instantiation: every L up to 80 with two stages needs no
// more, and radices 12, 14 and 16 raise the slice passes from 46-49 to 64-72 registers in FP32 and
// from 73-79 to 105-121 in FP64 (60 x 60 x 160: 24.4 us against 25.2).
constexpr int kFftNarrow = 10;

// n / d by a 32-bit reciprocal: m = floor((2^32 - 1) / d) + 1 = (2^32 + e) / d with 0 <= e < d, so
// the result is exact while n d < 2^32 (the FFT's counts and extents are below 2^16).
struct Div32 {
    uint32_t d, m;
    __host__ __device__ void init(uint32_t dd) {
        d = dd;
        m = 0xffffffffu / dd + 1u;   // d = 1: unused
    }
    __host__ __device__ __forceinline__ uint32_t div(uint32_t n) const {
        return d == 1u ? n : uint32_t((uint64_t(n) * m) >> 32);
    }
};

// A stage of radix r on sub-length ni: butterflies at positions b ni + n1 + M q, q < r, of a line,
// M = ni / r, 0 <= n1 < M.
struct FftStage {
    int radix, ni;
    Div32 M;        // ni / radix
    Div32 nb;       // butterflies of a line: n / radix
};

// Computed on the host; the kernels read it from the lattice's tables.
struct FftPlan {
    int n;                      // transform length
    int nst;                    // number of radix stages
    FftStage st[kFftMaxStages]; // stage 0 (outermost) ... nst - 1
    Div32 dn;                   // division by n
    Div32 dout;                 // slice lengths: division by n * (n / last radix), see fft_slice_pos
};

// The radices of length n: the fewest stages, of those the smallest largest radix (then the
// smallest first).  False if n has a prime factor above 7.
inline bool fft_radices(int n, int nst, int cap, int* out) {
    if (nst == 0) return n == 1;
    for (int r = 2; r <= cap; ++r) {
        if (n % r != 0 || r == 11 || r == 13 || r == 15) continue;
        out[0] = r;
        if (fft_radices(n / r, nst - 1, cap, out + 1)) return true;
    }
    return false;
}

inline bool make_fft_plan(int n, FftPlan& p) {
    p = FftPlan{};
    p.n = n;
    if (n < 1) return false;
    int m = n;
    for (int f : {2, 3, 5, 7})
        while (m % f == 0) m /= f;
    if (m != 1) return false;
    int r[kFftMaxStages] = {};
    bool ok = n == 1;
    for (int nst = 1; !ok && nst <= kFftMaxStages; ++nst) {
        long long most = 1;
        for (int i = 0; i < nst; ++i) most *= kFftMaxRadix;
        if (most < n) continue;
        for (int cap = 2; !ok && cap <= kFftMaxRadix; ++cap) {
            long long reach = 1;
            for (int i = 0; i < nst; ++i) reach *= cap;
            if (reach < n) continue;
            ok = fft_radices(n, nst, cap, r);
            if (ok) p.nst = nst;
        }
    }
    if (!ok) return false;
    int len = n;
    for (int s = 0; s < p.nst; ++s) {
        p.st[s].radix = r[s];
        p.st[s].ni = len;
        p.st[s].M.init(uint32_t(len / r[s]));
        p.st[s].nb.init(uint32_t(n / r[s]));
        len /= r[s];
    }
    p.dn.init(uint32_t(n));
    // an L only: the square of a time extent does not fit 32 bits
    p.dout.init(uint32_t(p.nst > 0 && n <= kMaxL ? n * (n / r[p.nst - 1]) : 1));
    return true;
}

// Frequency held at position pos after the forward transform.
__host__ __device__ inline int fft_freq(const FftPlan& pl, int pos) {
    int k = 0, mult = 1;
    for (int i = 0; i < pl.nst; ++i) {
        const int M = int(pl.st[i].M.d);
        const int d = pos / M;
        pos -= d * M;
        k += d * mult;
        mult *= pl.st[i].radix;
    }
    return k;
}

// ------------------------------------------------------------------------------------
// Small DFTs of compile-time length in registers, v_k <- sum_m v_m exp(-2 pi i m k / N).

// cos and sin of 2 pi k / n as constants: Taylor series on [0, pi / 4] after reduction.
constexpr double ct_series(double x, bool sine) {
    double term = sine ? x : 1.0, sum = term;
    for (int i = 1; i < 14; ++i) {
        const int k = 2 * i + (sine ? 1 : 0);
        term *= -x * x / double(k * (k - 1));
        sum += term;
    }
    return sum;
}
constexpr double ct_cos(int k, int n) {
    k %= n;
    if (k < 0) k += n;
    if (2 * k > n) k = n - k;
    constexpr double two_pi = 6.283185307179586476925286766559;
    if (4 * k > n) return -ct_cos(n - 2 * k, 2 * n);
    if (8 * k > n) return ct_series(two_pi * double(n - 4 * k) / double(4 * n), true);
    return ct_series(two_pi * double(k) / double(n), false);
}
constexpr double ct_sin(int k, int n) { return ct_cos(4 * k - n, 4 * n); }

// v exp(-2 pi i K / N)
template <typename R, int K, int N>
__host__ __device__ __forceinline__ C2<R> mul_root(C2<R> v) {
    if constexpr (K % N == 0) return v;
    else if constexpr (4 * (K % N) == N) return mk<R>(v.y, -v.x);
    else if constexpr (2 * (K % N) == N) return mk<R>(-v.x, -v.y);
    else if constexpr (4 * (K % N) == 3 * N) return mk<R>(-v.y, v.x);
    else {
        constexpr R c = R(ct_cos(K % N, N)), s = R(ct_sin(K % N, N));
        return mk<R>(c * v.x + s * v.y, c * v.y - s * v.x);
    }
}

// The small functions below hold register arrays by reference: every one of them has to be inlined,
// or the arrays would go to scratch memory.
#define HMC_FLAT __attribute__((always_inline))

// Compile-time loop: f(integral_constant 0) ... f(integral_constant N - 1).
template <int N, int I = 0, class F>
__host__ __device__ __forceinline__ void ct_for(const F& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        ct_for<N, I + 1>(f);
    }
}

constexpr int ct_inverse(int a, int m) {     // a^-1 mod m
    for (int i = 1; i < m; ++i)
        if (a * i % m == 1) return i;
    return 0;
}

template <typename R, int N>
__host__ __device__ __forceinline__ void dft(C2<R> (&v)[N]) {
    if constexpr (N == 1) {
    } else if constexpr (N == 2) {
        const C2<R> a = v[0], b = v[1];
        v[0] = add<R>(a, b);
        v[1] = sub<R>(a, b);
    } else if constexpr (N == 4) {
        const C2<R> a = v[0], b = v[1], c = v[2], d = v[3];
        const C2<R> s0 = add<R>(a, c), d0 = sub<R>(a, c), s1 = add<R>(b, d), d1 = sub<R>(b, d);
        const C2<R> jd1 = mk<R>(d1.y, -d1.x);
        v[0] = add<R>(s0, s1);
        v[1] = add<R>(d0, jd1);
        v[2] = sub<R>(s0, s1);
        v[3] = sub<R>(d0, jd1);
    } else if constexpr (N == 3 || N == 5 || N == 7) {
        // the sums and differences of the pairs (j, N - j); X_k, X_{N-k} = a_k -+ i b_k
        constexpr int H = N / 2;
        C2<R> t[H], d[H], x0 = v[0];
        ct_for<H>([&](auto j) HMC_FLAT {
            t[j] = add<R>(v[j + 1], v[N - 1 - j]);
            d[j] = sub<R>(v[j + 1], v[N - 1 - j]);
            x0 = add<R>(x0, t[j]);
        });
        C2<R> out[N];
        ct_for<H>([&](auto k) HMC_FLAT {
            C2<R> a = v[0], b = mk<R>(R(0), R(0));
            ct_for<H>([&](auto j) HMC_FLAT {
                constexpr int e = (decltype(j)::value + 1) * (decltype(k)::value + 1);
                constexpr R c = R(ct_cos(e, N)), s = R(ct_sin(e, N));
                a = axpy<R>(c, t[j], a);
                if constexpr (decltype(j)::value == 0) b = scl<R>(s, d[j]);
                else b = axpy<R>(s, d[j], b);
            });
            out[k + 1] = mk<R>(a.x + b.y, a.y - b.x);
            out[N - 1 - k] = mk<R>(a.x - b.y, a.y + b.x);
        });
        v[0] = x0;
        ct_for<N - 1>([&](auto k) HMC_FLAT { v[k + 1] = out[k + 1]; });
    } else {
        constexpr int A = N == 8 ? 4 : N == 9 ? 3 : N == 16 ? 4 : N == 12 ? 4 : 2, B = N / A;
        C2<R> w[N];
        if constexpr (N == 8 || N == 9 || N == 16) {
            // N = A B: the DFTs of length A over every B-th input, the roots, those of length B
            ct_for<B>([&](auto b) HMC_FLAT {
                C2<R> u[A];
                ct_for<A>([&](auto a) HMC_FLAT { u[a] = v[b + B * a]; });
                dft<R, A>(u);
                ct_for<A>([&](auto a) HMC_FLAT { w[b * A + a] = mul_root<R, decltype(b)::value * decltype(a)::value, N>(u[a]); });
            });
            ct_for<A>([&](auto a) HMC_FLAT {
                C2<R> u[B];
                ct_for<B>([&](auto b) HMC_FLAT { u[b] = w[b * A + a]; });
                dft<R, B>(u);
                ct_for<B>([&](auto b) HMC_FLAT { v[a + A * b] = u[b]; });
            });
        } else {
            // A and B coprime: index maps instead of roots (the prime-factor form)
            constexpr int ea = B * ct_inverse(B % A, A), eb = A * ct_inverse(A % B, B);
            ct_for<B>([&](auto b) HMC_FLAT {
                C2<R> u[A];
                ct_for<A>([&](auto a) HMC_FLAT { u[a] = v[(a * B + b * A) % N]; });
                dft<R, A>(u);
                ct_for<A>([&](auto a) HMC_FLAT { w[b * A + a] = u[a]; });
            });
            ct_for<A>([&](auto a) HMC_FLAT {
                C2<R> u[B];
                ct_for<B>([&](auto b) HMC_FLAT { u[b] = w[b * A + a]; });
                dft<R, B>(u);
                ct_for<B>([&](auto b) HMC_FLAT { v[(a * ea + b * eb) % N] = u[b]; });
            });
        }
    }
}
// The same with exp(+2 pi i m k / N): real and imaginary parts change places before and after.
template <typename R, bool INV, int N>
__host__ __device__ __forceinline__ void dft_dir(C2<R> (&v)[N]) {
    if constexpr (INV) ct_for<N>([&](auto k) HMC_FLAT { v[k] = mk<R>(v[k].y, v[k].x); });
    dft<R, N>(v);
    if constexpr (INV) ct_for<N>([&](auto k) HMC_FLAT { v[k] = mk<R>(v[k].y, v[k].x); });
}

// ------------------------------------------------------------------------------------
// Execution policies: the device one spreads work over the workgroup and synchronises it; the
// host one runs sequentially (CPU tests).
struct ExDevice {
    template <class F>
    __device__ __forceinline__ void for_each(int n, const F& f) const {
#pragma unroll 1
        for (int i = threadIdx.x; i < n; i += blockDim.x) f(i);
    }
    __device__ __forceinline__ void sync() const { __syncthreads(); }
};
struct ExHost {
    template <class F>
    void for_each(int n, const F& f) const {
        for (int i = 0; i < n; ++i) f(i);
    }
    void sync() const {}
};

// A set of lines in the working copy: line c (c < cnt) of set s starts at s * sp + c * cs, its
// elements es apart.
struct Lines {
    int cnt, es, cs, sp, nset;
    Div32 dcnt;
};

// One radix-RAD stage of every line.  A work item is one butterfly of one line, consecutive items
// consecutive lines.  Elements come from ld(set, item of the set, butterfly, line, q, position) and
// go to st(...) of the same arguments, q < RAD; the default accessors are the working copy itself.
// tw: exp(-2 pi i e / n), e < n.
template <typename R, bool INV, int RAD, class Ex, class Ld, class St>
__host__ __device__ __forceinline__ void fft_stage(const Ex& ex, const FftPlan& pl, const FftStage& sg, const Lines& ln,
                                                   const C2<R>* tw, const Ld& ld, const St& st) {
    const int nb = int(sg.nb.d), M = int(sg.M.d), per_set = ln.cnt * nb, fold = pl.n / sg.ni;
    ex.for_each(ln.nset * per_set, [&](int i) HMC_FLAT {
        int t = int(ln.dcnt.div(uint32_t(i)));
        const int c = i - t * ln.cnt;
        int set = 0;
        if (ln.nset > 1) {
            set = int(sg.nb.div(uint32_t(t)));
            t -= set * nb;
        }
        const int b = int(sg.M.div(uint32_t(t))), n1 = t - b * M;
        const int base = b * sg.ni + n1, it = i - set * per_set;
        C2<R> v[RAD];
        ct_for<RAD>([&](auto q) HMC_FLAT { v[q] = ld(set, it, c, int(q), base + M * q); });
        // Forward (DIF): small DFT, then times W_n^{e k}.  Inverse: the conjugate transpose of
        // that map.  The exponent e k stays below n because n1 < ni / RAD and k < RAD.  The last
        // stage (M = 1) has no factors.
        const int e = fold * n1;
        if constexpr (!INV) dft_dir<R, false, RAD>(v);
        if (M > 1)
            ct_for<RAD - 1>([&](auto k) HMC_FLAT {
                const C2<R> w = tw[e * (k + 1)];
                v[k + 1] = INV ? cmulc<R>(v[k + 1], w) : cmul<R>(v[k + 1], w);
            });
        if constexpr (INV) dft_dir<R, true, RAD>(v);
        ct_for<RAD>([&](auto q) HMC_FLAT { st(set, it, c, int(q), base + M * q, v[q]); });
    });
}

// Stage s of the plan on the lines.  MAXR is the largest radix compiled in (kFftNarrow or
// kFftMaxRadix): a kernel's register allocation covers every stage it can reach, and the largest
// radices need twice the registers, so kernels for lattices without them leave them out.
template <typename R, bool INV, int MAXR, class Ex, class Ld, class St>
__host__ __device__ __forceinline__ void fft_one_stage(const Ex& ex, const FftPlan& pl, int s, const Lines& ln,
                                                       const C2<R>* tw, const Ld& ld, const St& st) {
    const FftStage sg = pl.st[s];
#define HMC_FFT_STAGE(RAD) \
    case RAD: fft_stage<R, INV, RAD>(ex, pl, sg, ln, tw, ld, st); break;
    switch (sg.radix) {
        HMC_FFT_STAGE(2)
        HMC_FFT_STAGE(3)
        HMC_FFT_STAGE(4)
        HMC_FFT_STAGE(5)
        HMC_FFT_STAGE(6)
        HMC_FFT_STAGE(7)
        HMC_FFT_STAGE(8)
        HMC_FFT_STAGE(9)
        HMC_FFT_STAGE(10)
        default:
            if constexpr (MAXR > kFftNarrow) {
                switch (sg.radix) {
                    HMC_FFT_STAGE(12)
                    HMC_FFT_STAGE(14)
                    HMC_FFT_STAGE(16)
                }
            }
            break;
    }
#undef HMC_FFT_STAGE
}

// Stages s0 <= s < s1 in place on the lines of buf, in transform order (ascending forward,
// descending inverse), each followed by a synchronisation.
template <typename R, bool INV, int MAXR = kFftMaxRadix, class Ex>
__host__ __device__ __forceinline__ void fft_lines(const Ex& ex, C2<R>* buf, const Lines& ln, const FftPlan& pl,
                                                   const C2<R>* tw, int s0, int s1) {
    auto ld = [&](int set, int, int c, int, int pos) HMC_FLAT { return buf[set * ln.sp + c * ln.cs + pos * ln.es]; };
    auto st = [&](int set, int, int c, int, int pos, C2<R> v) HMC_FLAT { buf[set * ln.sp + c * ln.cs + pos * ln.es] = v; };
#pragma unroll 1
    for (int k = s0; k < s1; ++k) {
        fft_one_stage<R, INV, MAXR>(ex, pl, INV ? s1 - 1 - (k - s0) : k, ln, tw, ld, st);
        ex.sync();
    }
}

// 2-D transform of ns slices of L x L (row-major x, y; slice s at s * LL): forward along x then
// y, from src(element) to dst(element); the inverse takes the same way back.  The first stage
// reads src and the last writes dst, each element once, so there is no copy in or out; the
// working copy in buf has rows of P elements (P = L + 1 keeps a column's elements in different
// LDS banks).
//
// The transformed slice is not stored row by row: its last stage, radix r along y, would write r
// neighbouring elements per thread, 8 r bytes apart between lanes.  Element q of item (butterfly
// b, row x) is stored at q * (LL / r) + b * L + x instead, so that lanes write (and the inverse
// reads) consecutive addresses; fft_slice_pos gives the (x, y) positions of an index.
__host__ __device__ __forceinline__ void fft_slice_pos(const FftPlan& pl, int i, int& px, int& py) {
    const FftStage& sg = pl.st[pl.nst - 1];
    const int q = int(pl.dout.div(uint32_t(i))), it = i - q * int(pl.dout.d);
    const int b = int(pl.dn.div(uint32_t(it)));
    px = it - b * pl.n;
    py = b * sg.radix + q;
}
// The two ways' middle, for callers that have or want the slices in the working copy: forward from
// the working copy, its stages along x from sx on, to dst(slice, element); the inverse from
// src(slice, element), its stages along x down to sx, into the working copy (synchronised).
template <typename R, int MAXR = kFftMaxRadix, class Ex, class Dst>
__host__ __device__ __forceinline__ void fft_slices_out(const Ex& ex, C2<R>* buf, const Dst& dst, int ns, int P,
                                                        const FftPlan& pl, const C2<R>* tw, int sx) {
    const int L = pl.n, nst = pl.nst;
    const Lines col{L, P, 1, L * P, ns, pl.dn}, row{L, 1, P, L * P, ns, pl.dn};
    const int per_out = int(pl.dout.d);      // items of a slice in the last stage along y
    fft_lines<R, false, MAXR>(ex, buf, col, pl, tw, sx, nst);
    fft_lines<R, false, MAXR>(ex, buf, row, pl, tw, 0, nst - 1);
    fft_one_stage<R, false, MAXR>(
        ex, pl, nst - 1, row, tw, [&](int set, int, int c, int, int pos) HMC_FLAT { return buf[set * row.sp + c * P + pos]; },
        [&](int set, int it, int, int q, int, C2<R> v) HMC_FLAT { dst(set, q * per_out + it, v); });
}
template <typename R, int MAXR = kFftMaxRadix, class Ex, class Src>
__host__ __device__ __forceinline__ void fft_slices_in(const Ex& ex, const Src& src, C2<R>* buf, int ns, int P,
                                                       const FftPlan& pl, const C2<R>* tw, int sx) {
    const int L = pl.n, nst = pl.nst;
    const Lines col{L, P, 1, L * P, ns, pl.dn}, row{L, 1, P, L * P, ns, pl.dn};
    const int per_out = int(pl.dout.d);
    fft_one_stage<R, true, MAXR>(
        ex, pl, nst - 1, row, tw, [&](int set, int it, int, int q, int) HMC_FLAT { return src(set, q * per_out + it); },
        [&](int set, int, int c, int, int pos, C2<R> v) HMC_FLAT { buf[set * row.sp + c * P + pos] = v; });
    ex.sync();
    fft_lines<R, true, MAXR>(ex, buf, row, pl, tw, 0, nst - 1);
    fft_lines<R, true, MAXR>(ex, buf, col, pl, tw, sx, nst);
}
template <typename R, bool INV, int MAXR = kFftMaxRadix, class Ex, class Src, class Dst>
__host__ __device__ __forceinline__ void fft_slices(const Ex& ex, const Src& src, C2<R>* buf, const Dst& dst, int ns,
                                                    int P, const FftPlan& pl, const C2<R>* tw) {
    const int L = pl.n, LL = L * L;
    const Lines col{L, P, 1, L * P, ns, pl.dn};
    if constexpr (!INV) {
        fft_one_stage<R, false, MAXR>(
            ex, pl, 0, col, tw, [&](int set, int, int c, int, int pos) HMC_FLAT { return src(set * LL + pos * L + c); },
            [&](int set, int, int c, int, int pos, C2<R> v) HMC_FLAT { buf[set * col.sp + c + pos * P] = v; });
        ex.sync();
        fft_slices_out<R, MAXR>(ex, buf, [&](int set, int i, C2<R> v) HMC_FLAT { dst(set * LL + i, v); }, ns, P, pl, tw, 1);
    } else {
        fft_slices_in<R, MAXR>(ex, [&](int set, int i) HMC_FLAT { return src(set * LL + i); }, buf, ns, P, pl, tw, 1);
        fft_one_stage<R, true, MAXR>(
            ex, pl, 0, col, tw, [&](int set, int, int c, int, int pos) HMC_FLAT { return buf[set * col.sp + c + pos * P]; },
            [&](int set, int, int c, int, int pos, C2<R> v) HMC_FLAT { dst(set * LL + pos * L + c, v); });
    }
}

// Largest radix a plan uses.
inline int fft_max_radix(const FftPlan& pl) {
    int m = 1;
    for (int i = 0; i < pl.nst; ++i) m = pl.st[i].radix > m ? pl.st[i].radix : m;
    return m;
}

// Per-lattice tables, computed once on the host in FP64 (pc_table_blob) and read by the
// passes of the preconditioner and of the metric:
//   twl[j]   = exp(-2 pi i j / L)          FFT twiddles of length L
//   twT[j]   = exp(-2 pi i j / N_tau)      FFT twiddles of length N_tau
//   cosx[p]  = cos(2 pi k / L) for the frequency k held at x (or y) position p
//   planL, planT: the FFT plans of L and N_tau
// Offsets (in doubles) of the tables in the flat blob.
struct PcBlob {
    int twl, twT, cosx, planL, planT, size;
};
constexpr int kPlanDoubles = int((sizeof(FftPlan) + 7) / 8);
__host__ __device__ __forceinline__ PcBlob pc_blob_layout(int L, int Lt) {
    PcBlob b;
    b.twl = 0;
    b.twT = 2 * L;
    b.cosx = b.twT + 2 * Lt;
    b.planL = b.cosx + L;
    b.planT = b.planL + kPlanDoubles;
    b.size = b.planT + kPlanDoubles;
    return b;
}
__host__ __device__ __forceinline__ const FftPlan& blob_plan(const double* blob, int at) {
    return *reinterpret_cast<const FftPlan*>(blob + at);
}

}  // namespace hmc
