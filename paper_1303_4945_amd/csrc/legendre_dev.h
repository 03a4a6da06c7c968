// Device helpers shared by the Legendre kernels (legendre.hip, legendre0.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "sht_internal.h"

namespace sht {

typedef double dv4 __attribute__((ext_vector_type(4)));
typedef float fv4 __attribute__((ext_vector_type(4)));

template <bool F32>
struct MT;
template <>
struct MT<false> {
    using T = double;
    using V = dv4;
};
template <>
struct MT<true> {
    using T = float;
    using V = fv4;
};

__device__ __forceinline__ dv4 mfma(double a, double b, dv4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ fv4 mfma(float a, float b, fv4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Row of the 16x16 result held in register r of this lane (column = lane & 15);
// the FP64 and FP32 instructions use different result layouts.
template <bool F32>
__device__ __forceinline__ int c_row(int lane, int r)
{
    return F32 ? 4 * (lane >> 4) + r : (lane >> 4) + 4 * r;
}

// base^p for base in [0, 1], p >= 0, as mantissa * 2^ex (mantissa in [0.5, 1)).
__device__ inline void xpow(double base, int p, double &mant, int &ex)
{
    mant = 1.0;
    ex = 0;
    if (p == 0) return;
    if (!(base > 0.0)) {
        mant = 0.0;
        return;
    }
    int eb;
    double mb = frexp(base, &eb);
    for (;;) {
        if (p & 1) {
            int d;
            mant = frexp(mant * mb, &d);
            ex += eb + d;
        }
        p >>= 1;
        if (!p) break;
        int d;
        mb = frexp(mb * mb, &d);
        eb = 2 * eb + d;
    }
}

// ---------------------------------------------------------------- recursion

// One recursion chain per lane.  A wavefront runs chains of a single sign
// (+s or -s), so the per-step coefficients are wave-uniform LDS broadcasts.
struct Chain {
    double x;      // cos t
    double ms2;    // -2 sin^2(t/2)
    double mu;     // mu_l
    double aux;    // mu_{l-1} (plain form) or mu_l - mu_{l-1} (difference form)
    int k;         // scale index (value = mu * 2^(S k)), k <= 0
};

__device__ inline Chain chain_init(const LegView &v, int m, int slot, int chain)
{
    Chain c;
    c.mu = 0.0;
    c.aux = 0.0;
    c.k = 0;
    c.x = 0.0;
    c.ms2 = 0.0;
    if (slot >= v.nslots) return c;
    const double x = v.slot_cos[slot], st = v.slot_sin[slot];
    const double sh = v.slot_shalf[slot];
    c.x = x;
    c.ms2 = -2.0 * sh * sh;
    if (v.polar_T >= 0.0) {
        const double s = v.crit_spin, mm = (double)m;
        double q = mm * mm + s * s - 2.0 * mm * s * x;
        double crit = sqrt(q > 0.0 ? q : 0.0) - v.crit_lmax * st;
        if (crit > v.polar_T) return c;   // skipped term (Sect. 3.3)
    }
    const StartCoef sc = v.start[2 * m + chain];
    double mc, ms;
    int ec, es;
    xpow(v.slot_chalf[slot], sc.p, mc, ec);
    xpow(sh, sc.q, ms, es);
    int d;
    double mant = frexp(sc.kmant * mc * ms, &d);
    if (mant == 0.0) return c;
    const int e = sc.kexp + ec + es + d;
    const int S = v.rescale_bits, T = v.thresh_bits;
    int kk = 0;
    if (e < T) kk = (T - e) / S;
    c.k = -kk;
    c.mu = (double)sc.sign * ldexp(mant, e + S * kk);
    return c;
}

// wavefronts with a slot of cos t above this use the difference form
constexpr double DIFF_FORM_COS = 0.7;

__device__ __forceinline__ bool not_finite(double x) { return !(fabs(x) < __builtin_inf()); }

__device__ __forceinline__ bool wave_any(bool p)
{
    return __builtin_amdgcn_ballot_w64(p) != 0;
}

// Orders the LDS traffic of one wavefront at this point (the LDS executes a
// wavefront's requests in issue order; this keeps the compiler from moving
// them across).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// work groups of a persistent launch on a device: every CU filled to the
// kernel's occupancy
template <typename K>
inline int persistent_groups(K kernel, int threads, int dev)
{
    int ncu = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kernel, threads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 1024;
    }
    const int g = ncu * (per_cu > 0 ? per_cu : 1);
    return g > 0 ? g : 1024;
}

// Row of degree offset t in a chunk: natural order, or (PSPLIT) the even offsets
// first and then the odd ones.
template <int LC, bool PSPLIT>
__device__ __forceinline__ int chunk_row(int t)
{
    return PSPLIT ? (t & 1) * (LC / 2) + (t >> 1) : t;
}

// A chunk of the one-step recursion, mu to out[row(t) stride]; cf: per degree alpha,
// beta, the difference form's constant, alpha.  GEN: before (degree offset 0 lies below
// l0: no output, no step) and lanes whose scale is below 0 (no output; rescaled).  The
// coefficients of two steps are read together, one pair ahead of their use: read where
// they are used, every step would wait for the LDS (130 cycles against the 24 of its
// arithmetic).  The degrees past lmax, with coefficients 0, write finite values that
// the caller does not use.
template <int LC, bool PSPLIT, bool DIFF, bool GEN, typename T>
__device__ __forceinline__ void chain_run(Chain &c, const double4 *cf, bool before, double thr, double down, T *out,
                                          int stride)
{
    const double *q0 = reinterpret_cast<const double *>(cf) + (DIFF ? 2 : 0);
    double2 q[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) q[0][i] = *reinterpret_cast<const double2 *>(q0 + 4 * i);
#pragma unroll
    for (int b = 0; b < LC / 2; ++b) {
        if (b + 1 < LC / 2)
#pragma unroll
            for (int i = 0; i < 2; ++i) q[(b + 1) & 1][i] = *reinterpret_cast<const double2 *>(q0 + 4 * (2 * b + 2 + i));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int t = 2 * b + i;
            const double2 qt = q[b & 1][i];
            const bool skip = GEN && t == 0 && before;
            out[chunk_row<LC, PSPLIT>(t) * stride] = GEN && (skip || c.k != 0) ? (T)0 : (T)c.mu;
            if (skip) continue;
            if (DIFF) {
                const double eps = fma(qt.y, c.ms2, qt.x);
                c.aux = fma(eps, c.mu, c.aux);
                c.mu += c.aux;
            } else {
                const double nx = fma(fma(qt.x, c.x, qt.y), c.mu, -c.aux);
                c.aux = c.mu;
                c.mu = nx;
            }
            if (GEN) {
                const bool up = c.k < 0 && fabs(c.mu) >= thr;
                c.mu = up ? c.mu * down : c.mu;
                c.aux = up ? c.aux * down : c.aux;
                c.k += up ? 1 : 0;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace sht
