// Spin 1 and 2 away from the poles as spin-0 transforms.
//
// sin^s t times the spin-s functions W, X = (s_lambda +- (-1)^s -s_lambda)/2 is a
// short band of scalar functions of the same m: with
//   eps_l = sqrt((l^2 - m^2) / (4 l^2 - 1)),   L = l (l + 1),
//   cos t lambda_l = eps_(l+1) lambda_(l+1) + eps_l lambda_(l-1),
//   sin t d/dt lambda_l = l eps_(l+1) lambda_(l+1) - (l + 1) eps_l lambda_(l-1),
// the spin-raising operators (Sect. 4.1, Sect. 4.3) give
//   s = 1:  sin t W_l = -[sqrt(l/(l+1)) eps_(l+1) lambda_(l+1)
//                         - sqrt((l+1)/l) eps_l lambda_(l-1)],
//           sin t X_l = m / sqrt(L) lambda_l,
//   s = 2:  sin^2 t W_l = g eps_(l+1) eps_(l+2) lambda_(l+2)
//                         + 2 sqrt((L-2)/L) (3 m^2 - L) / (4 L - 3) lambda_l
//                         + (1/g) eps_l eps_(l-1) lambda_(l-2),
//           g = sqrt(l (l-1) / ((l+1) (l+2))),
//           sin^2 t X_l = -2 m [sqrt((l-1)/(l (l+1) (l+2))) eps_(l+1) lambda_(l+1)
//                               - sqrt((l+2)/((l-1) l (l+1))) eps_l lambda_(l-1)].
// So Q_m = -(sum E W + i sum B X) and U_m = -(sum B W - i sum E X) are, times
// sin^s t, spin-0 sums over l = m .. lmax + s with banded coefficients: half the
// products and a quarter of the recursion work of the two spin chains.  The
// division by sin^s t costs precision towards the poles, so the slots there
// keep the spin kernels.  The analysis is the transpose: spin-0 sums of Q and U
// over sin^s t, then the same band from lmax + s degrees back to lmax.
//
// The band kernels move the coefficients once each way (HBM bound: at sixteen
// spin-2 transforms of lmax 4095, 8.6 GB); the factors come from a per-degree
// table and four square roots of exact integers per (m, l), shared by the
// transforms of a plan.
#include <hip/hip_runtime.h>

#include <cmath>
#include <vector>

#include "sht_internal.h"

namespace sht {

// Factors of degree l (0 below the spin, and above lmax: those degrees hold no
// coefficient): r = 1/sqrt(4 l^2 - 1) for every l; up, dn: -W onto l + s, l - s;
// mid: -W (spin 2, times 3 m^2 - L) or X (spin 1, times m) onto l; xu, xd: X
// (spin 2) onto l + 1, l - 1; L = l (l + 1); d = sqrt(L) (derivative maps)
struct BandL {
    double r, up, dn, mid, xu, xd, L, d;
};

int band_upload(Plan &p)
{
    const int s = p.spin, n = p.lmax + 2 * s + 3;
    std::vector<BandL> t(n);
    for (int i = 0; i < n; ++i) {
        const long double l = i, L = l * (l + 1.0L);
        BandL b{};
        b.r = i > 0 ? (double)(1.0L / sqrtl(4.0L * l * l - 1.0L)) : 0.0;
        b.L = (double)L;
        if (i >= s && i <= p.lmax) {
            b.d = (double)sqrtl(L);
            if (s == 1) {
                b.up = (double)sqrtl(l / (l + 1.0L));
                b.dn = (double)(-sqrtl((l + 1.0L) / l));
                b.mid = (double)(1.0L / sqrtl(L));
            } else {
                const long double g = sqrtl(l * (l - 1.0L) / ((l + 1.0L) * (l + 2.0L)));
                b.up = (double)(-g);
                b.dn = (double)(-1.0L / g);
                b.mid = (double)(-2.0L * sqrtl((L - 2.0L) / L) / (4.0L * L - 3.0L));
                b.xu = (double)(-2.0L * sqrtl((l - 1.0L) / (l * (l + 1.0L) * (l + 2.0L))));
                b.xd = (double)(2.0L * sqrtl((l + 2.0L) / ((l - 1.0L) * l * (l + 1.0L))));
            }
        }
        t[i] = b;
    }
    int rc;
    if ((rc = dev_alloc((void **)&p.d_band, t.size() * sizeof(BandL), "band factors"))) return rc;
    return dev_upload(p.d_band, t.data(), t.size() * sizeof(BandL), "upload");
}

// sqrt(l^2 - m^2) r_l, 0 at l <= m
__device__ __forceinline__ double band_eps(const BandL *__restrict__ b, int l, int m)
{
    return l > m ? sqrt((double)(l - m) * (double)(l + m)) * b[l].r : 0.0;
}

// The five weights that take the coefficients of degrees l - 2 .. l + 2 to the
// scalar coefficient of degree l (FORWARD), or the scalar sums of degrees l - 2
// .. l + 2 to degree l (transpose): c[0..4] for degree offsets -2 .. 2, -W at
// offsets of the spin's parity, X at the others.
template <int S, bool FORWARD>
__device__ __forceinline__ void band_weights(const BandL *__restrict__ b, int l, int m, double (&c)[5])
{
    const double mm = (double)m;
    if (S == 1) {
        const double e0 = band_eps(b, l, m), e1 = band_eps(b, l + 1, m);
        c[0] = c[4] = 0.0;
        if (FORWARD) {
            c[1] = l > m ? b[l - 1].up * e0 : 0.0;
            c[3] = b[l + 1].dn * e1;
        } else {
            c[1] = b[l].dn * e0;
            c[3] = b[l].up * e1;
        }
        c[2] = b[l].mid * mm;
    } else {
        const double em = band_eps(b, l - 1, m), e0 = band_eps(b, l, m), e1 = band_eps(b, l + 1, m),
                     e2 = band_eps(b, l + 2, m);
        if (FORWARD) {
            c[0] = l > m + 1 ? b[l - 2].up * (em * e0) : 0.0;
            c[1] = l > m ? b[l - 1].xu * mm * e0 : 0.0;
            c[3] = b[l + 1].xd * mm * e1;
            c[4] = b[l + 2].dn * (e1 * e2);
        } else {
            c[0] = b[l].dn * (em * e0);
            c[1] = b[l].xd * mm * e0;
            c[3] = b[l].xu * mm * e1;
            c[4] = b[l].up * (e1 * e2);
        }
        c[2] = b[l].mid * (3.0 * mm * mm - b[l].L);
    }
}

// values a, x at the five degree offsets -> -(W a + i X x), the first component
// of either direction, or (SECOND) -(W a - i X x), the second (c: -W and X).  m = 0: X
// is 0 and the imaginary parts are never used; 0 x takes an Inf or NaN of x along.
template <int S, bool SECOND>
__device__ __forceinline__ double2 band_apply(const double (&c)[5], const double2 (&a)[5], const double2 (&x)[5], int m)
{
    double2 o = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if (S == 1 && (i == 0 || i == 4)) continue;
        const bool w = S == 1 ? (i != 2) : !(i & 1);
        if (w) {
            o.x = fma(c[i], a[i].x, o.x);
            o.y = fma(c[i], a[i].y, o.y);
        } else {
            o.x = fma(SECOND ? -c[i] : c[i], m ? x[i].y : x[i].x, o.x);
            o.y = fma(SECOND ? c[i] : -c[i], x[i].x, o.y);
        }
    }
    return o;
}

// alm [ntrans][ncin][nalm] -> q [ntrans][2][nalm_q] (band limit lmax + S): one
// thread per (m, l), looping over the transforms.  Degrees below the spin and
// Im a_l0 are never used; the derivative synthesis (S = 1, ncin = 1) takes
// E = sqrt(l (l + 1)) a_lm, B = 0.
template <int S>
__global__ __launch_bounds__(256) void k_band_synth(const double2 *__restrict__ alm, double2 *__restrict__ q,
                                                    const BandL *__restrict__ b, int lmax, int64_t nalm,
                                                    int64_t nalm_q, int ntrans, int deriv)
{
    const int m = blockIdx.y;
    const int l = m + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (l > lmax + S) return;
    const int64_t src = (int64_t)m * (2 * (int64_t)lmax + 1 - m) / 2;
    const int64_t dst = (int64_t)m * (2 * (int64_t)(lmax + S) + 1 - m) / 2 + l;
    const int l0 = m > S ? m : S;
    double c[5];
    band_weights<S, true>(b, l, m, c);
    bool ok[5];
    int64_t at[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int k = l + i - 2;
        ok[i] = k >= l0 && k <= lmax;
        at[i] = src + (ok[i] ? k : l0);
        if (S == 1 && deriv && ok[i]) c[i] *= b[k].d;
    }
    const int ncin = deriv ? 1 : 2;
    for (int t = 0; t < ntrans; ++t) {
        const double2 *pe = alm + (int64_t)t * ncin * nalm, *pb = pe + nalm;
        double2 e[5], bb[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (S == 1 && (i == 0 || i == 4)) continue;
            const double2 ev = pe[at[i]];
            const double2 bv = deriv ? make_double2(0.0, 0.0) : pb[at[i]];
            e[i] = ok[i] ? make_double2(ev.x, m ? ev.y : 0.0) : make_double2(0.0, 0.0);
            bb[i] = ok[i] ? make_double2(bv.x, m ? bv.y : 0.0) : make_double2(0.0, 0.0);
        }
        q[(int64_t)t * 2 * nalm_q + dst] = band_apply<S, false>(c, e, bb, m);
        q[((int64_t)t * 2 + 1) * nalm_q + dst] = band_apply<S, true>(c, bb, e, m);
    }
}

// Scalar sums q [ntrans][2][nalm_q] -> alm [ntrans][ncout][nalm]: the transpose,
// times fac_m (gradient) and, for the adjoint of the derivative synthesis,
// sqrt(l (l + 1)) and E alone; added to what the spin kernels stored for m <=
// mown, stored elsewhere (degrees below the spin and Im a_l0: zero).
template <int S>
__global__ __launch_bounds__(256) void k_band_anal(const double2 *__restrict__ q, double2 *__restrict__ alm,
                                                   const BandL *__restrict__ b, int lmax, int64_t nalm,
                                                   int64_t nalm_q, int ntrans, int mode, int mown)
{
    const int m = blockIdx.y;
    const int l = m + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (l > lmax) return;
    const int64_t dst = (int64_t)m * (2 * (int64_t)lmax + 1 - m) / 2 + l;
    const int64_t src = (int64_t)m * (2 * (int64_t)(lmax + S) + 1 - m) / 2;
    const bool deriv = mode & ANA_MODE_DERIV, add = m <= mown;
    const int ncout = deriv ? 1 : 2;
    if (l < S) {
        if (!add)
            for (int r = 0; r < ntrans * ncout; ++r) alm[(int64_t)r * nalm + dst] = make_double2(0.0, 0.0);
        return;
    }
    double c[5];
    band_weights<S, false>(b, l, m, c);
    const double f = ((mode & ANA_MODE_GRAD) && m > 0 ? 2.0 : 1.0) * (deriv ? b[l].d : 1.0);
    bool ok[5];
    int64_t at[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int k = l + i - 2;
        ok[i] = k >= m;   // k <= lmax + S by the range of l
        at[i] = src + (ok[i] ? k : m);
        c[i] *= f;
    }
    for (int t = 0; t < ntrans; ++t) {
        const double2 *pq = q + (int64_t)t * 2 * nalm_q, *pu = pq + nalm_q;
        double2 sq[5], su[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (i < 2 - S || i > 2 + S) continue;
            const double2 qv = pq[at[i]], uv = pu[at[i]];
            sq[i] = ok[i] ? qv : make_double2(0.0, 0.0);
            su[i] = ok[i] ? uv : make_double2(0.0, 0.0);
        }
        double2 *oe = alm + (int64_t)t * ncout * nalm + dst;
        double2 v = band_apply<S, false>(c, sq, su, m);
        if (m == 0) v.y = 0.0;
        if (add) v = make_double2(oe->x + v.x, oe->y + v.y);
        *oe = v;
        if (deriv) continue;
        oe += nalm;
        v = band_apply<S, true>(c, su, sq, m);
        if (m == 0) v.y = 0.0;
        if (add) v = make_double2(oe->x + v.x, oe->y + v.y);
        *oe = v;
    }
}

int launch_band_synth(const Plan &p, const double *alm, double *q, bool deriv, hipStream_t s)
{
    const dim3 grid((unsigned)((p.lmax + p.spin + 1 + 255) / 256), (unsigned)(p.mmax + 1));
    const double2 *a = reinterpret_cast<const double2 *>(alm);
    double2 *o = reinterpret_cast<double2 *>(q);
    if (p.spin == 1)
        hipLaunchKernelGGL(k_band_synth<1>, grid, dim3(256), 0, s, a, o, p.d_band, p.lmax, p.nalm, p.eq->nalm,
                           p.ntrans, deriv ? 1 : 0);
    else
        hipLaunchKernelGGL(k_band_synth<2>, grid, dim3(256), 0, s, a, o, p.d_band, p.lmax, p.nalm, p.eq->nalm,
                           p.ntrans, 0);
    return check_hip(hipGetLastError(), "band synthesis launch");
}

int launch_band_anal(const Plan &p, const double *q, double *alm, int mode, hipStream_t s)
{
    const dim3 grid((unsigned)((p.lmax + 1 + 255) / 256), (unsigned)(p.mmax + 1));
    const double2 *a = reinterpret_cast<const double2 *>(q);
    double2 *o = reinterpret_cast<double2 *>(alm);
    if (p.spin == 1)
        hipLaunchKernelGGL(k_band_anal<1>, grid, dim3(256), 0, s, a, o, p.d_band, p.lmax, p.nalm, p.eq->nalm,
                           p.ntrans, mode, p.own_mlim);
    else
        hipLaunchKernelGGL(k_band_anal<2>, grid, dim3(256), 0, s, a, o, p.d_band, p.lmax, p.nalm, p.eq->nalm,
                           p.ntrans, mode, p.own_mlim);
    return check_hip(hipGetLastError(), "band analysis launch");
}

}  // namespace sht
