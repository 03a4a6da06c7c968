// Spin synthesis on the matrix cores (Eqs. 4, 5), FP64 and FP32 products.
#include <hip/hip_runtime.h>

#include "legendre_dev.h"
#include "sht_internal.h"

namespace sht {

// Work group = (m, 32 NW slots from tile it.tile, 16 NCB columns (4 NCB transforms)
// from it.t0); wavefront w takes slots 32 w .. and all columns.
//
// Recursion: lane = chain * 32 + slot (chain 0 = +s, 1 = -s); each chunk of 16
// degrees of mu_l goes to the wavefront's own LDS rows.  Products (Eq. 4) on 16x16x4
// matrix-core tiles, rows = 16 slots, columns (transform, Q_re, Q_im, U_re, U_im), k =
// 4 degrees of one parity class: A rows W = -(lambda_+ + lambda_-)/2 and X =
// (lambda_+ - lambda_-)/2, B_W[o] = (E_re, E_im, B_re, B_im)[o], B_X[o] = s_o
// B_W[3 - o], s = (+, -, -, +).  The group stages c f_l a_lm (c = 1/2) in LDS once for
// its wavefronts, times tau_o = (+, +, -, +): tau_o tau_(3-o) = s_o, so X reads column
// 3 - o of the same rows and the sums hold tau_o times the result.  Class 0 collects
// the terms whose mirror-ring sign is +1 (W at l + m even, X at l + m odd), class 1
// the others; ring t gets A0 + A1, ring pi - t gets A0 - A1.
//
// What bounds it: where few wavefronts are in flight, the latency of a chunk (the
// recursion's coefficients, read from LDS two steps ahead; its vector instructions,
// which wait for another wavefront's matrix instruction each and run at raised
// priority); else the matrix cores and, with FP32 products, the vector instructions
// per product.  The kernel of one wavefront per group with its operands in registers
// (loads, scaling, conversion and lane exchange per wavefront; coefficients read where
// they are used) has 7 of them per product, this one 4.5.  Chunks whose lambda
// underflow take no products.  Sixteen spin-2 transforms at lmax 2047, FP32 products:
// 8.2 -> 6.7 ms; four spin-3 transforms at lmax 511: 122 -> 92 us.
constexpr int SS_LC = 16;
constexpr int SS_LROW = 64 + 8;   // one degree, 64 chains (rows two apart share no bank)

template <int NCB, bool F32, int NW>
struct SynSpinShared {
    using T = typename MT<F32>::T;
    static constexpr int BROW = NCB * 16 + 8;
    T lam[NW][SS_LC][SS_LROW];
    T b[2][SS_LC][BROW];
    double4 cf[2][2][SS_LC];   // per chain: alpha, +-beta, alpha +- beta - 2, alpha
    int bad;                   // a coefficient of this item is Inf or NaN: no chunk is left out
};

template <int NCB, bool F32, int NW>
__device__ __forceinline__ void synth_spin_item(const LegView &v, const WaveItem it, const double *__restrict__ alm,
                                                double *__restrict__ phase, int flush_chunks, int deriv,
                                                SynSpinShared<NCB, F32, NW> &sh)
{
    using T = typename MT<F32>::T;
    using V = typename MT<F32>::V;
    constexpr int LC = SS_LC, NT = 64 * NW;
    constexpr int NST = (LC * 8 * NCB + NT - 1) / NT;   // staged (re, im) pairs per thread
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i16 = lane & 15, kk = lane >> 4;
    if (it.m < 0) return;
    const int m = it.m, lmax = v.lmax;
    const int l0 = v.spin > m ? v.spin : m;
    const double ssign = (v.spin & 1) ? -1.0 : 1.0;   // sigma = (-1)^s of the mirror ring
    const int lstart = l0 - ((l0 + m) & 1);
    const double4 *coef = v.coef + v.coef_ofs[m];
    const double *flm = v.fl + v.coef_ofs[m];
    const int64_t mbase = (int64_t)m * (2 * (int64_t)lmax + 1 - m) / 2;
    const double thr = ldexp(1.0, v.thresh_bits), down = ldexp(1.0, -v.rescale_bits);
    const int tile = it.tile + wave;
    const bool act = tile < v.ntiles && v.tile_mlim[tile < v.ntiles ? tile : 0] >= m;

    Chain cs = chain_init(v, m, act ? tile * 32 + (lane & 31) : v.nslots, lane >> 5);
    const bool diff = wave_any(cs.x > DIFF_FORM_COS);
    if (diff) cs.aux = cs.mu;
    bool slow = wave_any(cs.k < 0);
    const bool live = wave_any(cs.mu != 0.0);

    // staging: thread -> degree tid % 16 of (transform, component) tid / 16 + (NT / 16) i.
    // Derivative synthesis (spin-1 plan): one input component per transform, taken as E
    // with B = 0, and f_l carries sqrt(l (l + 1)).
    const int sdeg = tid & 15, stc = tid >> 4;
    const int ncin = deriv ? 1 : 2;
    const double2 *src = reinterpret_cast<const double2 *>(alm) + mbase;
    double2 nb[NST];
    double nf = 0.0;
    double4 nq = double4{0, 0, 0, 0};
    auto fetch = [&](int lc) {
        const int l = lc + sdeg, lcl = l < l0 ? l0 : (l > lmax ? lmax : l);   // clamped address, masked when staged
        nf = flm[lcl] * 0.5 * (deriv ? v.dfac[lcl] : 1.0);
        if (tid < 2 * LC) nq = coef[lcl];
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int tc = stc + NT / 16 * i, t = it.t0 + (tc >> 1), comp = tc & 1;
            nb[i] = src[(int64_t)(t < v.ntrans && comp < ncin ? t * ncin + comp : 0) * v.nalm + lcl];
        }
    };
    auto stage = [&](int buf, int lc) {
        const int l = lc + sdeg;
        if (tid < 2 * LC) {
            const bool minus = tid >= LC;
            sh.cf[buf][minus ? 1 : 0][sdeg] =
                l >= l0 && l < lmax ? double4{nq.x, minus ? -nq.y : nq.y, minus ? nq.w : nq.z, nq.x} : double4{0, 0, 0, 0};
        }
        bool bad = false;
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int tc = stc + NT / 16 * i, comp = tc & 1;
            const bool ok = l >= l0 && l <= lmax && it.t0 + (tc >> 1) < v.ntrans && comp < ncin;
            const T x = ok ? (T)(nb[i].x * (comp ? -nf : nf)) : (T)0, y = ok && m ? (T)(nb[i].y * nf) : (T)0;
            bad = bad || not_finite(x) || not_finite(y);
            if (NST * NT == LC * 8 * NCB || tc < 8 * NCB) {
                sh.b[buf][sdeg][2 * tc] = x;
                sh.b[buf][sdeg][2 * tc + 1] = y;
            }
        }
        if (bad) sh.bad = 1;
    };

    V acc[2][2][NCB];   // class, 16-slot block, column block
    double acc64[F32 ? 2 : 1][F32 ? 2 : 1][F32 ? NCB : 1][4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                acc[p][sb][cb] = V{0, 0, 0, 0};
                if constexpr (F32)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc64[p][sb][cb][r] = 0.0;
            }

    if (tid == 0) sh.bad = 0;
    fetch(lstart);
    __syncthreads();
    stage(0, lstart);
    __syncthreads();
    T *const lout = &sh.lam[wave][0][lane];
    int buf = 0, chunk = 0;
    for (int lc = lstart; lc <= lmax; lc += LC, buf ^= 1, ++chunk) {
        const bool more = lc + LC <= lmax;
        if (more) fetch(lc + LC);
        if (act) {
            __builtin_amdgcn_s_setprio(2);
            const double4 *cf = sh.cf[buf][lane >> 5];
            const bool before = lc < l0;
            bool now = live;
            if (slow || before) {
                if (diff) chain_run<LC, false, true, true>(cs, cf, before, thr, down, lout, SS_LROW);
                else chain_run<LC, false, false, true>(cs, cf, before, thr, down, lout, SS_LROW);
                slow = wave_any(cs.k < 0);
                now = wave_any(cs.k == 0 && (cs.mu != 0.0 || cs.aux != 0.0));
            } else if (diff) {
                chain_run<LC, false, true, false>(cs, cf, false, thr, down, lout, SS_LROW);
            } else {
                chain_run<LC, false, false, false>(cs, cf, false, thr, down, lout, SS_LROW);
            }
            now = now || sh.bad;
            __builtin_amdgcn_s_setprio(0);
            wave_sync();
            if (now)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int te = 8 * h + 2 * kk;
                    T bwe[NCB], bwo[NCB], bxe[NCB], bxo[NCB];
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        bwe[cb] = sh.b[buf][te][16 * cb + i16];
                        bwo[cb] = sh.b[buf][te + 1][16 * cb + i16];
                        bxe[cb] = sh.b[buf][te][16 * cb + (i16 ^ 3)];
                        bxo[cb] = sh.b[buf][te + 1][16 * cb + (i16 ^ 3)];
                    }
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb) {
                        const T *le = &sh.lam[wave][te][sb * 16 + i16], *lo = le + SS_LROW;
                        const T upe = le[0], ume = le[32], upo = lo[0], umo = lo[32];
                        const T awe = -(upe + ume), axe = upe - ume;
                        const T awo = -(upo + umo), axo = upo - umo;
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb) {
                            acc[0][sb][cb] = mfma(awe, bwe[cb], acc[0][sb][cb]);
                            acc[0][sb][cb] = mfma(axo, bxo[cb], acc[0][sb][cb]);
                            acc[1][sb][cb] = mfma(awo, bwo[cb], acc[1][sb][cb]);
                            acc[1][sb][cb] = mfma(axe, bxe[cb], acc[1][sb][cb]);
                        }
                    }
                }
            wave_sync();
            if constexpr (F32) {
                if ((chunk + 1) % flush_chunks == 0) {
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
                            for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) acc64[p][sb][cb][r] += (double)acc[p][sb][cb][r];
                                acc[p][sb][cb] = V{0, 0, 0, 0};
                            }
                }
            }
        }
        if (more) stage(buf ^ 1, lc + LC);
        __syncthreads();
    }

    // ring t = A0 + A1, ring pi - t = sigma (A0 - A1), both times tau_o
    if (!act) return;
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
        int yn[4], ys[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int slot = tile * 32 + sb * 16 + c_row<F32>(lane, r);   // inside the padded tables
            yn[r] = v.slot_yn[slot];
            ys[r] = v.slot_ys[slot];
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const int col = i16 + 16 * cb, t = it.t0 + col / 4, o = col % 4;
            if (t >= v.ntrans) continue;
            const double ts = o == 2 ? -1.0 : 1.0;
            double *dst = phase + ((((int64_t)t * 2 + (o >> 1)) * v.nrings) * (v.mmax + 1) + m) * 2 + (o & 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double c0, c1;
                if constexpr (F32) {
                    c0 = acc64[0][sb][cb][r] + (double)acc[0][sb][cb][r];
                    c1 = acc64[1][sb][cb][r] + (double)acc[1][sb][cb][r];
                } else {
                    c0 = acc[0][sb][cb][r];
                    c1 = acc[1][sb][cb][r];
                }
                if (yn[r] >= 0) dst[(int64_t)yn[r] * (v.mmax + 1) * 2] = ts * (c0 + c1);
                if (ys[r] >= 0) dst[(int64_t)ys[r] * (v.mmax + 1) * 2] = (ssign * ts) * (c0 - c1);
            }
        }
    }
}

template <int NCB, bool F32, int NW>
__global__ __launch_bounds__(64 * NW, NCB == 1 ? 4 : NW == 1 ? 2 : 3) void k_legendre_synth_spin(LegView v, const WaveItem *__restrict__ items,
                                                                   const double *__restrict__ alm,
                                                                   double *__restrict__ phase, int flush_chunks,
                                                                   int deriv)
{
    __shared__ SynSpinShared<NCB, F32, NW> sh;
    synth_spin_item<NCB, F32, NW>(v, items[blockIdx.x], alm, phase, flush_chunks, deriv, sh);
}

// ---------------------------------------------------------------- launchers

template <int NCB, bool F32, int NW>
static void launch_t(const Plan &p, const double *alm, double *phase, int deriv, hipStream_t s)
{
    hipLaunchKernelGGL((k_legendre_synth_spin<NCB, F32, NW>), dim3((unsigned)p.synth_items.size()), dim3(64 * NW), 0, s,
                       make_leg_view(p), p.d_synth_items, alm, phase, p.flush_chunks, deriv);
}

// Wavefronts (32 slots each) per work group; 0: the one-wavefront kernel, which
// keeps its operands in registers, is the better one.  Spin 3, 501, 801 and 1501 rings
// (8, 13, 24 tiles), us, that kernel / 1 / 2 / 4 wavefronts per group:
//   FP64, 4 transforms   118 / 93 / 92 / 90,  271 / 272 / 252 / 303,  1311 / 1457 / 1253 / 1312
//   FP64, 8 transforms   153 / 139 / 132 / 124,  368 / 418 / 408 / 454,  1981 / 2316 / 2118 / 1957
//   FP64, 16 transforms  220 / 238 / 224 / 232,  698 / 844 / 798 / 838
//   FP32, 8 transforms   119 / 117 / 103 / 95,  334 / 390 / 291 / 325,  1732 / 1867 / 1447 / 1427
// 32 FP64 columns leave three wavefronts per SIMD whatever the kernel, and from 4.5
// wavefronts per SIMD on (4600 in all) the barriers cost what the staging saves; groups
// of four lose to empty wavefronts where the tiles do not fill them.
int synth_spin_waves(const Plan &p)
{
    const bool f32 = p.precision == SHT_FP32_MFMA, wide = p.tune.synth_ncb == 2;
    if (!f32 && wide && (int64_t)(p.mmax + 1) * p.ntiles * ((p.ntrans + 7) / 8) > 4600) return 0;
    if (!f32 && !wide) return p.ntiles == 1 ? 1 : 2;
    if ((p.ntiles + 3) / 4 * 4 * 100 <= p.ntiles * 115) return 4;
    return f32 && p.ntiles > 1 ? 2 : 1;
}

int launch_legendre_synth_spin(const Plan &p, const double *alm, double *phase, int deriv, hipStream_t s)
{
    const bool wide = p.tune.synth_ncb == 2;
    const int nw = synth_spin_waves(p);
    if (p.precision == SHT_FP32_MFMA) {
        if (wide && nw == 4) launch_t<2, true, 4>(p, alm, phase, deriv, s);
        else if (wide && nw == 2) launch_t<2, true, 2>(p, alm, phase, deriv, s);
        else if (wide) launch_t<2, true, 1>(p, alm, phase, deriv, s);
        else if (nw == 4) launch_t<1, true, 4>(p, alm, phase, deriv, s);
        else if (nw == 2) launch_t<1, true, 2>(p, alm, phase, deriv, s);
        else launch_t<1, true, 1>(p, alm, phase, deriv, s);
    } else if (wide) {
        if (nw == 4) launch_t<2, false, 4>(p, alm, phase, deriv, s);
        else launch_t<2, false, 1>(p, alm, phase, deriv, s);
    } else {
        if (nw == 2) launch_t<1, false, 2>(p, alm, phase, deriv, s);
        else launch_t<1, false, 1>(p, alm, phase, deriv, s);
    }
    return check_hip(hipGetLastError(), "legendre synthesis launch");
}

}  // namespace sht
