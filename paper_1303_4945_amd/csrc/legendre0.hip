// Spin-0 Legendre step in FP64 on the matrix cores (Eqs. 4, 5): plans of several
// scalar transforms, and the scalar part of spin-1 and spin-2 plans.
//
// lambda_lm runs by the two-step recursion inside each parity class of l + m,
//   mu_{l+2} = t_l mu_l - mu_{l-2},   lambda_l = f_l mu_l,
// so a wavefront covers 32 ring-pair slots with its 64 lanes: lane = class * 32 +
// slot.  Always in difference form, where t is near 2 (poles) or near -2
// (equator) and the small part is known to full relative precision:
//   cos^2 t > 1/2:  d_{l+2} = (t_l - 2) mu_l + d_l,  mu_{l+2} = mu_l + d_{l+2},
//                   t_l - 2 = (a_l + b_l - 2) - a_l sin^2 t;
//   else the same for (-1)^k mu (k the step), with -(t_l + 2) = -(b_l + 2) - a_l cos^2 t.
// Each lane takes the form of its own slot: about the pole a colatitude is held to
// 2^-54 tan t, which next to the equator has no bound.  (Wavefronts of one form by any
// slot's cos^2 t > 1/2, GL rings at lmax 63, where one wavefront has them all: relative
// error 2.0e-15 against 0.7e-15, 1.2e-14 at the ring next to the equator.)
// Extended exponent as in the other kernels (a lane contributes while its scale
// is 0); a chunk of degrees in which no lane of a wavefront has reached scale 0
// takes no products (5% of the chunks at lmax 777, 12% at 4095).
//
// What bounds both kernels: the matrix cores.  v_mfma_f64_16x16x4f64 issues every
// 68 cycles of a SIMD, 68 TFLOP/s over the device at the 2.27 GHz it runs at, and
// FP64 vector instructions take their 4 cycles beside it, not under it.  So the
// shape keeps the recursion small against the products (32 columns per wavefront:
// 96 of 1120 cycles per 16 degrees), and the registers at 128 for four wavefronts
// per SIMD, whose recursion, LDS and load latencies hide under each other's
// products.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "legendre_dev.h"
#include "sht_internal.h"

namespace sht {

// f(std::integral_constant 0), f(1), .. f(N - 1)
template <int N, int I = 0, typename F>
__device__ __forceinline__ void for_each_of(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        for_each_of<N, I + 1>(f);
    }
}

struct Chain2 {
    double w;    // sin^2 t (pole form) or -cos^2 t (equator form): the sign bit tells the form
    double mu;   // mu_l (equator form: times (-1)^k)
    double d;    // difference
    int k;       // scale index (value = mu 2^(S k)), k <= 0
    __device__ bool eq() const { return __double2hiint(w) < 0; }
};

__device__ __forceinline__ Chain2 chain2_init(const LegView &v, int m, int slot, int par, double thr, double down)
{
    const Chain c = chain_init(v, m, slot, 0);
    const bool eq = !(c.x * c.x > 0.5);
    Chain2 r;
    r.w = slot < v.nslots ? (eq ? -v.slot_c2[slot] : v.slot_s2[slot]) : -0.0;
    r.k = c.k;
    // lambda_{m+1} = sqrt(2 m + 3) cos t lambda_m
    r.mu = par ? c.mu * (c.x * sqrt((double)(2 * m + 3))) : c.mu;
    if (r.k < 0 && fabs(r.mu) >= thr) {
        r.mu *= down;
        r.k += 1;
    }
    r.d = r.mu;
    return r;
}

// Step j of a chunk (an even number of steps, from an even step of the chain) with
// the step coefficients q of the lane's form: returns mu_l (0 while the scale is below
// 0, SLOW) and moves on by two degrees.
template <bool SLOW>
__device__ __forceinline__ double chain2_step(Chain2 &c, const double2 q, int j, double thr, double down)
{
    const double eps = fma(-q.x, fabs(c.w), q.y);
    double out = SLOW ? (c.k == 0 ? c.mu : 0.0) : c.mu;
    if (j & 1)   // (by integer instructions, which run beside matrix instructions)
        out = __hiloint2double(__double2hiint(out) ^ (__double2hiint(c.w) & (int)0x80000000), __double2loint(out));
    c.d = fma(eps, c.mu, c.d);
    c.mu += c.d;
    if (SLOW) {
        const bool up = c.k < 0 && fabs(c.mu) >= thr;
        c.mu = up ? c.mu * down : c.mu;
        c.d = up ? c.d * down : c.d;
        c.k += up ? 1 : 0;
    }
    return out;
}

// NS steps (a chunk) into out[j stride]; cf: staged (a, a + b - 2, a, -(b + 2)) of the
// chunk's degrees, this class's at 2 j, of which a lane reads its form's pair.  The
// coefficients of NB steps are read together, one batch ahead of the steps that use
// them: read where they are used, every step would wait for the LDS (130 cycles against
// the 24 of its arithmetic).
template <int NS, int NB, bool SLOW>
__device__ __forceinline__ void chain2_run(Chain2 &c, const double4 *cf, double thr, double down, double *out,
                                           int stride)
{
    const double *q0 = reinterpret_cast<const double *>(cf) + (c.eq() ? 2 : 0);
    double2 q[2][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) q[0][i] = *reinterpret_cast<const double2 *>(q0 + 8 * i);
#pragma unroll
    for (int b = 0; b < NS / NB; ++b) {
        if (b + 1 < NS / NB)
#pragma unroll
            for (int i = 0; i < NB; ++i) q[(b + 1) & 1][i] = *reinterpret_cast<const double2 *>(q0 + 8 * ((b + 1) * NB + i));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int j = b * NB + i;
            out[j * stride] = chain2_step<SLOW>(c, q[b & 1][i], j, thr, down);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// (the masks by a branch that every lane takes alike)
template <int NS, int NB>
__device__ __forceinline__ void chain2_chunk(Chain2 &c, bool slow, const double4 *cf, double thr, double down,
                                             double *out, int stride)
{
    if (slow) chain2_run<NS, NB, true>(c, cf, thr, down, out, stride);
    else chain2_run<NS, NB, false>(c, cf, thr, down, out, stride);
}

// After a chunk: whether any lane contributed (or may have); live: some lane's
// chain is not zero throughout.
__device__ __forceinline__ bool chain2_done(const Chain2 &c, bool live, bool &slow)
{
    if (!slow) return live;
    slow = wave_any(c.k < 0);
    return wave_any(c.k == 0 && (c.mu != 0.0 || c.d != 0.0));   // (mu can be 0 between two degrees that are not)
}

__device__ __forceinline__ double4 chain2_coef(const double4 q) { return double4{q.x, q.y, q.x, q.z}; }

// ---------------------------------------------------------------- synthesis
//
// Work group = (m, 32 NW slots from tile it.tile, 16 NCB columns (8 NCB
// transforms) from it.t0); wavefront w takes slots 32 w .. and all columns.  Per
// chunk of 16 degrees the group stages f_l a_lm in LDS once for its wavefronts
// (loaded a chunk ahead, double-buffered, one barrier per chunk); each wavefront
// runs its recursion into its own LDS rows, then multiplies: A = lambda (16 slots x
// 4 degrees of one class), B = the staged coefficients.  Measured, sixteen spin-2
// transforms at lmax 4095 (32 scalar ones, 88% of the slots): 44.7 ms in the
// one-step kernel of 64 slots x 16 columns, 31.5 here; recursion of chunk c + 1
// interleaved with the products of chunk c and half the wavefronts per SIMD 32.5; 64
// columns per wavefront 32.1.  (In the whole transform, 86% of the slots: 33.7 ms, matrix
// cores busy 0.58 of the cycles; 0.44 with one column block.)  The recursion's few instructions run at raised
// priority: beside another wavefront's matrix instructions each of them waits for
// one to end (72 cycles; 137 at equal priority).
constexpr int S0_LC = 16;
constexpr int S0_LROW = 40;   // row of lambda: 32 slots + 8 (two rows two apart share no bank)

template <int NCB, int NW>
struct Syn0Shared {
    static constexpr int BROW = NCB * 16 + 8;
    double lam[NW][S0_LC][S0_LROW];
    double b[2][S0_LC][BROW];
    double4 cf[2][S0_LC];
    int bad;   // a coefficient of this item is Inf or NaN: no chunk is left out
};

template <int NCB, int NW>
__device__ __forceinline__ void synth0_item(const LegView &v, const WaveItem it, const double *__restrict__ alm,
                                            double *__restrict__ phase, Syn0Shared<NCB, NW> &sh)
{
    constexpr int LC = S0_LC;
    constexpr int NT = 64 * NW;
    constexpr int NST = (LC * 8 * NCB + NT - 1) / NT;   // staged values per thread
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i16 = lane & 15, kk = lane >> 4;
    if (it.m < 0) return;
    const int m = it.m, lmax = v.lmax;
    const double4 *coef = v.coef2 + v.coef_ofs[m];
    const int64_t mbase = (int64_t)m * (2 * (int64_t)lmax + 1 - m) / 2;
    const double thr = ldexp(1.0, v.thresh_bits), down = ldexp(1.0, -v.rescale_bits);
    const int slot0 = it.tile * 64 + 32 * wave;
    const bool act = slot0 < v.nslots && v.tile_mlim[slot0 >> 6] >= m;

    Chain2 cs = chain2_init(v, m, act ? slot0 + (lane & 31) : v.nslots, lane >> 5, thr, down);
    bool slow = wave_any(cs.k < 0);
    const bool live = wave_any(cs.mu != 0.0);

    // staging: thread -> degree tid % 16 of transforms tid / 16 + (NT / 16) i
    const int sdeg = tid & 15, st = tid >> 4;
    const double2 *src = reinterpret_cast<const double2 *>(alm) + mbase;
    double2 nb[NST];
    double nf = 0.0;
    double4 nq = double4{0, 0, 0, 0};
    auto fetch = [&](int lc) {
        const int l = lc + sdeg, lcl = l > lmax ? lmax : l;   // clamped address, masked when staged
        nf = coef[lcl].w;
        if (tid < LC) nq = coef[lcl];
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int t = it.t0 + st + NT / 16 * i;
            nb[i] = src[(int64_t)(t < v.ntrans ? t : 0) * v.nalm + lcl];
        }
    };
    auto stage = [&](int buf, int lc) {
        const bool in = lc + sdeg <= lmax;
        if (tid < LC) sh.cf[buf][tid] = in ? chain2_coef(nq) : double4{0, 0, 0, 0};
        bool bad = false;
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int tl = st + NT / 16 * i;
            const bool ok = in && it.t0 + tl < v.ntrans;
            const double2 c = make_double2(ok ? nb[i].x * nf : 0.0, ok && m ? nb[i].y * nf : 0.0);
            bad = bad || not_finite(c.x) || not_finite(c.y);
            if (NST * NT == LC * 8 * NCB || tl < 8 * NCB) *reinterpret_cast<double2 *>(&sh.b[buf][sdeg][2 * tl]) = c;
        }
        if (bad) sh.bad = 1;
    };
    dv4 acc[2][2][NCB];   // class, 16-slot block, column block
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) acc[p][rb][cb] = dv4{0, 0, 0, 0};

    // operands and products of class p, degrees 8 h + 2 kk + p of the chunk in buf
    struct Ops {
        double a[2], b[NCB];
    };
    auto load = [&](int buf, int h, int p) {
        const int row = 8 * h + 2 * kk + p;
        Ops o;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) o.a[rb] = sh.lam[wave][row][rb * 16 + i16];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) o.b[cb] = sh.b[buf][row][cb * 16 + i16];
        return o;
    };
    auto product = [&](const Ops &o, int p) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) acc[p][rb][cb] = mfma(o.a[rb], o.b[cb], acc[p][rb][cb]);
    };
    if (tid == 0) sh.bad = 0;
    fetch(m);
    __syncthreads();
    stage(0, m);
    __syncthreads();
    double *const lout = &sh.lam[wave][lane >> 5][lane & 31];
    constexpr int LSTEP = 2 * S0_LROW;
    int buf = 0;
    for (int lc = m; lc <= lmax; lc += LC, buf ^= 1) {
        const bool more = lc + LC <= lmax;
        if (more) fetch(lc + LC);
        if (act) {
            __builtin_amdgcn_s_setprio(2);
            chain2_chunk<LC / 2, 2>(cs, slow, &sh.cf[buf][lane >> 5], thr, down, lout, LSTEP);
            const bool now = chain2_done(cs, live, slow) || sh.bad;
            __builtin_amdgcn_s_setprio(0);
            wave_sync();
            if (now) {
#pragma unroll 1   // (unrolled, the operands of both halves are kept at once and registers spill)
                for (int h = 0; h < 2; ++h) {
                    product(load(buf, h, 0), 0);
                    product(load(buf, h, 1), 1);
                }
            }
            wave_sync();
        }
        if (more) stage(buf ^ 1, lc + LC);
        __syncthreads();
    }

    // ring t = A0 + A1, ring pi - t = A0 - A1, times the slot's factor
    if (!act) return;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        int yn[4], ys[4];
        double sc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int slot = slot0 + rb * 16 + c_row<false>(lane, r);   // inside the padded tables
            yn[r] = v.slot_yn[slot];
            ys[r] = v.slot_ys[slot];
            sc[r] = v.slot_scale[slot];
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const int col = i16 + 16 * cb, t = it.t0 + (col >> 1);
            if (t >= v.ntrans) continue;
            double *dst = phase + (((int64_t)t * v.nrings) * (v.mmax + 1) + m) * 2 + (col & 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double c0 = acc[0][rb][cb][r], c1 = acc[1][rb][cb][r];
                if (yn[r] >= 0) dst[(int64_t)yn[r] * (v.mmax + 1) * 2] = sc[r] * (c0 + c1);
                if (ys[r] >= 0) dst[(int64_t)ys[r] * (v.mmax + 1) * 2] = sc[r] * (c0 - c1);
            }
        }
    }
}

template <int NCB, int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_legendre_synth0(LegView v, const WaveItem *__restrict__ items,
                                                               const double *__restrict__ alm,
                                                               double *__restrict__ phase)
{
    __shared__ Syn0Shared<NCB, NW> sh;
    synth0_item<NCB, NW>(v, items[blockIdx.x], alm, phase, sh);
}

// ---------------------------------------------------------------- analysis
//
// Work group = one m and 16 NCB columns; eight wavefronts walk the m's active
// slots 256 at a time (four 64-slot tiles, eight regions of 32).  lambda of a
// chunk of 32 degrees is held in LDS for all of them; wavefront w runs the
// recursion of region w and multiplies one 16-degree (class) x 16-column block of
// the outputs over its share of the slots: A = the stationary phases G_t +-
// G_(pi-t) of its class, in registers for the pass (64, 128 or 256 slots with 1, 2
// or 4 column blocks: 32, 64 or 128 VGPRs), B = lambda.  Recursion, products and
// output of a chunk follow each other between barriers, all wavefronts in step: the
// matrix instructions then meet no vector instructions of a neighbour (each waits
// for a matrix instruction to end).  The 64-slot partial sums are added in a fixed
// order, (P0 + P1) + (P2 + P3), so the result does not depend on NCB; a lane holds
// four columns of one degree, and each share adds the totals of its NCB of them,
// times f_l, to a_lm, whose earlier value it loads before the recursion (8
// transforms at lmax 4096 on HEALPix N_side 2048, NCB = 1: 27.5 ms with all of it in
// the first share and the load after the products, 24.9 so).  256 slots per pass keep the read-modify-write of
// a_lm at 1/16 of the bytes that 16 slots would take.  Measured, sixteen spin-2
// transforms at lmax 4095 (64 scalar columns): 42.2 ms in the one-step kernel of 64
// slots x 16 columns on the same slots, 39.2 here; a chunk takes 13.3-14.6k cycles, of
// which 8.8k are matrix instructions at their issue rate, 2.0-2.6k the recursion,
// 1.6k the sums into a_lm.  (In the whole transform: 43.4 ms, matrix cores busy 0.46 of
// the cycles, partly filled passes and the ends of the launch included; 0.41 with one
// column block.)  The recursion of chunk c + 1 interleaved with the
// products of chunk c (two buffers of lambda) was no faster, two groups of 32 columns
// 7% slower.
constexpr int A0_LC = 32;
constexpr int A0_NW = 8;

// Row of lambda (one degree, 32 slots).  A product reads 16 rows x 2 slots at a
// time: rows of 34 put them on different banks; with one column block the partial
// sums leave two groups of a CU room for 33 (two-way conflicts, beside the fewer
// products of that shape).
template <int NCB>
constexpr int a0_lrow() { return NCB == 1 ? 33 : 34; }

template <int NCB>
struct Ana0Shared {
    static constexpr int NR = NCB;                  // columns of a lane that its wavefront sums up and puts out
    union {
        double lam[8][A0_LC * a0_lrow<NCB>()];      // region: [class * 16 + degree / 2][slot]
        double g[2][128 * 16 * NCB];                // phases of a class on their way to the registers
    };
    double part[NCB == 4 ? 1 : A0_NW][4 - NR ? 4 - NR : 1][64];   // the others, on their way to the other shares
    double4 cf[A0_LC];
    double f[2][A0_LC];
    int on[8];                                      // the region's lambda is not all zero in the chunk
};

template <int NCB>
__device__ __forceinline__ void anal0_item(const LegView &v, const int m, const int t0,
                                           const double *__restrict__ phase, double *__restrict__ alm, int mode,
                                           Ana0Shared<NCB> &sh)
{
    constexpr int LC = A0_LC;
    constexpr int LROW = a0_lrow<NCB>();
    constexpr int NQ = NCB;                      // 64-slot tiles per wavefront
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i16 = lane & 15, kk = lane >> 4;
    const int par = wave & 1;                    // class of the wavefront's output block
    const int cb = (wave >> 1) & (NCB - 1);      // its column block
    const int share = (wave >> 1) / NCB;         // its tiles: share * NQ ..
    const int lmax = v.lmax;
    const double4 *coef = v.coef2 + v.coef_ofs[m];
    const int64_t mbase = (int64_t)m * (2 * (int64_t)lmax + 1 - m) / 2;
    const double thr = ldexp(1.0, v.thresh_bits), down = ldexp(1.0, -v.rescale_bits);
    const double fac = ((mode & ANA_MODE_GRAD) && m > 0) ? 2.0 : 1.0;   // fac_m of the real-field gradient
    const int rpar = lane >> 5, rslot = lane & 31;                      // recursion role

    // a lane's sums: columns 16 cb + kk + 4 r, r < 4 (transform t0 + 8 cb + kk / 2 + 2 r),
    // degree lc + par + 2 i16; this share puts out NR of them from r0 on
    constexpr int NR = Ana0Shared<NCB>::NR;
    const int r0 = share * NR, ot = t0 + 8 * cb + (kk >> 1) + 2 * r0;
    const int nout = (v.ntrans - ot + 1) / 2;               // r < nout: the transform exists
    double *const obase = alm + ((int64_t)(ot < v.ntrans ? ot : 0) * v.nalm + mbase) * 2 + (kk & 1);
    const int64_t ostride = 4 * v.nalm;
    const bool imz = m == 0 && (kk & 1);                    // Im a_l0

    int ntiles_act = 0;
    for (int t = 0; t < v.ntiles; ++t) ntiles_act += v.tile_mlim[t] >= m;
    int tcount = 0, tscan = 0;
    bool first = true;
    while (tcount < ntiles_act || first) {
        int tile[4];   // this pass's 64-slot tiles (-1: none)
        {
            int k = 0;
            tile[0] = tile[1] = tile[2] = tile[3] = -1;
            for (; tscan < v.ntiles && k < 4; ++tscan) {
                if (v.tile_mlim[tscan] < m) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k == i) tile[i] = tscan;
                ++k;
            }
            tcount += k;
        }
        auto tile_at = [&](int i) {   // i uniform
            return i == 0 ? tile[0] : i == 1 ? tile[1] : i == 2 ? tile[2] : tile[3];
        };
        const int rtile = tile_at(wave >> 1);      // this wavefront's recursion region
        const bool ract = rtile >= 0;
        Chain2 cs = chain2_init(v, m, ract ? rtile * 64 + 32 * (wave & 1) + rslot : v.nslots, rpar, thr, down);
        bool slow = wave_any(cs.k < 0);
        const bool live = wave_any(cs.mu != 0.0);

        // step coefficients and f_l of a chunk, staged by the first 32 threads
        double4 nq = double4{0, 0, 0, 0};
        auto fetch = [&](int lc) {
            if (tid < LC) nq = coef[lc + tid > lmax ? lmax : lc + tid];
        };
        auto stage = [&](int c, int lc) {
            if (tid < LC) {
                const bool in = lc + tid <= lmax;
                sh.cf[tid] = in ? chain2_coef(nq) : double4{0, 0, 0, 0};
                sh.f[c & 1][tid] = in ? nq.w * fac : 0.0;
            }
        };

        // stationary phases, 128 slots at a time.  Thread -> transform tid % (8 NCB)
        // and every (64 / NCB)th slot: both rings' (re, im) pairs are loaded at once,
        // combined, and handed through LDS to the wavefronts that hold them (missing
        // rings, slots and transforms: zero)
        double gw[NQ][16];
        bool nonfin = false;
#pragma unroll
        for (int rd = 0; rd < 2; ++rd) {
            constexpr int TPG = 8 * NCB, SPI = 64 * A0_NW / TPG, NI = 128 / SPI;
            const int tl = tid % TPG, t = t0 + tl;
            const bool tok = t < v.ntrans;
            const double2 *src =
                reinterpret_cast<const double2 *>(phase) + (((int64_t)(tok ? t : 0) * v.nrings) * (v.mmax + 1) + m);
            double2 gn[NI], gs[NI];
            double sc[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int s = 128 * rd + tid / TPG + SPI * i, gt = tile_at(s >> 6);
                const int slot = (gt >= 0 ? gt : 0) * 64 + (s & 63);   // inside the padded tables
                const bool ok = tok && gt >= 0 && slot < v.nslots;
                const int yn = ok ? v.slot_yn[slot] : -1, ys = ok ? v.slot_ys[slot] : -1;
                sc[i] = v.slot_scale[slot];
                gn[i] = src[(int64_t)(yn >= 0 ? yn : 0) * (v.mmax + 1)];
                gs[i] = src[(int64_t)(ys >= 0 ? ys : 0) * (v.mmax + 1)];
                if (yn < 0) gn[i] = make_double2(0.0, 0.0);
                if (ys < 0) gs[i] = make_double2(0.0, 0.0);
            }
            __syncthreads();   // the previous pass is done with lambda, the previous round with g
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int s = tid / TPG + SPI * i;
                double2 *d = reinterpret_cast<double2 *>(&sh.g[0][s * 16 * NCB + 2 * tl]);
                d[0] = make_double2(sc[i] * (gn[i].x + gs[i].x), sc[i] * (gn[i].y + gs[i].y));
                d[sizeof(sh.g[0]) / sizeof(double2)] = make_double2(sc[i] * (gn[i].x - gs[i].x), sc[i] * (gn[i].y - gs[i].y));
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if ((share * NQ + q) >> 1 != rd) continue;
#pragma unroll
                for (int ks = 0; ks < 16; ++ks) {
                    const double g = sh.g[par][(64 * ((share * NQ + q) & 1) + 4 * ks + kk) * 16 * NCB + 16 * cb + i16];
                    nonfin = nonfin || not_finite(g);
                    gw[q][ks] = g;
                }
            }
        }
        __syncthreads();
        const bool force = wave_any(nonfin);   // an Inf or NaN: no chunk is left out

        fetch(m);
        stage(0, m);
        __syncthreads();
        // products of half hf of tile q (this wavefront's)
        dv4 acc[NQ];
        auto product = [&](int q, int hf) {
            const int rg = 2 * (share * NQ + q) + hf;
            if (!__builtin_amdgcn_readfirstlane(sh.on[rg]) && !(force && tile_at(share * NQ + q) >= 0)) return;
            const double *lam = sh.lam[rg] + (par * 16 + i16) * LROW + kk;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) acc[q] = mfma(gw[q][8 * hf + ks], lam[4 * ks], acc[q]);
        };
        double *const lout = sh.lam[wave] + rpar * 16 * LROW + rslot;
        int c = 0;
        for (int lc = m; lc <= lmax; lc += LC, ++c) {
            fetch(lc + LC);
            // the earlier passes' sums: in flight during recursion and products
            const int ol = lc + par + 2 * i16;
            double *const o = obase + 2 * (int64_t)(ol > lmax ? lmax : ol);
            double prev[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) prev[r] = !first && r < nout ? o[r * ostride] : 0.0;
            if (ract) chain2_chunk<LC / 2, NCB == 4 ? 4 : 2>(cs, slow, &sh.cf[rpar], thr, down, lout, LROW);
            const bool any = ract && chain2_done(cs, live, slow);
            if (lane == 0) sh.on[wave] = any ? 1 : 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] = dv4{0, 0, 0, 0};
            for_each_of<2 * NQ>([&](auto g) { product(decltype(g)::value >> 1, decltype(g)::value & 1); });
            stage(c + 1, lc + LC);   // (every wavefront is done with chunk c's recursion)
            dv4 sum = acc[0];
            if constexpr (NQ >= 2) sum = acc[0] + acc[1];
            if constexpr (NQ == 4) sum = sum + (acc[2] + acc[3]);
            double mine[NR];   // sum[r0 + r]
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                mine[r] = sum[r];
#pragma unroll
                for (int h = 1; h < 4 / NR; ++h) mine[r] = share == h ? sum[h * NR + r] : mine[r];
            }
            if constexpr (NR < 4) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (r / NR != share) sh.part[wave][r < r0 ? r : r - NR][lane] = sum[r];
            }
            __syncthreads();
            if (ol <= lmax) {
                const double f = sh.f[c & 1][par + 2 * i16];
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    double s = mine[r];
                    if constexpr (NR < 4) {
                        double ps[4 / NR];
#pragma unroll
                        for (int h = 0; h < 4 / NR; ++h) {   // (its own place in part: not written, not used)
                            const double x = sh.part[par + 2 * (cb + NCB * h)][h < share ? r0 - NR + r : r0 % (4 - NR) + r][lane];
                            ps[h] = h == share ? mine[r] : x;
                        }
                        s = ps[0] + ps[1];
                        if constexpr (NR == 1) s += ps[2] + ps[3];
                    }
                    s = first ? f * s : fma(f, s, prev[r]);
                    if (imz) s = 0.0;
                    if (r < nout) o[r * ostride] = s;
                }
            }
        }
        first = false;
    }
}

template <int NCB>
__global__ __launch_bounds__(64 * A0_NW, NCB == 4 ? 2 : 4) void k_legendre_anal0(LegView v, const int *__restrict__ mlist,
                                                                 const double *__restrict__ phase,
                                                                 double *__restrict__ alm, int mode)
{
    __shared__ Ana0Shared<NCB> sh;
    anal0_item<NCB>(v, mlist[blockIdx.x], (int)blockIdx.y * 8 * NCB, phase, alm, mode, sh);
}

// ---------------------------------------------------------------- batches

// Persistent analysis over a batch's queue (atomic counter; every work group
// reaches the exit test, so the grid drains).
template <int NCB>
__global__ __launch_bounds__(64 * A0_NW, 4) void k_legendre_anal0_batch(const LegView *__restrict__ views,
                                                                       const BatchAnaItem *__restrict__ items,
                                                                       int nitems, BatchPtrs ptrs, int mode,
                                                                       unsigned *counter)
{
    __shared__ Ana0Shared<NCB> sh;
    __shared__ unsigned sidx;
    for (;;) {
        if (threadIdx.x == 0) sidx = atomicAdd(counter, 1u);
        __syncthreads();
        const unsigned idx = __builtin_amdgcn_readfirstlane(sidx);
        __syncthreads();
        if (idx >= (unsigned)nitems) break;
        const BatchAnaItem bi = items[idx];
        for (int k = 0; k < (bi.m2 >= 0 ? 2 : 1); ++k) {
            anal0_item<NCB>(views[bi.plan], k ? bi.m2 : bi.m, bi.t0, ptrs.in[bi.plan], ptrs.out[bi.plan], mode, sh);
            __syncthreads();
        }
    }
}

// Persistent synthesis: one queue segment per die, as the other kernels' (a work
// group drains its die's segment, then takes from the others).
template <int NCB>
__global__ __launch_bounds__(256, 4) void k_legendre_synth0_batch(const LegView *__restrict__ views,
                                                                 const BatchSynItem *__restrict__ items, SynQueues q,
                                                                 BatchPtrs ptrs, unsigned *counters)
{
    __shared__ Syn0Shared<NCB, 4> sh;
    __shared__ unsigned sidx;
    const int die = (int)(blockIdx.x % NUM_XCD);
    int k = 0;
    for (;;) {
        const int d = (die + k) % NUM_XCD;
        const unsigned n = (unsigned)(q.ofs[d + 1] - q.ofs[d]);
        if (threadIdx.x == 0) sidx = atomicAdd(counters + 16 * d, 1u);
        __syncthreads();
        const unsigned idx = __builtin_amdgcn_readfirstlane(sidx);
        __syncthreads();
        if (idx >= n) {
            if (++k == NUM_XCD) break;   // every segment empty
            continue;
        }
        const BatchSynItem bi = items[q.ofs[d] + idx];
        for (int i = 0; i < (bi.m2 >= 0 ? 2 : 1); ++i) {
            synth0_item<NCB, 4>(views[bi.plan], WaveItem{i ? bi.m2 : bi.m, bi.tile, bi.t0, 0}, ptrs.in[bi.plan],
                                ptrs.out[bi.plan], sh);
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------- launchers

// wavefronts (32 slots each) of a synthesis work group: as many as the plan's slots fill
int synth0_waves(const Plan &p) { return p.nslots <= 32 ? 1 : p.nslots <= 64 ? 2 : 4; }

template <int NCB>
static void launch_synth0_t(const Plan &p, const LegView &v, const double *alm, double *phase, hipStream_t s)
{
    const dim3 grid((unsigned)p.synth_items.size());
    switch (synth0_waves(p)) {
    case 1: hipLaunchKernelGGL((k_legendre_synth0<NCB, 1>), grid, dim3(64), 0, s, v, p.d_synth_items, alm, phase); break;
    case 2: hipLaunchKernelGGL((k_legendre_synth0<NCB, 2>), grid, dim3(128), 0, s, v, p.d_synth_items, alm, phase); break;
    default: hipLaunchKernelGGL((k_legendre_synth0<NCB, 4>), grid, dim3(256), 0, s, v, p.d_synth_items, alm, phase); break;
    }
}

int launch_legendre_synth0(const Plan &p, const double *alm, double *phase, hipStream_t s)
{
    const LegView v = make_leg_view(p);
    if (p.tune.synth_ncb == 2) launch_synth0_t<2>(p, v, alm, phase, s);
    else launch_synth0_t<1>(p, v, alm, phase, s);
    return check_hip(hipGetLastError(), "legendre synthesis launch");
}

// Column blocks.  A wider work group runs the recursion for more columns, a narrower
// one leaves fewer columns empty and fills the chip at smaller sizes; the results are
// the same bit for bit.  NCB = 1 where its work groups are fewer than five per CU;
// else the smallest product of groups and time per group, from the times at lmax 1500
// and 24, 32, 64 transforms: synthesis 1961, 2639, 5406 us with NCB = 1, 2027, 2125,
// 4310 with 2; analysis 2454, 3255, 6477 with 1, 2802, 3014, 5981 with 2, 2578, 2732,
// 5341 with 4.  32 transforms (64 columns) at lmax 200, 804 groups with NCB = 1:
// synthesis 28.1 / 28.6, analysis 45.5 / 55.0 / 48.0; at lmax 350, 1404 groups of the
// analysis: 99 / 95 / 86.
constexpr int NCB_GROUPS = 5 * 256;

static int blocks16(const Plan &p) { return (2 * p.ntrans + 15) / 16; }

int synth0_ncb(const Plan &p)
{
    const int n = blocks16(p);
    const int64_t groups = (int64_t)(p.mmax + 1) * ((p.nslots + 127) / 128) * n;
    return n == 1 || n == 3 || groups < NCB_GROUPS ? 1 : 2;   // 2 blocks together: 1.6 times one
}

// time of the analysis in groups of one block
static double anal0_cost(int n, int ncb) { return ((n + ncb - 1) / ncb) * (ncb == 4 ? 3.35 : ncb == 2 ? 1.85 : 1.0); }

static int anal0_ncb(const Plan &p)
{
    const int n = blocks16(p);
    if (p.tune.anal_ncb == 1 || (int64_t)(p.mmax + 1) * n < NCB_GROUPS) return 1;
    int best = 1;
    for (int ncb : {2, 4})
        if (anal0_cost(n, ncb) < anal0_cost(n, best)) best = ncb;
    return best;
}

int anal0_batch_ncb(const Batch &b)
{
    double c1 = 0.0, c2 = 0.0;
    int64_t groups = 0;
    for (const Plan *p : b.plans) {
        const double work = (double)p->nalm * p->nslots;
        c1 += work * anal0_cost(blocks16(*p), 1);
        c2 += work * anal0_cost(blocks16(*p), 2);
        groups += (int64_t)(p->mmax + 1) * blocks16(*p);
    }
    return groups < NCB_GROUPS || c1 <= c2 ? 1 : 2;
}

template <int NCB>
static void launch_anal0_t(const Plan &p, const LegView &v, const double *phase, double *alm, int mode, hipStream_t s)
{
    const dim3 grid((unsigned)p.anal_ms.size(), (unsigned)((p.ntrans + 8 * NCB - 1) / (8 * NCB)));
    hipLaunchKernelGGL(k_legendre_anal0<NCB>, grid, dim3(64 * A0_NW), 0, s, v, p.d_anal_ms, phase, alm, mode);
}

int launch_legendre_anal0(const Plan &p, const double *phase, double *alm, int mode, hipStream_t s)
{
    const LegView v = make_leg_view(p);
    const int ncb = anal0_ncb(p);
    log_msg(3, "two-step Legendre analysis plan %llu: %d column blocks", (unsigned long long)p.serial, ncb);
    switch (ncb) {
    case 4: launch_anal0_t<4>(p, v, phase, alm, mode, s); break;
    case 2: launch_anal0_t<2>(p, v, phase, alm, mode, s); break;
    default: launch_anal0_t<1>(p, v, phase, alm, mode, s); break;
    }
    return check_hip(hipGetLastError(), "legendre analysis launch");
}

int anal0_batch_groups(int ncb, int dev)
{
    return ncb == 2 ? persistent_groups(k_legendre_anal0_batch<2>, 64 * A0_NW, dev)
                    : persistent_groups(k_legendre_anal0_batch<1>, 64 * A0_NW, dev);
}

int synth0_batch_groups(int ncb, int dev)
{
    return ncb == 2 ? persistent_groups(k_legendre_synth0_batch<2>, 256, dev)
                    : persistent_groups(k_legendre_synth0_batch<1>, 256, dev);
}

// (the counters are reset by the caller)
void launch_anal0_batch(const Batch &b, const BatchPtrs &ptrs, int mode, hipStream_t s)
{
    const dim3 grid((unsigned)b.ana_groups), block(64 * A0_NW);
    if (b.ana_ncb == 2)
        hipLaunchKernelGGL(k_legendre_anal0_batch<2>, grid, block, 0, s, b.d_views, b.d_ana, b.nana, ptrs, mode,
                           b.d_counter);
    else
        hipLaunchKernelGGL(k_legendre_anal0_batch<1>, grid, block, 0, s, b.d_views, b.d_ana, b.nana, ptrs, mode,
                           b.d_counter);
}

void launch_synth0_batch(const Batch &b, const BatchPtrs &ptrs, const SynQueues &q, unsigned *counters, hipStream_t s)
{
    const dim3 grid((unsigned)b.syn_groups);
    if (b.syn_ncb == 2)
        hipLaunchKernelGGL(k_legendre_synth0_batch<2>, grid, dim3(256), 0, s, b.d_views, b.d_syn, q, ptrs, counters);
    else
        hipLaunchKernelGGL(k_legendre_synth0_batch<1>, grid, dim3(256), 0, s, b.d_views, b.d_syn, q, ptrs, counters);
}

}  // namespace sht
