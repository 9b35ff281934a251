// Legendre recurrence kernels of the general SHT on gfx950: the "synthesis" and
// "doubling" steps of Sect. 3 and their adjoints ("undoubling" and "adjoint
// synthesis"), FP64 throughout.
//
// For each m and each ring pair (theta_q, pi - theta_q) of the equidistant grid
// theta_q = pi q / (ntheta - 1), one lane runs the three-term recurrence in l of
// the spin-weighted harmonic, normalised as p_l = sY_lm / N_l so that
//     p_{l+1} = (a_l cos(theta) + sigma b_l) p_l - p_{l-1},
// for both channels sigma = +s (a) and sigma = -s (b).  The south ring reuses the
// north recurrence through sY_lm(pi - theta) = (-1)^(l+m) (-s)Y_lm(theta), and the
// column -m of a spin-s field through sY_{l,-m} = (-1)^(s+m) (-s)Y_lm.
//
// Start values at l0 = max(m, s) can lie far below the double range, and on each ring
// the values stay negligible until l sin(theta) comes near m.  A table holds, for every
// (m, ring pair), the first 8-degree block at whose start each channel has reached 2^-100
// and its two recurrence values there; the kernels start each wave at the first such block
// of its rings, keep a lane's values at 0 until its own block, and then simply set them.
// A channel just below 2^-100 at the start of a block is dropped up to its end, so the
// dropped terms reach 2^-77 at spins up to 10, 2^-64 at spin 100 and 2^-61 at any spin (the
// recurrence run over every accepted size), against values of order 1 in the oscillating
// region: 24 (8) bits below the rounding of the sums they would enter.  The stage entry
// points, whose callers see the rings and coefficients themselves, take 2^-900 (rings) and
// 2^-256 (adjoint) instead, so that small values come out right, too.
//
// Work decomposition: one wave per (m, chunk); a chunk is R slices of 64 consecutive
// ring pairs counted from the equator, lane L of slice r owning position 64 (R chunk +
// r) + L.  Degrees advance in blocks of 8 without masks or scaling, and only a final
// partial block checks the degree bound.
#include "legendre_device.hpp"

namespace gsht {

// ---- recurrence starts ----------------------------------------------------------------

// A channel enters at the first multiple of START_DEG degrees above l0 at which its
// value has reached 2^inx (gsht_plan::start_exp).  At lmax 4096 (spin 2) 77 % of the (m, l,
// ring) volume in waves of 128 rings lies past the entry at inx = -100; -256 would make it
// 81 %, -900 90 %, -64 76 %.

// true value = p 2^ex; ex == 0 <=> at least 2^inx, otherwise ex <= -512 is a multiple of
// 512.
__device__ inline void to_scaled(const XD &v, int inx, double &p, int &ex)
{
    if (v.m == 0.0) {
        p = 0.0;
        ex = -512;
    } else if (v.e >= inx + 1) {
        p = ldexp(v.m, v.e);
        ex = 0;
    } else {
        const int t = v.e + 256;
        ex = t < 0 ? 512 * (-((-t + 511) / 512)) : -512;
        p = ldexp(v.m, v.e - ex);
    }
}

// Fold to ex = 0 once |p| 2^ex >= 2^inx; step the offset when |p| has grown past 2^256.
// START_DEG degrees multiply |p| by at most 2^37 at lmax 1000, 2^45 at 4096 and 2^57 at
// 32766 for small spins, and by 2^109 at spin 20000; a block starts with |p| < 2^(inx + 512)
// at ex = -512 and with |p| < 2^256 at smaller ex, so |p| stays below 2^(412 + 109).
__device__ inline void rescale_channel(double &p0, double &p1, int &ex, int inx)
{
    if (ex == 0)
        return;
    if (fabs(p1) >= ldexp(1.0, ex < -1024 ? 1023 : inx - ex)) {
        p0 = ldexp(p0, ex);
        p1 = ldexp(p1, ex);
        ex = 0;
    } else if (ex < -512 && fabs(p1) >= 0x1p256) {
        p0 *= 0x1p-512;
        p1 *= 0x1p-512;
        ex += 512;
    }
}

// One lane per (m, ring pair), the pair's position counted from the equator.  Runs the
// recurrence with exponent offsets through the degrees where the values are negligible;
// done once per plan (or in each Legendre launch), 2 ms at lmax 4096.
template <bool SPIN>
__global__ __launch_bounds__(64) void leg_starts_kernel(
    const double *__restrict__ ab, const StartInfo *__restrict__ st, int lmax, int inx, int m0,
    int ntheta, int npairs, int np, double2 *__restrict__ sta, double2 *__restrict__ stb,
    int32_t *__restrict__ stk)
{
    const int m = m0 + blockIdx.y, e = blockIdx.x * 64 + threadIdx.x;
    const StartInfo si = st[m];
    const int l0 = si.l0;
    const bool valid = e < npairs && l0 <= lmax;
    double x, sh, ch;
    ring_geom(valid ? npairs - 1 - e : 0, ntheta, x, sh, ch);
    double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;
    int ea = -512, eb = -512;
    if (valid) {
        to_scaled(start_value(si.mant_p, si.ex_p, si.a_p, si.b_p, sh, ch), inx, a1, ea);
        if (SPIN)
            to_scaled(start_value(si.mant_m, si.ex_m, si.a_m, si.b_m, sh, ch), inx, b1, eb);
    }
    const size_t idx = (size_t)blockIdx.y * np + e;
    int ka = START_NEVER, kb = START_NEVER;
    double2 va = make_double2(0.0, 0.0), vb = va;
    bool wa = valid && a1 != 0.0, wb = SPIN && valid && b1 != 0.0;  // still waiting
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    for (int lb = l0, k = 0; lb <= lmax; lb += START_DEG, ++k) {
        if (wa && ea == 0) {
            va = make_double2(a0, a1);
            ka = k;
            wa = false;
        }
        if (SPIN && wb && eb == 0) {
            vb = make_double2(b0, b1);
            kb = k;
            wb = false;
        }
        if (!__any(wa || wb) || lb + START_DEG > lmax)
            break;
#pragma unroll
        for (int d = 0; d < START_DEG; ++d) {
            const double2 c = rec_coef<SPIN>(ab, base + lb + d);
            const double na = fma(fma(c.x, x, c.y), a1, -a0);
            a0 = a1;
            a1 = na;
            if (SPIN) {
                const double nb = fma(fma(c.x, x, -c.y), b1, -b0);
                b0 = b1;
                b1 = nb;
            }
        }
        if (wa)
            rescale_channel(a0, a1, ea, inx);
        if (SPIN && wb)
            rescale_channel(b0, b1, eb, inx);
    }
    if (e >= np)
        return;
    sta[idx] = va;
    if (SPIN)
        stb[idx] = vb;
    stk[idx] = (int32_t)((unsigned)ka | ((unsigned)kb << 16));
}

size_t leg_start_bytes(const gsht_plan &p)
{
    return (size_t)p.leg.np * ((p.spin ? 2 : 1) * sizeof(double2) + sizeof(int32_t));
}

hipError_t launch_leg_starts(const gsht_plan &p, int m0, int nm, hipStream_t s)
{
    dim3 blk(64), grd((p.leg.np + 63) / 64, nm);
    if (p.spin)
        hipLaunchKernelGGL(leg_starts_kernel<true>, grd, blk, 0, s, p.leg.ab, p.leg.start, p.lmax,
                           p.start_exp, m0, p.ntheta, p.npairs, p.leg.np, p.leg.sta, p.leg.stb, p.leg.stk);
    else
        hipLaunchKernelGGL(leg_starts_kernel<false>, grd, blk, 0, s, p.leg.ab, p.leg.start, p.lmax,
                           p.start_exp, m0, p.ntheta, p.npairs, p.leg.np, p.leg.sta, p.leg.stb, p.leg.stk);
    return hipGetLastError();
}

// Accumulators of one ring pair: spin s -> N+ (0,1), S+ (2,3), N- (4,5), S- (6,7);
// spin 0 -> the sums E (0,1) over even and O (2,3) over odd l - l0, N = E + O and
// S = E - O.  SG = (-1)^(l - l0).
template <bool SPIN, int SG>
__device__ inline void synth_acc(double (&c)[8], double va, double vb, const double *u)
{
    if (SPIN) {
        c[0] = fma(u[0], va, c[0]);
        c[1] = fma(u[1], va, c[1]);
        c[2] = fma(SG * u[0], vb, c[2]);
        c[3] = fma(SG * u[1], vb, c[3]);
        c[4] = fma(u[2], vb, c[4]);
        c[5] = fma(u[3], vb, c[5]);
        c[6] = fma(SG * u[2], va, c[6]);
        c[7] = fma(SG * u[3], va, c[7]);
    } else {
        constexpr int o = SG > 0 ? 0 : 2;
        c[o] = fma(u[0], va, c[o]);
        c[o + 1] = fma(u[1], va, c[o + 1]);
    }
}

// Spin 0: parity sums E, O -> ring values N, S.
__device__ inline void parity_rings(double (&c)[8])
{
    const double e0 = c[0], e1 = c[1], o0 = c[2], o1 = c[3];
    c[0] = e0 + o0;
    c[1] = e1 + o1;
    c[2] = e0 - o0;
    c[3] = e1 - o1;
}

// Gradient-only spin s (C = 0): u- = (-1)^s conj(u+), so the four ring sums follow
// from the products of u+ with both channels, kept per degree parity:
// E_a (0,1), E_b (2,3) for SG = +1 and O_a (4,5), O_b (6,7) for SG = -1;
//   N+ = E_a + O_a,  S+ = E_b - O_b,  N- = (-1)^s conj(E_b + O_b),
//   S- = (-1)^s conj(E_a - O_a)
// (4 FMA per ring pair and degree instead of 8).
template <int SG>
__device__ inline void synth_acc_grad(double (&c)[8], double va, double vb, const double *u)
{
    constexpr int o = SG > 0 ? 0 : 4;
    c[o + 0] = fma(u[0], va, c[o + 0]);
    c[o + 1] = fma(u[1], va, c[o + 1]);
    c[o + 2] = fma(u[0], vb, c[o + 2]);
    c[o + 3] = fma(u[1], vb, c[o + 3]);
}

template <bool SPIN, bool GRAD, int SG>
__device__ inline void synth_acc_any(double (&c)[8], double va, double vb, const double *u)
{
    if constexpr (GRAD)
        synth_acc_grad<SG>(c, va, vb, u);
    else
        synth_acc<SPIN, SG>(c, va, vb, u);
}

constexpr int LB = START_DEG;  // degrees per block

// One wave per (m, chunk), R slices per lane: 12 FMA per ring pair and degree for spin s
// (4 of them the two channels' recurrences), 4 for spin 0, the coefficients through
// scalar loads.  Bound by the FP64 vector rate: 4.6 ms at lmax 4096, spin 2 (6.9 ms when
// every wave ran all degrees from l0 with masks and exponent offsets and waited for the
// coefficients), 1.64 ms for spin 0.  The offsets and masks gone, R = 2 takes 71 and
// R = 4 124 registers.
template <typename T, bool SPIN, int R, bool GRAD = false>
__global__ __launch_bounds__(64) void leg_synth_kernel(
    const double *__restrict__ ab, const double *__restrict__ u, const StartInfo *__restrict__ st,
    RingStarts tab, int lmax, int mend, int mmax, int s, int ntheta, int nd, int dbl, int npairs, int nchunk,
    typename cplxk<T>::type *__restrict__ D)
{
    static_assert(SPIN || !GRAD, "gradient-only needs spin > 0");
    constexpr int US = (SPIN && !GRAD) ? 4 : 2;
    __shared__ double2 ent[R][SPIN ? 2 : 1][64];
    int m, chunk;
    xcd_map(tab.m0, nchunk, m, chunk);
    if (m >= mend)
        return;
    const int lane = threadIdx.x;
    const int l0 = st[m].l0;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;

    Ring rg[R];
    RingStart rs[R];
    double c[R][8];
    int first[R], kmax;
    rings_init<SPIN>(rg, rs, ent, tab, m, chunk * 64 * R, ntheta, npairs, l0 <= lmax, first, kmax);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < 8; ++k)
            c[r][k] = 0.0;
    if (kmax >= 0) {
        // Degrees in groups of G, their coefficients loaded one group ahead so that the
        // scalar loads overlap the previous group's arithmetic (as many as two groups'
        // worth of scalar registers hold).
        constexpr int G = US == 4 ? 2 : 4;
        struct Group {
            double2 c[G];
            double u[G * US];
        };
        auto load_group = [&](int l) {
            Group q;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                q.c[g] = rec_coef<SPIN>(ab, base + l + g);
#pragma unroll
                for (int k = 0; k < US; ++k)
                    q.u[g * US + k] = u[US * (base + l + g) + k];
            }
            return q;
        };
        // Slice r joins at the first entry block of its rings: spans with 1, 2, .., R
        // slices follow one another.
        int kb = first[0], lb = l0 + LB * kb;
        const int kfull = (lmax + 1 - l0) / LB;  // full blocks
        float ta = stream_touch<SPIN ? 2 : 1>(ab, base, lb, lmax);
        float tu = stream_touch<US>(u, base, lb, lmax);
        int lpf = lb;  // at degree lpf the stretch from lpf + PF_DEG is fetched
        if (kb < kfull) {  // at least one full block, so lb + LB - 1 <= lmax
            const int lsafe = lmax + 1 - G;  // last degree a whole group can be read at
            Group cur = load_group(lb);
            for_counts<R>([&](auto nr) {
                constexpr int NR = decltype(nr)::value;
                const int kend = NR < R ? min(first[NR < R ? NR : 0], kfull) : kfull;
                for (; kb < kend; lb += LB, ++kb) {
                    if (kb <= kmax)
                        rings_enter<SPIN, NR>(rg, rs, ent, kb);
                    if (lb >= lpf) {
                        asm volatile("" ::"v"(ta), "v"(tu));
                        lpf += PF_DEG;
                        ta = stream_touch<SPIN ? 2 : 1>(ab, base, lpf, lmax);
                        tu = stream_touch<US>(u, base, lpf, lmax);
                    }
#pragma unroll
                    for (int b = 0; b < LB; b += G) {
                        const Group nxt = load_group(min(lb + b + G, lsafe));
#pragma unroll
                        for (int r = 0; r < NR; ++r)
#pragma unroll
                            for (int g = 0; g < G; g += 2) {
                                const double *ug = cur.u + g * US;
                                synth_acc_any<SPIN, GRAD, 1>(c[r], rg[r].a1, rg[r].b1, ug);
                                ring_advance<SPIN>(rg[r], cur.c[g].x, cur.c[g].y);
                                synth_acc_any<SPIN, GRAD, -1>(c[r], rg[r].a1, rg[r].b1, ug + US);
                                ring_advance<SPIN>(rg[r], cur.c[g + 1].x, cur.c[g + 1].y);
                            }
                        cur = nxt;
                    }
                }
            });
        }
        if (lb <= lmax) {
            if (kb <= kmax)
                rings_enter<SPIN, R>(rg, rs, ent, kb);
            auto degree = [&](int l, auto sign) {
                constexpr int SG = decltype(sign)::value;
                const double2 cf = rec_coef<SPIN>(ab, base + l);
                const double *ul = u + US * (base + l);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    synth_acc_any<SPIN, GRAD, SG>(c[r], rg[r].a1, rg[r].b1, ul);
                    ring_advance<SPIN>(rg[r], cf.x, cf.y);
                }
            };
#pragma unroll 1
            for (; lb <= lmax; lb += 2) {
                degree(lb, count<1>());
                if (lb + 1 <= lmax)
                    degree(lb + 1, count<-1>());
            }
        }
    }
    // south values carry (-1)^(l+m) = (-1)^(l0+m) (-1)^(l-l0)
    const double sfix = ((l0 + m) & 1) ? -1.0 : 1.0;
    const double ms = ((s + m) & 1) ? -1.0 : 1.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int q = npairs - 1 - (chunk * 64 * R + 64 * r + lane);
        if (q < 0)
            continue;
        if constexpr (!SPIN)
            parity_rings(c[r]);
        if constexpr (GRAD) {  // parity sums -> N+, S+, N-, S- (see synth_acc_grad)
            const double sg = (s & 1) ? -1.0 : 1.0;
            double (&v)[8] = c[r];
            const double ea0 = v[0], ea1 = v[1], eb0 = v[2], eb1 = v[3];
            const double oa0 = v[4], oa1 = v[5], ob0 = v[6], ob1 = v[7];
            v[0] = ea0 + oa0;
            v[1] = ea1 + oa1;
            v[2] = eb0 - ob0;
            v[3] = eb1 - ob1;
            v[4] = sg * (eb0 + ob0);
            v[5] = -sg * (eb1 + ob1);
            v[6] = sg * (ea0 - oa0);
            v[7] = -sg * (ea1 - oa1);
        }
        const int jn = q, js = ntheta - 1 - q;
        typename cplxk<T>::type *colp = D + (size_t)(SPIN ? m + mmax : m) * nd;
        put_ring<T>(colp, jn, ntheta, nd, dbl, ms, c[r][0], c[r][1]);
        if (js != jn)
            put_ring<T>(colp, js, ntheta, nd, dbl, ms, sfix * c[r][2], sfix * c[r][3]);
        if (SPIN && m > 0) {
            typename cplxk<T>::type *colm = D + (size_t)(mmax - m) * nd;
            put_ring<T>(colm, jn, ntheta, nd, dbl, ms, c[r][4], c[r][5]);
            if (js != jn)
                put_ring<T>(colm, js, ntheta, nd, dbl, ms, sfix * c[r][6], sfix * c[r][7]);
        }
    }
}

template <int R>
static void synth_launch(const gsht_plan &p, const RingStarts &tab, int nm, void *Dout, bool grad,
                         hipStream_t s)
{
    dim3 blk(64), grd(xcd_grid(nm, p.syn_nchunk));
#define GSHT_LEG_SYNTH(T, SP, G, C)                                                              \
    hipLaunchKernelGGL((leg_synth_kernel<T, SP, R, G>), grd, blk, 0, s, p.leg.ab, p.uprep,       \
                       p.leg.start, tab, p.lmax, tab.m0 + nm, p.mmax, p.spin, p.ntheta, p.ds,     \
                       p.colmode != 2, p.npairs, p.syn_nchunk, (C *)Dout)
    if (p.prec == GSHT_F64) {
        if (p.spin && grad) GSHT_LEG_SYNTH(double, true, true, double2);
        else if (p.spin) GSHT_LEG_SYNTH(double, true, false, double2);
        else GSHT_LEG_SYNTH(double, false, false, double2);
    } else {
        if (p.spin && grad) GSHT_LEG_SYNTH(float, true, true, float2);
        else if (p.spin) GSHT_LEG_SYNTH(float, true, false, float2);
        else GSHT_LEG_SYNTH(float, false, false, float2);
    }
#undef GSHT_LEG_SYNTH
}

hipError_t launch_leg_synth(const gsht_plan &p, void *Dout, bool grad, hipStream_t s)
{
    if (p.syn_r != 1 && p.syn_r != 2 && p.syn_r != 4)
        return hipErrorInvalidValue;
    return leg_bands(p, s, [&](const RingStarts &tab, int nm) {
        switch (p.syn_r) {
        case 1: synth_launch<1>(p, tab, nm, Dout, grad, s); break;
        case 2: synth_launch<2>(p, tab, nm, Dout, grad, s); break;
        default: synth_launch<4>(p, tab, nm, Dout, grad, s); break;
        }
    });
}

// ---- synthesis of several maps sharing one geometry --------------------------------

// NM maps at once: the recurrence (both channels) runs once per ring pair and
// degree and feeds the sums of every map; coefficients are interleaved per degree
// as u[idx][map][US].  Chunks, starts and blocks are the single-map kernel's.  Map k's
// columns start at D + k dstride.
template <typename T, bool SPIN, int R, int NM>
__global__ __launch_bounds__(64) void leg_synth_multi_kernel(
    const double *__restrict__ ab, const double *__restrict__ u, const StartInfo *__restrict__ st,
    RingStarts tab, int lmax, int mend, int mmax, int s, int ntheta, int nd, int dbl, int npairs, int nchunk,
    size_t dstride, typename cplxk<T>::type *__restrict__ D)
{
    constexpr int US = SPIN ? 4 : 2;
    constexpr int UD = NM * US;  // doubles per degree
    __shared__ double2 ent[R][SPIN ? 2 : 1][64];
    int m, chunk;
    xcd_map(tab.m0, nchunk, m, chunk);
    if (m >= mend)
        return;
    const int lane = threadIdx.x;
    const int l0 = st[m].l0;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;

    Ring rg[R];
    RingStart rs[R];
    double c[R][NM][8];
    int first[R], kmax;
    rings_init<SPIN>(rg, rs, ent, tab, m, chunk * 64 * R, ntheta, npairs, l0 <= lmax, first, kmax);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < NM; ++k)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                c[r][k][j] = 0.0;
    auto degree = [&](int l, auto sign) {
        constexpr int SG = decltype(sign)::value;
        const double2 cf = rec_coef<SPIN>(ab, base + l);
        const double *ul = u + UD * (base + l);
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int k = 0; k < NM; ++k)
                synth_acc<SPIN, SG>(c[r][k], rg[r].a1, rg[r].b1, ul + US * k);
            ring_advance<SPIN>(rg[r], cf.x, cf.y);
        }
    };
    if (kmax >= 0) {
        int lb = l0 + LB * first[0];
#pragma unroll 1
        for (; lb <= lmax; lb += 2) {
            const int d = lb - l0;
            if ((d & (LB - 1)) == 0 && d / LB <= kmax)
                rings_enter<SPIN, R>(rg, rs, ent, d / LB);
            degree(lb, count<1>());
            if (lb + 1 <= lmax)
                degree(lb + 1, count<-1>());
        }
    }
    const double sfix = ((l0 + m) & 1) ? -1.0 : 1.0;
    const double ms = ((s + m) & 1) ? -1.0 : 1.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int q = npairs - 1 - (chunk * 64 * R + 64 * r + lane);
        if (q < 0)
            continue;
        const int jn = q, js = ntheta - 1 - q;
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            if constexpr (!SPIN)
                parity_rings(c[r][k]);
            typename cplxk<T>::type *Dk = D + k * dstride;
            typename cplxk<T>::type *colp = Dk + (size_t)(SPIN ? m + mmax : m) * nd;
            put_ring<T>(colp, jn, ntheta, nd, dbl, ms, c[r][k][0], c[r][k][1]);
            if (js != jn)
                put_ring<T>(colp, js, ntheta, nd, dbl, ms, sfix * c[r][k][2], sfix * c[r][k][3]);
            if (SPIN && m > 0) {
                typename cplxk<T>::type *colm = Dk + (size_t)(mmax - m) * nd;
                put_ring<T>(colm, jn, ntheta, nd, dbl, ms, c[r][k][4], c[r][k][5]);
                if (js != jn)
                    put_ring<T>(colm, js, ntheta, nd, dbl, ms, sfix * c[r][k][6], sfix * c[r][k][7]);
            }
        }
    }
}

template <int R, int NM>
static void synth_multi_launch(const gsht_plan &p, const RingStarts &tab, int nm, const double *u,
                               void *Dout, size_t dstride, hipStream_t s)
{
    const int nchunk = (p.npairs + 64 * R - 1) / (64 * R);
    dim3 blk(64), grd(xcd_grid(nm, nchunk));
#define GSHT_LEG_SYNTH_M(T, SP, C)                                                               \
    hipLaunchKernelGGL((leg_synth_multi_kernel<T, SP, R, NM>), grd, blk, 0, s, p.leg.ab, u,      \
                       p.leg.start, tab, p.lmax, tab.m0 + nm, p.mmax, p.spin, p.ntheta, p.ds,     \
                       p.colmode != 2, p.npairs, nchunk, dstride, (C *)Dout)
    if (p.prec == GSHT_F64) {
        if (p.spin) GSHT_LEG_SYNTH_M(double, true, double2);
        else GSHT_LEG_SYNTH_M(double, false, double2);
    } else {
        if (p.spin) GSHT_LEG_SYNTH_M(float, true, float2);
        else GSHT_LEG_SYNTH_M(float, false, float2);
    }
#undef GSHT_LEG_SYNTH_M
}

// nm maps (2 or 4) at once; slices per lane as the plan's synthesis, at most 2.
hipError_t launch_leg_synth_multi(const gsht_plan &p, int nm, const double *u, void *Dout,
                                  size_t dstride, hipStream_t s)
{
    const int key = 10 * (p.syn_r < 2 ? p.syn_r : 2) + nm;
    if (key != 12 && key != 14 && key != 22 && key != 24)
        return hipErrorInvalidValue;
    return leg_bands(p, s, [&](const RingStarts &tab, int n) {
        switch (key) {
        case 12: synth_multi_launch<1, 2>(p, tab, n, u, Dout, dstride, s); break;
        case 14: synth_multi_launch<1, 4>(p, tab, n, u, Dout, dstride, s); break;
        case 22: synth_multi_launch<2, 2>(p, tab, n, u, Dout, dstride, s); break;
        default: synth_multi_launch<2, 4>(p, tab, n, u, Dout, dstride, s); break;
        }
    });
}

// ---- adjoint -----------------------------------------------------------------------

// Per-ring adjoint inputs.  Spin 0: e = F(N) + F(S'), o = F(N) - F(S') (even / odd
// l - l0).  Spin s: F+(N), F+(S'), conj F-(N), conj F-(S'), S' = (-1)^(l0+m) S.
struct RingIn {
    double v[8];
};

// One ring's contribution to the per-degree sums cb[0..NC-1]:
//   spin s: S+ += a F+(N) + SG b F+(S'),  S- += b cF-(N) + SG a cF-(S')
//   spin 0: b_l += a (SG > 0 ? e : o)
template <bool SPIN, int SG>
__device__ inline void adj_acc(double *cb, const RingIn &in, double va, double vb)
{
    if (SPIN) {
        cb[0] = fma(va, in.v[0], cb[0]);
        cb[1] = fma(va, in.v[1], cb[1]);
        cb[0] = fma(SG * vb, in.v[2], cb[0]);
        cb[1] = fma(SG * vb, in.v[3], cb[1]);
        cb[2] = fma(vb, in.v[4], cb[2]);
        cb[3] = fma(vb, in.v[5], cb[3]);
        cb[2] = fma(SG * va, in.v[6], cb[2]);
        cb[3] = fma(SG * va, in.v[7], cb[3]);
    } else {
        cb[0] = fma(va, in.v[SG > 0 ? 0 : 2], cb[0]);
        cb[1] = fma(va, in.v[SG > 0 ? 1 : 3], cb[1]);
    }
}

// Gradient-only spin s: only T = S+ + (-1)^s S- is needed (G = -T / 2).  With the
// ring inputs precombined as X = F+(N) + SG sg cF-(S'), Y = SG F+(S') + sg cF-(N)
// (sg = (-1)^s, one pair per degree parity SG), T += a X + b Y; a and b go to
// separate sums (0,1) and (2,3), added before the lane reduction.
template <int SG>
__device__ inline void adj_acc_grad(double *cb, const RingIn &in, double va, double vb)
{
    constexpr int o = SG > 0 ? 0 : 2;
    cb[0] = fma(va, in.v[o + 0], cb[0]);
    cb[1] = fma(va, in.v[o + 1], cb[1]);
    cb[2] = fma(vb, in.v[o + 4], cb[2]);
    cb[3] = fma(vb, in.v[o + 5], cb[3]);
}

template <bool SPIN, bool GRAD, int SG>
__device__ inline void adj_acc_any(double *cb, const RingIn &in, double va, double vb)
{
    if constexpr (GRAD)
        adj_acc_grad<SG>(cb, in, va, vb);
    else
        adj_acc<SPIN, SG>(cb, in, va, vb);
}

// a' = [a(0..31), b(0..31)], b' = [a(32..63), b(32..63)] (v_permlane32_swap on both
// halves of the doubles); returns a' + b': lanes 0..31 hold a summed over lanes L
// and L + 32, lanes 32..63 hold b summed likewise.
__device__ inline double swap_add32(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32),
                                                     false, false);
    const double a2 = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    const double b2 = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
    return a2 + b2;
}

// Same with v_permlane16_swap (odd rows of a <-> even rows of b): rows 0 and 2 end
// with a summed over rows (0,1) resp. (2,3), rows 1 and 3 with b likewise.
__device__ inline double swap_add16(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32),
                                                     false, false);
    const double a2 = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    const double b2 = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
    return a2 + b2;
}

// The value of the lane whose number within the quad differs in bit 1 (0: bit 0).
template <int CTRL>
__device__ inline double quad_perm(double x)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_mov_dpp((unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp((unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double quad_xor2(double x) { return quad_perm<0x4e>(x); }

// Even lanes: a summed over the lane pair, odd lanes: b.
__device__ inline double quad_swap_add(double a, double b)
{
    const bool odd = threadIdx.x & 1;
    const double send = odd ? a : b, keep = odd ? b : a;
    return keep + quad_perm<0xb1>(send);
}

// Degrees per partial block at the end of the adjoint's range.
constexpr int ADJ_TAIL_B = 4;

// Waves per SIMD each adjoint shape is compiled for.
template <int R, int B>
constexpr int adj_waves()
{
    return R == 3 ? 3 : 1;
}

// One wave per (m, chunk).  Per block of B degrees the V = B NR per-lane sums are
// reduced over the 64 lanes: two swap-add stages in registers leave V/4 values per
// lane, each value spread over the 16 lanes of one row; these go through LDS in pairs
// and are joined there and across a few lanes.  The results are added to
// acc[idx][0..NR-1] with one FP64 atomic per (degree, component).
// Bound by the FP64 vector rate and, at few slices per wave, by the reduction (a fixed
// cost per block: at lmax 4096, spin 2, the launch takes 5.7 ms + 5 ms / R).  R = 5: 6.7 ms
// against 9.2 ms of R = 3 with masked blocks, exponent offsets and all degrees from l0.
// Reducing through LDS alone (whole rows of 16 values per lane, no swaps) took 8.1
// instead of 7.4 ms at R = 3: LDS bandwidth then binds.
template <typename T, bool SPIN, int R, int B, bool GRAD = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(adj_waves<R, B>())))
void leg_adjoint_kernel(
    const double *__restrict__ ab, const StartInfo *__restrict__ st, RingStarts tab,
    const typename cplxk<T>::type *__restrict__ D, int lmax, int mend, int mmax, int s, int ntheta,
    int nd, int dbl, int npairs, int nchunk, double *__restrict__ acc)
{
    static_assert(SPIN || !GRAD, "gradient-only needs spin > 0");
    constexpr int NC = SPIN ? 4 : 2;         // per-lane sums per degree
    constexpr int NR = GRAD ? 2 : NC;        // reduced values per degree
    constexpr int V = B * NR;
    constexpr int BM = ADJ_TAIL_B < B ? ADJ_TAIL_B : B;  // degrees per partial block
    static_assert(64 % V == 0 && V >= 8, "block values must divide the wave");
    static_assert(LB % B == 0, "entry blocks start with reduction blocks");
    __shared__ double2 red[V * 8];
    __shared__ double2 ent[R][SPIN ? 2 : 1][64];
    int m, chunk;
    xcd_map(tab.m0, nchunk, m, chunk);
    if (m >= mend)
        return;
    const int lane = threadIdx.x;
    const int l0 = st[m].l0;
    Ring rg[R];
    RingStart rs[R];
    int first[R], kmax;
    rings_init<SPIN>(rg, rs, ent, tab, m, chunk * 64 * R, ntheta, npairs, l0 <= lmax, first, kmax);
    if (kmax < 0)
        return;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const double ms = ((s + m) & 1) ? -1.0 : 1.0;
    const double sfix = ((l0 + m) & 1) ? -1.0 : 1.0;

    RingIn in[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int q = npairs - 1 - (chunk * 64 * R + 64 * r + lane);
        const bool active = q >= 0;
        double2 fpn = make_double2(0, 0), fps = fpn, fmn = fpn, fms = fpn;
        if (active) {
            const int jn = q, js = ntheta - 1 - q;
            const typename cplxk<T>::type *colp = D + (size_t)(SPIN ? m + mmax : m) * nd;
            fpn = ring_in<T>(colp, jn, ntheta, nd, dbl, ms);
            if (js != jn) {
                fps = ring_in<T>(colp, js, ntheta, nd, dbl, ms);
                fps.x *= sfix;
                fps.y *= sfix;
            }
            if (SPIN) {
                const typename cplxk<T>::type *colm = D + (size_t)(mmax - m) * nd;
                fmn = ring_in<T>(colm, jn, ntheta, nd, dbl, ms);
                if (js != jn) {
                    fms = ring_in<T>(colm, js, ntheta, nd, dbl, ms);
                    fms.x *= sfix;
                    fms.y *= sfix;
                }
            }
        }
        if (GRAD) {  // X_e, X_o, Y_e, Y_o (see adj_acc_grad)
            const double sg = (s & 1) ? -1.0 : 1.0;
            in[r].v[0] = fpn.x + sg * fms.x; in[r].v[1] = fpn.y - sg * fms.y;
            in[r].v[2] = fpn.x - sg * fms.x; in[r].v[3] = fpn.y + sg * fms.y;
            in[r].v[4] = fps.x + sg * fmn.x; in[r].v[5] = fps.y - sg * fmn.y;
            in[r].v[6] = -fps.x + sg * fmn.x; in[r].v[7] = -fps.y - sg * fmn.y;
        } else if (SPIN) {
            in[r].v[0] = fpn.x; in[r].v[1] = fpn.y;
            in[r].v[2] = fps.x; in[r].v[3] = fps.y;
            in[r].v[4] = fmn.x; in[r].v[5] = -fmn.y;
            in[r].v[6] = fms.x; in[r].v[7] = -fms.y;
        } else {
            in[r].v[0] = fpn.x + fps.x; in[r].v[1] = fpn.y + fps.y;
            in[r].v[2] = fpn.x - fps.x; in[r].v[3] = fpn.y - fps.y;
            in[r].v[4] = in[r].v[5] = in[r].v[6] = in[r].v[7] = 0.0;
        }
    }
    // Reduce the block sums cb (VB values: VB / NR degrees) over the wave and add them
    // to acc (degrees lb..).
    auto reduce_add = [&](auto &cb, int lb) {
        constexpr int VB = std::extent<std::remove_reference_t<decltype(cb)>>::value;
        static_assert(64 % VB == 0 && VB >= 8 && VB <= V, "block values must divide the wave");
        // stage 1: lanes L, L + 32 -> VB/2 values; value k + (L / 32) VB/2 in slot k
        double c1[VB / 2];
#pragma unroll
        for (int k = 0; k < VB / 2; ++k)
            c1[k] = swap_add32(cb[k], cb[k + VB / 2]);
        // stage 2: rows (0,1), (2,3) -> VB/4 values per lane; slot k of row g holds
        // value k + (g & 1) VB/4 + (g >> 1) VB/2, partially summed over 4 lanes
        double c2[VB / 4];
#pragma unroll
        for (int k = 0; k < VB / 4; ++k)
            c2[k] = swap_add16(c1[k], c1[k + VB / 4]);
        // stage 3: pairs of slots go through LDS ([pair][lane]); SUB lanes of a group sum
        // the 16 lanes of one (pair, row), first each its 16 / SUB entries (read in an
        // order that keeps the groups on different banks), then across the group
        constexpr int NP = VB / 8;          // pairs per row
        constexpr int SUB = 64 / (4 * NP);  // lanes per group: lane bits 0, 1, then 5, 4
        static_assert(SUB == 4 || SUB == 8 || SUB == 16, "8, 16 or 32 values");
        double2 *const buf = red;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NP; ++k)
            buf[k * 64 + lane] = make_double2(c2[2 * k], c2[2 * k + 1]);
        __syncthreads();
        const int G = SUB == 4 ? lane >> 2 : SUB == 8 ? (lane >> 2) & 7 : (lane >> 2) & 3;
        const int sub = SUB == 4   ? lane & 3
                        : SUB == 8 ? (lane & 3) | ((lane >> 5) << 2)
                                   : (lane & 3) | ((lane >> 4) << 2);
        const int g = G & 3, pr = G >> 2;
        constexpr int NE = 16 / SUB;
        const double2 *src = buf + pr * 64 + 16 * g + NE * sub;
        double2 t = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const double2 v = src[(i + G) & (NE - 1)];
            t.x += v.x;
            t.y += v.y;
        }
        double sum = quad_swap_add(t.x, t.y);  // even lanes .x, odd lanes .y
        sum += quad_xor2(sum);
        if constexpr (SUB >= 8)
            sum = swap_add32(sum, sum);
        if constexpr (SUB == 16)
            sum = swap_add16(sum, sum);
        const int v = 2 * pr + (lane & 1) + (g & 1) * (VB / 4) + (g >> 1) * (VB / 2);
        constexpr int idle = 2 | (SUB >= 8 ? 32 : 0) | (SUB == 16 ? 16 : 0);
        if ((lane & idle) == 0 && lb + v / NR <= lmax)
            unsafeAtomicAdd(acc + (base + lb) * NR + v, sum);
    };
    // per-lane sums of a block of BB = size / NC degrees -> the values reduced over
    // the wave
    auto reduce_block = [&](auto &cf, int lb) {
        constexpr int BB = std::extent<std::remove_reference_t<decltype(cf)>>::value / NC;
        if constexpr (GRAD) {
            double cr[2 * BB];
#pragma unroll
            for (int b = 0; b < BB; ++b) {
                cr[2 * b] = cf[4 * b] + cf[4 * b + 2];
                cr[2 * b + 1] = cf[4 * b + 1] + cf[4 * b + 3];
            }
            reduce_add(cr, lb);
        } else {
            reduce_add(cf, lb);
        }
    };
    // Full blocks, in spans with 1, 2, .., R slices (slice r joins at the first entry
    // block of its rings); the coefficients of each degree pair are loaded one pair ahead
    // (across block ends too), so the scalar loads overlap the current pair's work.
    int lb = l0 + LB * first[0];
    if (lb + B - 1 <= lmax) {
        const int lfull = l0 + (lmax + 1 - l0) / B * B;
        float ta = stream_touch<SPIN ? 2 : 1>(ab, base, lb, lmax);
        int lpf = lb;  // at degree lpf the stretch from lpf + PF_DEG is fetched
        double2 q0 = rec_coef<SPIN>(ab, base + lb), q1 = rec_coef<SPIN>(ab, base + lb + 1);
        for_counts<R>([&](auto nr) {
            constexpr int N = decltype(nr)::value;
            const int lend = N < R ? min(l0 + LB * first[N < R ? N : 0], lfull) : lfull;
            for (; lb < lend; lb += B) {
                const int d = lb - l0;
                if ((B == LB || (d & (LB - 1)) == 0) && d / LB <= kmax)
                    rings_enter<SPIN, N>(rg, rs, ent, d / LB);
                if (lb >= lpf) {
                    asm volatile("" ::"v"(ta));
                    lpf += PF_DEG;
                    ta = stream_touch<SPIN ? 2 : 1>(ab, base, lpf, lmax);
                }
                double cb[B * NC];
#pragma unroll
                for (int k = 0; k < B * NC; ++k)
                    cb[k] = 0.0;
#pragma unroll
                for (int b = 0; b < B; b += 2) {
                    const int ln = lb + b + 2;                    // next pair
                    const int lc = ln + 1 <= lmax ? ln : lb + b;  // stays inside this m's table
                    const double2 n0 = rec_coef<SPIN>(ab, base + lc), n1 = rec_coef<SPIN>(ab, base + lc + 1);
#pragma unroll
                    for (int r = 0; r < N; ++r) {
                        adj_acc_any<SPIN, GRAD, 1>(cb + b * NC, in[r], rg[r].a1, rg[r].b1);
                        ring_advance<SPIN>(rg[r], q0.x, q0.y);
                        adj_acc_any<SPIN, GRAD, -1>(cb + (b + 1) * NC, in[r], rg[r].a1, rg[r].b1);
                        ring_advance<SPIN>(rg[r], q1.x, q1.y);
                    }
                    q0 = n0;
                    q1 = n1;
                }
                reduce_block(cb, lb);
            }
        });
    }
    // partial blocks at the end
    for (; lb <= lmax; lb += BM) {
        const int d = lb - l0;
        if ((d & (LB - 1)) == 0 && d / LB <= kmax)
            rings_enter<SPIN, R>(rg, rs, ent, d / LB);
        double cb[BM * NC];
#pragma unroll
        for (int k = 0; k < BM * NC; ++k)
            cb[k] = 0.0;
#pragma unroll
        for (int b = 0; b < BM; b += 2) {
            const int l = lb + b;
            if (l > lmax)
                break;
            const double2 c0 = rec_coef<SPIN>(ab, base + l);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                adj_acc_any<SPIN, GRAD, 1>(cb + b * NC, in[r], rg[r].a1, rg[r].b1);
                ring_advance<SPIN>(rg[r], c0.x, c0.y);
            }
            if (l + 1 > lmax)
                break;
            const double2 c1 = rec_coef<SPIN>(ab, base + l + 1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                adj_acc_any<SPIN, GRAD, -1>(cb + (b + 1) * NC, in[r], rg[r].a1, rg[r].b1);
                ring_advance<SPIN>(rg[r], c1.x, c1.y);
            }
        }
        reduce_block(cb, lb);
    }
}

template <int R, int B>
static void adj_launch(const gsht_plan &p, const RingStarts &tab, int nm, const void *Din, bool grad,
                       hipStream_t s)
{
    dim3 blk(64), grd(xcd_grid(nm, p.adj_nchunk));
#define GSHT_LEG_ADJ(T, SP, G, C)                                                                \
    hipLaunchKernelGGL((leg_adjoint_kernel<T, SP, R, B, G>), grd, blk, 0, s, p.leg.ab,           \
                       p.leg.start, tab, (const C *)Din, p.lmax, tab.m0 + nm, p.mmax, p.spin,     \
                       p.ntheta, p.ds, p.colmode != 2, p.npairs, p.adj_nchunk, p.acc)
    if (p.prec == GSHT_F64) {
        if (p.spin && grad) GSHT_LEG_ADJ(double, true, true, double2);
        else if (p.spin) GSHT_LEG_ADJ(double, true, false, double2);
        else GSHT_LEG_ADJ(double, false, false, double2);
    } else {
        if (p.spin && grad) GSHT_LEG_ADJ(float, true, true, float2);
        else if (p.spin) GSHT_LEG_ADJ(float, true, false, float2);
        else GSHT_LEG_ADJ(float, false, false, float2);
    }
#undef GSHT_LEG_ADJ
}

hipError_t launch_zero(void *ptr, size_t bytes, hipStream_t s);

hipError_t launch_leg_adjoint(const gsht_plan &p, const void *Din, bool grad, hipStream_t s)
{
    hipError_t e = launch_zero(p.acc, sizeof(double) * (size_t)p.nalm * 2 * p.ncomp, s);
    if (e != hipSuccess)
        return e;
    const int key = p.adj_r * 100 + p.adj_b;
    if (key != 108 && key != 208 && key != 204 && key != 404 && key != 308 && key != 304 &&
        key != 408 && key != 508)
        return hipErrorInvalidValue;
    return leg_bands(p, s, [&](const RingStarts &tab, int nm) {
        switch (key) {
        case 108: adj_launch<1, 8>(p, tab, nm, Din, grad, s); break;
        case 208: adj_launch<2, 8>(p, tab, nm, Din, grad, s); break;
        case 204: adj_launch<2, 4>(p, tab, nm, Din, grad, s); break;
        case 404: adj_launch<4, 4>(p, tab, nm, Din, grad, s); break;
        case 508: adj_launch<5, 8>(p, tab, nm, Din, grad, s); break;
        case 308: adj_launch<3, 8>(p, tab, nm, Din, grad, s); break;
        case 304: adj_launch<3, 4>(p, tab, nm, Din, grad, s); break;
        default: adj_launch<4, 8>(p, tab, nm, Din, grad, s); break;
        }
    });
}

}  // namespace gsht
