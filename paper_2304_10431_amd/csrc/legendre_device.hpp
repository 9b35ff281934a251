// Device helpers shared by the Legendre kernels (single-map, several-map and
// matrix-core forms): start values with a separate binary exponent, the per-ring
// recurrence state and its range handling, the XCD-aware work mapping and the
// doubled-column stores.  The conventions are described in legendre_kernels.hip.
#pragma once

#include <type_traits>

#include "gsht_internal.hpp"

namespace gsht {

template <typename T> struct cplxk;
template <> struct cplxk<float> { using type = float2; };
template <> struct cplxk<double> { using type = double2; };

// ---- start values -----------------------------------------------------------------

struct XD {
    double m;
    int e;
};

__device__ inline void xnorm(XD &x)
{
    int k;
    x.m = frexp(x.m, &k);
    x.e += k;
}

// base^n (base >= 0, n >= 0) with a separate binary exponent; 0^0 = 1.
__device__ inline XD xpow(double base, int n)
{
    XD r{1.0, 0};
    if (n == 0)
        return r;
    if (base == 0.0)
        return XD{0.0, 0};
    XD b{base, 0};
    xnorm(b);
    while (n) {
        if (n & 1) {
            r.m *= b.m;
            r.e += b.e;
            xnorm(r);
        }
        b.m *= b.m;
        b.e *= 2;
        xnorm(b);
        n >>= 1;
    }
    return r;
}

// One channel's value at l0: mant 2^ex0 sin(theta/2)^a cos(theta/2)^b.
__device__ inline XD start_value(double mant, int ex0, int a, int b, double sh, double ch)
{
    XD v{mant, ex0};
    const XD ps = xpow(sh, a), pc = xpow(ch, b);
    v.m *= ps.m;
    v.e += ps.e;
    xnorm(v);
    v.m *= pc.m;
    v.e += pc.e;
    xnorm(v);
    return v;
}

__device__ inline void ring_geom(int q, int ntheta, double &x, double &sh, double &ch)
{
    const double t = (double)q / (double)(ntheta - 1);
    x = cospi(t);
    sh = sinpi(0.5 * t);
    ch = cospi(0.5 * t);
}

// ---- work mapping -------------------------------------------------------------------

// Workgroups are dispatched round-robin over the MI355X's 8 XCDs.  All chunks of one
// m are kept on one XCD, so that XCD's L2 serves the m's coefficient stream to all of
// them (spread over every XCD, each 4 MB L2 would hold dozens of streams and thrash),
// and the m values are dealt to the XCDs round-robin, largest work first on each.
constexpr int NXCD = 8;

__device__ inline void xcd_map(int m0, int nchunk, int &m, int &chunk)
{
    const int x = blockIdx.x % NXCD, k = blockIdx.x / NXCD;
    const int g = k / nchunk;
    chunk = k - g * nchunk;
    m = m0 + x + NXCD * g;
}

// Workgroups for a band of nm values of m.
inline unsigned xcd_grid(int nm, int nchunk)
{
    return (unsigned)(NXCD * ((nm + NXCD - 1) / NXCD) * nchunk);
}

// ---- per-ring recurrence state ------------------------------------------------------

// Ring pairs are counted from the equator: position e is the pair q = npairs - 1 - e.
// A wave's chunk of 64 R consecutive positions then holds rings that enter the sums at
// similar degrees, and the one partly filled chunk of an m lies at the pole, where the
// sums are shortest (counted from the pole it lay at the equator and ran all degrees).
struct Ring {
    double x;
    double a0, a1, b0, b1;  // p_{l-1}, p_l of channels +s and -s
};

// Start of one ring pair's recurrences (see leg_starts_kernel): k is the 8-degree block,
// counted from l0, at which a channel enters; before it the channel's values are 0.
constexpr int START_DEG = 8;  // degrees per entry block

struct RingStart {
    int ka, kb;
};

__device__ inline RingStart ring_start(const RingStarts &t, int m, int e, bool spin)
{
    const unsigned k = (unsigned)t.k[(size_t)(m - t.m0) * t.np + e];
    return RingStart{(int)(k & 0xffffu), spin ? (int)(k >> 16) : START_NEVER};
}

// first[r]: the smallest entry block among a wave's slices r, r + 1, ... (slices nearer
// the pole enter later, so normally that of slice r); kmax: the largest entry block below
// START_NEVER (-1: none).
template <int R>
__device__ inline void wave_start_range(const RingStart (&rs)[R], int (&first)[R], int &kmax)
{
    int hi = -1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        first[r] = min(rs[r].ka, rs[r].kb);
        hi = max(hi, rs[r].ka < START_NEVER ? rs[r].ka : -1);
        hi = max(hi, rs[r].kb < START_NEVER ? rs[r].kb : -1);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            first[r] = min(first[r], __shfl_xor(first[r], d, 64));
        hi = max(hi, __shfl_xor(hi, d, 64));
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        first[r] = __builtin_amdgcn_readfirstlane(first[r]);
#pragma unroll
    for (int r = R - 2; r >= 0; --r)
        first[r] = min(first[r], first[r + 1]);
    kmax = __builtin_amdgcn_readfirstlane(hi);
}

__device__ inline double ring_x(int q, int ntheta)
{
    return cospi((double)q / (double)(ntheta - 1));
}

// Enter the channels whose block is k.
template <bool SPIN>
__device__ inline void ring_enter(Ring &r, const RingStart &rs, int k, const double2 &va,
                                  const double2 &vb)
{
    if (rs.ka == k) {
        r.a0 = va.x;
        r.a1 = va.y;
    }
    if (SPIN && rs.kb == k) {
        r.b0 = vb.x;
        r.b1 = vb.y;
    }
}

// Recurrence coefficients (a_l, b_l) at coefficient index i: interleaved for spin > 0;
// spin 0 has b_l = 0 and keeps a_l alone, which halves that scalar stream.
template <bool SPIN>
__device__ inline double2 rec_coef(const double *__restrict__ ab, int64_t i)
{
    if constexpr (SPIN)
        return *reinterpret_cast<const double2 *>(ab + 2 * i);
    else
        return make_double2(ab[i], 0.0);
}

// Sets the recurrence state of a wave's rings to "not entered" and loads their entry
// blocks; the entry values wait in LDS (each lane reads back its own).
template <bool SPIN, int R>
__device__ inline void rings_init(Ring (&rg)[R], RingStart (&rs)[R], double2 (&ent)[R][SPIN ? 2 : 1][64],
                                  const RingStarts &tab, int m, int e0, int ntheta, int npairs,
                                  bool live, int (&first)[R], int &kmax)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = e0 + 64 * r + lane;
        const bool in = live && e < npairs;
        rs[r] = in ? ring_start(tab, m, e, SPIN) : RingStart{START_NEVER, START_NEVER};
        rg[r].x = ring_x(in ? npairs - 1 - e : 0, ntheta);
        rg[r].a0 = rg[r].a1 = rg[r].b0 = rg[r].b1 = 0.0;
        const size_t idx = (size_t)(m - tab.m0) * tab.np + e;
        if (rs[r].ka < START_NEVER)
            ent[r][0][lane] = tab.a[idx];
        if (SPIN && rs[r].kb < START_NEVER)
            ent[r][1][lane] = tab.b[idx];
    }
    wave_start_range(rs, first, kmax);
}

// Enters the channels whose block is k (a wave-uniform test first: most blocks have none).
template <bool SPIN, int NR, int R>
__device__ inline void rings_enter(Ring (&rg)[R], const RingStart (&rs)[R],
                                   const double2 (&ent)[R][SPIN ? 2 : 1][64], int k)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (__any(rs[r].ka == k || (SPIN && rs[r].kb == k)))
            ring_enter<SPIN>(rg[r], rs[r], k, ent[r][0][lane], ent[r][SPIN ? 1 : 0][lane]);
}

template <bool SPIN>
__device__ inline void ring_advance(Ring &r, double a, double b)
{
    const double ta = SPIN ? fma(a, r.x, b) : a * r.x;
    const double na = fma(ta, r.a1, -r.a0);
    r.a0 = r.a1;
    r.a1 = na;
    if (SPIN) {
        const double tb = fma(a, r.x, -b);
        const double nb = fma(tb, r.b1, -r.b0);
        r.b0 = r.b1;
        r.b1 = nb;
    }
}

// Pulls the coefficient stream of one m into the XCD's L2 ahead of the scalar loads,
// which otherwise wait for HBM about once per pair of degrees (all chunks of an m run
// close together, so none of them finds the line already there).  One lane per touched
// line; W doubles per degree, PF_DEG degrees per call.  The value is dropped: the empty
// asm only keeps the load, and names it as an input one call later.
constexpr int PF_DEG = 256;

template <int W>
__device__ inline float stream_touch(const double *p, int64_t base, int l, int lmax)
{
    const int lane = threadIdx.x & 63;
    const int ll = min(l + lane * (PF_DEG / 64), lmax);
    return *reinterpret_cast<const float *>(p + W * (base + ll));
}

template <int N>
using count = std::integral_constant<int, N>;

// f(count<1>()), ..., f(count<N>()) in order.
template <int N, typename F>
__device__ inline void for_counts(F &&f)
{
    if constexpr (N > 1)
        for_counts<N - 1>(f);
    f(count<N>());
}

template <bool B>
using flag = std::integral_constant<bool, B>;

// ---- synthesis -------------------------------------------------------------------

template <typename T>
__device__ inline void store_c(typename cplxk<T>::type *p, double re, double im)
{
    typename cplxk<T>::type v;
    v.x = (T)re;
    v.y = (T)im;
    *p = v;
}

// Ring value and, with dbl and for interior rings, its doubled mirror with sign ms.  (A
// plan whose column stage takes pairs of columns wants the rings alone; nd is then only
// the stride of its columns.)
template <typename T>
__device__ inline void put_ring(typename cplxk<T>::type *col, int j, int ntheta, int nd, int dbl,
                                double ms, double re, double im)
{
    store_c<T>(col + j, re, im);
    if (dbl && j > 0 && j < ntheta - 1)
        store_c<T>(col + (nd - j), ms * re, ms * im);
}

template <typename T>
__device__ inline double2 ld_c(const typename cplxk<T>::type *p)
{
    const typename cplxk<T>::type v = *p;
    return make_double2((double)v.x, (double)v.y);
}

// Ring value H(j) of the adjoint: the undoubled sum of a doubled column (dbl), or the
// entry itself.
template <typename T>
__device__ inline double2 ring_in(const typename cplxk<T>::type *col, int j, int ntheta, int nd,
                                  int dbl, double ms)
{
    double2 v = ld_c<T>(col + j);
    if (dbl && j > 0 && j < ntheta - 1) {
        const double2 w = ld_c<T>(col + (nd - j));
        v.x += ms * w.x;
        v.y += ms * w.y;
    }
    return v;
}

}  // namespace gsht
