// Column FFT stage of the general SHT on gfx950 (Sect. 3: the FFT of the
// doubled meridians, the deconvolution / zero padding of the NUFFT, and the
// oversampled theta transform), with one workgroup per column (two neighbouring columns
// where both transforms fit) and its columns held in LDS, so that each column crosses HBM
// once on the way in and once on the way out.
//
//   forward:  D[col][0..nd)  --FFT_nd(-)-->  D^  --f(k,m), zero pad-->  E^[0..n1)
//             --FFT_n1(+)-->  E[col][a]   (only the torus rows the grid keeps)
//   adjoint:  E[col][kept rows]  --FFT_n1(-)-->  E^  --f(k,m)-->  D^[0..nd)
//             --FFT_nd(+)-->  D[col]
//
// f(k, m) = kfac1[|k|] kfac2[|m|] for |k| <= lmax and 0 otherwise, the same real
// factors both ways, so the adjoint stays the exact transpose of the forward.
// When n1 does not fit in LDS (FP64 at large n1) only the nd transform and the
// deconvolution are fused here and the theta transform runs separately on E.
//
// The FFTs are in-place mixed-radix decimation-in-frequency passes over LDS (radices
// 8, 4, 2, 3, 5, 7): pass i splits sub-transforms of length L into radix r_i
// butterflies of stride s = L / r_i, each followed by the twiddles w_L^(q j).  The
// result sits in digit-reversed order; a host-built table gives the LDS position of
// every frequency.  Twiddles come from per-pass tables in the working precision,
// read contiguously per butterfly.
#include <algorithm>

#include "gsht_internal.hpp"

namespace gsht {

namespace {

constexpr int COL_THREADS = 1024;

// largest radix of the in-LDS transforms (a radix-16 pass, 16 complex values plus 15
// twiddles, does not fit the 128 registers of either precision's workgroups)
constexpr int COL_MAXR = 8;

template <typename T> struct cx;
template <> struct cx<float> { using type = float2; };
template <> struct cx<double> { using type = double2; };
template <typename C> struct cx2;  // two complex values
template <> struct cx2<float2> { using type = float4; };
template <> struct cx2<double2> { using type = double4; };

// Mode 2 (split theta transform): threads per workgroup at most, and the largest nd or
// n1 / 2 it takes; each thread stages up to col_half_maxn / threads values in
// registers.  At lmax 4096 two FP32 workgroups of 512 threads (2 x 66 KB of LDS) share a
// CU, and one FP64 workgroup of 1024 threads (132 KB) fills it (18 % faster than 512
// threads with radix-16 passes).  Either way 16 waves per CU and 128 VGPRs.
template <typename T>
constexpr int col_half_threads()
{
    return sizeof(T) == 4 ? 512 : 1024;
}
constexpr int COL_HALF_WAVES = 4;  // waves per SIMD
template <typename T>
constexpr int col_half_maxn()
{
    return sizeof(T) == 4 ? 17 * 512 : 20 * 512;
}

template <typename C>
__device__ inline C cadd(C a, C b) { a.x += b.x; a.y += b.y; return a; }
template <typename C>
__device__ inline C csub(C a, C b) { a.x -= b.x; a.y -= b.y; return a; }

// ---- small DFTs in registers (DIR = -1 forward e^{-2 pi i}, +1 backward) ------

// cos, sin of 2 pi k / 16 for k < 8
__device__ constexpr double C16[8] = {1.0, 0.92387953251128675613, 0.70710678118654752440,
                                      0.38268343236508977173, 0.0, -0.38268343236508977173,
                                      -0.70710678118654752440, -0.92387953251128675613};
__device__ constexpr double S16[8] = {0.0, 0.38268343236508977173, 0.70710678118654752440,
                                      0.92387953251128675613, 1.0, 0.92387953251128675613,
                                      0.70710678118654752440, 0.38268343236508977173};

// b * w_16^(DIR * idx) with w_16 = e^{2 pi i / 16}; idx is a compile-time constant
// after unrolling, so the trivial factors cost nothing.
template <typename C, int DIR>
__device__ inline C tw16(C b, int idx)
{
    using T = decltype(b.x);
    if (idx == 0)
        return b;
    C o;
    if (idx == 4) {  // multiply by DIR * i
        o.x = -DIR * b.y;
        o.y = DIR * b.x;
        return o;
    }
    const T c = (T)C16[idx], s = (T)(DIR * S16[idx]);
    o.x = b.x * c - b.y * s;
    o.y = b.x * s + b.y * c;
    return o;
}

template <int R>
__device__ constexpr int bitrev(int i)
{
    int r = 0;
    for (int b = 1; b < R; b <<= 1) {
        r = (r << 1) | (i & 1);
        i >>= 1;
    }
    return r;
}

// Radix-2 decimation in time over R <= 16 values (bit-reversed load, natural output).
template <typename C, int R, int DIR>
__device__ inline void dft_pow2(C (&v)[R])
{
    C w[R];
#pragma unroll
    for (int i = 0; i < R; ++i)
        w[bitrev<R>(i)] = v[i];
#pragma unroll
    for (int m = 2; m <= R; m <<= 1)
#pragma unroll
        for (int k0 = 0; k0 < R; k0 += m)
#pragma unroll
            for (int j = 0; j < m / 2; ++j) {
                const C a = w[k0 + j];
                const C b = tw16<C, DIR>(w[k0 + j + m / 2], j * (16 / m));
                w[k0 + j] = cadd(a, b);
                w[k0 + j + m / 2] = csub(a, b);
            }
#pragma unroll
    for (int i = 0; i < R; ++i)
        v[i] = w[i];
}

template <int R> struct OddTab;
template <> struct OddTab<3> {
    static constexpr double c[3] = {1.0, -0.5, -0.5};
    static constexpr double s[3] = {0.0, 0.86602540378443864676, -0.86602540378443864676};
};
template <> struct OddTab<5> {
    static constexpr double c[5] = {1.0, 0.30901699437494742410, -0.80901699437494742410,
                                    -0.80901699437494742410, 0.30901699437494742410};
    static constexpr double s[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917,
                                    -0.58778525229247312917, -0.95105651629515357212};
};
template <> struct OddTab<7> {
    static constexpr double c[7] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                    -0.90096886790241912624, -0.90096886790241912624,
                                    -0.22252093395631440429, 0.62348980185873353053};
    static constexpr double s[7] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                    0.43388373911755812048, -0.43388373911755812048,
                                    -0.97492791218182360702, -0.78183148246802980871};
};

// Odd prime R: X_q = v0 + sum_t [(v_t + v_{R-t}) cos(2 pi t q / R)
//                                 + DIR i (v_t - v_{R-t}) sin(2 pi t q / R)].
template <typename C, int R, int DIR>
__device__ inline void dft_odd(C (&v)[R])
{
    using T = decltype(v[0].x);
    constexpr int H = (R - 1) / 2;
    C sp[H], sm[H];
#pragma unroll
    for (int t = 1; t <= H; ++t) {
        sp[t - 1] = cadd(v[t], v[R - t]);
        sm[t - 1] = csub(v[t], v[R - t]);
    }
    C y[R];
    y[0] = v[0];
#pragma unroll
    for (int t = 0; t < H; ++t)
        y[0] = cadd(y[0], sp[t]);
#pragma unroll
    for (int q = 1; q <= H; ++q) {
        C a = v[0], b;
        b.x = 0;
        b.y = 0;
#pragma unroll
        for (int t = 1; t <= H; ++t) {
            const int k = (t * q) % R;
            const T c = (T)OddTab<R>::c[k], s = (T)OddTab<R>::s[k];
            a.x += c * sp[t - 1].x;
            a.y += c * sp[t - 1].y;
            b.x += s * sm[t - 1].x;
            b.y += s * sm[t - 1].y;
        }
        // X_q = a + DIR i b,  X_{R-q} = a - DIR i b
        y[q].x = a.x - DIR * b.y;
        y[q].y = a.y + DIR * b.x;
        y[R - q].x = a.x + DIR * b.y;
        y[R - q].y = a.y - DIR * b.x;
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        v[i] = y[i];
}

template <typename C, int R, int DIR>
__device__ inline void dft(C (&v)[R])
{
    if constexpr ((R & (R - 1)) == 0)
        dft_pow2<C, R, DIR>(v);
    else
        dft_odd<C, R, DIR>(v);
}

// One decimation-in-frequency pass over NT threads: butterflies b < n / R over
// sub-transforms of length L = R s; butterfly (sub, j) reads positions
// sub L + j + t s, t < R, and its twiddles w_L^(q j) from tw[j (R - 1) + q - 1]
// (conjugated for DIR > 0): a lane's twiddles are contiguous.
template <typename C, int R, int DIR, int NT>
__device__ inline void dif_pass(C *X, const C *__restrict__ tw, int n, int s, int sh)
{
    const int L = R * s, nb = n / R;
    const double rs = 1.0 / (double)s;  // b / s by an FP64 product: exact for b < 2^26
    for (int b = threadIdx.x; b < nb; b += NT) {
        const int sub = (int)(((double)b + 0.5) * rs), j = b - sub * s;
        const int base = sub * L + j;
        C v[R];
#pragma unroll
        for (int t = 0; t < R; ++t)
            v[t] = X[lds_pos(base + t * s, sh)];
        dft<C, R, DIR>(v);
        if (j != 0) {
#pragma unroll
            for (int q = 1; q < R; ++q) {
                C w = tw[j * (R - 1) + q - 1];
                if (DIR > 0)
                    w.y = -w.y;
                const C a = v[q];
                v[q].x = a.x * w.x - a.y * w.y;
                v[q].y = a.x * w.y + a.y * w.x;
            }
        }
#pragma unroll
        for (int t = 0; t < R; ++t)
            X[lds_pos(base + t * s, sh)] = v[t];
    }
}

// Whole transform in LDS (the block must hold the column before the call; the
// result is in digit-reversed order when it returns, after a barrier).
template <typename C, int DIR, int NT>
__device__ void lds_fft(C *X, const ColFFT &f)
{
    int L = f.n;
    for (int p = 0; p < f.npass; ++p) {
        const int r = f.radix[p];
        const int s = L / r;
        const C *tw = reinterpret_cast<const C *>(f.tw) + f.twoff[p];
        switch (r) {
        case 8: dif_pass<C, 8, DIR, NT>(X, tw, f.n, s, f.psh); break;
        case 4: dif_pass<C, 4, DIR, NT>(X, tw, f.n, s, f.psh); break;
        case 2: dif_pass<C, 2, DIR, NT>(X, tw, f.n, s, f.psh); break;
        case 3: dif_pass<C, 3, DIR, NT>(X, tw, f.n, s, f.psh); break;
        case 5: dif_pass<C, 5, DIR, NT>(X, tw, f.n, s, f.psh); break;
        case 7: dif_pass<C, 7, DIR, NT>(X, tw, f.n, s, f.psh); break;
        default: break;
        }
        L = s;
        __syncthreads();
    }
}

__device__ inline bool row_kept(int a, int n1, int nrows, int a_min)
{
    int r = a - a_min;
    if (r >= n1)
        r -= n1;
    return r < nrows;  // a_min <= 0 and a < n1, so r >= 0
}

template <typename C>
__device__ inline C scale_c(C v, double f)
{
    using T = decltype(v.x);
    v.x = (T)(f * (double)v.x);
    v.y = (T)(f * (double)v.y);
    return v;
}

template <typename C>
__device__ inline C cmul(C a, C b)
{
    C o;
    o.x = a.x * b.x - a.y * b.y;
    o.y = a.x * b.y + a.y * b.x;
    return o;
}

template <typename C>
__device__ inline C cmulc(C a, C b)  // a * conj(b)
{
    C o;
    o.x = a.x * b.x + a.y * b.y;
    o.y = a.y * b.x - a.x * b.y;
    return o;
}

// LDS of mode 2: the column buffer (the transforms of lengths nd and nh = n1 / 2).
__host__ __device__ inline int col_half_lds_n(int nd, int nh) { return nd > nh ? nd : nh; }

struct ColArgs {
    const double *kf1, *kf2;
    int lmax, mmax, spin, ncol, nd, ds, n1, nrows, a_min;
};

__device__ inline int col_m(const ColArgs &a, int col) { return a.spin ? col - a.mmax : col; }

// The kept torus rows as row pairs (2i, 2i + 1): pair j < kept_pairs is i = j + floor(a_min
// / 2) modulo n1 / 2 (the first and the last may hold one kept row).
__device__ inline int first_pair(const ColArgs &a) { return -((1 - a.a_min) / 2); }
__device__ inline int kept_pairs(const ColArgs &a)
{
    return (a.a_min + a.nrows - 1) / 2 - first_pair(a) + 1;
}
__device__ inline int pair_row(int j, const ColArgs &a, int nh)
{
    const int i = j + first_pair(a);
    return i < 0 ? i + nh : i;
}

// Register slots for the kept pairs of one column where nh <= MAXV threads: at most
// nh / 2 + w / 2 + 2 pairs (w <= 16).
template <int MAXV>
constexpr int kept_slots()
{
    return MAXV / 2 + 1;
}

// Rows 2i (value ev) and 2i + 1 (od) of an E column, those of them the grid keeps;
// one 2-element store when both are kept (E columns have even length, so the pair is
// aligned to its own size).
template <typename C>
__device__ inline void store_rows(C *ec, int i, C ev, C od, const ColArgs &a)
{
    using C2 = typename cx2<C>::type;
    const bool ke = row_kept(2 * i, a.n1, a.nrows, a.a_min);
    const bool ko = row_kept(2 * i + 1, a.n1, a.nrows, a.a_min);
    if (ke && ko) {
        C2 p;
        p.x = ev.x;
        p.y = ev.y;
        p.z = od.x;
        p.w = od.y;
        reinterpret_cast<C2 *>(ec)[i] = p;
    } else if (ke) {
        ec[2 * i] = ev;
    } else if (ko) {
        ec[2 * i + 1] = od;
    }
}

// Rows 2i and 2i + 1 of an E column as (ev, od), zero where the grid keeps no row.
template <typename C>
__device__ inline void load_rows(const C *ec, int i, C &ev, C &od, const ColArgs &a)
{
    using C2 = typename cx2<C>::type;
    const bool ke = row_kept(2 * i, a.n1, a.nrows, a.a_min);
    const bool ko = row_kept(2 * i + 1, a.n1, a.nrows, a.a_min);
    ev.x = ev.y = od.x = od.y = 0;
    if (ke && ko) {
        const C2 p = reinterpret_cast<const C2 *>(ec)[i];
        ev.x = p.x;
        ev.y = p.y;
        od.x = p.z;
        od.y = p.w;
    } else if (ke) {
        ev = ec[2 * i];
    } else if (ko) {
        od = ec[2 * i + 1];
    }
}

// Mode 2 takes two neighbouring columns per workgroup.  The doubled meridian of column m
// is f_m(-theta) = sigma_m f_m(theta) with sigma_m = (-1)^(s + m), so of the columns m and
// m + 1 one is even and one odd, and so are their transforms (the deconvolution in theta
// is even in k): the two run as one complex transform z = f_m + f_{m+1} and separate at
// the end by f_m[a] = (z[a] + sigma_m z[-a]) / 2, f_{m+1}[a] = (z[a] - sigma_m z[-a]) / 2.
// The two thereby share the transforms' rounding, relative to the larger of them (an empty
// column next to a full one is no longer exactly zero); the phi transform, which follows or
// precedes, mixes all columns at the same level, and the errors of whole calls against 64
// bits did not move.
// D then holds the ntheta rings alone, not the doubled meridian.  Half the transforms and half the traffic of D; at lmax
// 4096, sigma 2: FP64 1.90 -> 1.12 ms forward, 1.80 -> 1.18 ms adjoint (sigma 1.5, FP32:
// 0.90 -> 0.48 and 0.96 -> 0.59 ms).
//
// Forward, D columns -> E columns (kept rows).  The oversampled theta transform is
// split by output parity: with nh = n1 / 2 and the spectrum c_k, |k| <= lmax,
//   E[2a'] = sum_k c_k e^{2 pi i k a' / nh},  E[2a' + 1] = sum_k (c_k t^k) e^{2 pi i k a' / nh},
// t = e^{2 pi i / n1}: two length-nh transforms of the spectra folded modulo nh (at
// most two k per residue, since nh > lmax), so the LDS buffer holds max(nd, nh)
// values.  twist[k] = e^{-2 pi i k / n1}, k < n1.
template <typename T, int NT, int MAXV>
__global__ __launch_bounds__(NT, COL_HALF_WAVES) void column_fwd_half_kernel(
    const typename cx<T>::type *__restrict__ D, typename cx<T>::type *__restrict__ E, ColArgs a,
    ColFFT fd, ColFFT fh, const typename cx<T>::type *__restrict__ twist)
{
    using C = typename cx<T>::type;
    constexpr int HV = kept_slots<MAXV>();
    extern __shared__ unsigned char smem_raw[];
    C *X = reinterpret_cast<C *>(smem_raw);
    const int sh = fd.psh;  // LDS padding shift
    const int c0 = 2 * blockIdx.x, tid = threadIdx.x, nh = fh.n;
    const bool two = c0 + 1 < a.ncol;
    const int m0 = col_m(a, c0);
    const T sg = ((a.spin + m0) & 1) ? (T)-1 : (T)1;
    const double f0 = 0.5 * a.kf2[m0 < 0 ? -m0 : m0];
    const double f1 = two ? 0.5 * a.kf2[m0 + 1 < 0 ? -(m0 + 1) : m0 + 1] : 0.0;
    const C *d0 = D + (size_t)c0 * a.ds, *d1 = d0 + a.ds;
    C *e0 = E + (size_t)c0 * a.n1, *e1 = e0 + a.n1;
    const int half = a.nd / 2;
    for (int i = tid; i <= half; i += NT) {
        const C x = d0[i];
        C y;
        y.x = y.y = 0;
        if (two)
            y = d1[i];
        X[lds_pos(i, sh)] = cadd(x, y);
        if (i > 0 && i < half) {
            C z = csub(x, y);
            z.x *= sg;
            z.y *= sg;
            X[lds_pos(a.nd - i, sh)] = z;
        }
    }
    __syncthreads();
    lds_fft<C, -1, NT>(X, fd);
    auto chat = [&](int k) {
        return scale_c(X[lds_pos(fd.perm[k < 0 ? k + a.nd : k], sh)], a.kf1[k < 0 ? -k : k]);
    };
    // Fold: residue i < nh receives c_i (i <= lmax) and c_{i - nh} (i >= nh - lmax);
    // absent terms count as zero.  The even-row input is ye = c_i + c_{i-nh}, the
    // odd-row input t^i (c_i - c_{i-nh}) (t^{-nh} = -1).  Both are formed in
    // registers before the odd input overwrites the spectrum in LDS; ye stays there
    // until the even transform.
    const int ov0 = nh - a.lmax;
    C ye[MAXV], yd[MAXV];
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        ye[v].x = ye[v].y = 0;
        yd[v] = ye[v];
        if (i < nh) {
            C c1, c2;
            c1.x = c1.y = 0;
            c2 = c1;
            if (i <= a.lmax)
                c1 = chat(i);
            if (i >= ov0)
                c2 = chat(i - nh);
            ye[v] = cadd(c1, c2);
            yd[v] = csub(c1, c2);
        }
    }
    __syncthreads();
    // odd rows
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        if (i < nh)
            X[lds_pos(i, sh)] = cmulc(yd[v], twist[i]);
    }
    __syncthreads();
    lds_fft<C, 1, NT>(X, fh);
    // f0 (z[i] + sg z[j]) and f1 (z[i] - sg z[j]) of the transform in LDS
    auto split = [&](int i, int j, C &v0, C &v1) {
        const C p = X[lds_pos(fh.perm[i], sh)];
        C q = X[lds_pos(fh.perm[j], sh)];
        q.x *= sg;
        q.y *= sg;
        v0 = scale_c(cadd(p, q), f0);
        v1 = scale_c(csub(p, q), f1);
    };
    // the odd rows (row 2i + 1 mirrors row 2 (nh - 1 - i) + 1) wait in registers until
    // the even rows are done, so that rows 2i and 2i + 1 leave as one contiguous store
    const int np = kept_pairs(a);
    C o0[HV], o1[HV];
#pragma unroll
    for (int v = 0; v < HV; ++v) {
        const int j = tid + v * NT;
        o0[v].x = o0[v].y = 0;
        o1[v] = o0[v];
        if (j < np) {
            const int i = pair_row(j, a, nh);
            split(i, nh - 1 - i, o0[v], o1[v]);
        }
    }
    __syncthreads();
    // even rows
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        if (i < nh)
            X[lds_pos(i, sh)] = ye[v];
    }
    __syncthreads();
    lds_fft<C, 1, NT>(X, fh);
#pragma unroll
    for (int v = 0; v < HV; ++v) {
        const int j = tid + v * NT;
        if (j < np) {
            const int i = pair_row(j, a, nh);
            C v0, v1;
            split(i, i ? nh - i : 0, v0, v1);
            store_rows(e0, i, v0, o0[v], a);
            if (two)
                store_rows(e1, i, v1, o1[v], a);
        }
    }
}

// Mode 2, E columns (kept rows; the rest counts as zero) -> D columns: the transpose
// of column_fwd_half_kernel (odd rows first, then even rows).  The rows of each column
// are first made even or odd, (g[a] + sigma g[-a]) / 2, which leaves the ring values
// H(j) = y[j] + sigma y[-j] unchanged: each kept row puts half its value, times the
// column's kfac2, into its own place and sigma times that into its mirror's.  (Where
// sigma = -1 the pole entries become 0; the harmonics vanish there.)
template <typename T, int NT, int MAXV>
__global__ __launch_bounds__(NT, COL_HALF_WAVES) void column_adj_half_kernel(
    const typename cx<T>::type *__restrict__ E, typename cx<T>::type *__restrict__ D, ColArgs a,
    ColFFT fd, ColFFT fh, const typename cx<T>::type *__restrict__ twist)
{
    using C = typename cx<T>::type;
    constexpr int HV = kept_slots<MAXV>();
    extern __shared__ unsigned char smem_raw[];
    C *X = reinterpret_cast<C *>(smem_raw);
    const int sh = fd.psh;  // LDS padding shift
    const int c0 = 2 * blockIdx.x, tid = threadIdx.x, nh = fh.n;
    const bool two = c0 + 1 < a.ncol;
    const int m0 = col_m(a, c0);
    const T sg = ((a.spin + m0) & 1) ? (T)-1 : (T)1;
    const double f0 = 0.5 * a.kf2[m0 < 0 ? -m0 : m0];
    const double f1 = two ? 0.5 * a.kf2[m0 + 1 < 0 ? -(m0 + 1) : m0 + 1] : 0.0;
    const C *e0 = E + (size_t)c0 * a.n1, *e1 = e0 + a.n1;
    C *d0 = D + (size_t)c0 * a.ds, *d1 = d0 + a.ds;
    // theta frequency k of output i (|k| <= lmax contributes) and its residue mod nh
    auto freq = [&](int i, int &k, int &kh) {
        k = (i <= a.nd / 2) ? i : i - a.nd;
        kh = k % nh;
        if (kh < 0)
            kh += nh;
        return (k < 0 ? -k : k) <= a.lmax;
    };
    const int np = kept_pairs(a);
    // X <- packed rows: x0 + x1 of row pair j at i, then sigma (x0 - x1) added at the
    // mirror of i (the kept places cover each i at most once, and so do the mirrors)
    auto put_packed = [&](const C (&x0)[HV], const C (&x1)[HV], auto mirror) {
        for (int i = np + tid; i < nh; i += NT) {
            C z;
            z.x = z.y = 0;
            X[lds_pos(pair_row(i, a, nh) % nh, sh)] = z;
        }
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            const int j = tid + v * NT;
            if (j < np && j < nh)
                X[lds_pos(pair_row(j, a, nh) % nh, sh)] = cadd(x0[v], x1[v]);
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            const int j = tid + v * NT;
            if (j < np && j < nh) {
                const int k = mirror(pair_row(j, a, nh) % nh);
                C z = csub(x0[v], x1[v]);
                z.x *= sg;
                z.y *= sg;
                X[lds_pos(k, sh)] = cadd(X[lds_pos(k, sh)], z);
            }
        }
        __syncthreads();
    };
    // rows 2i and 2i + 1 arrive as one load; the odd rows go first, the even rows
    // wait in registers
    C ev0[HV], ev1[HV];
    {
        C od0[HV], od1[HV];
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            const int j = tid + v * NT;
            ev0[v].x = ev0[v].y = 0;
            ev1[v] = od0[v] = od1[v] = ev0[v];
            if (j < np) {
                const int i = pair_row(j, a, nh);
                load_rows(e0, i, ev0[v], od0[v], a);
                if (two)
                    load_rows(e1, i, ev1[v], od1[v], a);
                ev0[v] = scale_c(ev0[v], f0);
                od0[v] = scale_c(od0[v], f0);
                ev1[v] = scale_c(ev1[v], f1);
                od1[v] = scale_c(od1[v], f1);
            }
        }
        put_packed(od0, od1, [&](int i) { return nh - 1 - i; });
    }
    lds_fft<C, -1, NT>(X, fh);
    C acc[MAXV];
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        acc[v].x = acc[v].y = 0;
        int k, kh;
        if (i < a.nd && freq(i, k, kh))
            acc[v] = cmul(X[lds_pos(fh.perm[kh], sh)], twist[k < 0 ? k + a.n1 : k]);
    }
    __syncthreads();
    // even rows
    put_packed(ev0, ev1, [&](int i) { return i ? nh - i : 0; });
    lds_fft<C, -1, NT>(X, fh);
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        int k, kh;
        if (i < a.nd && freq(i, k, kh))
            acc[v] = scale_c(cadd(acc[v], X[lds_pos(fh.perm[kh], sh)]), a.kf1[k < 0 ? -k : k]);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < MAXV; ++v) {
        const int i = tid + v * NT;
        if (i < a.nd)
            X[lds_pos(i, sh)] = acc[v];
    }
    __syncthreads();
    lds_fft<C, 1, NT>(X, fd);
    const int half = a.nd / 2;
    for (int j = tid; j <= half; j += NT) {
        const C p = X[lds_pos(fd.perm[j], sh)];
        C q;
        q.x = q.y = 0;
        if (j > 0 && j < half)
            q = X[lds_pos(fd.perm[a.nd - j], sh)];
        q.x *= sg;
        q.y *= sg;
        const bool pole = j == 0 || j == half;
        C h0 = cadd(p, q), h1 = csub(p, q);
        if (pole && sg < 0)
            h0.x = h0.y = 0;
        if (pole && sg > 0)
            h1.x = h1.y = 0;
        d0[j] = h0;
        if (two)
            d1[j] = h1;
    }
}

// Mode 1, D column -> zero-padded, deconvolved spectrum over all n1 entries (the
// theta transform follows in the library FFT).
template <typename T>
__global__ __launch_bounds__(COL_THREADS) void column_fwd_kernel(
    const typename cx<T>::type *__restrict__ D, typename cx<T>::type *__restrict__ E, ColArgs a,
    ColFFT fd)
{
    using C = typename cx<T>::type;
    extern __shared__ unsigned char smem_raw[];
    C *X = reinterpret_cast<C *>(smem_raw);
    const int sh = fd.psh;  // LDS padding shift
    const int col = blockIdx.x, tid = threadIdx.x;
    const int m = col_m(a, col);
    const double fm = a.kf2[m < 0 ? -m : m];
    const C *dc = D + (size_t)col * a.nd;
    C *ec = E + (size_t)col * a.n1;
    for (int i = tid; i < a.nd; i += COL_THREADS)
        X[lds_pos(i, sh)] = dc[i];
    __syncthreads();
    lds_fft<C, -1, COL_THREADS>(X, fd);
    for (int i = tid; i < a.n1; i += COL_THREADS) {
        C o;
        o.x = 0;
        o.y = 0;
        const int k = (i <= a.n1 / 2) ? i : i - a.n1;
        const int ak = k < 0 ? -k : k;
        if (ak <= a.lmax)
            o = scale_c(X[lds_pos(fd.perm[k < 0 ? k + a.nd : k], sh)], a.kf1[ak] * fm);
        ec[i] = o;
    }
}

// Mode 1, theta spectrum E^ -> deconvolution and nd transform -> D column.
template <typename T>
__global__ __launch_bounds__(COL_THREADS) void column_adj_kernel(
    const typename cx<T>::type *__restrict__ E, typename cx<T>::type *__restrict__ D, ColArgs a,
    ColFFT fd)
{
    using C = typename cx<T>::type;
    extern __shared__ unsigned char smem_raw[];
    C *X = reinterpret_cast<C *>(smem_raw);
    const int sh = fd.psh;  // LDS padding shift
    const int col = blockIdx.x, tid = threadIdx.x;
    const int m = col_m(a, col);
    const double fm = a.kf2[m < 0 ? -m : m];
    const C *ec = E + (size_t)col * a.n1;
    C *dc = D + (size_t)col * a.nd;
    for (int i = tid; i < a.nd; i += COL_THREADS) {
        C o;
        o.x = 0;
        o.y = 0;
        const int k = (i <= a.nd / 2) ? i : i - a.nd;
        const int ak = k < 0 ? -k : k;
        if (ak <= a.lmax)
            o = scale_c(ec[k < 0 ? k + a.n1 : k], a.kf1[ak] * fm);
        X[lds_pos(i, sh)] = o;
    }
    __syncthreads();
    lds_fft<C, 1, COL_THREADS>(X, fd);
    for (int i = tid; i < a.nd; i += COL_THREADS)
        dc[i] = X[lds_pos(fd.perm[i], sh)];
}

ColArgs col_args(const gsht_plan &p)
{
    ColArgs a;
    a.kf1 = p.kfac1;
    a.kf2 = p.kfac2;
    a.lmax = p.lmax;
    a.mmax = p.mmax;
    a.spin = p.spin;
    a.ncol = p.ncol;
    a.nd = p.nd;
    a.ds = p.ds;
    a.n1 = p.n1;
    a.nrows = p.nrows;
    a.a_min = p.a_min;
    return a;
}

template <typename T>
size_t col_lds(const gsht_plan &p)
{
    const int sh = p.lds_psh;
    const int n = p.colmode == 2 ? lds_pad_n(col_half_lds_n(p.nd, p.n1 / 2), sh)
                                 : lds_pad_n(p.nd, sh);
    return sizeof(typename cx<T>::type) * (size_t)n;
}

// Threads of the mode-2 workgroups (one per pair of columns).  A pass of an n-point
// transform has n / 8 butterflies, so large workgroups leave most of their waves idle on
// short columns; but while all pairs fit the chip at once (1024 / NT workgroups per CU),
// more threads shorten each of them.  So: the most threads with which every pair is
// resident, and enough for 12 (FP32) or 9 (FP64) values per thread.  That is 256 to 1024
// threads (FP32: 512): more than 1024 pairs have columns too long for fewer than 256.
// Forward + adjoint, spin 2: FP64 lmax 512 (513 pairs) 256 threads 0.061, 512 0.081, 1024
// 0.106 ms; lmax 255 (256 pairs) 0.039, 0.037, 0.039; FP32 lmax 700 256 threads 0.064, 512
// 0.081 ms; lmax 1024 256 threads 0.107, 512 0.130 ms.
template <typename T>
int half_threads(const gsht_plan &p)
{
    constexpr int top = col_half_threads<T>(), per = sizeof(T) == 4 ? 12 : 9;
    const int nh = p.n1 / 2, n = p.nd > nh ? p.nd : nh, pairs = (p.ncol + 1) / 2;
    int nt = top;
    while (nt > 256 && pairs > 256 * (1024 / nt) && n <= per * (nt / 2))
        nt /= 2;
    return nt;
}

// Calls f(kernel, threads, slots) with the mode-2 instance for this plan, forward or
// adjoint.  MAXV register slots per thread hold the forward's n1 / 2 or the adjoint's
// max(nd, n1 / 2) values; slots beyond that cost registers (FP64 with the most, 10, spills
// 36 to scratch: at lmax 4096 the forward took 1.70 instead of 1.61 ms, single columns).
// The lists below hold the counts that accepted plans come to (n1 / 2 is 1, 3 or 5 times a
// power of two, so the forward skips some; its 10 needs columns without LDS padding).
template <typename T, bool ADJ, int NT, int MAXV, int... MORE, typename F>
hipError_t with_slots(int v, F &&f)
{
    if constexpr (sizeof...(MORE) > 0)
        if (v > MAXV)
            return with_slots<T, ADJ, NT, MORE...>(v, f);
    if (v > MAXV)
        return hipErrorInvalidValue;
    if constexpr (ADJ)
        return f(column_adj_half_kernel<T, NT, MAXV>, NT, MAXV);
    else
        return f(column_fwd_half_kernel<T, NT, MAXV>, NT, MAXV);
}

template <typename T, bool ADJ, typename F>
hipError_t with_half(const gsht_plan &p, F &&f)
{
    const int nt = half_threads<T>(p), nh = p.n1 / 2;
    const int v = ((ADJ && p.nd > nh ? p.nd : nh) + nt - 1) / nt;
    if constexpr (sizeof(T) == 4) {
        if (nt == 256)
            return with_slots<T, ADJ, 256, 9, 12>(v, f);
        return with_slots<T, ADJ, 512, 9, 12, 17>(v, f);
    } else if constexpr (ADJ) {
        switch (nt) {
        case 256: return with_slots<T, ADJ, 256, 6, 8, 9>(v, f);
        case 512: return with_slots<T, ADJ, 512, 6, 8, 9>(v, f);
        default: return with_slots<T, ADJ, 1024, 4, 5, 6, 7, 8, 9, 10>(v, f);
        }
    } else {
        switch (nt) {
        case 256: return with_slots<T, ADJ, 256, 6, 8>(v, f);
        case 512: return with_slots<T, ADJ, 512, 6, 8>(v, f);
        default: return with_slots<T, ADJ, 1024, 4, 5, 6, 8, 10>(v, f);
        }
    }
}

template <typename T>
hipError_t set_lds(const gsht_plan &p)
{
    const int b = (int)col_lds<T>(p);
    hipError_t e;
    if (p.colmode == 2) {
        auto attr = [&](auto kern, int, int) {
            return hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, b);
        };
        e = with_half<T, false>(p, attr);
        if (e == hipSuccess)
            e = with_half<T, true>(p, attr);
    } else {
        e = hipFuncSetAttribute((const void *)column_fwd_kernel<T>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, b);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)column_adj_kernel<T>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, b);
    }
    return e;
}

template <typename T>
void launch_fwd(const gsht_plan &p, hipStream_t s)
{
    using C = typename cx<T>::type;
    const ColArgs a = col_args(p);
    const size_t b = col_lds<T>(p);
    if (p.colmode == 2) {
        (void)with_half<T, false>(p, [&](auto kern, int nt, int) {
            hipLaunchKernelGGL(kern, dim3((p.ncol + 1) / 2), dim3(nt), b, s, (const C *)p.D, (C *)p.E, a,
                               p.cf_d, p.cf_h, (const C *)p.twist);
            return hipSuccess;
        });
    } else {
        hipLaunchKernelGGL((column_fwd_kernel<T>), dim3(p.ncol), dim3(COL_THREADS), b, s,
                           (const C *)p.D, (C *)p.E, a, p.cf_d);
    }
}

template <typename T>
void launch_adj(const gsht_plan &p, hipStream_t s)
{
    using C = typename cx<T>::type;
    const ColArgs a = col_args(p);
    const size_t b = col_lds<T>(p);
    if (p.colmode == 2) {
        (void)with_half<T, true>(p, [&](auto kern, int nt, int) {
            hipLaunchKernelGGL(kern, dim3((p.ncol + 1) / 2), dim3(nt), b, s, (const C *)p.E, (C *)p.D, a,
                               p.cf_d, p.cf_h, (const C *)p.twist);
            return hipSuccess;
        });
    } else {
        hipLaunchKernelGGL((column_adj_kernel<T>), dim3(p.ncol), dim3(COL_THREADS), b, s,
                           (const C *)p.E, (C *)p.D, a, p.cf_d);
    }
}

}  // namespace

hipError_t column_set_lds(const gsht_plan &p)
{
    return p.prec == GSHT_F64 ? set_lds<double>(p) : set_lds<float>(p);
}

int column_half_maxn(int prec) { return prec == GSHT_F64 ? col_half_maxn<double>() : col_half_maxn<float>(); }

int column_max_radix(int) { return COL_MAXR; }

void column_shape(const gsht_plan &p, int &threads, int &fwd, int &adj)
{
    auto get = [&](int &slots) {
        return [&](auto, int nt, int v) {
            threads = nt;
            slots = v;
            return hipSuccess;
        };
    };
    threads = fwd = adj = 0;
    if (p.colmode != 2)
        return;
    if (p.prec == GSHT_F64) {
        (void)with_half<double, false>(p, get(fwd));
        (void)with_half<double, true>(p, get(adj));
    } else {
        (void)with_half<float, false>(p, get(fwd));
        (void)with_half<float, true>(p, get(adj));
    }
}

size_t column_lds_bytes(const gsht_plan &p)
{
    return p.prec == GSHT_F64 ? col_lds<double>(p) : col_lds<float>(p);
}

hipError_t launch_column_fwd(const gsht_plan &p, hipStream_t s)
{
    if (p.prec == GSHT_F64)
        launch_fwd<double>(p, s);
    else
        launch_fwd<float>(p, s);
    return hipGetLastError();
}

hipError_t launch_column_adj(const gsht_plan &p, hipStream_t s)
{
    if (p.prec == GSHT_F64)
        launch_adj<double>(p, s);
    else
        launch_adj<float>(p, s);
    return hipGetLastError();
}

}  // namespace gsht
