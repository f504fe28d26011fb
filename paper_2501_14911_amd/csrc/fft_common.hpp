// Pieces shared by the runtime-length and the fixed-length FFT kernels:
// small DFT butterflies (radices 2, 3, 4, 5, 7, 8 and the composite 10, 20, 21,
// 25 of the compiled lengths), the real split on bin pairs, the workgroup-to-tile
// map, resident grids and the active length of a right-hand side.
#pragma once
#include <algorithm>

#include "common.hpp"

namespace p2o {

// ---------------------------------------------------------------- butterflies
// cos(2 pi m / R) and sin(2 pi m / R), m = 1 .. (R - 1) / 2, for the odd
// prime radices (to 21 significant digits).
template <typename T, int R>
__device__ __forceinline__ constexpr T prime_cos(int m) {
    if constexpr (R == 3) return T(-0.5);
    if constexpr (R == 5) return m == 1 ? T(0.309016994374947424102) : T(-0.809016994374947424102);
    return m == 1 ? T(0.623489801858733530525) : m == 2 ? T(-0.222520933956314404289) : T(-0.900968867902419126236);
}
template <typename T, int R>
__device__ __forceinline__ constexpr T prime_sin(int m) {
    if constexpr (R == 3) return T(0.866025403784438646764);
    if constexpr (R == 5) return m == 1 ? T(0.951056516295153572116) : T(0.587785252292473129169);
    return m == 1 ? T(0.781831482468029808708) : m == 2 ? T(0.974927912181823607018) : T(0.433883739117558120476);
}

// cos and sin of 2 pi m / R at compile time (Taylor series after reduction to at
// most pi / 4), for the inner twiddles of the composite radices.
constexpr double kPi = 3.14159265358979323846264338327950288;
constexpr double series_sin(double x) {
    double t = x, s = x;
    for (int k = 1; k < 14; ++k) { t *= -x * x / ((2 * k) * (2 * k + 1)); s += t; }
    return s;
}
constexpr double series_cos(double x) {
    double t = 1.0, s = 1.0;
    for (int k = 1; k < 14; ++k) { t *= -x * x / ((2 * k - 1) * (2 * k)); s += t; }
    return s;
}
constexpr double root_cos(int m, int R) {             // cos(2 pi m / R), 0 <= m < R
    if (2 * m > R) return root_cos(R - m, R);
    if (4 * m > R) return -root_cos(R - 2 * m, 2 * R);
    return 8 * m > R ? series_sin(kPi * (R - 4 * m) / (2.0 * R)) : series_cos(2.0 * kPi * m / R);
}
constexpr double root_sin(int m, int R) {
    if (2 * m > R) return -root_sin(R - m, R);
    if (4 * m > R) return root_sin(R - 2 * m, 2 * R);
    return 8 * m > R ? series_cos(kPi * (R - 4 * m) / (2.0 * R)) : series_sin(2.0 * kPi * m / R);
}
struct Roots25 {                                       // of e^{-2 pi i m / 25}, m <= 16
    double c[17], s[17];
};
constexpr Roots25 roots25() {
    Roots25 r{};
    for (int m = 0; m < 17; ++m) {
        r.c[m] = root_cos(m, 25);
        r.s[m] = root_sin(m, 25);
    }
    return r;
}
constexpr int inverse_mod(int a, int m) {
    for (int x = 1; x < m; ++x)
        if (a * x % m == 1) return x;
    return 0;
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_small(cplx<T>* a) {
    using Z = cplx<T>;
    if constexpr (R == 10 || R == 20 || R == 21) {
        // coprime factors A B: with inputs n = (B p + A q) mod R and outputs k = p mod
        // A = q mod B, A transforms of B and B of A without twiddles in between
        // (Good-Thomas)
        constexpr int A = R == 10 ? 2 : R == 20 ? 4 : 3, B = R / A;
        constexpr int ea = B * inverse_mod(B % A, A), eb = A * inverse_mod(A % B, B);
        Z v[A][B];
#pragma unroll
        for (int p = 0; p < A; ++p) {
#pragma unroll
            for (int q = 0; q < B; ++q) v[p][q] = a[(B * p + A * q) % R];
            dft_small<T, B, INV>(v[p]);
        }
#pragma unroll
        for (int q = 0; q < B; ++q) {
            Z c[A];
#pragma unroll
            for (int p = 0; p < A; ++p) c[p] = v[p][q];
            dft_small<T, A, INV>(c);
#pragma unroll
            for (int p = 0; p < A; ++p) a[(ea * p + eb * q) % R] = c[p];
        }
    } else if constexpr (R == 25) {
        // 5 x 5: inputs 5 p + q, a transform over p, twiddles e^{-2 pi i q k / 25}, a
        // transform over q, outputs k + 5 l
        constexpr Roots25 W = roots25();
        Z v[5][5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
#pragma unroll
            for (int p = 0; p < 5; ++p) v[q][p] = a[5 * p + q];
            dft_small<T, 5, INV>(v[q]);
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            Z c[5];
            c[0] = v[0][k];
#pragma unroll
            for (int q = 1; q < 5; ++q) {
                const T wr = (T)W.c[q * k], wi = (T)(INV ? W.s[q * k] : -W.s[q * k]);
                c[q] = k == 0 ? v[q][k] : cmk<T>(v[q][k].x * wr - v[q][k].y * wi, v[q][k].x * wi + v[q][k].y * wr);
            }
            dft_small<T, 5, INV>(c);
#pragma unroll
            for (int l = 0; l < 5; ++l) a[k + 5 * l] = c[l];
        }
    } else if constexpr (R == 2) {
        Z t = a[0];
        a[0] = cadd(t, a[1]);
        a[1] = csub(t, a[1]);
    } else if constexpr (R == 4) {
        Z t0 = cadd(a[0], a[2]), t1 = csub(a[0], a[2]);
        Z t2 = cadd(a[1], a[3]), t3 = csub(a[1], a[3]);
        a[0] = cadd(t0, t2);
        a[2] = csub(t0, t2);
        if constexpr (!INV) {   // multiply t3 by -i
            a[1] = cmk<T>(t1.x + t3.y, t1.y - t3.x);
            a[3] = cmk<T>(t1.x - t3.y, t1.y + t3.x);
        } else {                // multiply t3 by +i
            a[1] = cmk<T>(t1.x - t3.y, t1.y + t3.x);
            a[3] = cmk<T>(t1.x + t3.y, t1.y - t3.x);
        }
    } else if constexpr (R == 8) {
        Z e[4] = {a[0], a[2], a[4], a[6]};
        Z o[4] = {a[1], a[3], a[5], a[7]};
        dft_small<T, 4, INV>(e);
        dft_small<T, 4, INV>(o);
        const T c = T(0.70710678118654752440084436210485);   // sqrt(2)/2
        Z o1, o2, o3;
        if constexpr (!INV) {   // e^{-i pi p / 4} o_p
            o1 = cmk<T>(c * (o[1].x + o[1].y), c * (o[1].y - o[1].x));
            o2 = cmk<T>(o[2].y, -o[2].x);
            o3 = cmk<T>(c * (o[3].y - o[3].x), -c * (o[3].x + o[3].y));
        } else {                // e^{+i pi p / 4} o_p
            o1 = cmk<T>(c * (o[1].x - o[1].y), c * (o[1].x + o[1].y));
            o2 = cmk<T>(-o[2].y, o[2].x);
            o3 = cmk<T>(-c * (o[3].x + o[3].y), c * (o[3].x - o[3].y));
        }
        a[0] = cadd(e[0], o[0]); a[4] = csub(e[0], o[0]);
        a[1] = cadd(e[1], o1);   a[5] = csub(e[1], o1);
        a[2] = cadd(e[2], o2);   a[6] = csub(e[2], o2);
        a[3] = cadd(e[3], o3);   a[7] = csub(e[3], o3);
    } else {
        // odd prime radix.  With s_q = a_q + a_{R-q}, d_q = a_q - a_{R-q} and
        // theta = 2 pi p q / R, output p of the forward DFT is
        //   a_0 + sum_q s_q cos(theta) - i sum_q d_q sin(theta)
        // and output R - p the same with + i (q, p = 1 .. (R - 1) / 2): real
        // coefficients instead of complex roots, a third of the multiplies.
        constexpr int H = (R - 1) / 2;
        Z sm[H + 1], df[H + 1];
        Z a0 = a[0], out0 = a[0];
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            sm[q] = cadd(a[q], a[R - q]);
            df[q] = csub(a[q], a[R - q]);
            out0 = cadd(out0, sm[q]);
        }
#pragma unroll
        for (int p = 1; p <= H; ++p) {
            T ar = a0.x, ai = a0.y, br = T(0), bi = T(0);
#pragma unroll
            for (int q = 1; q <= H; ++q) {
                const int m = (p * q) % R;
                const T c = prime_cos<T, R>(m <= H ? m : R - m);
                const T sn = m <= H ? prime_sin<T, R>(m) : -prime_sin<T, R>(R - m);
                ar += c * sm[q].x;
                ai += c * sm[q].y;
                br += sn * df[q].x;
                bi += sn * df[q].y;
            }
            if constexpr (!INV) {
                a[p] = cmk<T>(ar + bi, ai - br);
                a[R - p] = cmk<T>(ar - bi, ai + br);
            } else {
                a[p] = cmk<T>(ar - bi, ai + br);
                a[R - p] = cmk<T>(ar + bi, ai - br);
            }
        }
        a[0] = out0;
    }
}


// ---------------------------------------------------------------- real <-> half spectrum, by bin pairs
// Bins k and M - k share their sums, differences and twiddle product (W^(M-k) =
// -conj W^k), so a pair costs 14 operations instead of 28.  hw = W^k / 2: the
// factor 1 / 2 of either direction is in the table and in the multiply-adds, which
// cost what additions do, so that no intermediate is larger than the transform's
// own (a factor left to a later scaling would halve the largest series that the
// precision can hold).
// Inverse pre-step: Z[k] = e + i o, Z[M-k] = conj e + i conj o, with e = (X[k] +
// conj X[M-k]) / 2, o = conj(W^k) (X[k] - conj X[M-k]) / 2.
template <typename T>
__device__ __forceinline__ void pre_pair(cplx<T> a, cplx<T> b, cplx<T> hw, cplx<T>& zk, cplx<T>& zm) {
    const T h = T(0.5), ex = a.x + b.x, ey = a.y - b.y;
    const cplx<T> o = cmul(cconj(hw), cmk<T>(a.x - b.x, a.y + b.y));
    zk = cmk<T>(h * ex - o.y, h * ey + o.x);
    zm = cmk<T>(h * ex + o.y, o.x - h * ey);
}

// Forward post-step: X[k] = s - i t, X[M-k] = conj s - i conj t, with s = (Z[k] +
// conj Z[M-k]) / 2, t = W^k (Z[k] - conj Z[M-k]) / 2.
template <typename T>
__device__ __forceinline__ void post_pair(cplx<T> a, cplx<T> b, cplx<T> hw, cplx<T>& xk, cplx<T>& xm) {
    const T h = T(0.5), sx = a.x + b.x, sy = a.y - b.y;
    const cplx<T> t = cmul(hw, cmk<T>(a.x - b.x, a.y + b.y));
    xk = cmk<T>(h * sx + t.y, h * sy - t.x);
    xm = cmk<T>(h * sx - t.y, -(h * sy) - t.x);
}

// ---------------------------------------------------------------- work items
// Workgroup id -> (tile, outer) such that consecutive ids on one XCD (ids are
// dealt to the 8 XCDs round-robin) take adjacent column tiles and share L2 lines.
struct ItemMap {
    int ntiles;   // column tiles per outer index
    int items;    // ntiles * outer count
    int Q;        // ceil(items / 8)
};

inline ItemMap item_map(int S, int sh, int outer) {     // S series per outer index in tiles of 1 << sh
    ItemMap im;
    im.ntiles = (S + (1 << sh) - 1) >> sh;
    im.items = im.ntiles * outer;
    im.Q = (im.items + 7) / 8;
    return im;
}

// Grid of the persistent kernels: `occ` resident workgroups on each CU, at most 8 Q.
inline dim3 resident_grid(int occ, const ItemMap& im) {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        ncu = 256;
    return dim3(8 * (unsigned)std::max(1, std::min(im.Q, (occ * ncu + 7) / 8)));
}

__device__ __forceinline__ bool fft_item(const ItemMap& im, int& tile, int& outer) {
    const int q = (int)(blockIdx.x & 7) * im.Q + (int)(blockIdx.x >> 3);
    if (q >= im.items) return false;
    outer = q / im.ntiles;
    tile = q - outer * im.ntiles;
    return true;
}

__device__ __forceinline__ int active_len(const SeriesIO& io, int outer) {
    int nt = io.Nt;
    if (io.nt_active) {
        const int a = io.nt_active[outer];
        nt = a < 0 ? 0 : (a < nt ? a : nt);
    }
    return nt;
}


// Misfit epilogue of the inverse transform (see k_c2r).
struct MisfitArgs {
    const void* d_obs;       // [outer][t][col], I/O type
    const double* var;       // noise variances
    int var_mode;            // 0: scalar, 1: per column (sensor), 2: per (t, col)
    double* partials;
};

enum { EPI_PLAIN = 0, EPI_MISFIT = 1 };

}  // namespace p2o
