// Batched real FFTs along time for many series, any transform length.
//
// The same transforms as the runtime-length kernels in fft.hip (section 4's
// circulant embedding; a tile of TW adjacent series x all bins in LDS, each
// real series of length L = 2M as one complex series of length M, Stockham
// passes of the plan's radices), for the parameter side, whose time is that of
// its memory accesses: a tile of 4 FP64 or 8 FP32 series reads 32-byte runs of
// a time step and writes 64-byte runs of a bin, which ran at 2.0-2.5 and 3.1
// TB/s where 128-byte runs reach 4-5.5.  So
//  - tiles are 32 (FP32) or 16 series wide where two of them fit a CU's LDS and
//    registers, half of that and a quarter for longer transforms, on 512-thread
//    workgroups (256 for short transforms);
//  - workgroups are persistent, so the twiddle tables (e^{-2 pi i n / M} for
//    the passes, e^{-2 pi i k / L}, k <= M / 2, for the real split) are staged
//    once; the split takes bins k and M - k together;
//  - the forward transform's first pass reads the time series and the inverse
//    transform's last pass writes them, and the re-pad, whose inverse runs the
//    radices in reverse order, merges its last inverse pass, the truncation and
//    its first forward pass in registers.
// Lengths with a compiled kernel (fft_fixed.hip) keep that one: 1.2-1.5 times as
// fast in FP32, whose time is its integer and LDS work as well (M = 420, 32 x
// 16384 series: r2c 0.63 against 0.89 ms, c2r 0.76 against 0.94, re-pad 0.98 against
// 1.47).  In FP64 it depends on the length (r2c / c2r / re-pad, ms, compiled against
// these kernels, 32 x 16384 series): M = 16, 0.04 / 0.04 / 0.05 against 0.11 / 0.11 /
// 0.18; M = 128, 0.33 / 0.49 / 0.53 against 0.34 / 0.41 / 0.51; M = 420, 1.67 / 2.02 /
// 2.32 against 1.50 / 1.62 / 2.58; M = 500, whose compiled FP64 tiles are 2 series
// wide, 4.51 / 3.11 / 4.26 against 2.07 / 2.22 / 3.39 (16 x 1000 series: 0.053 / 0.051 /
// 0.092 against 0.057 / 0.063 / 0.106).  The one order for both types is as it was before
// these kernels: FP64 batches of many series at M = 420 and 500 would gain here.
// gfx950, against the 4 to 8-series tiles: FP64, M = 250, 32 x 16384 series, r2c
// 1.25 -> 0.84, c2r 1.23 -> 0.88, re-pad 2.09 -> 1.42 ms (3.7, 3.6 and 2.9 TB/s);
// FP32, M = 243, 1.18 -> 0.51, 1.02 -> 0.54, 1.80 -> 0.89 ms; M = 375, 16 x 10007
// series, 0.43 -> 0.28, 0.37 -> 0.30, 0.64 -> 0.44 ms.
#include <algorithm>

#include "common.hpp"
#include "fft_common.hpp"
#include "kernels.hpp"

namespace p2o {
namespace {

constexpr size_t kWideLds = 80 * 1024;                   // two workgroups per CU
// Tiles that a launch should have at least: two for each CU (M = 243, FP32, 4096
// series, re-pad: 23.5 us with this line at 512, 28 at 256 and at 1024).
constexpr int kWideTiles = 512;

// Complex tile entries per thread.
template <typename T> constexpr int kMaxV = sizeof(T) == 4 ? 16 : 8;

template <typename E>
__device__ __forceinline__ E ld(const E* base, uint32_t off) {
    return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(base) + off);
}
template <typename E>
__device__ __forceinline__ void st(E* base, uint32_t off, E v) {
    *reinterpret_cast<E*>(reinterpret_cast<char*>(base) + off) = v;
}

template <int SH> constexpr int kRS = (1 << SH) + 1;     // LDS row stride (odd: spreads banks)
template <int SH, int NT> constexpr int kJS = NT >> SH;  // bins or butterflies per sweep of the workgroup

// j / d for j < 2^16 (uniform magic of d).
__device__ __forceinline__ int div_by(int j, int d, uint32_t magic) {
    return d > 1 ? (int)__umulhi((uint32_t)j, magic) : j;
}

// Butterflies j = j0 + u JS of one pass from the tile, twiddled.
template <typename T, int SH, int NT, int R, bool INV, int NU>
__device__ __forceinline__ void gather(cplx<T> (&v)[NU][R], const cplx<T>* buf, const cplx<T>* tm, int M, int Ns,
                                       uint32_t magic, int s, int j0) {
    using Z = cplx<T>;
    const int MR = M / R, step = MR / Ns;
    const Z* rb = buf + j0 * kRS<SH> + s;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int j = j0 + u * kJS<SH, NT>;
        if (j < MR) {
#pragma unroll
            for (int q = 0; q < R; ++q) v[u][q] = rb[(u * kJS<SH, NT> + q * MR) * kRS<SH>];
            if (Ns > 1) {
                const int k = (j - div_by(j, Ns, magic) * Ns) * step;
#pragma unroll
                for (int q = 1; q < R; ++q) {
                    const Z t = tm[q * k];
                    v[u][q] = cmul(v[u][q], INV ? cconj(t) : t);
                }
            }
        }
    }
}

template <typename T, int SH, int NT, int R, bool INV>
__device__ __forceinline__ void tile_pass(cplx<T>* buf, const cplx<T>* tm, int M, int Ns, int s, int j0) {
    using Z = cplx<T>;
    constexpr int NU = (kMaxV<T> + R - 1) / R;
    const uint32_t magic = Ns > 1 ? 0xFFFFFFFFu / (uint32_t)Ns + 1u : 0u;
    const int MR = M / R;
    Z v[NU][R];
    gather<T, SH, NT, R, INV, NU>(v, buf, tm, M, Ns, magic, s, j0);
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (j0 + u * kJS<SH, NT> < MR) dft_small<T, R, INV>(v[u]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int j = j0 + u * kJS<SH, NT>;
        if (j < MR) {
            const int k = j - div_by(j, Ns, magic) * Ns;
            Z* wb = buf + ((j - k) * R + k) * kRS<SH> + s;
#pragma unroll
            for (int p = 0; p < R; ++p) wb[p * Ns * kRS<SH>] = v[u][p];
        }
    }
    __syncthreads();
}

template <typename T, int SH, int NT, bool INV>
__device__ __forceinline__ void any_pass(int R, cplx<T>* buf, const cplx<T>* tm, int M, int Ns, int s, int j0) {
    switch (R) {
        case 2: tile_pass<T, SH, NT, 2, INV>(buf, tm, M, Ns, s, j0); break;
        case 3: tile_pass<T, SH, NT, 3, INV>(buf, tm, M, Ns, s, j0); break;
        case 4: tile_pass<T, SH, NT, 4, INV>(buf, tm, M, Ns, s, j0); break;
        case 5: tile_pass<T, SH, NT, 5, INV>(buf, tm, M, Ns, s, j0); break;
        case 7: tile_pass<T, SH, NT, 7, INV>(buf, tm, M, Ns, s, j0); break;
        default: tile_pass<T, SH, NT, 8, INV>(buf, tm, M, Ns, s, j0); break;
    }
}

// First forward pass (Ns = 1) of butterflies given by `fill(u, j, v)`, onto
// the tile; `free_tile`: wait for readers of the tile first.
template <typename T, int SH, int NT, int R, typename Fill>
__device__ __forceinline__ void first_pass(cplx<T>* buf, int M, int s, int j0, bool free_tile, Fill&& fill) {
    using Z = cplx<T>;
    constexpr int NU = (kMaxV<T> + R - 1) / R;
    const int MR = M / R;
    Z v[NU][R];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int j = j0 + u * kJS<SH, NT>;
        if (j < MR) fill(u, j, v[u]);
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (j0 + u * kJS<SH, NT> < MR) dft_small<T, R, false>(v[u]);
    if (free_tile) __syncthreads();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int j = j0 + u * kJS<SH, NT>;
        if (j < MR) {
            Z* wb = buf + j * R * kRS<SH> + s;
#pragma unroll
            for (int p = 0; p < R; ++p) wb[p * kRS<SH>] = v[u][p];
        }
    }
    __syncthreads();
}

// z[n] = x[2n] + i x[2n+1], x[t] = 0 for t >= nt or a series past S (ok false),
// through the first pass.
template <typename T, typename TIN, int SH, int NT, int R>
__device__ __forceinline__ void from_time(cplx<T>* buf, int M, const TIN* __restrict__ src, long long t_stride, bool ok,
                                          int nt, int s, int j0, bool* bad = nullptr) {
    const uint32_t ts = (uint32_t)t_stride * (uint32_t)sizeof(TIN);
    const uint32_t o0 = 2u * (uint32_t)j0 * ts + (uint32_t)s * (uint32_t)sizeof(TIN);
    const int MR = M / R;
    first_pass<T, SH, NT, R>(buf, M, s, j0, false, [&](int u, int j, cplx<T> (&v)[R]) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int t0 = 2 * (j + q * MR);
            const TIN* sb = src + (long long)(2 * (u * kJS<SH, NT> + q * MR)) * t_stride;
            T x0 = T(0), x1 = T(0);
            if (ok && t0 < nt) x0 = (T)ld(sb, o0);
            if (ok && t0 + 1 < nt) x1 = (T)ld(sb, o0 + ts);
            if (bad) *bad |= !isfinite(x0) || !isfinite(x1);
            v[q] = cmk<T>(x0, x1);
        }
    });
}

// Last inverse pass (Ns = M / R) to the time series, truncated to Nt steps and
// zero past the active length.
template <typename T, typename TOUT, int SH, int NT, int R>
__device__ __forceinline__ void to_time(const cplx<T>* buf, const cplx<T>* tm, int M, TOUT* __restrict__ dst,
                                        long long t_stride, bool ok, int nt, int Nt, int s, int j0) {
    using Z = cplx<T>;
    constexpr int NU = (kMaxV<T> + R - 1) / R;
    const int MR = M / R;
    const T inv = T(1) / T(M);
    const uint32_t ts = (uint32_t)t_stride * (uint32_t)sizeof(TOUT);
    const uint32_t o0 = 2u * (uint32_t)j0 * ts + (uint32_t)s * (uint32_t)sizeof(TOUT);
    Z v[NU][R];
    // j < MR = Ns: butterfly j has k = j
    gather<T, SH, NT, R, true, NU>(v, buf, tm, M, MR, MR > 1 ? 0xFFFFFFFFu / (uint32_t)MR + 1u : 0u, s, j0);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int j = j0 + u * kJS<SH, NT>;
        if (j < MR) {
            dft_small<T, R, true>(v[u]);
#pragma unroll
            for (int p = 0; p < R; ++p) {
                const int t0 = 2 * (j + p * MR);
                TOUT* db = dst + (long long)(2 * (u * kJS<SH, NT> + p * MR)) * t_stride;
                if (ok && t0 < Nt) st(db, o0, t0 < nt ? (TOUT)(v[u][p].x * inv) : TOUT(0));
                if (ok && t0 + 1 < Nt) st(db, o0 + ts, t0 + 1 < nt ? (TOUT)(v[u][p].y * inv) : TOUT(0));
            }
        }
    }
}

// The re-pad's merged pass: last inverse pass, truncation to the active length,
// first forward pass (both of radix R over the same index sets).
template <typename T, int SH, int NT, int R>
__device__ __forceinline__ void repad_pass(cplx<T>* buf, const cplx<T>* tm, int M, int nt, int s, int j0) {
    using Z = cplx<T>;
    const int MR = M / R;
    const T inv = T(1) / T(M);
    const Z* rb = buf + j0 * kRS<SH> + s;
    first_pass<T, SH, NT, R>(buf, M, s, j0, true, [&](int u, int j, Z (&v)[R]) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            v[q] = rb[(u * kJS<SH, NT> + q * MR) * kRS<SH>];
            if (q > 0) v[q] = cmul(v[q], cconj(tm[q * j]));
        }
        dft_small<T, R, true>(v);
#pragma unroll
        for (int p = 0; p < R; ++p) {
            const int t0 = 2 * (j + p * MR);
            v[p].x = t0 < nt ? v[p].x * inv : T(0);
            v[p].y = t0 + 1 < nt ? v[p].y * inv : T(0);
        }
    });
}

#define P2O_ANY_RADIX(R, CALL)          \
    switch (R) {                        \
        case 2: { constexpr int RR = 2; CALL; } break; \
        case 3: { constexpr int RR = 3; CALL; } break; \
        case 4: { constexpr int RR = 4; CALL; } break; \
        case 5: { constexpr int RR = 5; CALL; } break; \
        case 7: { constexpr int RR = 7; CALL; } break; \
        default: { constexpr int RR = 8; CALL; } break; \
    }

// Tables: tm[n] = e^{-2 pi i n / M} (n < M), tq[k] = e^{-2 pi i k / L} / 2 (k <= M / 2).
template <typename T, int NT>
__device__ __forceinline__ void stage_tables(cplx<T>* tm, cplx<T>* tq, const cplx<T>* __restrict__ twg, int M) {
    for (int n = threadIdx.x; n < M; n += NT) tm[n] = twg[2 * n];
    for (int k = threadIdx.x; k <= M / 2; k += NT) tq[k] = cscale(twg[k], T(0.5));
}

// Half spectra X[0..M] (partials summed in order; zero for a series past S)
// to Z[0..M-1] on the tile, bins k and M - k together.
template <typename T, int SH, int NT>
__device__ __forceinline__ void load_split(cplx<T>* buf, const cplx<T>* tq, int M, const cplx<T>* __restrict__ src,
                                           const SeriesIO& io, bool ok, int s, int j0) {
    using Z = cplx<T>;
    constexpr int NU = kMaxV<T> / 2 + 1, JS = kJS<SH, NT>;
    const int np = M / 2 + 1;
    const uint32_t fs = (uint32_t)io.f_stride * (uint32_t)sizeof(Z), so = (uint32_t)s * (uint32_t)sizeof(Z);
    const uint32_t oa = (uint32_t)j0 * fs + so, ob = (uint32_t)(JS - 1 - j0) * fs + so;
    Z xa[NU], xb[NU];
    auto read = [&](const Z* sp, Z (&va)[NU], Z (&vb)[NU]) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (j0 + u * JS < np) {
                va[u] = ld(sp + (long long)(u * JS) * io.f_stride, oa);
                vb[u] = ld(sp + (long long)(M - (JS - 1) - u * JS) * io.f_stride, ob);
            }
    };
    if (ok) {
        read(src, xa, xb);
        for (int part = 1; part < io.nparts; ++part) {
            Z va[NU], vb[NU];
            read(src + (long long)part * io.f_part, va, vb);
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (j0 + u * JS < np) {
                    xa[u] = cadd(xa[u], va[u]);
                    xb[u] = cadd(xb[u], vb[u]);
                }
        }
    } else {
#pragma unroll
        for (int u = 0; u < NU; ++u) xa[u] = xb[u] = cmk<T>(T(0), T(0));
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int k = j0 + u * JS;
        if (k < np) {
            Z a = xa[u], b = xb[u];
            if (k == 0) { a.y = T(0); b.y = T(0); }
            Z zk, zm;
            pre_pair<T>(a, b, tq[k], zk, zm);
            buf[k * kRS<SH> + s] = zk;
            if (k > 0 && 2 * k != M) buf[(M - k) * kRS<SH> + s] = zm;
        }
    }
    __syncthreads();
}

// Half spectra X[0..M] from Z on the tile to row[k f_stride + s0 + s]
// (complex, or quad BF16 hi / lo); the wavefront's largest |re|, |im| to amax_slot.
template <typename T, int SH, int NT>
__device__ __forceinline__ void split_store(const cplx<T>* buf, const cplx<T>* tq, int M, const SeriesIO& io,
                                            cplx<T>* row, int s0, int s, int j0, float* amax_slot) {
    using Z = cplx<T>;
    constexpr int NU = kMaxV<T> / 2 + 1, JS = kJS<SH, NT>;
    const int np = M / 2 + 1;
    const bool ok = s0 + s < io.S_pad;
    bool quad = false;
    if constexpr (sizeof(T) == 4) quad = io.quad != 0;
    Z* const rb = row + s0;
    const uint32_t fs = (uint32_t)io.f_stride * (uint32_t)sizeof(Z);
    const uint32_t so = quad ? (uint32_t)(8 * (s >> 2) + (s & 3)) * 4u : (uint32_t)s * (uint32_t)sizeof(Z);
    const uint32_t oa = (uint32_t)j0 * fs + so, ob = (uint32_t)(JS - 1 - j0) * fs + so;
    float vmax = 0.f;
    auto put = [&](Z* base, uint32_t off, Z X) {
        if constexpr (sizeof(T) == 4) {
            vmax = fmaxf(vmax, fmaxf(fabsf(X.x), fabsf(X.y)));
            if (quad) {
                const uint32_t hi = pack_bf16_rne(X.x, X.y);
                const uint32_t lo = pack_bf16_rne(X.x - __uint_as_float(hi << 16), X.y - __uint_as_float(hi & 0xffff0000u));
                st(reinterpret_cast<uint32_t*>(base), off, hi);
                st(reinterpret_cast<uint32_t*>(base), off + 16u, lo);
                return;
            }
        }
        st(base, off, X);
    };
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int k = j0 + u * JS;
        if (k < np && ok) {
            const Z a = buf[k * kRS<SH> + s], b = buf[(k == 0 ? 0 : M - k) * kRS<SH> + s];
            Z xk, xm;
            post_pair<T>(a, b, tq[k], xk, xm);
            put(rb + (long long)(u * JS) * io.f_stride, oa, xk);
            if (2 * k != M) put(rb + (long long)(M - (JS - 1) - u * JS) * io.f_stride, ob, xm);
        }
    }
    if constexpr (sizeof(T) == 4) {
        if (amax_slot) wave_amax_store(vmax, amax_slot);
    }
}

// Persistent workgroups: workgroup b takes items of XCD b % 8.  The lane indices
// and M are opaque to the compiler in each item, so that it does not compute
// every address of the loop body before the loop (and spill them).
#define P2O_WIDE_INDEX                                                                          \
    int s = threadIdx.x & ((1 << SH) - 1), j0 = threadIdx.x >> SH, M = pl.M;                    \
    asm volatile("" : "+v"(s), "+v"(j0), "+s"(M));
#define P2O_WIDE_SETUP                                                                          \
    extern __shared__ __align__(16) unsigned char smem_raw[];                                   \
    using Z = cplx<T>;                                                                          \
    Z* buf = reinterpret_cast<Z*>(smem_raw);                                                    \
    Z* tm = buf + (pl.M + 1) * kRS<SH>;                                                         \
    Z* tq = tm + pl.M;                                                                          \
    stage_tables<T, NT>(tm, tq, twg, pl.M);                                                         \
    __syncthreads();

template <typename T, typename TIN, int SH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
void k_r2c_wide(FftPlan pl, SeriesIO io, const TIN* __restrict__ in, cplx<T>* __restrict__ out,
                const cplx<T>* __restrict__ twg, ItemMap im) {
    P2O_WIDE_SETUP
    for (int it = blockIdx.x >> 3; it < im.Q; it += gridDim.x >> 3) {
        const int q = (int)(blockIdx.x & 7) * im.Q + it;
        if (q >= im.items) break;
        P2O_WIDE_INDEX
        const int outer = q / im.ntiles, tile = q - outer * im.ntiles, s0 = tile << SH;
        const int nt = active_len(io, outer);
        const TIN* src = in + (long long)outer * io.t_outer + s0;
        const bool ok = s0 + s < io.S;
        P2O_ANY_RADIX(pl.radix[0], (from_time<T, TIN, SH, NT, RR>(buf, M, src, io.t_stride, ok, nt, s, j0)))
        int Ns = pl.radix[0];
        for (int p = 1; p < pl.npass; ++p) {
            any_pass<T, SH, NT, false>(pl.radix[p], buf, tm, M, Ns, s, j0);
            Ns *= pl.radix[p];
        }
        float* slot = io.amax_part ? io.amax_part + (long long)outer * io.amax_slots + tile * (NT / 64) : nullptr;
        split_store<T, SH, NT>(buf, tq, M, io, out + (long long)outer * io.f_outer, s0, s, j0, slot);
        __syncthreads();
    }
}

template <typename T, int SH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
void k_c2r_wide(FftPlan pl, SeriesIO io, const cplx<T>* __restrict__ in, T* __restrict__ out,
                const cplx<T>* __restrict__ twg, ItemMap im) {
    P2O_WIDE_SETUP
    for (int it = blockIdx.x >> 3; it < im.Q; it += gridDim.x >> 3) {
        const int q = (int)(blockIdx.x & 7) * im.Q + it;
        if (q >= im.items) break;
        P2O_WIDE_INDEX
        const int outer = q / im.ntiles, tile = q - outer * im.ntiles, s0 = tile << SH;
        const int nt = active_len(io, outer);
        const bool ok = s0 + s < io.S;
        load_split<T, SH, NT>(buf, tq, M, in + (long long)outer * io.f_outer + s0, io, ok, s, j0);
        int Ns = 1;
        for (int p = 0; p < pl.npass - 1; ++p) {
            any_pass<T, SH, NT, true>(pl.radix[p], buf, tm, M, Ns, s, j0);
            Ns *= pl.radix[p];
        }
        T* dst = out + (long long)outer * io.t_outer + s0;
        P2O_ANY_RADIX(pl.radix[pl.npass - 1],
                      (to_time<T, T, SH, NT, RR>(buf, tm, M, dst, io.t_stride, ok, nt, io.Nt, s, j0)))
        __syncthreads();
    }
}

template <typename T, int SH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
void k_project_wide(FftPlan pl, SeriesIO io, cplx<T>* in_out, const cplx<T>* __restrict__ twg, ItemMap im) {
    P2O_WIDE_SETUP
    for (int it = blockIdx.x >> 3; it < im.Q; it += gridDim.x >> 3) {
        const int q = (int)(blockIdx.x & 7) * im.Q + it;
        if (q >= im.items) break;
        P2O_WIDE_INDEX
        const int outer = q / im.ntiles, tile = q - outer * im.ntiles, s0 = tile << SH;
        const int nt = active_len(io, outer);
        Z* base = in_out + (long long)outer * io.f_outer;
        load_split<T, SH, NT>(buf, tq, M, base + s0, io, s0 + s < io.S, s, j0);
        int Ns = 1;
        for (int p = pl.npass - 1; p > 0; --p) {
            any_pass<T, SH, NT, true>(pl.radix[p], buf, tm, M, Ns, s, j0);
            Ns *= pl.radix[p];
        }
        P2O_ANY_RADIX(pl.radix[0], (repad_pass<T, SH, NT, RR>(buf, tm, M, nt, s, j0)))
        Ns = pl.radix[0];
        for (int p = 1; p < pl.npass; ++p) {
            any_pass<T, SH, NT, false>(pl.radix[p], buf, tm, M, Ns, s, j0);
            Ns *= pl.radix[p];
        }
        float* slot = io.amax_part ? io.amax_part + (long long)outer * io.amax_slots + tile * (NT / 64) : nullptr;
        split_store<T, SH, NT>(buf, tq, M, io, base, s0, s, j0, slot);
        __syncthreads();
    }
}

// Transform of the time-domain blocks for storage, in FP64: item = (row, tile of
// columns).  PASS 0: the largest |re|, |im| of each (bin, scale block), as float
// bits (exact and order independent): a bin of an item always meets the same 1 <<
// SH lanes, so it is kept in a register over the workgroup's items and joins the
// others' when the block changes; and a non-finite flag.  PASS 1: round and store.
// Bound: LDS and FP64 work of the two transforms (with 4-column tiles, an LDS
// atomic per value in pass 0 and an exponent per value in pass 1: 64 x 16384 x
// 128, FP32 blocks into FP16, 2.0 -> 1.4 ms; 33 x 8200 x 420, 5.1 -> 2.3 ms; the
// blocks twice and the spectrum once would take 0.3 and 0.25).
template <typename TIN, int PASS, int SH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
void k_load_wide(FftPlan pl, LoadArgs la, int prec, const TIN* __restrict__ in, const double2* __restrict__ twg,
                 ItemMap im) {
    using T = double;
    constexpr int JS = kJS<SH, NT>, NU = kMaxV<T> / 2 + 1;
    P2O_WIDE_SETUP
    const bool scaled = prec == kBF16 || prec == kFP16;
    float mk[NU], mm[NU];                                // PASS 0: maxima of bins k and M - k
    int ek[NU], em[NU];                                  // PASS 1: their exponents
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        mk[u] = mm[u] = 0.f;
        ek[u] = em[u] = 0;
    }
    // Between items, through the free tile, so that consecutive lanes join the maxima
    // of consecutive bins: atomics of the lanes that hold them, one bin in 1 << SH
    // lanes, were up to 16 times as many transactions on the few lines of `scales`
    // that all workgroups share.
    unsigned* smax = reinterpret_cast<unsigned*>(la.scales);
    auto flush = [&](int blk) {
        unsigned* lm = reinterpret_cast<unsigned*>(smem_raw);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
#pragma unroll
            for (int o = (1 << SH) / 2; o > 0; o >>= 1) {
                mk[u] = fmaxf(mk[u], __shfl_xor(mk[u], o));
                mm[u] = fmaxf(mm[u], __shfl_xor(mm[u], o));
            }
            const int k = (int)(threadIdx.x >> SH) + u * JS;
            if ((threadIdx.x & ((1 << SH) - 1)) == 0 && k <= pl.M / 2) {
                if (2 * k == pl.M) mk[u] = mm[u] = fmaxf(mk[u], mm[u]);
                lm[k] = __float_as_uint(mk[u]);
                lm[pl.M - k] = __float_as_uint(mm[u]);
            }
            mk[u] = mm[u] = 0.f;
        }
        __syncthreads();
        for (int k = threadIdx.x; k <= pl.M; k += NT) atomicMax(smax + (long long)k * la.nblk + blk, lm[k]);
        __syncthreads();
    };
    int cur = -1;
    bool bad = false;
    for (int it = blockIdx.x >> 3; it < im.Q; it += gridDim.x >> 3) {
        const int q = (int)(blockIdx.x & 7) * im.Q + it;
        if (q >= im.items) break;
        P2O_WIDE_INDEX
        const int row = q / im.ntiles, tile = q - row * im.ntiles, s0 = tile << SH;
        const int np = M / 2 + 1, blk = (int)((la.col0 + s0) / kScaleBlock);
        const bool ok = s0 + s < la.ncols;
        if (scaled && blk != cur) {
            if constexpr (PASS == 0) {
                if (cur >= 0) flush(cur);
            } else {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int k = j0 + u * JS;
                    if (k < np) {
                        ek[u] = storage_exponent(la.scales[(long long)k * la.nblk + blk], prec);
                        em[u] = storage_exponent(la.scales[(long long)(M - k) * la.nblk + blk], prec);
                    }
                }
            }
            cur = blk;
        }
        const TIN* src = in + (long long)row * la.ncols + s0;
        bool odd = false;
        P2O_ANY_RADIX(pl.radix[0], (from_time<T, TIN, SH, NT, RR>(buf, M, src, la.t_stride, ok, la.Nt, s, j0, &odd)))
        bad |= odd;
        int Ns = pl.radix[0];
        for (int p = 1; p < pl.npass; ++p) {
            any_pass<T, SH, NT, false>(pl.radix[p], buf, tm, M, Ns, s, j0);
            Ns *= pl.radix[p];
        }
        auto put = [&](int k, int ex, Z X) {
            const long long off = ((long long)k * la.Nd + row) * la.pitch + la.col0 + s0 + s;
            if (prec == kFP64) {
                reinterpret_cast<double2*>(la.fhat)[off] = X;
            } else if (prec == kFP32) {
                reinterpret_cast<float2*>(la.fhat)[off] = make_float2((float)X.x, (float)X.y);
            } else {
                const float re = f64_to_f32_odd(ldexp(X.x, ex)), im2 = f64_to_f32_odd(ldexp(X.y, ex));
                reinterpret_cast<uint32_t*>(la.fhat)[off] =
                    prec == kBF16 ? f32_to_bf16_rne(re) | (f32_to_bf16_rne(im2) << 16)
                                  : f32_to_f16_rne(re) | (f32_to_f16_rne(im2) << 16);
            }
        };
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = j0 + u * JS;
            if (k < np && ok) {
                const Z a = buf[k * kRS<SH> + s], b = buf[(k == 0 ? 0 : M - k) * kRS<SH> + s];
                Z xk, xm;
                post_pair<T>(a, b, tq[k], xk, xm);
                if constexpr (PASS == 0) {
                    mk[u] = fmaxf(mk[u], (float)fmax(fabs(xk.x), fabs(xk.y)));
                    mm[u] = fmaxf(mm[u], (float)fmax(fabs(xm.x), fabs(xm.y)));
                } else {
                    put(k, ek[u], xk);
                    if (2 * k != M) put(M - k, em[u], xm);
                }
            }
        }
        __syncthreads();
    }
    if constexpr (PASS == 0) {
        if (cur >= 0) flush(cur);
    }
    if (bad) atomicOr(la.flag, 1u);
}

// ---------------------------------------------------------------- host side
size_t wide_lds(int M, int sh, size_t z) { return ((size_t)(M + 1) * ((1 << sh) + 1) + M + M / 2 + 1) * z; }

// 256-thread workgroups where their registers hold the tile (short transforms:
// a pass of a larger workgroup would leave threads without a butterfly: M =
// 128, 32 x 16384 FP32 series in tiles of 16, r2c 320 -> 215 us), else 512.
template <typename T>
int wide_threads(int M, int sh) { return (M << sh) <= 256 * kMaxV<T> ? 256 : 512; }

// Resident workgroups (two per CU by LDS, more where LDS and registers allow),
// at most one per item.
template <auto K, int NT>
dim3 wide_grid(size_t lds, const ItemMap& im) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, K, NT, lds) != hipSuccess || occ < 1) occ = 1;
    return resident_grid(occ, im);
}

bool fits32(long long rows, long long stride, size_t esz) { return (rows * stride + 64) * (long long)esz < (1LL << 32); }

template <auto K, int NT, typename... A>
hipError_t wide_go(size_t lds, const ItemMap& im, hipStream_t st, A... a) {
    hipLaunchKernelGGL(K, (wide_grid<K, NT>(lds, im)), dim3(NT), lds, st, a..., im);
    return hipGetLastError();
}

// f(tile shift, workgroup size) for element type T
template <typename T, typename F>
hipError_t by_tile(int M, int sh, F&& f) {
    const bool small = wide_threads<T>(M, sh) == 256;
    auto with = [&](auto c) {
        return small ? f(c, std::integral_constant<int, 256>{}) : f(c, std::integral_constant<int, 512>{});
    };
    if constexpr (sizeof(T) == 4)
        if (sh == 5) return with(std::integral_constant<int, 5>{});
    if (sh == 4) return with(std::integral_constant<int, 4>{});
    if (sh == 3) return with(std::integral_constant<int, 3>{});
    if constexpr (sizeof(T) == 8)
        if (sh == 2) return with(std::integral_constant<int, 2>{});
    return hipErrorInvalidValue;
}

template <typename T, typename TIN>
hipError_t r2c_go(const FftPlan& pl, const SeriesIO& io, const void* in, void* out, const void* tw, int sh,
                  hipStream_t st) {
    const ItemMap im = item_map(io.S_pad, sh, io.outer_count);
    return by_tile<T>(pl.M, sh, [&](auto s, auto n) {
        constexpr int SH = decltype(s)::value, NT = decltype(n)::value;
        return wide_go<k_r2c_wide<T, TIN, SH, NT>, NT>(wide_lds(pl.M, sh, 2 * sizeof(T)), im, st, pl, io, (const TIN*)in,
                                                       (cplx<T>*)out, (const cplx<T>*)tw);
    });
}

template <typename T>
hipError_t c2r_go(const FftPlan& pl, const SeriesIO& io, const void* in, void* out, const void* tw, int sh,
                  hipStream_t st) {
    const ItemMap im = item_map(io.S, sh, io.outer_count);
    return by_tile<T>(pl.M, sh, [&](auto s, auto n) {
        constexpr int SH = decltype(s)::value, NT = decltype(n)::value;
        return wide_go<k_c2r_wide<T, SH, NT>, NT>(wide_lds(pl.M, sh, 2 * sizeof(T)), im, st, pl, io, (const cplx<T>*)in,
                                                  (T*)out, (const cplx<T>*)tw);
    });
}

template <typename T>
hipError_t project_go(const FftPlan& pl, const SeriesIO& io, void* in_out, const void* tw, int sh, hipStream_t st) {
    const ItemMap im = item_map(io.S_pad, sh, io.outer_count);
    return by_tile<T>(pl.M, sh, [&](auto s, auto n) {
        constexpr int SH = decltype(s)::value, NT = decltype(n)::value;
        return wide_go<k_project_wide<T, SH, NT>, NT>(wide_lds(pl.M, sh, 2 * sizeof(T)), im, st, pl, io, (cplx<T>*)in_out,
                                                      (const cplx<T>*)tw);
    });
}

// Wavefront maxima of these tiles fit the caller's slots.
bool slots_fit(const SeriesIO& io, int sh, int waves) {
    return !io.amax_part || (long long)((io.S_pad + (1 << sh) - 1) >> sh) * waves <= io.amax_slots;
}

template <typename TIN>
hipError_t load_go(int pass, const FftPlan& pl, const LoadArgs& la, int prec, const void* in, const void* tw, int sh,
                   hipStream_t st) {
    const ItemMap im = item_map(la.ncols, sh, la.Nd);
    const size_t lds = wide_lds(pl.M, sh, 16);
    return by_tile<double>(pl.M, sh, [&](auto s, auto n) {
        constexpr int SH = decltype(s)::value, NT = decltype(n)::value;
        return pass == 0
            ? wide_go<k_load_wide<TIN, 0, SH, NT>, NT>(lds, im, st, pl, la, prec, (const TIN*)in, (const double2*)tw)
            : wide_go<k_load_wide<TIN, 1, SH, NT>, NT>(lds, im, st, pl, la, prec, (const TIN*)in, (const double2*)tw);
    });
}

}  // namespace

// One pass over a chunk of blocks with the widest tiles; false where the chunk has
// too few tiles, the transform too few entries for the threads, or an offset does
// not fit.  Tiles of two or three entries per thread leave most of the workgroup
// idle in a pass: faster than 32-column tiles of fft.hip while their rows are a
// chain there, not where these are in flight by the thousand.  Those run fewer
// passes with a radix 8 and an LDS atomic per value for the maxima of 16-bit
// spectra, so the line lies lower and higher (whole loads of 4096 columns, us here
// / there: FP32, M = 32, 96 rows 146 / 166, 112 169 / 166, 300 534 / 367; M = 48, 128
// 276 / 281, 152 333 / 313; M = 45, 160 278 / 319, 208 360 / 354; FP16, M = 32, 112
// 330 / 351, 128 354 / 340; M = 45, 208 about 625 / 740, 256 770 / 732; M = 60, 4
// entries: 0.8 of the time there).  The narrow tiles' time goes in steps of 256 rows,
// so just past one the line errs by up to a sixth (M = 45, FP32, 288 rows: 493 / 562).
static bool few_rows(int prec, int M, long long tiles) {
    const bool r8 = M % 8 == 0, maxima = prec == kBF16 || prec == kFP16;
    return tiles <= (r8 ? (maxima ? 960LL : 768LL) : (maxima ? 1400LL : 1152LL)) * M;
}

bool launch_wide_load(int pass, int prec, bool in_f64, const FftPlan& pl, const LoadArgs& la, const void* in,
                      const void* tw, hipStream_t st, hipError_t* err) {
    if ((long long)la.ncols * la.Nd >= (1LL << 31)) return false;
    const int sh = fft_wide_shift(true, pl, la.ncols, la.Nd);
    if (sh < 0 || (pl.M << sh) < 512) return false;
    if ((pl.M << sh) < 800 && !few_rows(prec, pl.M, (long long)((la.ncols + (1 << sh) - 1) >> sh) * la.Nd)) return false;
    if (!fits32(2 * (512 >> sh), la.t_stride, in_f64 ? 8 : 4)) return false;
    *err = in_f64 ? load_go<double>(pass, pl, la, prec, in, tw, sh, st) : load_go<float>(pass, pl, la, prec, in, tw, sh, st);
    return true;
}

int fft_wide_waves(bool f64, const FftPlan& pl, int sh) {
    return (f64 ? wide_threads<double>(pl.M, sh) : wide_threads<float>(pl.M, sh)) / 64;
}

// Tile shift of the wide kernels for `outer` x S series, or -1: the widest
// tile (32 to 8 series, FP64 16 to 4) two of which fit a CU and whose entries
// fit the threads' registers, when there are tiles for every CU (below that,
// the smaller tiles of fft.hip spread the work over more of them).
int fft_wide_shift(bool f64, const FftPlan& pl, int S, int outer) {
    if (pl.npass < 2) return -1;
    const size_t z = f64 ? 16 : 8;
    const int cap = 512 * (f64 ? kMaxV<double> : kMaxV<float>);
    for (int sh = f64 ? 4 : 5; sh >= (f64 ? 2 : 3); --sh)
        if ((pl.M << sh) <= cap && wide_lds(pl.M, sh, z) <= kWideLds)
            if ((long long)((S + (1 << sh) - 1) >> sh) * outer >= kWideTiles) return sh;
    return -1;
}

// (offsets are checked for the largest sweep, of 512 threads)
bool launch_wide_r2c(bool f64, bool in_f64, const FftPlan& pl, const SeriesIO& io, const void* in, void* out,
                     const void* tw, int sh, hipStream_t st, hipError_t* err) {
    if (!fits32(2 * (512 >> sh), io.t_stride, in_f64 ? 8 : 4) || !fits32(512 >> sh, io.f_stride, f64 ? 16 : 8) ||
        !slots_fit(io, sh, fft_wide_waves(f64, pl, sh)))
        return false;
    *err = !f64 ? r2c_go<float, float>(pl, io, in, out, tw, sh, st)
         : in_f64 ? r2c_go<double, double>(pl, io, in, out, tw, sh, st)
                  : r2c_go<double, float>(pl, io, in, out, tw, sh, st);
    return true;
}

bool launch_wide_c2r(bool f64, const FftPlan& pl, const SeriesIO& io, const void* in, void* out, const void* tw, int sh,
                     hipStream_t st, hipError_t* err) {
    if (!fits32(2 * (512 >> sh), io.t_stride, f64 ? 8 : 4) || !fits32(512 >> sh, io.f_stride, f64 ? 16 : 8)) return false;
    *err = f64 ? c2r_go<double>(pl, io, in, out, tw, sh, st) : c2r_go<float>(pl, io, in, out, tw, sh, st);
    return true;
}

bool launch_wide_project(bool f64, const FftPlan& pl, const SeriesIO& io, void* in_out, const void* tw, int sh,
                         hipStream_t st, hipError_t* err) {
    if (!fits32(512 >> sh, io.f_stride, f64 ? 16 : 8) || !slots_fit(io, sh, fft_wide_waves(f64, pl, sh))) return false;
    *err = f64 ? project_go<double>(pl, io, in_out, tw, sh, st) : project_go<float>(pl, io, in_out, tw, sh, st);
    return true;
}

}  // namespace p2o
