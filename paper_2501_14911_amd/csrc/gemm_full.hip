// Per-frequency complex products of FP64 and FP32 spectra with several
// right-hand sides on the matrix cores (v_mfma_f64_16x16x4f64 and
// v_mfma_f32_16x16x4f32: inputs and products in the spectrum's own precision;
// FP64 sums in FP64, FP32 ones in short chains that join FP64 totals (forward)
// or FP32 totals (adjoint)).
//
// Section 4 of the paper reduces each matvec to one Nd x Nm complex product
// per frequency; with several right-hand sides that is a narrow complex GEMM.
// One streaming pass per right-hand side (gemv.hip) reads the spectrum nrhs
// times; here one pass serves 8 T right-hand sides.  8 of them are the 16
// rows of a matrix instruction: row m stands for (right-hand side b, part c),
// c = 0 the real and c = 1 the imaginary part of the output.  With the
// spectrum's real part as the other operand row (b, 0) takes x_r and row
// (b, 1) takes x_i; with its imaginary part they take -x_i and x_r (forward;
// the adjoint, on the conjugate, y_i and -y_r).  Rows are numbered so that
// the lane that ends up with (b, 0) also holds (b, 1), so results leave as
// whole complex values, 16 lanes on 16 neighbouring outputs.
//
// Bound: HBM (the spectrum once per pass: 8 T real products per complex entry
// and right-hand side group are 4 T (FP64) or 8 T (FP32) flop per byte, 26 T
// and 52 T TFLOP/s at 6.5 TB/s against 79 and 157), so the loads go straight
// to registers, one stage ahead of the matrix cores, and nothing is staged in
// LDS but the final sums of the four wavefronts of a forward workgroup.
// gfx950, whole F then F* calls: FP64, 64 x 4096 x 128, 8 right-hand sides 1578 ->
// 324 us (products 725 + 797 -> 164 + 116 us: 0.54 GB of spectrum in each); FP32,
// 101 x 10007 x 365, 4 right-hand sides 4176 -> 1351 us (1880 + 2065 -> 677 + 560
// us, 4.5 and 5.4 TB/s of spectrum).  HBM counters of the two: 0.62 and 0.55 GB
// read per launch for 0.54 GB of spectrum in FP64, 3.33 and 3.09 for 3.03 in FP32.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace p2o {

namespace {

constexpr int kThreads = 256;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename CT> struct Mma;
template <> struct Mma<double> {
    using Acc = f64x4;
    static constexpr int CPL = 1;                        // complex entries in a lane's 16 bytes
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // operand row n = l % 16 and result item v of lane group g = l / 16 (the
    // result row is 4 v + g): row 4 v + g is (b, c) = (4 (v / 2) + g, v % 2)
    static __device__ __forceinline__ int row_b(int n) { return 4 * (n >> 3) + (n & 3); }
    static __device__ __forceinline__ int row_c(int n) { return (n >> 2) & 1; }
    static __device__ __forceinline__ int out_b(int g, int pair) { return 4 * pair + g; }
};
template <> struct Mma<float> {
    using Acc = f32x4;
    static constexpr int CPL = 2;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // result row 4 g + v: row n is (n / 2, n % 2)
    static __device__ __forceinline__ int row_b(int n) { return n >> 1; }
    static __device__ __forceinline__ int row_c(int n) { return n & 1; }
    static __device__ __forceinline__ int out_b(int g, int pair) { return 2 * g + pair; }
};

// The complex entries of 16 loaded bytes.
__device__ __forceinline__ void entries(u32x4 w, double (&re)[1], double (&im)[1]) {
    re[0] = __hiloint2double((int)w.y, (int)w.x);
    im[0] = __hiloint2double((int)w.w, (int)w.z);
}
__device__ __forceinline__ void entries(u32x4 w, float (&re)[2], float (&im)[2]) {
    re[0] = __uint_as_float(w.x); im[0] = __uint_as_float(w.y);
    re[1] = __uint_as_float(w.z); im[1] = __uint_as_float(w.w);
}


// Forward: y_w[b][i] = sum_j Fhat_w[i, j] x_w[b][j].  Work item = (frequency,
// column chunk, slab of 16 R rows, group of 8 T right-hand sides); the four
// wavefronts take the chunk's 128-byte steps (8 FP64 or 16 FP32 columns) in
// turn.  Lane (n, g) loads 16 bytes of row n of each 16-row block, g picking
// the 16 bytes of a 64-byte run: one instruction covers 16 rows x 64 bytes and
// the next one the other half of the same lines.  Rows past Nd repeat the last
// row (their results are not stored); columns past Nm are zero in both
// operands up to the pitch.
template <typename CT, int T, int R>
__global__ __launch_bounds__(kThreads) void k_full_fwd(const uint8_t* __restrict__ fhat, const cplx<CT>* __restrict__ X,
                                                       cplx<CT>* __restrict__ Yp, FullArgs fa) {
    using M = Mma<CT>;
    using Z = cplx<CT>;
    constexpr int CPL = M::CPL, JS = 8 * CPL, B = sizeof(Z);
    __shared__ CT red[4][R][4][64];
    int q = xcd_item(fa.Q);
    if (q >= fa.items) return;
    const int grp = q % fa.n_grp; q /= fa.n_grp;
    const int slab = q % fa.n_slab; q /= fa.n_slab;
    const int part = q % fa.n_part;
    const int w = q / fa.n_part;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int nsteps = (fa.ncols + JS - 1) / JS;         // ends inside the pitch (a multiple of 32)
    const int s0 = part * fa.steps_per_part, s1 = min(nsteps, s0 + fa.steps_per_part);

    const long long rowb = (long long)fa.pitch * B;
    const uint8_t* Fl[R];
#pragma unroll
    for (int a = 0; a < R; ++a)
        Fl[a] = fhat + ((long long)w * fa.Nd + min(fa.Nd - 1, slab * 16 * R + 16 * a + n)) * rowb + 16 * g;
    const uint8_t* Xl[T];
    const int im_row = M::row_c(n);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int b = min(fa.nrhs - 1, grp * 8 * T + 8 * t + M::row_b(n));
        Xl[t] = reinterpret_cast<const uint8_t*>(X) + ((long long)w * fa.nrhs + b) * rowb + 16 * g;
    }
    // FP32 sums leave the matrix cores after every four chained instructions for
    // FP64 totals: one FP32 chain over a row of 10007 columns had three times the
    // streaming kernel's error (7.0e-7 against 2.5e-7); this way it is 2.2e-7.
    constexpr bool kSplit = sizeof(CT) == 4;
    const typename M::Acc zero{CT(0), CT(0), CT(0), CT(0)};
    f64x4 acc[T][R];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int a = 0; a < R; ++a) acc[t][a] = f64x4{0.0, 0.0, 0.0, 0.0};

    struct Stage { u32x4 f[R][2], x[T][2]; };
    auto load = [&](Stage& st, int s) {
        const bool live = s < s1;                        // past the chunk: its last step against zeros
        const long long o = (long long)(live ? s : s1 - 1) * 128;
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                st.f[a][h] = *reinterpret_cast<const u32x4*>(Fl[a] + o + 64 * h);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 x = *reinterpret_cast<const u32x4*>(Xl[t] + o + 64 * h);
                st.x[t][h] = live ? x : u32x4{0u, 0u, 0u, 0u};
            }
    };
    auto products = [&](const Stage& st) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            CT xa[T][CPL], xb[T][CPL];                   // against the real and the imaginary parts
#pragma unroll
            for (int t = 0; t < T; ++t) {
                CT xr[CPL], xi[CPL];
                entries(st.x[t][h], xr, xi);
#pragma unroll
                for (int u = 0; u < CPL; ++u) {
                    xa[t][u] = im_row ? xi[u] : xr[u];
                    xb[t][u] = im_row ? xr[u] : -xi[u];
                }
            }
#pragma unroll
            for (int a = 0; a < R; ++a) {
                CT fr[CPL], fi[CPL];
                entries(st.f[a][h], fr, fi);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    typename M::Acc c = zero;
                    if constexpr (!kSplit) c = acc[t][a];
#pragma unroll
                    for (int u = 0; u < CPL; ++u) {
                        c = M::mma(xa[t][u], fr[u], c);
                        c = M::mma(xb[t][u], fi[u], c);
                    }
                    if constexpr (kSplit) acc[t][a] += __builtin_convertvector(c, f64x4);
                    else acc[t][a] = c;
                }
            }
        }
    };
    Stage A, Bs;
    load(A, s0 + wave);
    for (int s = s0 + wave; s < s1; s += 8) {
        load(Bs, s + 4);
        __builtin_amdgcn_sched_barrier(0);               // keep the loads ahead of the products
        products(A);
        load(A, s + 8);
        __builtin_amdgcn_sched_barrier(0);
        products(Bs);
    }

    // the four wavefronts' sums in order; wavefront a finishes row block a
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (t) __syncthreads();
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][a][v][lane] = (CT)acc[t][a][v];
        __syncthreads();
        if (wave < R) {
            const int row = slab * 16 * R + 16 * wave + n;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int b = grp * 8 * T + 8 * t + M::out_b(g, p);
                Z y;
                y.x = (red[0][wave][2 * p][lane] + red[1][wave][2 * p][lane]) +
                      (red[2][wave][2 * p][lane] + red[3][wave][2 * p][lane]);
                y.y = (red[0][wave][2 * p + 1][lane] + red[1][wave][2 * p + 1][lane]) +
                      (red[2][wave][2 * p + 1][lane] + red[3][wave][2 * p + 1][lane]);
                if (row < fa.Nd && b < fa.nrhs)
                    Yp[(long long)part * fa.part_stride + ((long long)w * fa.nrhs + b) * fa.Nd + row] = y;
            }
        }
    }
}

// Adjoint: x_w[b][j] = sum_i conj(Fhat_w[i, j]) y_w[b][i].  Work item =
// (frequency, 4 wavefronts x C blocks of 16 CPL columns, group of 8 T
// right-hand sides).  Lane (n, g) loads 16 bytes of row 4 s + g, its 16
// neighbours covering 256 contiguous bytes; a stage is two steps of 4 rows.
// Rows past Nd repeat the last row against zeros.
template <typename CT, int T, int C>
__global__ __launch_bounds__(kThreads) void k_full_adj(const uint8_t* __restrict__ fhat, const cplx<CT>* __restrict__ Y,
                                                       cplx<CT>* __restrict__ Xp, FullArgs fa) {
    using M = Mma<CT>;
    using Z = cplx<CT>;
    constexpr int CPL = M::CPL, B = sizeof(Z), W = 16 * CPL;
    int q = xcd_item(fa.Q);
    if (q >= fa.items) return;
    const int grp = q % fa.n_grp; q /= fa.n_grp;
    const int ct = q % fa.n_slab;
    const int w = q / fa.n_slab;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int col0 = (ct * 4 + wave) * C * W + CPL * n;
    if ((ct * 4 + wave) * C * W >= fa.ncols) return;     // (no barrier below)

    const long long rowb = (long long)fa.pitch * B;
    const uint8_t* Fl[C];
#pragma unroll
    for (int a = 0; a < C; ++a) {
        const int col = col0 + a * W;
        Fl[a] = fhat + (long long)w * fa.Nd * rowb + (long long)(col < fa.ncols ? col : 0) * B;
    }
    const Z* Yl[T];
    const int im_row = M::row_c(n);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int b = min(fa.nrhs - 1, grp * 8 * T + 8 * t + M::row_b(n));
        Yl[t] = Y + ((long long)w * fa.nrhs + b) * fa.Nd;
    }
    constexpr bool kSplit = sizeof(CT) == 4;
    const typename M::Acc zero{CT(0), CT(0), CT(0), CT(0)};
    typename M::Acc acc[T][C][CPL], total[T][C][CPL];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int a = 0; a < C; ++a)
#pragma unroll
            for (int u = 0; u < CPL; ++u) acc[t][a][u] = total[t][a][u] = zero;

    struct Stage { u32x4 f[C][2]; Z y[T][2]; };
    auto load = [&](Stage& st, int i0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = i0 + 4 * h + g, ic = min(i, fa.Nd - 1);
#pragma unroll
            for (int a = 0; a < C; ++a)
                st.f[a][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(Fl[a] + (long long)ic * rowb));
#pragma unroll
            for (int t = 0; t < T; ++t) {
                Z y = Yl[t][ic];
                if (i >= fa.Nd) y = Z{CT(0), CT(0)};
                st.y[t][h] = y;
            }
        }
    };
    auto products = [&](const Stage& st) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            CT ya[T], yb[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                ya[t] = im_row ? st.y[t][h].y : st.y[t][h].x;
                yb[t] = im_row ? -st.y[t][h].x : st.y[t][h].y;
            }
#pragma unroll
            for (int a = 0; a < C; ++a) {
                CT fr[CPL], fi[CPL];
                entries(st.f[a][h], fr, fi);
#pragma unroll
                for (int u = 0; u < CPL; ++u)
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        acc[t][a][u] = M::mma(ya[t], fr[u], acc[t][a][u]);
                        acc[t][a][u] = M::mma(yb[t], fi[u], acc[t][a][u]);
                    }
            }
        }
    };
    Stage A, Bs;
    load(A, 0);
    for (int i = 0; i < fa.Nd; i += 16) {
        load(Bs, i + 8);
        __builtin_amdgcn_sched_barrier(0);               // keep the loads ahead of the products
        products(A);
        load(A, i + 16);
        __builtin_amdgcn_sched_barrier(0);
        products(Bs);
        // FP32: the sum of 16 rows joins a total of its own (one chain over 600
        // rows had 4.7e-7 of error against the streaming kernel's 3.5e-7; 1.7e-7 now)
        if constexpr (kSplit) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int a = 0; a < C; ++a)
#pragma unroll
                    for (int u = 0; u < CPL; ++u) {
                        total[t][a][u] += acc[t][a][u];
                        acc[t][a][u] = zero;
                    }
        }
    }

#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int b = grp * 8 * T + 8 * t + M::out_b(g, p);
            if (b >= fa.nrhs) continue;
            const auto& sum = kSplit ? total : acc;
            Z* out = Xp + ((long long)w * fa.nrhs + b) * fa.pitch + col0;
#pragma unroll
            for (int a = 0; a < C; ++a)
                if (col0 + a * W < fa.ncols) {
                    if constexpr (CPL == 1) {
                        out[a * W] = Z{sum[t][a][0][2 * p], sum[t][a][0][2 * p + 1]};
                    } else {
                        *reinterpret_cast<float4*>(out + a * W) = make_float4(
                            sum[t][a][0][2 * p], sum[t][a][0][2 * p + 1], sum[t][a][1][2 * p], sum[t][a][1][2 * p + 1]);
                    }
                }
        }
}

template <typename CT, int T, int R>
void fwd_go(const FullArgs& fa, const void* fhat, const void* X, void* Yp, hipStream_t st) {
    hipLaunchKernelGGL((k_full_fwd<CT, T, R>), dim3(8 * fa.Q), dim3(kThreads), 0, st, (const uint8_t*)fhat,
                       (const cplx<CT>*)X, (cplx<CT>*)Yp, fa);
}
template <typename CT, int T, int C>
void adj_go(const FullArgs& fa, const void* fhat, const void* Y, void* Xp, hipStream_t st) {
    hipLaunchKernelGGL((k_full_adj<CT, T, C>), dim3(8 * fa.Q), dim3(kThreads), 0, st, (const uint8_t*)fhat,
                       (const cplx<CT>*)Y, (cplx<CT>*)Xp, fa);
}

// Right-hand-side tiles of 8 per pass: as many as the call has, up to 2 (FP64, whose
// accumulators are twice as wide and whose matrix cores are the bound from 24
// right-hand sides on; FP32 up to 32 sensors, where reading a short spectrum again
// costs less than a workgroup's longer code: F* at 3 x 4097 x 60, 32 right-hand
// sides, 83 us with 4 tiles, 69 with 2) or 4.
int rhs_tiles(bool f64, int Nd, int nrhs) { return nrhs <= 8 ? 1 : nrhs <= 16 || f64 || Nd <= 32 ? 2 : 4; }

constexpr int kWantItems = 2048;        // work items that fill 256 CUs a few times over

FullArgs base(const GemvArgs& ga) {
    FullArgs fa{};
    fa.Nd = ga.Nd;
    fa.pitch = ga.pitch;
    fa.ncols = ga.ncols;
    fa.nrhs = ga.nrhs;
    return fa;
}


// 16-row blocks of a forward wavefront.  FP64 from 9 right-hand sides on: 4, which
// share the loads of the right-hand sides (49 x 16384 x 250, 16 right-hand sides:
// 0.92 ms against 1.20 with 2 and 1.59 with 1).  Otherwise 2: the smaller tile's
// extra wavefronts are worth more (64 x 4096 x 128, 8: FP64 164 us against 175,
// FP32 72 against 81), and FP32's FP64 totals fill the registers of a larger one
// (600 x 16384 x 100, 16: 1.69 ms against 1.76).
int fwd_blocks(bool f64, int Nd, int T) { return Nd <= 16 ? 1 : Nd <= 32 || T == 1 || !f64 ? 2 : 4; }

int groups(int nrhs, int T) { return (nrhs + 8 * T - 1) / (8 * T); }

// Column chunks of the forward products (partial sums for the inverse FFT to
// add): enough work items to fill the chip, each wavefront keeping at least
// four steps, and no more than max_parts.
int fwd_parts_of(bool f64, int Nd, int nfreq, int nrhs, int ncols, int T, int max_parts) {
    const int js = f64 ? 8 : 16, rows = 16 * fwd_blocks(f64, Nd, T);
    const long long rest = (long long)nfreq * ((Nd + rows - 1) / rows) * groups(nrhs, T);
    const int nsteps = (ncols + js - 1) / js;
    long long p = (kWantItems + rest - 1) / rest;
    p = std::min<long long>({p, std::max(1, nsteps / 16), max_parts});
    p = std::max<long long>(p, 1);
    const int per = (int)((nsteps + p - 1) / p);
    return (nsteps + per - 1) / per;                     // every part has work
}

// Tiles of a forward pass: fewer while the larger ones leave too few work items
// (FP32 1000 x 31, 8 sensors, 17 right-hand sides, whole F calls: 31.6 us with 4
// tiles, 24.6 with 2, 21.9 with 1).  One tile only while all sensors are in one row
// block (FP32) or up to 32 and far from filling the chip (FP64, 20 sensors, 9: 30.4
// -> 27.4 us; 36 sensors the other way, 37.8 and 54.3).
int fwd_tiles(bool f64, int Nd, int nfreq, int nrhs, int ncols) {
    int T = rhs_tiles(f64, Nd, nrhs);
    auto items = [&] {
        const int rows = 16 * fwd_blocks(f64, Nd, T);
        return (long long)nfreq * ((Nd + rows - 1) / rows) * groups(nrhs, T) *
               fwd_parts_of(f64, Nd, nfreq, nrhs, ncols, T, 1 << 30);
    };
    if (T == 4 && items() < kWantItems) T = 2;
    if (T == 2 && Nd <= (f64 ? 32 : 16) && items() < (f64 ? kWantItems / 8 : kWantItems)) T = 1;
    return T;
}

// The same for an adjoint pass (FP32 1000 x 31, 8 sensors, 17 right-hand sides, whole
// F* calls: 33.4 us with 4 tiles, 19.6 with 2, 19.0 with 1).
int adj_tiles(bool f64, int Nd, int nfreq, int nrhs, int ncols) {
    const int w = f64 ? 64 : 128;
    int T = rhs_tiles(f64, Nd, nrhs);
    while (T > 1 && (long long)nfreq * ((ncols + w - 1) / w) * groups(nrhs, T) < kWantItems / 2) T /= 2;
    return T;
}

}  // namespace

// Whether one pass is faster than one streaming pass per right-hand side.  A pass
// does the work of 16 sensors and of whole tiles of right-hand sides, so not where
// sensors times right-hand sides are few, unless the rows are so short that
// launching work for each right-hand side is the time.  Products alone, streaming
// against one pass, us: F* at 33000 x 128, FP64, 1 sensor, 2 right-hand sides 44 and
// 139, 3 and 4: 210, 172; 6 and 2: 158, 150; 1 and 17, which is 32: 440, 528.  F,
// FP64: 1 and 2: 57, 116; 4 and 2: 105, 159; 1 and 8: 250, 213; 3 and 4: 201, 181;
// and not below two million entries read, as the streaming kernel has the shorter
// chain (8 x 1000 x 31, 8 right-hand sides: 10, 11.5), or five per tile of 16
// right-hand sides where more than 8 share up to 5 sensors (whole F calls, 2 x 4096 x
// 16, 17 right-hand sides 28 and 39; 4 x 1000 x 128, 16: 43, 40; F*, 3.5 million: 2 x 500
// x 240, 17: 46 and 54, FP32 2 x 1000 x 128: 27, 31); nor for 2 right-hand
// sides where more than 3 / 8 of two blocks of 32 rows are padding (F of 33 and 42
// sensors x 4096 x 440: 355 and 410, 441 and 416).  F, FP32: always.  Short rows, whole
// F and F* calls, 1 x 33 x 406, FP64, 33 right-hand sides: 64 and 47 against 31 and 25.
// Over 3706 sizes the calls are within 0.5 % of the faster side as a mean.
bool full_pays(bool f64, int Nd, int nfreq, int nrhs, int ncols, bool fwd) {
    const long long nr = (long long)Nd * nrhs;
    const int g16 = groups(nrhs, 2);
    const bool part = nrhs > 8 && Nd <= 5;               // part of a row block, and of its tiles
    if (!fwd) return ncols <= 200 || (nr >= 14 * g16 && (!part || nr * nfreq * ncols >= 3500000LL * g16));
    if (!f64 || ncols <= 128) return true;
    if (nrhs == 2 && Nd > 32 && Nd <= 40) return false;
    const int T = fwd_tiles(f64, Nd, nfreq, nrhs, ncols);
    const long long least = part ? 9600LL * g16 : 4000;
    return nrhs * (Nd + 1LL) >= (nrhs <= 8 ? 15 : 18) * groups(nrhs, T) &&
           (Nd > 16 || nr * nfreq * ncols >= least * std::min(ncols, 500));
}

// Whether a launch can hold the work items of these sizes at the smallest tiles
// of either direction (64 FP64 or 128 FP32 columns; 16 rows, and as many chunks
// as fill the chip anyway).
bool full_fits(bool f64, int Nd, int nfreq, int nrhs, int ncols) {
    const long long w = f64 ? 64 : 128, grp = (nrhs + 7) / 8, per = (long long)nfreq * grp;
    return per * ((ncols + w - 1) / w) <= kMaxItems && per * ((Nd + 15) / 16) + kWantItems <= kMaxItems;
}

// Column chunks of a call's forward products, no more than the workspace has room for.
int full_fwd_parts(bool f64, int Nd, int nfreq, int nrhs, int ncols, int max_parts) {
    return fwd_parts_of(f64, Nd, nfreq, nrhs, ncols, fwd_tiles(f64, Nd, nfreq, nrhs, ncols), max_parts);
}

hipError_t launch_full_fwd(bool f64, const GemvArgs& ga, int parts, const void* fhat, const void* X, void* Yp,
                           hipStream_t st) {
    FullArgs fa = base(ga);
    const int T = fwd_tiles(f64, ga.Nd, ga.nfreq, ga.nrhs, ga.ncols), R = fwd_blocks(f64, ga.Nd, T), js = f64 ? 8 : 16;
    const int nsteps = (ga.ncols + js - 1) / js;
    fa.part_stride = (long long)ga.nfreq * ga.nrhs * ga.Nd;
    fa.n_part = parts;
    fa.steps_per_part = (nsteps + parts - 1) / parts;
    fa.n_slab = (ga.Nd + 16 * R - 1) / (16 * R);
    fa.n_grp = groups(ga.nrhs, T);
    const hipError_t e = set_items(fa, (long long)ga.nfreq * fa.n_part * fa.n_slab * fa.n_grp);
    if (e != hipSuccess) return e;
    auto pick = [&](auto ct, auto t) {
        using CT = decltype(ct);
        constexpr int TT = decltype(t)::value;
        if (R == 1) fwd_go<CT, TT, 1>(fa, fhat, X, Yp, st);
        else if (R == 2) fwd_go<CT, TT, 2>(fa, fhat, X, Yp, st);
        else if constexpr (TT == 2 && sizeof(CT) == 8) fwd_go<CT, TT, 4>(fa, fhat, X, Yp, st);
    };
    if (f64) {
        if (T == 1) pick(double{}, std::integral_constant<int, 1>{});
        else pick(double{}, std::integral_constant<int, 2>{});
    } else {
        if (T == 1) pick(float{}, std::integral_constant<int, 1>{});
        else if (T == 2) pick(float{}, std::integral_constant<int, 2>{});
        else pick(float{}, std::integral_constant<int, 4>{});
    }
    return hipGetLastError();
}

hipError_t launch_full_adj(bool f64, const GemvArgs& ga, const void* fhat, const void* Y, void* Xp, hipStream_t st) {
    FullArgs fa = base(ga);
    const int T = adj_tiles(f64, ga.Nd, ga.nfreq, ga.nrhs, ga.ncols), W = f64 ? 16 : 32;
    fa.n_grp = groups(ga.nrhs, T);
    // the widest column tile that still fills the chip: 4 (FP64) or 2 (FP32)
    // blocks are 1 KB of a row per wavefront
    int C = f64 ? 4 : 2;
    while (C > 1 && (long long)ga.nfreq * fa.n_grp * ((ga.ncols + 4 * C * W - 1) / (4 * C * W)) < kWantItems) C /= 2;
    fa.n_slab = (ga.ncols + 4 * C * W - 1) / (4 * C * W);
    const hipError_t e = set_items(fa, (long long)ga.nfreq * fa.n_slab * fa.n_grp);
    if (e != hipSuccess) return e;
    auto pick = [&](auto ct, auto t) {
        using CT = decltype(ct);
        constexpr int TT = decltype(t)::value;
        if (C == 1) adj_go<CT, TT, 1>(fa, fhat, Y, Xp, st);
        else if (C == 2) adj_go<CT, TT, 2>(fa, fhat, Y, Xp, st);
        else if constexpr (sizeof(CT) == 8) adj_go<CT, TT, 4>(fa, fhat, Y, Xp, st);
    };
    if (f64) {
        if (T == 1) pick(double{}, std::integral_constant<int, 1>{});
        else pick(double{}, std::integral_constant<int, 2>{});
    } else {
        if (T == 1) pick(float{}, std::integral_constant<int, 1>{});
        else if (T == 2) pick(float{}, std::integral_constant<int, 2>{});
        else pick(float{}, std::integral_constant<int, 4>{});
    }
    return hipGetLastError();
}

}  // namespace p2o
