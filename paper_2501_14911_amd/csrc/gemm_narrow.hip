// Per-frequency complex products of BF16 and FP16 spectra with few right-hand
// sides (or few sensors) on the matrix cores.
//
// The LDS-ring kernels of gemm_mfma.hip work on tiles of 32 or 64 right-hand
// sides and at least 64 sensors; below that most of their matrix work, LDS
// traffic and right-hand-side loads is padding.  Here 8 right-hand sides are the
// 16 rows of v_mfma_f32_16x16x32 (row 2 b + c: right-hand side b, c = 0 the real,
// 1 the imaginary part of the result), and the spectrum goes from memory to the
// matrix cores without LDS:
//  - forward: 16 bytes of a spectrum row are 4 complex columns = the 8 values of a
//    lane's operand.  Lane (n, g) loads those of row n at column 4 g of a run of
//    16; a step is two such runs, one 128-byte line of each of 16 R rows.  The
//    right-hand sides enter as (x_r, -x_i) in rows c = 0 and (x_i, x_r) in rows c =
//    1, made from the loaded words by a lane's own rotation and sign.
//  - adjoint: lane (n, g) loads 4 columns of 4 sensor rows 4 g ..; the words of one
//    column are the operand for it, so the 4 x 4 block needs no transposition.
//    (y_r, y_i) and (y_i, -y_r) are the other operand.
// BF16 right-hand sides are hi + lo pairs (two products), FP16 ones are scaled
// per right-hand side and rounded once, as in the ring kernels; sums are FP32.
// Bound: HBM.  the figures are at narrow_on.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace p2o {

namespace {

constexpr int kThreads = 256;           // adjoint; forward: 64 NW

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Right-hand-side storage: quad BF16 hi / lo (BF16 spectrum), complex FP32 with a
// scale per right-hand side, or FP16 (re, im) pairs already scaled (FP16 spectrum).
enum { kQuad = 0, kScaled = 1, kPairs = 2 };

template <int K>
__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (K == kQuad)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pair_f16(uint32_t re, uint32_t im, float s) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{__uint_as_float(re) * s, __uint_as_float(im) * s}, f16x2));
}

// Four right-hand-side words as loaded (a, and b for the second 16 bytes of quad
// and complex FP32 storage), as (re, im) words: hi in w[0], lo in w[1] (quad only).
template <int K>
__device__ __forceinline__ void words(u32x4 a, u32x4 b, float s, u32x4 (&w)[2]) {
    if constexpr (K == kScaled)
        w[0] = u32x4{pair_f16(a.x, a.y, s), pair_f16(a.z, a.w, s), pair_f16(b.x, b.y, s), pair_f16(b.z, b.w, s)};
    else
        w[0] = a;
    if constexpr (K == kQuad) w[1] = b;
}
template <int K> constexpr int kHalves = K == kQuad ? 2 : 1;

// A row's own form of (re, im) words: rotated by `rot` (0 or 16) bits, sign bits `neg`.
__device__ __forceinline__ u32x4 form(u32x4 w, uint32_t rot, uint32_t neg) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_alignbit(w[i], w[i], rot) ^ neg;
    return r;
}

__device__ __forceinline__ u32x4 ld16(const uint8_t* p) { return *reinterpret_cast<const u32x4*>(p); }

// Forward: work item = (frequency, column chunk = one scale block, slab of 16 R
// rows, group of 8 T right-hand sides); the NW wavefronts take the chunk's
// 32-column steps in turn and their sums are added in order in LDS.  Rows past Nd
// repeat the last row (not stored); columns past Nm are zero up to the pitch.
template <int K, int T, int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_narrow_fwd(const uint8_t* __restrict__ fhat, const float* __restrict__ scales,
                                                         const uint8_t* __restrict__ X, const float* __restrict__ rhs_scale,
                                                         float2* __restrict__ Yp, FullArgs fa) {
    constexpr int XB = K == kPairs ? 4 : 8;              // bytes per right-hand-side value
    __shared__ float red[NW][R][4][64];
    int q = xcd_item(fa.Q);
    if (q >= fa.items) return;
    const int grp = q % fa.n_grp; q /= fa.n_grp;
    const int slab = q % fa.n_slab; q /= fa.n_slab;
    const int part = q % fa.n_part;
    const int w = q / fa.n_part;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int nsteps = (fa.ncols + 31) / 32;
    const int s0 = part * fa.steps_per_part, s1 = min(nsteps, s0 + fa.steps_per_part);
    const uint32_t rot = n & 1 ? 16u : 0u, neg = n & 1 ? 0u : 0x80000000u;   // (x_i, x_r) or (x_r, -x_i)

    const uint8_t* Fl[R];
#pragma unroll
    for (int a = 0; a < R; ++a)
        Fl[a] = fhat + ((long long)w * fa.Nd + min(fa.Nd - 1, slab * 16 * R + 16 * a + n)) * fa.pitch * 4 + 16 * g;
    const uint8_t* Xl[T];
    float xs[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int b = min(fa.nrhs - 1, grp * 8 * T + 8 * t + (n >> 1));
        Xl[t] = X + (((long long)w * fa.nrhs + b) * fa.pitch + 4 * g) * XB;
        xs[t] = K == kScaled ? rhs_scale[b] : 1.f;
    }
    f32x4 acc[T][R];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int a = 0; a < R; ++a) acc[t][a] = f32x4{0.f, 0.f, 0.f, 0.f};

    struct Stage { u32x4 f[R][2], xa[T][2], xb[T][2]; };
    auto load = [&](Stage& st, int s) {
        const bool live = s < s1;                        // past the chunk: its last step against zeros
        const long long c = (long long)(live ? s : s1 - 1) * 32;
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h) st.f[a][h] = ld16(Fl[a] + (c + 16 * h) * 4);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint8_t* p = Xl[t] + (c + 16 * h) * XB;
                const u32x4 zero = {0u, 0u, 0u, 0u}, a = ld16(p);
                st.xa[t][h] = live ? a : zero;
                if constexpr (K != kPairs) {
                    const u32x4 b = ld16(p + 16);
                    st.xb[t][h] = live ? b : zero;
                }
            }
    };
    auto products = [&](const Stage& st) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                u32x4 x[2];
                words<K>(st.xa[t][h], st.xb[t][h], xs[t], x);
#pragma unroll
                for (int l = 0; l < kHalves<K>; ++l) {
                    const u32x4 op = form(x[l], rot, neg);
#pragma unroll
                    for (int a = 0; a < R; ++a) acc[t][a] = mma<K>(op, st.f[a][h], acc[t][a]);
                }
            }
    };
    Stage A, B;
    load(A, s0 + wave);
    for (int s = s0 + wave; s < s1; s += 2 * NW) {
        load(B, s + NW);
        __builtin_amdgcn_sched_barrier(0);               // keep the loads ahead of the products
        products(A);
        load(A, s + 2 * NW);
        __builtin_amdgcn_sched_barrier(0);
        products(B);
    }

    const float sc = scales[(long long)w * fa.nblk + s0 * 32 / kScaleBlock];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (t) __syncthreads();
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][a][v][lane] = acc[t][a][v];
        __syncthreads();
        if (wave < R) {
            const int row = slab * 16 * R + 16 * wave + n;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int b = grp * 8 * T + 8 * t + 2 * g + p;
                if (row >= fa.Nd || b >= fa.nrhs) continue;
                const float s = K == kQuad ? sc : sc * (1.f / rhs_scale[b]);
                auto sum = [&](int v) {
                    float y = red[0][wave][v][lane];
#pragma unroll
                    for (int k = 1; k < NW; ++k) y += red[k][wave][v][lane];
                    return y;
                };
                Yp[(long long)part * fa.part_stride + ((long long)w * fa.nrhs + b) * fa.Nd + row] =
                    make_float2(sum(2 * p) * s, sum(2 * p + 1) * s);
            }
        }
    }
}

// Adjoint: work item = (frequency, 4 wavefronts x 64 columns, group of 8 T
// right-hand sides); a stage is two steps of 16 sensor rows (rows past Nd repeat
// the last one against the zeros of the padded right-hand sides).  Results as
// complex FP32, or (kHalf) as FP16 pairs multiplied by out_scale[b].
template <int K, int T, bool kHalf>
__global__ __launch_bounds__(kThreads) void k_narrow_adj(const uint8_t* __restrict__ fhat, const float* __restrict__ scales,
                                                         const uint8_t* __restrict__ Y, const float* __restrict__ rhs_scale,
                                                         const float* __restrict__ out_scale, void* __restrict__ Xp,
                                                         FullArgs fa) {
    int q = xcd_item(fa.Q);
    if (q >= fa.items) return;
    const int grp = q % fa.n_grp; q /= fa.n_grp;
    const int ct = q % fa.n_slab;
    const int w = q / fa.n_slab;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int base = (ct * 4 + wave) * 64, col = base + 4 * n;
    if (base >= fa.ncols) return;                        // (no barrier below)
    const uint32_t rot = n & 1 ? 16u : 0u, neg = n & 1 ? 0x80000000u : 0u;   // (y_i, -y_r) or (y_r, y_i)
    const int ld = (fa.Nd + 15) / 16 * 16;               // padded right-hand-side rows

    const long long rowb = (long long)fa.pitch * 4;
    const uint8_t* F = fhat + (long long)w * fa.Nd * rowb + (long long)(col < fa.ncols ? col : 0) * 4;
    const uint8_t* Yl[T];
    float ys[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int b = min(fa.nrhs - 1, grp * 8 * T + 8 * t + (n >> 1));
        Yl[t] = Y + (((long long)w * fa.nrhs + b) * ld + 4 * g) * 8;
        ys[t] = K == kScaled ? rhs_scale[b] : 1.f;
    }
    f32x4 acc[T][4];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};

    struct Stage { u32x4 f[2][4], ya[T][2], yb[T][2]; };
    auto load = [&](Stage& st, int i0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = i0 + 16 * h;
            const bool live = i < ld;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                st.f[h][r] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4*>(F + (long long)min(i + 4 * g + r, fa.Nd - 1) * rowb));
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint8_t* p = Yl[t] + (live ? i : 0) * 8;
                const u32x4 zero = {0u, 0u, 0u, 0u}, a = ld16(p), b = ld16(p + 16);
                st.ya[t][h] = live ? a : zero;
                st.yb[t][h] = live ? b : zero;
            }
        }
    };
    auto products = [&](const Stage& st) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 op[T][2];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                u32x4 y[2];
                words<K>(st.ya[t][h], st.yb[t][h], ys[t], y);
#pragma unroll
                for (int l = 0; l < kHalves<K>; ++l) op[t][l] = form(y[l], rot, neg);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const u32x4 f = {st.f[h][0][c], st.f[h][1][c], st.f[h][2][c], st.f[h][3][c]};
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int l = 0; l < kHalves<K>; ++l) acc[t][c] = mma<K>(op[t][l], f, acc[t][c]);
            }
        }
    };
    Stage A, B;
    load(A, 0);
    for (int i = 0; i < ld; i += 64) {
        load(B, i + 32);
        __builtin_amdgcn_sched_barrier(0);               // keep the loads ahead of the products
        products(A);
        load(A, i + 64);
        __builtin_amdgcn_sched_barrier(0);
        products(B);
    }

    if (col >= fa.ncols) return;
    const float sc = scales[(long long)w * fa.nblk + col / kScaleBlock];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int b = grp * 8 * T + 8 * t + 2 * g + p;
            if (b >= fa.nrhs) continue;
            float s = K == kQuad ? sc : sc * (1.f / rhs_scale[b]);
            if constexpr (kHalf) s *= out_scale[b];
            const long long at = ((long long)w * fa.nrhs + b) * fa.pitch + col;
            float v[8];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                v[2 * c] = acc[t][c][2 * p] * s;
                v[2 * c + 1] = acc[t][c][2 * p + 1] * s;
            }
            if constexpr (kHalf) {
                u32x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    o[c] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{v[2 * c], v[2 * c + 1]}, f16x2));
                *reinterpret_cast<u32x4*>(reinterpret_cast<uint32_t*>(Xp) + at) = o;
            } else {
                float4* o = reinterpret_cast<float4*>(reinterpret_cast<float2*>(Xp) + at);
                o[0] = make_float4(v[0], v[1], v[2], v[3]);
                o[1] = make_float4(v[4], v[5], v[6], v[7]);
            }
        }
}

// (4 tiles: forward products of at most 16 sensors only)
int rhs_tiles(int nrhs) { return nrhs <= 8 ? 1 : nrhs <= 16 ? 2 : 4; }
int row_blocks(int Nd) { return Nd <= 16 ? 1 : Nd <= 32 ? 2 : Nd <= 48 ? 3 : 4; }

FullArgs base(const GemmArgs& ga) {
    FullArgs fa{};
    fa.Nd = ga.Nd;
    fa.pitch = ga.pitch;
    fa.ncols = ga.ncols;
    fa.nrhs = ga.nrhs;
    fa.nblk = ga.nblk;
    fa.n_grp = (ga.nrhs + 8 * rhs_tiles(ga.nrhs) - 1) / (8 * rhs_tiles(ga.nrhs));
    return fa;
}

// Below, 8 wavefronts share a forward item instead of 4 where its rows are a whole
// chunk (200 x 4097, L = 64, 2 right-hand sides, F calls: 52 us against 81; shorter rows
// are up to a quarter slower that way: 200 x 257, L = 972, 9: 109 and 76).
constexpr int kFewItems = 2048;

template <typename F>
void by_tiles(int T, F&& f) {
    if (T == 1) f(std::integral_constant<int, 1>{});
    else if (T == 2) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{});
}

}  // namespace

// Whether calls without a forced or tuned ring variant take these kernels.  FP16
// spectra, us, here against the fastest ring variant (BF16 alike):
//   forward, 2 / 8 / 16 right-hand sides: 8 sensors x 16384, L = 500: 43 / 89 / 163
//   against 149 / 182 / 212 (64: 438 against 430); 37 x 5003, L = 486: 50 / 63 / 85
//   against 100 / 131 / 135; 200 x 8192, L = 256: 219 / 243 / 287 against 263 / 284 /
//   304; 300 x 16384, L = 120: 242 / 271 / 314 against 196 / 246 / 261; 37 x 5003
//   at 64: 255 against 211.
//   adjoint: 8 sensors 100 / 147 / 255 against 192 / 212 / 229; 37: 45 / 57 / 86 against
//   90 / 97 / 107; 200: 139 / 167 / 202 against 196 / 207 / 217 (BF16 at 16: 207
//   against 194); 600 x 16384, L = 120: 380 / 437 / 500 against 412 / 423 / 437.
// Forward rows of few columns are a step or two per wavefront, while the ring's larger
// tiles of sensors and right-hand sides read the other operand less often, so it keeps
// rows shorter than this: past 64 sensors with the frequencies, as its workgroups are few
// below that (products, FP16, L = 1000, ring against here, us: 65 x 400, 4 right-hand sides
// 19 and 26, x 512: 23, 25; 256 x 512, L = 500, 9: 27, 30, 2: 26, 26; L = 120, 65 x 256, 4
// the other way, 1 and 0.78; whole F calls, FP16, L = 972, 16 x 257, 33: 59, 64, x 512: 81,
// 80; as means over L = 64 .. 972 the two are equal near the lines).
static int min_cols(int Nd, int nfreq, int nrhs) {
    if (Nd > 64) return nfreq > 100 ? 448 : 200;
    return nrhs > 32 ? 448 : nrhs > 16 || (Nd > 32 && nrhs > 8) ? 200 : 0;
}

bool narrow_on(int Nd, int nfreq, int nrhs, int ncols, bool fwd) {
    const bool fast = fwd ? (Nd <= 16 || (Nd <= 256 && nrhs <= 16)) && ncols >= min_cols(Nd, nfreq, nrhs)
                          : nrhs <= 8 ? Nd <= 256 : nrhs <= 16 && Nd > 16 && Nd <= 128;
    // a launch's work items at the smallest tiles
    const long long per = (long long)nfreq * ((nrhs + 7) / 8);
    return fast && per * ((ncols + 255) / 256) <= kMaxItems && per * ((Nd + 15) / 16) * ((ncols + kScaleBlock - 1) / kScaleBlock) <= kMaxItems / 2;
}

hipError_t launch_narrow_fwd(const GemmArgs& ga, const void* fhat, const float* scales, const void* X, void* Yp,
                             hipStream_t st) {
    if (ga.a_f16 && !ga.rhs_scale) return hipErrorInvalidValue;      // FP16 products read per-RHS scales
    FullArgs fa = base(ga);
    const int T = rhs_tiles(ga.nrhs), R = row_blocks(ga.Nd);
    fa.part_stride = ga.part_stride;
    fa.n_part = gemm_fwd_kchunks(ga.ncols);
    fa.steps_per_part = kScaleBlock / 32;
    fa.n_slab = (ga.Nd + 16 * R - 1) / (16 * R);
    hipError_t e = set_items(fa, (long long)ga.nfreq * fa.n_part * fa.n_slab * fa.n_grp);
    if (e != hipSuccess) return e;
    auto go = [&](auto k, auto t, auto r) {
        constexpr int K = decltype(k)::value, TT = decltype(t)::value, RR = decltype(r)::value;
        auto with = [&](auto nw) {
            constexpr int NW = decltype(nw)::value;
            hipLaunchKernelGGL((k_narrow_fwd<K, TT, RR, NW>), dim3(8 * fa.Q), dim3(64 * NW), 0, st, (const uint8_t*)fhat,
                               scales, (const uint8_t*)X, ga.rhs_scale, (float2*)Yp, fa);
        };
        if (fa.items < kFewItems && ga.ncols >= kScaleBlock) with(std::integral_constant<int, 8>{});
        else with(std::integral_constant<int, 4>{});
    };
    auto kind = [&](auto k) {
        by_tiles(T, [&](auto t) {
            if (R == 1) go(k, t, std::integral_constant<int, 1>{});
            else if constexpr (decltype(t)::value == 4) e = hipErrorInvalidValue;
            else if (R == 2) go(k, t, std::integral_constant<int, 2>{});
            else if (R == 3) go(k, t, std::integral_constant<int, 3>{});
            else go(k, t, std::integral_constant<int, 4>{});
        });
    };
    if (!ga.a_f16) kind(std::integral_constant<int, kQuad>{});
    else if (ga.b_f16) kind(std::integral_constant<int, kPairs>{});
    else kind(std::integral_constant<int, kScaled>{});
    return e != hipSuccess ? e : hipGetLastError();
}

hipError_t launch_narrow_adj(const GemmArgs& ga, const void* fhat, const float* scales, const void* Y, void* Xp,
                             hipStream_t st) {
    if (ga.a_f16 && !ga.rhs_scale) return hipErrorInvalidValue;      // FP16 products read per-RHS scales
    FullArgs fa = base(ga);
    fa.n_slab = (ga.ncols + 255) / 256;
    const hipError_t e = set_items(fa, (long long)ga.nfreq * fa.n_slab * fa.n_grp);
    if (e != hipSuccess) return e;
    auto go = [&](auto k, auto t, auto h) {
        hipLaunchKernelGGL((k_narrow_adj<decltype(k)::value, decltype(t)::value, decltype(h)::value>), dim3(8 * fa.Q),
                           dim3(kThreads), 0, st, (const uint8_t*)fhat, scales, (const uint8_t*)Y, ga.rhs_scale,
                           ga.out_scale, Xp, fa);
    };
    auto kind = [&](auto t) {
        if (!ga.a_f16) go(std::integral_constant<int, kQuad>{}, t, std::false_type{});
        else if (ga.out_scale) go(std::integral_constant<int, kScaled>{}, t, std::true_type{});
        else go(std::integral_constant<int, kScaled>{}, t, std::false_type{});
    };
    if (rhs_tiles(ga.nrhs) == 1) kind(std::integral_constant<int, 1>{});
    else if (rhs_tiles(ga.nrhs) == 2) kind(std::integral_constant<int, 2>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace p2o
