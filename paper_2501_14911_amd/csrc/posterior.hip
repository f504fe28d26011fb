// Kernels of the offline and online phases built on the p2o map (section 4,
// Phases 2-4): assembly of the data-space matrix K = Gamma_noise + F G*
// from batched operator columns, its Cholesky factorisation K = L L^T, the
// triangular solves with L, and the small elementwise steps of the MAP point
// and posterior-covariance actions.
//
// Dense matrices are FP64 and column-major with a leading dimension: entry
// (i, j) at A[j * lda + i].  The data-space index is j = t * Nd + s (the
// time-major order of the data series).
//
// Cholesky (right-looking, panels of 256 or 512 columns made of blocks of kCB =
// 128):
//   for each 128-column block k of a panel: factor its diagonal block in LDS
//   (one workgroup, 16 columns at a time); solve the rows below it against
//   L_kk^T (16 rows per wavefront, on the matrix cores); subtract its P P^T
//   from the panel's remaining columns.  After the panel: subtract the
//   panel's product from the lower tiles of the trailing matrix.
//   Both updates run on v_mfma_f64_16x16x4f64 (128 x 128 tiles, the panel
//   columns staged in LDS 16 at a time, the tile accumulated in registers
//   and written once).
// The factor is also written transposed into the strict upper triangle
// (entry (i, j), i < j, receives L(j, i)), so that both triangular solves
// read whole contiguous column runs: the forward solve columns of L, the
// backward solve columns of L^T.
#include "common.hpp"
#include "kernels.hpp"

namespace p2o {

namespace {

constexpr int kNB = 64;                 // solve block size

__device__ __forceinline__ double noise_var_at(const double* var, int mode, long long i, int Nd) {
    return mode == 0 ? var[0] : mode == 1 ? var[i % Nd] : var[i];
}

// ---------------------------------------------------------------- K assembly
// E[b][i] = value at i = j0 + b, zero elsewhere (b < ncols, i < N).
template <typename T>
__global__ void k_unit_vectors(T* __restrict__ E, long long N, long long j0, int ncols, T value) {
    const long long n = N * ncols;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / N, i = e - b * N;
        E[e] = (i == j0 + b) ? value : T(0);
    }
}

// K[:, j0 + b] = H[b] + Gamma_noise e_{j0+b}: the operator columns (FP32 or
// FP64) widened to FP64, the noise variance added on the diagonal.
template <typename T>
__global__ void k_K_columns(const T* __restrict__ H, long long N, double* __restrict__ K, long long ldk, long long j0,
                            int ncols, const double* __restrict__ var, int var_mode, int Nd) {
    const long long n = N * ncols;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / N, i = e - b * N;
        double v = (double)H[e];
        if (i == j0 + b) v += noise_var_at(var, var_mode, i, Nd);
        K[(j0 + b) * ldk + i] = v;
    }
}

// ---------------------------------------------------------------- elementwise steps of the online phase
// D = gamma d / var (nrhs data series of N values).
template <typename T>
__global__ void k_weight_data(const T* __restrict__ d, T* __restrict__ D, long long N, int nrhs,
                              const double* __restrict__ var, int var_mode, int Nd, double gamma) {
    const long long n = N * nrhs;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long i = e % N;
        D[e] = (T)(gamma * (double)d[e] / noise_var_at(var, var_mode, i, Nd));
    }
}

// Z[b][i] = Y[b][i] widened to FP64 (Z rows ldz apart).
template <typename T>
__global__ void k_to_f64(const T* __restrict__ Y, double* __restrict__ Z, long long N, int nrhs, long long ldz) {
    const long long n = N * nrhs;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / N, i = e - b * N;
        Z[b * ldz + i] = (double)Y[e];
    }
}

// D[b][i] = a0 * D[b][i] + a1 * Z[b][i]   (Z rows ldz apart).
// (a0 = 0 does not read D, so stale contents never reach the result.)
template <typename T>
__global__ void k_combine(T* __restrict__ D, const double* __restrict__ Z, long long N, int nrhs, long long ldz,
                          double a0, double a1) {
    const long long n = N * nrhs;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / N, i = e - b * N;
        const double z = a1 * Z[b * ldz + i];
        D[e] = (T)(a0 == 0.0 ? z : a0 * (double)D[e] + z);
    }
}

// out = a0 * out + a1 * v (a0 = 0 does not read out).
template <typename T>
__global__ void k_axpby(const T* __restrict__ v, T* __restrict__ out, long long n, double a0, double a1) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const double y = a1 * (double)v[e];
        out[e] = (T)(a0 == 0.0 ? y : a0 * (double)out[e] + y);
    }
}

// ---------------------------------------------------------------- multi-rate (QoI) series
// A plan observed every r-th step (QoI series, section 2 remark on distinct
// temporal discretisations; section 5: QoIs at 1 Hz, parameters at 10 Hz)
// exchanges series of Nt / r steps, step i standing for fine step r (i+1) - 1.
// Y[b][t][s] = q[b][t / r][s] at those steps, 0 elsewhere.
template <typename T>
__global__ void k_qoi_scatter(const T* __restrict__ q, T* __restrict__ Y, int Nt, int Nd, int r, int nrhs) {
    const long long n = (long long)nrhs * Nt * Nd;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / ((long long)Nt * Nd);
        const int rem = (int)(e - b * Nt * Nd), t = rem / Nd, s = rem - t * Nd;
        Y[e] = (t % r == r - 1) ? q[(b * (Nt / r) + t / r) * Nd + s] : T(0);
    }
}

// q[b][i][s] = Y[b][r (i + 1) - 1][s]; with f64 output (C given), column
// c0 + b of C (leading dimension ldc) receives alpha q[b] (added when accum).
template <typename T>
__global__ void k_qoi_gather(const T* __restrict__ Y, T* __restrict__ q, double* __restrict__ C, long long ldc,
                             long long c0, double alpha, int accum, int Nt, int Nd, int r, int nrhs) {
    const int Ntq = Nt / r;
    const long long n = (long long)nrhs * Ntq * Nd;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / ((long long)Ntq * Nd);
        const int rem = (int)(e - b * Ntq * Nd), i = rem / Nd, s = rem - i * Nd;
        const T v = Y[(b * Nt + (long long)r * (i + 1) - 1) * Nd + s];
        if (C) {
            double* c = C + (c0 + b) * ldc + rem;
            *c = accum ? *c + alpha * (double)v : alpha * (double)v;
        } else {
            q[e] = v;
        }
    }
}

// Rows r0 + b of the data-to-QoI map: Q[(r0 + b) ldq + i] =
// gamma (y[b][i] - h[b][i]) / var_i.
template <typename T>
__global__ void k_d2q_rows(const T* __restrict__ y, const T* __restrict__ h, long long N, int nrows,
                           double* __restrict__ Q, long long ldq, long long r0, const double* __restrict__ var,
                           int var_mode, int Nd, double gamma) {
    const long long n = N * nrows;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long b = e / N, i = e - b * N;
        Q[(r0 + b) * ldq + i] = gamma * ((double)y[e] - (double)h[e]) / noise_var_at(var, var_mode, i, Nd);
    }
}

// q[b][r] = sum_j Q[r ldq + j] d[b][j]: TEAM lanes (a workgroup or a wavefront) per
// (row, RB right-hand sides), striding over j (coalesced) with kU loads of the row
// in flight each, fixed-order reduction.  Bound: HBM (Q once per RB right-hand
// sides).  A workgroup per row fills the chip at a few hundred rows: 400 x 12250, 1
// right-hand side 57.9 -> 11.5 us against a wavefront per row; 800 x 24500, 115 ->
// 39 us, 8 right-hand sides 158 -> 99 us.  For short rows see launch_d2q_apply.
template <int RB, int TEAM>
__global__ __launch_bounds__(256) void k_d2q_apply(const double* __restrict__ Q, long long nq, long long N,
                                                   long long ldq, const double* __restrict__ d, double* __restrict__ q,
                                                   int nrhs) {
    constexpr int kU = RB == 1 ? 8 : 4, kTeams = 256 / TEAM;
    __shared__ double red[RB][4];
    const int b0 = blockIdx.y * RB;
    const double* x[RB];                                  // (a right-hand side past the last repeats it)
#pragma unroll
    for (int b = 0; b < RB; ++b) x[b] = d + (long long)min(b0 + b, nrhs - 1) * N;
    for (long long r = (long long)blockIdx.x * kTeams + threadIdx.x / TEAM; r < nq; r += (long long)gridDim.x * kTeams) {
        const double* row = Q + r * ldq;
        double acc[RB][kU];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int u = 0; u < kU; ++u) acc[b][u] = 0.0;
        long long j = threadIdx.x % TEAM;
        for (; j + (kU - 1) * TEAM < N; j += kU * TEAM) {
            double v[kU], w[RB][kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                v[u] = row[j + u * TEAM];
#pragma unroll
                for (int b = 0; b < RB; ++b) w[b][u] = x[b][j + u * TEAM];
            }
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int u = 0; u < kU; ++u) acc[b][u] += v[u] * w[b][u];
        }
        for (; j < N; j += TEAM) {
            const double v = row[j];
#pragma unroll
            for (int b = 0; b < RB; ++b) acc[b][0] += v * x[b][j];
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            double t = acc[b][0];
#pragma unroll
            for (int u = 1; u < kU; ++u) t += acc[b][u];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
            if constexpr (TEAM == 64) {
                if ((threadIdx.x & 63) == b && b0 + b < nrhs) q[(long long)(b0 + b) * nq + r] = t;
            } else {
                if ((threadIdx.x & 63) == 0) red[b][threadIdx.x >> 6] = t;
            }
        }
        if constexpr (TEAM == 256) {                      // (uniform: every lane has the same rows)
            __syncthreads();
            if (threadIdx.x < RB && b0 + (int)threadIdx.x < nrhs) {
                const double* t = red[threadIdx.x];
                q[(long long)(b0 + threadIdx.x) * nq + r] = (t[0] + t[1]) + (t[2] + t[3]);
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mma(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- Cholesky
// 16 x 16 Cholesky of the rows a[c], c <= m, of lanes m (all lane groups alike),
// the pivots' inverses in lane j of dv.  Returns the first column (1-based) whose
// pivot was not positive, or 0.  kExact: sqrt and a division.  Otherwise the
// hardware's 1 / sqrt estimate and two Newton steps (each squares its relative
// error), the root corrected by its own residual off the chain: no branch, so the
// updates of later columns fill the gaps of the chain; `odd` reports a pivot
// outside the range where no intermediate over- or underflows.
template <bool kExact>
__device__ __forceinline__ int factor16(double (&a)[16], double& dv, int m, bool& odd) {
    int bad = 0;
    dv = 1.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const double d = readlane_f64(a[j], j);
        if (!(d > 0.0) && bad == 0) bad = j + 1;
        double piv, inv;
        if constexpr (kExact) {
            piv = sqrt(d);
            inv = 1.0 / piv;
        } else {
            odd |= !(d > 1e-280 && d < 1e280);
            inv = __builtin_amdgcn_rsq(d);
            const double dh = 0.5 * d;
#pragma unroll
            for (int it = 0; it < 2; ++it) inv = fma(inv, fma(-dh * inv, inv, 0.5), inv);
            const double r = d * inv;
            piv = fma(0.5 * inv, fma(-r, r, d), r);
        }
        const double col = a[j] * inv;                 // (rows past j; row j's own value is not used)
#pragma unroll
        for (int c = j + 1; c < 16; ++c) a[c] -= (m > j ? col : 0.0) * readlane_f64(col, c);
        a[j] = m == j ? piv : (m > j ? col : 0.0);
        dv = m == j ? inv : dv;
    }
    return bad;
}

// Factor the diagonal block at (k, k) of nb <= kCB rows in place: one workgroup,
// the block in LDS (rows from nb up to a multiple of 16 are those of the identity, and
// there are no steps past those: a call with n = 16 or 64 takes 25 or 44 us, with all
// 128 columns 60 or 64), 16 columns at a time.  One wavefront factors the 16 x 16
// diagonal block in registers (lane = row; the pivot and the column's entries are
// broadcast with v_readlane), the rows below are solved against it one row per lane,
// and their product leaves the rest on the matrix cores.  A pivot that is not positive (or not a number) records k +
// j + 1 in *info if nothing was recorded before (*info is reset by the call with k
// = 0).  L is also written transposed into the upper triangle of the block.
// Bound: latency of the 128 dependent columns: 45 us, where 64 columns in the
// registers of one wavefront took 35 us.  Without the chain of the 16-column blocks
// 28 us, without any of the three steps 13.
constexpr int kCB = 2 * kNB;            // diagonal block and panel solve width
constexpr int kCS = kCB + 16;           // LDS column stride (doubles): 4 columns of 16 rows on distinct banks
constexpr int kCholThreads = 512;
__global__ __launch_bounds__(kCholThreads) void k_potrf_block(double* __restrict__ A, long long lda, int k, int nb,
                                                              int* __restrict__ info) {
    extern __shared__ __align__(16) double S[];        // S[c * kCS + r], then 16 inverse pivots
    double* dinv = S + kCB * kCS;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int prev = (info && k > 0) ? *info : 0;
    const int nc = (nb + 15) / 16 * 16;                // columns of the 16-column blocks that hold the nb
#pragma unroll 8
    for (int e = tid; e < kCB * nc; e += kCholThreads) {
        const int c = e / kCB, r = e % kCB;
        S[c * kCS + r] = r < nb && c < nb ? (r >= c ? A[(long long)(k + c) * lda + k + r] : 0.0) : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    int bad = 0;                                       // first non-positive pivot of the block (1-based; wavefront 0)
    auto diagonal = [&](int c0) {                      // by wavefront 0
        double* D = S + c0 * kCS + c0;
        double a[16], dv;
        auto fetch = [&] {
#pragma unroll
            for (int c = 0; c < 16; ++c) a[c] = c <= m ? D[c * kCS + m] : 0.0;
        };
        bool odd = false;
        fetch();
        int b = factor16<false>(a, dv, m, odd);
        if (odd) {
            fetch();
            b = factor16<true>(a, dv, m, odd);
        }
        if (b && bad == 0) bad = c0 + b;
        if (lane < 16) {
            dinv[m] = dv;
#pragma unroll
            for (int c = 0; c < 16; ++c)
                if (c <= m) D[c * kCS + m] = a[c];
        }
    };
    if (wave == 0) diagonal(0);
    __syncthreads();
    for (int c0 = 0; c0 < nc - 16; c0 += 16) {
        double* D = S + c0 * kCS + c0;                 // D[c * kCS + r]: the 16 x 16 diagonal block
        if (tid < nc - c0 - 16) {                      // rows below it, one per lane
            double* X = D + 16 + tid;
            double x[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) x[c] = X[c * kCS];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                x[j] *= dinv[j];
#pragma unroll
                for (int c = j + 1; c < 16; ++c) x[c] -= x[j] * D[j * kCS + c];
            }
#pragma unroll
            for (int c = 0; c < 16; ++c) X[c * kCS] = x[c];
        }
        __syncthreads();
        // the remaining 16-row blocks' tiles: wavefront 0 takes the next diagonal block and
        // factors it while the others take the rest
        const int nt = (nc - c0 - 16) / 16;
        const double* P = S + c0 * kCS + c0 + 16;
        auto update = [&](int q) {
            int tj = 0;
            while (q >= nt - tj) q -= nt - tj++;
            const int R = 16 * (tj + q), C = 16 * tj;
            f64x4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u)
                acc = mma(P[(4 * u + g) * kCS + C + m], P[(4 * u + g) * kCS + R + m], acc);
            double* T = S + (c0 + 16 + C) * kCS + c0 + 16 + R + m;
#pragma unroll
            for (int v = 0; v < 4; ++v) T[(4 * v + g) * kCS] -= acc[v];
        };
        if (wave == 0) {
            update(0);
            diagonal(c0 + 16);
        } else {
            for (int q = wave; q < nt * (nt + 1) / 2; q += kCholThreads / 64 - 1) update(q);
        }
        __syncthreads();
    }
#pragma unroll 8
    for (int e = tid; e < kCB * nc; e += kCholThreads) {
        const int c = e / kCB, r = e % kCB;
        if (r < nb && r >= c) A[(long long)(k + c) * lda + k + r] = S[c * kCS + r];
    }
    // L^T: row k + c, column k + r, by 8 x 8 squares (lanes along c alone would meet in one LDS bank)
#pragma unroll 8
    for (int e = tid; e < kCB * nc; e += kCholThreads) {
        const int q = e >> 6, c = 8 * (q % (kCB / 8)) + (e & 7), r = 8 * (q / (kCB / 8)) + ((e >> 3) & 7);
        if (r < nb && r > c) A[(long long)(k + r) * lda + k + c] = S[c * kCS + r];
    }
    if (tid == 0 && info) {
        if (k == 0) *info = bad;
        else if (prev == 0 && bad) *info = k + bad;
    }
}

// Rows r in [k + kCB, n) of the panel: x L_kk^T = a for each row, L_kk of kCB
// rows.  A wavefront takes 16 rows, their kCB entries as 8 transposed 16 x 16
// tiles in the matrix cores' result layout (lane (m, g): row m, columns 4 v + g),
// which is also the layout of their second operand, so the whole solve runs in
// registers: column tile s is multiplied by the inverse of its 16 x 16 diagonal
// block, corrected once by its residual (x += (t - x L_ss^T) L_ss^-T, so that the
// explicit inverse costs no accuracy), and its product with L_js leaves the tiles j
// > s, L_js loaded one s ahead.  The 16 lane groups of the workgroup invert a
// diagonal block each beforehand (two groups the same one).
// Bound: latency (208 matrix instructions of 64 cycles in each of the SIMDs' one
// wavefront, launch, loads): 21 us for 128 columns, N = 4096 to 8192, against 46 us for 64 with
// one row per lane (44 us with 8 wavefronts per workgroup: two on a SIMD, half of
// the CUs).
constexpr int kTrsmThreads = 256;
__global__ __launch_bounds__(kTrsmThreads) void k_trsm_block(double* __restrict__ A, long long lda, int n, int k) {
    constexpr int NS = kCB / 16;
    __shared__ double ld[NS][16][17], li[NS][16][17];  // [block][row][column] of L_ss and its inverse
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const long long row = (long long)k + kCB + blockIdx.x * (kTrsmThreads / 4) + 16 * wave + m;
    const bool live = row < n;
    f64x4 t[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) t[s][v] = live ? A[(long long)(k + 16 * s + 4 * v + g) * lda + row] : 0.0;
    double lj[2][NS - 1][4];                           // L_js of this s and the next
    auto load = [&](double (&l)[NS - 1][4], int s) {
#pragma unroll
        for (int j = 1; j < NS; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (j > s) l[j - 1][u] = -A[(long long)(k + 16 * s + 4 * u + g) * lda + k + 16 * j + m];
    };
    load(lj[0], 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const double* D = A + (long long)(k + 16 * (2 * wave + h)) * (lda + 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = 4 * v + g;
            ld[2 * wave + h][m][c] = m >= c ? D[(long long)c * lda + m] : 0.0;
        }
    }
    __syncthreads();
    {
        const int b = 2 * wave + (g & 1);              // column m of the inverse of block b
        const double dm = 1.0 / ld[b][m][m];
        double y[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            double a = r == m ? 1.0 : 0.0;
#pragma unroll
            for (int c = 0; c < r; ++c) a -= ld[b][r][c] * y[c];
            y[r] = a * __shfl(dm, 16 * g + r);
        }
        if (g < 2)
#pragma unroll
            for (int r = 0; r < 16; ++r) li[b][r][m] = y[r];
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s + 1 < NS) load(lj[(s + 1) & 1], s + 1);
        __builtin_amdgcn_sched_barrier(0);
        double iv[4], lv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            iv[u] = li[s][m][4 * u + g];
            lv[u] = -ld[s][m][4 * u + g];
        }
        f64x4 x{0.0, 0.0, 0.0, 0.0}, r = t[s];
#pragma unroll
        for (int u = 0; u < 4; ++u) x = mma(iv[u], t[s][u], x);
#pragma unroll
        for (int u = 0; u < 4; ++u) r = mma(lv[u], x[u], r);
#pragma unroll
        for (int u = 0; u < 4; ++u) x = mma(iv[u], r[u], x);
        t[s] = x;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = s + 1; j < NS; ++j) t[j] = mma(lj[s & 1][j - 1][u], x[u], t[j]);
    }
    if (!live) return;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            A[(long long)(k + 16 * s + 4 * v + g) * lda + row] = t[s][v];
            A[row * lda + k + 16 * s + 4 * v + g] = t[s][v];           // L^T: row k + c, column r
        }
}

// 128 x 128 tile products on the FP64 matrix cores, P_j P_i^T for two panels of
// 128 rows: a workgroup's four wavefronts take 64 x 64 each (4 x 4 blocks of 16 x
// 16, in registers).  The panels pass through two LDS buffers kKC columns at a
// time: while the matrix cores work on one, the next columns are loaded into
// registers and then written to the other, so a step has one barrier.  The
// products are taken as the transposed block so that lane l of a block holds rows
// l % 16 of four columns: stores cover 128 contiguous bytes per 16 lanes.
// Bound: the matrix cores: K from the blocks, N = 8192, 4096 columns, 5.87 -> 5.59 ms
// (49 TFLOP/s; a large product reaches 72); the Cholesky updates at N = 8192 (63
// launches) 7.11 -> 6.05 ms, less well because a tile has 16 to 32 steps only and
// the last panels have fewer tiles than CUs.
// load(k0, si, sj) fills this thread's entries e = t + 256 u of the next columns,
// row_of(e) and col_of(e) say which they are; SP: LDS row stride.
constexpr int kST = 128;                // tile
constexpr int kKC = 16;                 // panel columns per LDS stage
constexpr int kNU = kKC * kST / 256;    // staged entries per thread and panel
template <int SP, typename Load, typename At>
__device__ __forceinline__ void tile_products(f64x4 (&acc)[4][4], int kd, double* lds, Load&& load, At&& at) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = (wave >> 1) * 64 + (lane & 15), wc = (wave & 1) * 64 + (lane & 15), lk = lane >> 4;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    double si[kNU], sj[kNU];
    auto stage = [&](double* buf) {
#pragma unroll
        for (int u = 0; u < kNU; ++u) {
            const int o = at(threadIdx.x + 256 * u);
            buf[o] = si[u];
            buf[kKC * SP + o] = sj[u];
        }
    };
    load(0, si, sj);
    stage(lds);
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < kd; k0 += kKC) {
        const bool more = k0 + kKC < kd;
        if (more) load(k0 + kKC, si, sj);              // in flight during the products
        const double* pi = lds + cur * 2 * kKC * SP + lk * SP;
        const double* pj = pi + kKC * SP;
        double vi[2][4], vj[2][4];
        auto frag = [&](int c0, double (&x)[4], double (&y)[4]) {
#pragma unroll
            for (int a = 0; a < 4; ++a) x[a] = pi[c0 * SP + wr + 16 * a];
#pragma unroll
            for (int b = 0; b < 4; ++b) y[b] = pj[c0 * SP + wc + 16 * b];
        };
        frag(0, vi[0], vj[0]);
#pragma unroll
        for (int c0 = 0; c0 < kKC; c0 += 4) {
            const int h = (c0 >> 2) & 1;
            if (c0 + 4 < kKC) frag(c0 + 4, vi[h ^ 1], vj[h ^ 1]);
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) acc[a][b] = mma(vj[h][b], vi[h][a], acc[a][b]);
        }
        if (more) {
            cur ^= 1;
            stage(lds + cur * 2 * kKC * SP);
            __syncthreads();
        }
    }
}

// Tiles numbered column by column: column tile tj has T - tj tiles (tile row >=
// tile column); tj is the largest column with S(tj) = tj (2T - tj + 1) / 2 <= q.
__device__ __forceinline__ void lower_tile(int T, int& ti, int& tj) {
    const long long q = blockIdx.x;
    const double b2 = 2.0 * T + 1.0;
    tj = (int)((b2 - sqrt(b2 * b2 - 8.0 * (double)q)) * 0.5);
    auto S = [&](long long c) { return c * (2LL * T - c + 1) / 2; };
    while (tj > 0 && S(tj) > q) --tj;
    while (S(tj + 1) <= q) ++tj;
    ti = tj + (int)(q - S(tj));
}

// C(i, j) += sign * products for the tile's entries on or below the diagonal,
// rows < m and columns < mc, C column-major at (row 0, column 0) = c0.  A
// wavefront's 16 columns of a row block are read together before any is written.
__device__ __forceinline__ void tile_add(const f64x4 (&acc)[4][4], double* __restrict__ c0, long long ld, int ri, int rj,
                                         int m, int mc, double sign) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi0 = ri + (wave >> 1) * 64 + (lane & 15), gj0 = rj + (wave & 1) * 64 + (lane >> 4);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int gi = gi0 + 16 * a;
        double v[4][4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int gj = gj0 + 16 * b + 4 * u;
                v[b][u] = gi < m && gj < mc && gi >= gj ? c0[(long long)gj * ld + gi] : 0.0;
            }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int gj = gj0 + 16 * b + 4 * u;
                if (gi < m && gj < mc && gi >= gj) c0[(long long)gj * ld + gi] = v[b][u] + sign * acc[a][b][u];
            }
    }
}

// Update A[t0 + i, t0 + j] -= sum_c P[i, c] P[j, c] over the 128 x 128
// tiles of rows [t0, n) and columns [t0, c_end) on or below the diagonal
// (tile row >= tile column), P = A[t0:n, pk0:pk0 + kd].
constexpr int kSyrkSP = kST + 16;       // LDS row stride: reads of 4 columns x 16 rows on distinct banks
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_syrk_update(double* __restrict__ A, long long lda, int n, int t0, int c_end, int pk0, int kd) {
    extern __shared__ __align__(16) double lds[];
    const int m = n - t0, mc = c_end - t0;
    int ti, tj;
    lower_tile((m + kST - 1) / kST, ti, tj);
    const int ri = ti * kST, rj = tj * kST;            // first rows (relative to t0)
    if (rj >= mc) return;
    f64x4 acc[4][4];
    // staging: column e / kST, row e % kST
    tile_products<kSyrkSP>(acc, kd, lds, [&](int k0, double (&si)[kNU], double (&sj)[kNU]) {
        const int kw = min(kKC, kd - k0);
#pragma unroll
        for (int u = 0; u < kNU; ++u) {
            const int e = threadIdx.x + 256 * u, c = e / kST, r = e % kST;
            const double* col = A + (long long)(pk0 + k0 + c) * lda + t0;
            si[u] = c < kw && ri + r < m ? col[ri + r] : 0.0;
            sj[u] = c < kw && rj + r < m ? col[rj + r] : 0.0;
        }
    }, [](int e) { return (e / kST) * kSyrkSP + e % kST; });
    tile_add(acc, A + (long long)t0 * (lda + 1), lda, ri, rj, m, mc, -1.0);
}

constexpr size_t tile_lds(int sp) { return (size_t)4 * kKC * sp * sizeof(double); }

static long long trapezoid_tiles(long long m, long long mc) {
    const long long T = (m + kST - 1) / kST, C = std::min(T, (mc + kST - 1) / kST);
    return C * (2 * T - C + 1) / 2;
}

// ---------------------------------------------------------------- K from the blocks' Gram matrix
// With the blocks F_k themselves at hand (not only their spectrum), the
// (i, j) block of F F^* is sum_{k <= min(i, j)} F_{i-k} F_{j-k}^T (F is
// block lower-triangular Toeplitz), i.e. for i >= j the sum over l <= j of
// G(i - j + l, l), G(p, q) = F_p F_q^T: prefix sums along the block
// diagonals of the Gram matrix G = A A^T of the stacked blocks
// A = [F_0; ...; F_{Nt-1}] (row t Nd + s = sensor s of F_t).  G is summed
// over column chunks of A as they are generated.

// G += B B^T on the lower 128 x 128 tiles (tile row >= tile column) of the
// N x N matrix G, B a chunk of A: N rows of kc columns, row r at B + r ldb.  The
// staging reads 16 consecutive columns (one 128-byte line) of each row.
constexpr int kGramSP = kST + 2;        // LDS row stride: writes of 16 columns x 4 rows spread over the banks
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_gram_update(const double* __restrict__ B, long long ldb, int N, int kc, double* __restrict__ G, long long ldg) {
    extern __shared__ __align__(16) double lds[];
    int ti, tj;
    lower_tile((N + kST - 1) / kST, ti, tj);
    const int ri = ti * kST, rj = tj * kST;
    f64x4 acc[4][4];
    // staging: row e / kKC, column e % kKC
    tile_products<kGramSP>(acc, kc, lds, [&](int k0, double (&si)[kNU], double (&sj)[kNU]) {
        const int kw = min(kKC, kc - k0);
#pragma unroll
        for (int u = 0; u < kNU; ++u) {
            const int e = threadIdx.x + 256 * u, r = e / kKC, c = e % kKC;
            si[u] = c < kw && ri + r < N ? B[(long long)(ri + r) * ldb + k0 + c] : 0.0;
            sj[u] = c < kw && rj + r < N ? B[(long long)(rj + r) * ldb + k0 + c] : 0.0;
        }
    }, [](int e) { return (e % kKC) * kGramSP + e / kKC; });
    tile_add(acc, G, ldg, ri, rj, N, N, 1.0);
}

// Prefix sums along the block diagonals of the lower triangle of G, in
// place: thread (d, p, q) walks block (d + j, j), j = 0 .. Nt - 1 - d, entry
// (p, q), keeping the running sum in a register (q <= p on the diagonal
// blocks, whose upper parts are not computed).
__global__ void k_gram_prefix(double* __restrict__ G, long long ldg, int Nt, int Nd) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long per = (long long)Nd * Nd;
    if (t >= (long long)Nt * per) return;
    const int d = (int)(t / per), e = (int)(t % per), q = e / Nd, p = e % Nd;
    if (d == 0 && p < q) return;
    double* g = G + (long long)q * ldg + (long long)d * Nd + p;    // block (d, 0), entry (p, q)
    const long long step = (long long)Nd * ldg + Nd;                 // to block (d + j + 1, j + 1)
    double sum = 0.0;
    for (int j = 0; j < Nt - d; ++j) {
        sum += *g;
        *g = sum;
        g += step;
    }
}

// K from the prefix-summed G: K = prior_var G + Gamma_noise on and below the
// diagonal, mirrored into the upper triangle (64 x 64 tiles through LDS;
// tile (ti, tj), ti >= tj, writes its transpose to tile (tj, ti)).
__global__ __launch_bounds__(256) void k_gram_finish(double* __restrict__ G, long long ldg, int N, double prior_var,
                                                     const double* __restrict__ var, int var_mode, int Nd) {
    __shared__ double t[64][65];
    const long long qd = blockIdx.x;
    int ti = (int)((sqrt(8.0 * (double)qd + 1.0) - 1.0) * 0.5);
    while ((long long)(ti + 1) * (ti + 2) / 2 <= qd) ++ti;
    while ((long long)ti * (ti + 1) / 2 > qd) --ti;
    const int tj = (int)(qd - (long long)ti * (ti + 1) / 2);
    const int r0 = ti * 64, c0 = tj * 64;
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int c = e / 64, r = e % 64, i = r0 + r, j = c0 + c;
        if (i < N && j < N && i >= j) {
            double v = prior_var * G[(long long)j * ldg + i];
            if (i == j) v += noise_var_at(var, var_mode, i, Nd);
            G[(long long)j * ldg + i] = v;
            t[c][r] = v;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int r = e / 64, c = e % 64, i = r0 + r, j = c0 + c;      // write K(j, i) = K(i, j), i > j
        if (i < N && j < N && i > j) G[(long long)i * ldg + j] = t[c][r];
    }
}

// ---------------------------------------------------------------- triangular solves with L
// One launch per panel of kPB = 128 rows and direction.  Launch j applies panel
// j - 1's solved entries (backward: panel j + 1's) and solves panel j:
//  - workgroup b < nrhs takes right-hand side b through panel j: four wavefronts
//    apply the entries to the panel's rows (64 x 64 blocks), then the panel's two
//    64-row blocks are solved one after the other, one wavefront each, with the
//    block between them applied by a third.  Every wavefront loads its 64 x 64
//    block into registers first (lane = row; column runs of 512 bytes), so all of
//    the panel's loads are in flight together; a solved entry is broadcast with
//    v_readlane, its row scaled by the inverse diagonal beforehand, so that the
//    chain has two readlanes and one fused multiply-add per entry.
//  - the other workgroups apply the same entries to 64 rows past panel j each
//    (forward; above it, backward) for up to 16 T right-hand sides, on the FP64
//    matrix cores (right-hand side x row, so that 16 lanes update 16 consecutive
//    rows), the 128 columns split over four wavefronts.
// Each row thus receives panel m's entries in the launch after m was solved.  The
// factor's transpose in the upper triangle makes every read of the backward solve
// a contiguous column run too.
// Bound: latency, one chain of 128 entries and its launch per panel (the factor,
// 4 N^2 bytes per direction, would take 0.1 ms at N = 12250).  A solve pair at N = 12250
// and 24500: one right-hand side 5.03 -> 1.79 and 10.4 -> 3.71 ms, 32 right-hand
// sides 11.3 -> 1.86 and 24.0 -> 4.93 ms (64-row blocks with separate launches for
// solve and update before).
constexpr int kPB = 2 * kNB;            // panel rows
constexpr int kSolveThreads = 512;

template <bool BWD>
__device__ __forceinline__ void trsv_panel_rhs(const double* __restrict__ L, long long lda, int n, int j,
                                               double* __restrict__ x, double* sh) {
    double* xs = sh;                                   // [kPB] the applied panel's entries
    double* part = sh + kPB;                           // [2][kPB] their products with the panel's rows
    double* sol = sh + 3 * kPB;                        // [kNB] solved entries of the first block
    double* off = sol + kNB;                           // [kNB] their products with the second block's rows
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int P = j * kPB, src = BWD ? j + 1 : j - 1, ks = src * kPB;
    const bool apply = BWD ? ks < n : src >= 0;
    const int first = BWD ? 1 : 0;                     // block solved first
    const int F0 = P + kNB * first, S0 = P + kNB * (1 - first);
    // wavefronts 0, 1: the diagonal blocks; 2: the block between them; 4..7: the applied panel's blocks
    const bool diag = wave < 2;
    const int rg = wave & 1, cg = (wave >> 1) & 1;
    const int row = (wave == 0 ? F0 : wave < 4 ? S0 : P + kNB * rg) + lane;
    const int col0 = wave == 1 ? S0 : wave < 4 ? F0 : ks + kNB * cg;
    const bool rowok = row < n && wave != 3 && (wave < 4 || apply);
    double a[kNB];
#pragma unroll
    for (int c = 0; c < kNB; ++c) {
        const bool ok = rowok && col0 + c < n && (!diag || (BWD ? c > lane : c < lane));
        a[c] = ok ? L[(long long)(col0 + c) * lda + row] : 0.0;
    }
    double inv = 1.0, xi = 0.0;
    if (diag && rowok) {
        inv = 1.0 / L[(long long)row * lda + row];
        xi = x[row];
    }
    if (apply && threadIdx.x < kPB) xs[threadIdx.x] = ks + (int)threadIdx.x < n ? x[ks + threadIdx.x] : 0.0;
    auto dot = [&](const double* v) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
        for (int c = 0; c < kNB; c += 4) {
            s0 += a[c] * v[c];
            s1 += a[c + 1] * v[c + 1];
            s2 += a[c + 2] * v[c + 2];
            s3 += a[c + 3] * v[c + 3];
        }
        return (s0 + s1) + (s2 + s3);
    };
    auto solve = [&](double b) {
        double y = b * inv;
#pragma unroll
        for (int c = 0; c < kNB; ++c) {
            const int q = BWD ? kNB - 1 - c : c;
            y -= a[q] * readlane_f64(y, q);
        }
        return y;
    };
    if (diag) {
#pragma unroll
        for (int c = 0; c < kNB; ++c) a[c] *= inv;
    }
    if (apply) {                                       // (uniform; the first panel has nothing to apply)
        __syncthreads();
        if (wave >= 4) part[cg * kPB + kNB * rg + lane] = dot(xs + kNB * cg);
        __syncthreads();
        if (diag) xi -= part[row - P] + part[kPB + row - P];
    }
    // a last panel of one block (P + kNB >= n): its wavefront, and no second chain
    const bool two = P + kNB < n;
    if (wave == (two ? 0 : first)) {
        xi = solve(xi);
        sol[lane] = xi;
        if (rowok) x[row] = xi;
    }
    if (!two) return;
    __syncthreads();
    if (wave == 2) off[lane] = dot(sol);
    __syncthreads();
    if (wave == 1) {
        xi = solve(xi - off[lane]);
        if (rowok) x[row] = xi;
    }
}

template <bool BWD, int T>
__device__ __forceinline__ void trsv_panel_rows(const double* __restrict__ L, long long lda, int n, int j, int item,
                                                int row_tiles, double* __restrict__ X, long long ldx, int nrhs,
                                                double* sh) {
    const int P = j * kPB, src = BWD ? j + 1 : j - 1, ks = src * kPB;
    if (BWD ? ks >= n : src < 0) return;               // nothing solved yet
    const int r0 = (BWD ? 0 : P + kPB) + 64 * (item % row_tiles), lim = BWD ? P : n;
    const int b0 = 16 * T * (item / row_tiles);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int rg = wave & 1, kg = wave >> 1;
    double a[8][2], xv[8][T];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int col = ks + 32 * kg + 4 * q + g;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = r0 + 32 * rg + 16 * h + m;
            a[q][h] = r < lim && col < n ? L[(long long)col * lda + r] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int b = b0 + 16 * t + m;
            xv[q][t] = b < nrhs && col < n ? X[(long long)b * ldx + col] : 0.0;
        }
    }
    f64x4 acc[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            acc[t][h] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 8; ++q)
                acc[t][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[q][t], a[q][h], acc[t][h], 0, 0, 0);
        }
    // lane l holds D[4 v + l / 16][l % 16] in item v: right-hand side 4 v + g, row m; the four
    // column quarters are added here, wavefront w finishing item v = w / 2 of its 32 rows
    auto red = [&](int k, int h, int v) -> double& { return sh[(((k * 2 + rg) * 2 + h) * 4 + v) * 64 + lane]; };
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (t) __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v) red(kg, h, v) = acc[t][h][v];
        __syncthreads();
        const int b = b0 + 16 * t + 4 * kg + g;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = r0 + 32 * rg + 16 * h + m;
            if (r < lim && b < nrhs)
                X[(long long)b * ldx + r] -= (red(0, h, kg) + red(1, h, kg)) + (red(2, h, kg) + red(3, h, kg));
        }
    }
}

template <bool BWD, int T>
__global__ __launch_bounds__(kSolveThreads) void k_trsv_panel(const double* __restrict__ L, long long lda, int n, int j,
                                                              int row_tiles, double* __restrict__ X, long long ldx,
                                                              int nrhs) {
    __shared__ double sh[4 * 2 * 2 * 4 * 64];
    if ((int)blockIdx.x < nrhs) trsv_panel_rhs<BWD>(L, lda, n, j, X + (long long)blockIdx.x * ldx, sh);
    else trsv_panel_rows<BWD, T>(L, lda, n, j, (int)blockIdx.x - nrhs, row_tiles, X, ldx, nrhs, sh);
}

dim3 grid_for(long long n) { return dim3((unsigned)std::max<long long>(1, std::min<long long>(4096, (n + 255) / 256))); }

}  // namespace

// ---------------------------------------------------------------- launchers
hipError_t launch_unit_vectors(bool f64, void* E, long long N, long long j0, int ncols, double value, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_unit_vectors<double>, grid_for(N * ncols), dim3(256), 0, st, (double*)E, N, j0, ncols, value);
    else
        hipLaunchKernelGGL(k_unit_vectors<float>, grid_for(N * ncols), dim3(256), 0, st, (float*)E, N, j0, ncols,
                           (float)value);
    return hipGetLastError();
}

hipError_t launch_K_columns(bool f64, const void* H, long long N, double* K, long long ldk, long long j0, int ncols,
                            const double* var, int var_mode, int Nd, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_K_columns<double>, grid_for(N * ncols), dim3(256), 0, st, (const double*)H, N, K, ldk, j0,
                           ncols, var, var_mode, Nd);
    else
        hipLaunchKernelGGL(k_K_columns<float>, grid_for(N * ncols), dim3(256), 0, st, (const float*)H, N, K, ldk, j0,
                           ncols, var, var_mode, Nd);
    return hipGetLastError();
}

hipError_t launch_weight_data(bool f64, const void* d, void* D, long long N, int nrhs, const double* var, int var_mode,
                              int Nd, double gamma, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_weight_data<double>, grid_for(N * nrhs), dim3(256), 0, st, (const double*)d, (double*)D, N,
                           nrhs, var, var_mode, Nd, gamma);
    else
        hipLaunchKernelGGL(k_weight_data<float>, grid_for(N * nrhs), dim3(256), 0, st, (const float*)d, (float*)D, N,
                           nrhs, var, var_mode, Nd, gamma);
    return hipGetLastError();
}

hipError_t launch_to_f64(bool f64, const void* Y, double* Z, long long N, int nrhs, long long ldz, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_to_f64<double>, grid_for(N * nrhs), dim3(256), 0, st, (const double*)Y, Z, N, nrhs, ldz);
    else
        hipLaunchKernelGGL(k_to_f64<float>, grid_for(N * nrhs), dim3(256), 0, st, (const float*)Y, Z, N, nrhs, ldz);
    return hipGetLastError();
}

hipError_t launch_combine(bool f64, void* D, const double* Z, long long N, int nrhs, long long ldz, double a0, double a1,
                          hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_combine<double>, grid_for(N * nrhs), dim3(256), 0, st, (double*)D, Z, N, nrhs, ldz, a0, a1);
    else
        hipLaunchKernelGGL(k_combine<float>, grid_for(N * nrhs), dim3(256), 0, st, (float*)D, Z, N, nrhs, ldz, a0, a1);
    return hipGetLastError();
}

hipError_t launch_axpby(bool f64, const void* v, void* out, long long n, double a0, double a1, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_axpby<double>, grid_for(n), dim3(256), 0, st, (const double*)v, (double*)out, n, a0, a1);
    else
        hipLaunchKernelGGL(k_axpby<float>, grid_for(n), dim3(256), 0, st, (const float*)v, (float*)out, n, a0, a1);
    return hipGetLastError();
}

hipError_t launch_qoi_scatter(bool f64, const void* q, void* Y, int Nt, int Nd, int r, int nrhs, hipStream_t st) {
    const long long n = (long long)nrhs * Nt * Nd;
    if (f64)
        hipLaunchKernelGGL(k_qoi_scatter<double>, grid_for(n), dim3(256), 0, st, (const double*)q, (double*)Y, Nt, Nd, r,
                           nrhs);
    else
        hipLaunchKernelGGL(k_qoi_scatter<float>, grid_for(n), dim3(256), 0, st, (const float*)q, (float*)Y, Nt, Nd, r,
                           nrhs);
    return hipGetLastError();
}

hipError_t launch_qoi_gather(bool f64, const void* Y, void* q, double* C, long long ldc, long long c0, double alpha,
                             bool accum, int Nt, int Nd, int r, int nrhs, hipStream_t st) {
    const long long n = (long long)nrhs * (Nt / r) * Nd;
    if (f64)
        hipLaunchKernelGGL(k_qoi_gather<double>, grid_for(n), dim3(256), 0, st, (const double*)Y, (double*)q, C, ldc, c0,
                           alpha, accum ? 1 : 0, Nt, Nd, r, nrhs);
    else
        hipLaunchKernelGGL(k_qoi_gather<float>, grid_for(n), dim3(256), 0, st, (const float*)Y, (float*)q, C, ldc, c0,
                           alpha, accum ? 1 : 0, Nt, Nd, r, nrhs);
    return hipGetLastError();
}

hipError_t launch_d2q_rows(bool f64, const void* y, const void* h, long long N, int nrows, double* Q, long long ldq,
                           long long r0, const double* var, int var_mode, int Nd, double gamma, hipStream_t st) {
    if (f64)
        hipLaunchKernelGGL(k_d2q_rows<double>, grid_for(N * nrows), dim3(256), 0, st, (const double*)y, (const double*)h,
                           N, nrows, Q, ldq, r0, var, var_mode, Nd, gamma);
    else
        hipLaunchKernelGGL(k_d2q_rows<float>, grid_for(N * nrows), dim3(256), 0, st, (const float*)y, (const float*)h, N,
                           nrows, Q, ldq, r0, var, var_mode, Nd, gamma);
    return hipGetLastError();
}

// A wavefront per row below 1024 columns, where a workgroup has less than its four
// loads per lane and its barriers and its launch are the time (20000 x 10, 1 and 64
// right-hand sides 15 and 668 us, with wavefronts 10 and 156; x 1000, 31 and 924,
// 30 and 848; 1600 x 1500, 8: 15, with wavefronts 18).
hipError_t launch_d2q_apply(const double* Q, long long nq, long long N, long long ldq, const double* d, double* q,
                            int nrhs, hipStream_t st) {
    auto go = [&](auto k, int rows_per_wg, int rb) {
        const long long rows = (nq + rows_per_wg - 1) / rows_per_wg;
        hipLaunchKernelGGL(k, dim3((unsigned)std::min<long long>(rows, 1 << 20), (unsigned)((nrhs + rb - 1) / rb)), dim3(256),
                           0, st, Q, nq, N, ldq, d, q, nrhs);
    };
    if (N < 1024)
        nrhs == 1 ? go(k_d2q_apply<1, 64>, 4, 1) : nrhs == 2 ? go(k_d2q_apply<2, 64>, 4, 2) : go(k_d2q_apply<4, 64>, 4, 4);
    else
        nrhs == 1 ? go(k_d2q_apply<1, 256>, 1, 1) : go(k_d2q_apply<4, 256>, 1, 4);
    return hipGetLastError();
}

hipError_t launch_gram_update(const double* B, long long ldb, long long N, int kc, double* G, long long ldg,
                              hipStream_t st) {
    if (N <= 0 || kc <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gram_update, dim3((unsigned)trapezoid_tiles(N, N)), dim3(256), tile_lds(kGramSP), st, B, ldb,
                       (int)N, kc, G, ldg);
    return hipGetLastError();
}

hipError_t launch_gram_to_K(double* G, long long ldg, int Nt, int Nd, double prior_var, const double* var,
                            int var_mode, hipStream_t st) {
    const long long N = (long long)Nt * Nd, nthr = (long long)Nt * Nd * Nd;
    hipLaunchKernelGGL(k_gram_prefix, dim3((unsigned)((nthr + 255) / 256)), dim3(256), 0, st, G, ldg, Nt, Nd);
    const long long T = (N + 63) / 64;
    hipLaunchKernelGGL(k_gram_finish, dim3((unsigned)(T * (T + 1) / 2)), dim3(256), 0, st, G, ldg, (int)N, prior_var,
                       var, var_mode, Nd);
    return hipGetLastError();
}

hipError_t launch_cholesky(double* A, long long n, long long lda, int* info, hipStream_t st) {
    constexpr size_t lds = (kCB * kCS + 16) * sizeof(double);
    long long width = 0;
    for (long long K0 = 0; K0 < n; K0 += width) {
        // panels of 256 columns; 512 where the trailing matrix is large, whose update
        // reads and writes every entry per panel (N = 12250: 25.0 ms with 256
        // throughout, 23.2 with 512; N = 4000: 3.92 against 4.03)
        width = n - K0 > 6144 ? 512 : 256;
        const long long pend = std::min<long long>(K0 + width, n);     // end of the panel
        for (long long k = K0; k < pend; k += kCB) {
            const int nb = (int)std::min<long long>(kCB, n - k);
            hipLaunchKernelGGL(k_potrf_block, dim3(1), dim3(kCholThreads), lds, st, A, lda, (int)k, nb, info);
            const long long below = n - k - nb;
            if (below <= 0) break;
            hipLaunchKernelGGL(k_trsm_block, dim3((unsigned)((below + kTrsmThreads / 4 - 1) / (kTrsmThreads / 4))),
                               dim3(kTrsmThreads), 0, st, A, lda, (int)n, (int)k);
            if (k + kCB < pend)                            // the panel's remaining columns, all rows below
                hipLaunchKernelGGL(k_syrk_update, dim3((unsigned)trapezoid_tiles(below, pend - k - kCB)), dim3(256),
                                   tile_lds(kSyrkSP), st, A, lda, (int)n, (int)(k + kCB), (int)pend, (int)k, kCB);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        if (pend < n)                                       // trailing matrix, the panel's rank
            hipLaunchKernelGGL(k_syrk_update, dim3((unsigned)trapezoid_tiles(n - pend, n - pend)), dim3(256),
                               tile_lds(kSyrkSP), st, A, lda, (int)n, (int)pend, (int)n, (int)K0, (int)(pend - K0));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

template <int T>
static void solve_panels(const double* L, long long n, long long lda, double* X, int nrhs, long long ldx,
                         hipStream_t st) {
    const int np = (int)((n + kPB - 1) / kPB), groups = (nrhs + 16 * T - 1) / (16 * T);
    for (int j = 0; j < np; ++j) {
        const long long past = j > 0 ? std::max(0LL, n - (long long)(j + 1) * kPB) : 0;
        const int tiles = (int)((past + 63) / 64);
        hipLaunchKernelGGL((k_trsv_panel<false, T>), dim3((unsigned)(nrhs + tiles * groups)), dim3(kSolveThreads), 0, st,
                           L, lda, (int)n, j, tiles, X, ldx, nrhs);
    }
    for (int j = np - 1; j >= 0; --j) {
        const int tiles = j < np - 1 ? j * (kPB / 64) : 0;
        hipLaunchKernelGGL((k_trsv_panel<true, T>), dim3((unsigned)(nrhs + tiles * groups)), dim3(kSolveThreads), 0, st,
                           L, lda, (int)n, j, tiles, X, ldx, nrhs);
    }
}

// Right-hand sides per pass over the factor: up to 64.
hipError_t launch_cholesky_solve(const double* L, long long n, long long lda, double* X, int nrhs, long long ldx,
                                 hipStream_t st) {
    if (nrhs <= 16) solve_panels<1>(L, n, lda, X, nrhs, ldx, st);
    else if (nrhs <= 32) solve_panels<2>(L, n, lda, X, nrhs, ldx, st);
    else solve_panels<4>(L, n, lda, X, nrhs, ldx, st);
    return hipGetLastError();
}

}  // namespace p2o
