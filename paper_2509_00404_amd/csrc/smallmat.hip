// One-workgroup fp64 factorizations of the small (k+p)x(k+p) matrices of the decomposition
// (Sec. 3.1): Cholesky + triangular inverse for CholeskyQR2 (thin QR Z = H R), and a
// one-sided Jacobi eigensolver for the Gram matrices of the reduced problem.
#include "smallmat.h"
#include <algorithm>
#include <cstdlib>
#include <utility>

// ---------------------------------------------------------------------------------------
// Blocked Cholesky in LDS, shared by both kernels below.  On entry W holds the lower triangle of a
// symmetric matrix column-major (element (i, c), i >= c, at W[c*ld + i]); on exit the same places
// hold L, and rinv[c] = 1 / L[c][c].  Panels of 16 columns, three workgroup barriers each:
//   1  a lane holds the 16 panel entries of one row below the diagonal block in registers, and every 16 lanes a copy of the
//      16 rows of the diagonal block (each group factors it for itself), so one pass over the columns factors the block and
//      solves the rows: a column's pivot and multipliers reach the 16 lanes by v_mov_b64 with a row broadcast,
//      with no LDS, no scalar registers and no barrier between columns;
//   2  the trailing matrix takes the rank-16 update on the fp64 matrix cores: four v_mfma_f64_16x16x4_f64 per 16x16 tile,
//      transposed, so that a tile's columns are read and written along the lanes.
// The chain of n dependent reciprocal square roots bounds it.  n = 80: 15 us, n = 64: 11 us; blocks of 4
// columns factored by every thread out of LDS, two barriers each, took 31 and 23 us.
// BAD_PIVOT_ZEROES: a pivot <= floor zeroes its column (semi-definite input, eigensolver); otherwise it is
// replaced by 1e-300 and its 1-based index is written to *info (CholeskyQR2's rank check).
// (Multipliers passed as scalars by v_readlane cost 27 cycles each, 3.4 us a panel.)
// ---------------------------------------------------------------------------------------
typedef double double4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double readlane64(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// x of lane N of each row of 16 lanes, in all 16
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
    return __longlong_as_double(__builtin_amdgcn_update_dpp((long long)0, __double_as_longlong(x), 0x150 + N, 0xF, 0xF, true));
}
template <class F, int... I>
__device__ __forceinline__ void for_each_block_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index is a compile-time constant
template <int N, class F>
__device__ __forceinline__ void for_each_block(F&& f) {
    for_each_block_impl(f, std::make_integer_sequence<int, N>{});
}

// 1 / sqrt(x) to ~1e-16: the hardware seed (~2^-23) and one third-order step
__device__ __forceinline__ double chol_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-(x * y), y, 1.0);
    return __builtin_fma(e * y, __builtin_fma(e, 0.375, 0.5), y);
}

// SMALL: the order is at most 4.  (Its own instances of the kernels: behind a test the path cost every order 0.5 us a launch.)
template <bool BAD_PIVOT_ZEROES, bool SMALL>
__device__ __forceinline__ void chol_blocked(double* __restrict__ W, int ld, int n, double* __restrict__ rinv, double floor_,
                             int32_t* __restrict__ info) {
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
    if constexpr (SMALL) {                               // (the same operations on one lane; a panel's 16 columns take 3 us)
        if (tid == 0) {
            double l[4][4], rv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c <= i; ++c) l[i][c] = i < n ? W[(size_t)c * ld + i] : (i == c ? 1.0 : 0.0);
            int bad = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double piv = l[c][c];
                if (BAD_PIVOT_ZEROES) {
                    rv[c] = piv > floor_ ? chol_rsqrt(piv) : 0.0;
                } else {
                    const bool ok = piv > 0.0;
                    bad = !ok && c < n ? c + 1 : bad;
                    piv = ok ? piv : 1e-300;
                    rv[c] = chol_rsqrt(piv);
                }
#pragma unroll
                for (int i = c; i < 4; ++i) l[i][c] *= rv[c];
#pragma unroll
                for (int t = c + 1; t < 4; ++t)
#pragma unroll
                    for (int i = t; i < 4; ++i) l[i][t] = __builtin_fma(-l[i][c], l[t][c], l[i][t]);
            }
            if (!BAD_PIVOT_ZEROES && bad && info) *info = bad;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < n) {
                    rinv[c] = rv[c];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i < n) W[(size_t)c * ld + i] = i >= c ? l[i >= c ? i : c][c] : 0.0;
                }
        }
        __syncthreads();
        return;
    }
    for (int k0 = 0; k0 < n; k0 += 16) {
        const int below = n - k0 - 16;                   // rows under the diagonal block
        const bool mine = wave == 0 || 64 * wave < below;      // uniform
        const int l16 = lane & 15, i = k0 + 16 + 64 * wave + lane;
        double d[16], x[16], rv = 0.0;                   // row k0 + l16 of the diagonal block, row i below it
        if (mine) {
            // (unconditional loads, then selects: a branch per entry would cost more than the column's arithmetic.)
            const int id = min(k0 + l16, n - 1), ix = min(i, n - 1);
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const double* col = W + (size_t)min(k0 + c, n - 1) * ld;
                d[c] = col[id];
                x[c] = col[ix];
            }
            if (below < 0) {                             // entries past n act as an identity block
#pragma unroll
                for (int c = 0; c < 16; ++c) d[c] = k0 + l16 >= n || k0 + c >= n ? (l16 == c ? 1.0 : 0.0) : d[c];
            }
        }
        __syncthreads();                                 // every wave holds the unfactored block
        if (mine) {
            int bad = 0;
            double r = 0.0;
            auto pivot = [&](auto C) {
                constexpr int c = decltype(C)::value;
                double piv = row_bcast<c>(d[c]);
                if (BAD_PIVOT_ZEROES) {
                    r = piv > floor_ ? chol_rsqrt(piv) : 0.0;
                } else {
                    const bool ok = piv > 0.0;
                    bad = !ok && k0 + c < n ? k0 + c + 1 : bad;
                    piv = ok ? piv : 1e-300;
                    r = chol_rsqrt(piv);
                }
            };
            pivot(std::integral_constant<int, 0>{});
            // (column c's first update feeds the next pivot's reciprocal square root, the others fill its latency; the fences
            // keep the compiler from postponing them into one long chain per column)
            for_each_block<16>([&](auto C) {
                constexpr int c = decltype(C)::value;
                __builtin_amdgcn_sched_barrier(0);
                rv = l16 == c ? r : rv;
                d[c] *= r;                               // the pivot's lane: sqrt(pivot), or 0 for a zeroed column
                x[c] *= r;
                for_each_block<15 - c>([&](auto T) {
                    constexpr int t = c + 1 + decltype(T)::value;
                    const double m = row_bcast<t>(d[c]);
                    d[t] = __builtin_fma(-d[c], m, d[t]);
                    if constexpr (t == c + 1) pivot(std::integral_constant<int, t>{});
                    x[t] = __builtin_fma(-x[c], m, x[t]);
                });
            });
            __builtin_amdgcn_sched_barrier(0);
            // (formed here, not in the branches below: sunk there, the rows would wait for the whole block with every multiplier
            // alive)
#pragma unroll
            for (int c = 0; c < 16; ++c) asm volatile("" : "+v"(x[c]), "+v"(d[c]));
            asm volatile("" : "+v"(rv));
            if (!BAD_PIVOT_ZEROES && bad && tid == 0 && info) *info = bad;
            if (i < n) {
#pragma unroll
                for (int c = 0; c < 16; ++c) W[(size_t)(k0 + c) * ld + i] = x[c];
            }
            if (tid < 16 && k0 + tid < n) {
#pragma unroll
                for (int c = 0; c < 16; ++c)             // above the diagonal: zeros
                    if (k0 + c < n) W[(size_t)(k0 + c) * ld + k0 + tid] = tid >= c ? d[c] : 0.0;
                rinv[k0 + tid] = rv;
            }
        }
        if (below <= 0) break;
        __syncthreads();
        // trailing update A22 -= L21 L21^T, lower 16 x 16 tiles, one per wave and round; rows: the tile's columns of A22
        const int t0 = k0 + 16, T = (below + 15) / 16, ntiles = T * (T + 1) / 2;
        for (int tile = wave; tile < ntiles; tile += nwaves) {
            int ti = 0, rem = tile;
            while (rem > ti) { rem -= ti + 1; ++ti; }       // tile -> (ti, tc), tc <= ti
            const int i0 = t0 + 16 * ti, c0 = t0 + 16 * rem, kq = lane >> 4;
            const int ib = min(i0 + (lane & 15), n - 1), ca = min(c0 + (lane & 15), n - 1);
            double av[4], bv[4];
            double4_t acc;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                const size_t col = (size_t)(k0 + 4 * kc + kq) * ld;
                av[kc] = -W[col + ca];
                bv[kc] = W[col + ib];
            }
            // D: lane l, element v -> (row 4 v + l / 16, column l % 16) of the tile; surplus ones are not stored
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] = W[(size_t)min(c0 + 4 * v + kq, n - 1) * ld + ib];
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[kc], bv[kc], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + (lane & 15), c = c0 + 4 * v + kq;
                if (i < n && c < n && i >= c) W[(size_t)c * ld + i] = acc[v];
            }
        }
        __syncthreads();
    }
    __syncthreads();                                     // the last panel is visible to the caller
}

// One 16x16 tile of sum_{kbeg <= k < kend} a(i, k) b(k, j) on the fp64 matrix cores (kbeg a multiple of 16); lane supplies
// row/column (lane & 15) and the k offset lane >> 4.  fa / fb read in-bounds elements; out-of-range rows, columns and k
// contribute zero.
template <class FA, class FB>
__device__ __forceinline__ double4_t tile_mma(int n, int ia, int jb, int kq, FA fa, FB fb, int kbeg, int kend) {
    const int ic = min(ia, n - 1), jc = min(jb, n - 1);
    const bool iok = ia < n, jok = jb < n;
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    if ((n & 15) == 0 && (kend & 15) == 0) {      // whole tiles: no guards, operands of four steps loaded ahead
        for (int k0 = kbeg; k0 < kend; k0 += 16) {
            double a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = fa(ia, k0 + 4 * u + kq);
                b[u] = fb(k0 + 4 * u + kq, jb);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
        }
        return acc;
    }
    for (int k0 = kbeg; k0 < kend; k0 += 16) {    // (a step at a time, its loads awaited, CHFIG)
        double a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + 4 * u + kq, kc = min(k, n - 1);
            const double x = fa(ic, kc), y = fb(kc, jc);
            a[u] = iok && k < kend ? x : 0.0;
            b[u] = jok && k < kend ? y : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    return acc;
}

// ---------------------------------------------------------------------------------------
// Cholesky G = L L^T and Linv = L^-1 (lower triangular), n <= SM_MAX_CHOL; optionally a second matrix F <- Linv F Linv^T (transform).
// LDS: L [n][n+1] doubles, X [n][n+1] doubles.
// ---------------------------------------------------------------------------------------
#define CI_THREADS 512               // 256 registers per lane: the panels take 140
// dinv: SM_MAX_CHOL doubles of LDS.  The workgroup's size is a multiple of 64, at least 512.
template <bool SMALL>
__device__ __forceinline__ void chol_inverse(const double* G, double* Linv, int32_t* info, int32_t* wellcond_out, double* transform, int n,
                                             double* __restrict__ sm, double* __restrict__ dinv) {
    const int ld = n + 1;
    double* L = sm;                              // column-major: L(i, c) at L[c*ld + i]
    double* X = sm + (size_t)n * ld;             // L^-1, row-major: X(t, c) at X[t*ld + c]
    const int tid = threadIdx.x, nthr = blockDim.x;
    for (int p = tid >> 4; p < n; p += nthr >> 4)             // G is symmetric: its row p is column p of L
        for (int i = tid & 15; i < n; i += 16) {
            L[p * ld + i] = G[(size_t)p * n + i];
            X[p * ld + i] = 0.0;
        }
    __syncthreads();
    chol_blocked<false, SMALL>(L, ld, n, dinv, 0.0, info);
    if (wellcond_out && tid < 64) {
        double lo = dinv[tid < n ? tid : 0], hi = lo;
        if (tid + 64 < n) { lo = fmin(lo, dinv[tid + 64]); hi = fmax(hi, dinv[tid + 64]); }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) { lo = fmin(lo, __shfl_xor(lo, o)); hi = fmax(hi, __shfl_xor(hi, o)); }
        if (tid == 0) *wellcond_out = (hi <= 1e3 * lo) ? 1 : 0;        // a replaced pivot has dinv = 1e150 and fails this
    }
    // L^-1 by 16 x 16 blocks.  The diagonal blocks are inverted by substitution (one thread per column, 16 steps in
    // registers); then, one block sub-diagonal after the other, X_ij = -X_ii (sum_k L_ik X_kj) on the fp64 matrix
    // cores, one wave per block.  The inner sum leaves the matrix instruction in exactly the register layout that
    // the second product wants for its right operand (accumulator element v = contraction chunk v), so it never
    // touches memory.  Rows and columns past n act as an identity.
    {
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
        const int T = (n + 15) / 16;
        const bool whole = (n & 15) == 0;             // no padding: the accessors need no tests
        auto Lat = [&](int i, int c2) { return (whole || (i < n && c2 < n)) ? L[min(c2, n - 1) * ld + min(i, n - 1)] : (i == c2 ? 1.0 : 0.0); };
        auto Xat = [&](int t, int c2) { return (whole || (t < n && c2 < n)) ? X[min(t, n - 1) * ld + min(c2, n - 1)] : (t == c2 ? 1.0 : 0.0); };
        if (tid < 16 * T) {
            const int b0 = 16 * (tid >> 4), cc = tid & 15, c = b0 + cc;
            if (c < n) {
                double x[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int i = b0 + q;
                    double v = q == cc ? 1.0 : 0.0;
#pragma unroll
                    for (int u = 0; u < q; ++u) v -= Lat(i, b0 + u) * x[u];
                    x[q] = (q >= cc && i < n) ? v * dinv[i] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (b0 + q < n) X[(b0 + q) * ld + c] = x[q];
            }
        }
        __syncthreads();
        const int r16 = lane & 15, kq = lane >> 4;
        for (int d = 1; d < T; ++d) {
            for (int blk0 = 0; blk0 < T - d; blk0 += nwaves) {
                // block (ib, jb); surplus waves sit the round out (`wave` is a scalar: a uniform branch, and waves that
                // repeated a block would queue on the same matrix pipes)
                if (blk0 + wave >= T - d) continue;
                const int jb = blk0 + wave, ib = jb + d;
                double4_t P = {0.0, 0.0, 0.0, 0.0};
                double xa[4];                     // X_ii for the second product, loaded ahead
#pragma unroll
                for (int kc = 0; kc < 4; ++kc) xa[kc] = Xat(16 * ib + r16, 16 * ib + 4 * kc + kq);
                for (int k = jb; k < ib; ++k) {
                    double a[4], b[4];            // the operands of a whole block product before its four instructions
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc) {
                        a[kc] = Lat(16 * ib + r16, 16 * k + 4 * kc + kq);
                        b[kc] = Xat(16 * k + 4 * kc + kq, 16 * jb + r16);
                    }
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc) P = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kc], b[kc], P, 0, 0, 0);
                }
                double4_t R = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int kc = 0; kc < 4; ++kc) R = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[kc], P[kc], R, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ib + 4 * v + kq, c2 = 16 * jb + r16;
                    if (i < n && c2 < n) X[i * ld + c2] = -R[v];
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
    for (int i = tid >> 4; i < n; i += nthr >> 4)
        for (int j = tid & 15; j < n; j += 16) Linv[(size_t)i * n + j] = X[i * ld + j];
    // F <- X F X^T, by way of L's place: X F first, row-major.  X is lower triangular: neither sum goes past its diagonal; F is
    // symmetric, and only its tiles on and right of the diagonal are written.
    if (transform) {
        double* F = transform;
        constexpr int TW = (((SM_MAX_CHOL + 15) / 16) * ((SM_MAX_CHOL + 15) / 16) + 7) / 8;      // tiles a wave
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
        const int T = (n + 15) / 16, r16 = lane & 15, kq = lane >> 4;
        double4_t acc[TW];
        auto product = [&](bool second, auto fb) {
#pragma unroll
            for (int t = 0; t < TW; ++t) {
                const int tile = wave + t * nwaves;
                if (tile >= T * T) continue;     // (uniform)
                const int ti = tile / T, tj = tile - ti * T;
                if (second && tj < ti) continue;
                acc[t] = tile_mma(n, 16 * ti + r16, 16 * tj + r16, kq, [&](int i, int k) { return fb(i, k, true); },
                                  [&](int k, int j) { return fb(k, j, false); }, 0, min(16 * (second ? tj : ti) + 16, n));
            }
        };
        auto each = [&](bool second, auto put) {
#pragma unroll
            for (int t = 0; t < TW; ++t) {
                const int tile = wave + t * nwaves;
                if (tile >= T * T) continue;
                const int ti = tile / T, tj = tile - ti * T;
                if (second && tj < ti) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + 4 * v + kq, j = 16 * tj + r16;
                    if (i < n && j < n) put(i, j, acc[t][v]);
                }
            }
        };
        __syncthreads();
        for (int i = tid >> 4; i < n; i += nthr >> 4)
            for (int j = tid & 15; j < n; j += 16) L[i * ld + j] = F[(size_t)i * n + j];
        __syncthreads();
        product(false, [&](int i, int j, bool left) { return left ? X[i * ld + j] : L[i * ld + j]; });
        __syncthreads();
        each(false, [&](int i, int j, double v) { L[i * ld + j] = v; });
        __syncthreads();
        product(true, [&](int i, int j, bool left) { return left ? L[i * ld + j] : X[j * ld + i]; });
        each(true, [&](int i, int j, double v) { F[(size_t)i * n + j] = v; });
    }
}

template <bool SMALL>
__global__ void __launch_bounds__(CI_THREADS)
k_chol_inv(const CholBatch batch, int n) {
    extern __shared__ double sm[];
    __shared__ double dinv[SM_MAX_CHOL];
    const CholProblem& prob = batch.p[blockIdx.x];
    chol_inverse<SMALL>(prob.G, prob.Linv, prob.info, prob.wellcond_out, nullptr, n, sm, dinv);
}

// ---------------------------------------------------------------------------------------
// One-sided Jacobi on a symmetric positive semi-definite G (n <= SM_MAX_N), applied to its
// Cholesky factor: rotate the columns of W = L until they are mutually orthogonal; then
// column j is sqrt(lambda_j) v_j.  1024 threads = 64 groups of 16 lanes, one column pair per group and
// step, round-robin ordering; dot products by 16-lane DPP rotations.
// Outputs (eigenvalues descending):
//   lam  [n]            eigenvalues
//   vec  [n][n]         vec[i*n + j] = component i of eigenvector j          (optional)
//   tmat [n][kk]        tmat[i*kk + c] = vec[i][c] / sqrt(lam_c), c < kk     (optional)
//   sval [kk]           (float) sqrt(lam_c)                                  (optional)
// ---------------------------------------------------------------------------------------
// ---- 8-lane all-reduce of a double with DPP (no LDS traffic) ----
template <int CTRL>
__device__ __forceinline__ double dpp_mov64(double x) {
    int lo = __double2loint(x), hi = __double2hiint(x);
    lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true);
    hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double group8_sum(double x) {
    x += dpp_mov64<0xB1>(x);      // quad_perm [1,0,3,2]
    x += dpp_mov64<0x4E>(x);      // quad_perm [2,3,0,1]
    x += dpp_mov64<0x141>(x);     // row_half_mirror: lane i <-> 7-i within each 8 lanes
    return x;
}

// 1/sqrt(x), 1/x for x > 0: hardware seed + one Newton step.  The rotation only has to be
// orthogonal to ~1e-13 (c and s come from the same t, so c^2 + s^2 = 1 up to the error of one rsqrt).
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    return y * (1.5 - 0.5 * x * y * y);
}
__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
    return y * (2.0 - x * y);
}

template <int JGL> __device__ __forceinline__ double group_sum(double x);
template <> __device__ __forceinline__ double group_sum<4>(double x) {
    x += dpp_mov64<0xB1>(x);      // quad_perm [1,0,3,2]
    x += dpp_mov64<0x4E>(x);      // quad_perm [2,3,0,1]
    return x;
}
template <> __device__ __forceinline__ double group_sum<8>(double x) { return group8_sum(x); }
template <> __device__ __forceinline__ double group_sum<16>(double x) {
    x = group8_sum(x);
    x += dpp_mov64<0x140>(x);     // row_mirror: lane i <-> 15-i within each 16 lanes
    return x;
}

// lanes per column pair: a step is bound by the latency of its chain of dependent operations, so the
// widest group (shortest per-lane column pieces) wins even though it needs the most waves; behind the preconditioner the
// workgroup keeps to 512 threads
#define JGL_PLAIN 16
#define PRE_JGL 8
// Column stride in doubles: at least n rounded up to 16 (the rows from n up exist and stay zero, so the
// column loads and stores need no bounds checks), and = l (mod 2 l), which shifts neighbouring columns
// by one group's width in the banks.
__host__ __device__ static inline int jacobi_ld(int n, int l) {
    const int rows = (n + 15) / 16 * 16;
    return rows % (2 * l) == l ? rows : rows + l;
}

// ---------------------------------------------------------------------------------------
// Eigenvector preconditioner for the one-sided Jacobi below.
//
// The cyclic rotations need ~log n sweeps before their quadratic convergence sets in.  If the columns
// of the factor are first multiplied by an orthogonal P that is close to the eigenvector matrix of
// L^T L, the very first sweep already finds (nearly) orthogonal columns and the sweeps only confirm and
// refine: W0 = L P has W0 W0^T = L L^T = G for ANY orthogonal P, so the accuracy of P only affects the
// number of sweeps, never the result (a P orthogonal to 1e-10 perturbs G multiplicatively, i.e. every
// eigenvalue by 1e-10 relative).  P comes from the classical dense symmetric path, all inside this
// workgroup:
//   1  A = L^T L                                       (fp64 matrix cores)
//   2  Householder tridiagonalisation  Q^T A Q = T     (a column a lane, the rows dealt over four waves, one barrier a step)
//   3  eigenvalues of T by multisection on Sturm counts (5 to 10 probes per eigenvalue and round)
//   4  eigenvectors of T by twisted factorisation       (two lanes per eigenvector, one from either end)
//   5  back-transformation  P = Q Z                     (blocks of 16 reflectors on the fp64 matrix cores)
//   6  Newton-Schulz polish  P <- P (I - (P^T P - I) / 2)  until orthogonal to 1e-10; if the computed
//      vectors are far from orthogonal (coincident or tiny eigenvalues) the preconditioner is dropped
//   7  W0 = L P                                         (fp64 matrix cores)
// What bounds all but 5 to 7 is one wave's issue (a dependent fp64 operation every 8.8 cycles, an independent one every
// 6.5, with a row broadcast or without; a second wave on the SIMD issues in between for nothing).  Thousands of cycles (2.4
// GHz) at order 80, and what the phase took before it was written this way:
//   2  141 (184: 8 lanes a row on four waves, two barriers a step)       3  64 (79: 3 probes, coefficients from LDS)
//   4  21 (53: one thread an eigenvector)      5  31 (48: 8 lanes a column and one reflector at a time)
//   6  30 (35)      7 and the check 29 (35)      the whole eigenproblem 375 (498)
// R1 holds L on entry (column-major, odd stride lda = n | 1: rows and columns both walk all banks); the result is left in
// R2 in the sweeps' layout (stride ld, ne + 1 columns).  gscr: n * lda doubles of global scratch for L.  sa: pre_doubles(n) doubles
// of LDS, 16-byte aligned.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmax(x, __shfl_xor(x, o));
    return x;
}
// the sum over the wave, in every lane
__device__ __forceinline__ double wave_sum(double x) {
    x = group_sum<16>(x);
    return (readlane64(x, 0) + readlane64(x, 16)) + (readlane64(x, 32) + readlane64(x, 48));
}
__device__ __forceinline__ double rcp_nr2(double x) {          // 1/x to ~1e-15 relative
    double y = __builtin_amdgcn_rcp(x);
    y = y * (2.0 - x * y);
    return y * (2.0 - x * y);
}
// acc += (x of lane N of the row of 16 lanes) * m.  A lane's own write of x needs two wait states before another lane of the row
// reads it: the caller puts dpp_settle(x) between the two.
template <int N>
__device__ __forceinline__ void fmac_row(double& acc, double x, double m) {
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(x), "v"(m), "n"(N));
}
__device__ __forceinline__ void dpp_settle(double& x) { asm volatile("s_nop 1" : "+v"(x)); }

// eigenvalues to 2^-38 of ||T||, eigenvectors orthogonal to ~1e-5 before the polish, which one Newton-Schulz step brings to
// ~1e-10; small ones of a graded spectrum go on to at most 2^-64
#define PRE_BITS 38
#define PRE_MAX_BITS 64

// row length of the tridiagonalisation's published vectors: a place for every lane's column, and one more
__host__ __device__ static constexpr int pre_row(int n16) { return (n16 > 64 ? n16 : 64) + 1; }
// doubles of LDS for the vectors of the phases below (the largest of what they keep one after the other)
__host__ __device__ static inline size_t pre_doubles(int n) {
    const size_t n16 = (n + 15) / 16 * 16, tri = 16 * pre_row((int)n16) + 128 * ((n16 + 63) / 64) + 4 + 65;
    return 4 * n16 + (tri > 17 * n16 ? tri : 17 * n16) + 1;  // dd, ee, tau, lam | the tridiagonalisation's; twisted pairs; T of the block reflectors
}

template <int NE>
__device__ __forceinline__ bool eig_precondition(double* __restrict__ R1, double* __restrict__ R2, int ld, int lda, int n, int ne,
                                 double* __restrict__ gscr, double* __restrict__ sa) {
    constexpr int N16 = 16 * NE;                  // the order in whole tiles
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, r16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
    const int T16 = (n + 15) / 16, ntiles = T16 * T16;
    double* dd = sa;                              // [N16] diagonal of T; past n: 4, outside the scaled spectrum
    double* ee = dd + N16;                        // [N16] ee[j] couples j and j+1; past n - 2: 0
    double* tauv = ee + N16;                      // [N16] Householder tau; past n - 3: 0
    double* lamv = tauv + N16;                    // [N16] eigenvalues of T, ascending
    double* scr = lamv + N16;                     // of the phase at work
    __shared__ unsigned long long err_s;
    __shared__ int fail_s;

    // ---- 0: L to global scratch (R1 is reused for the eigenvectors) ----
    for (int e = tid; e < n * lda; e += nthr) gscr[e] = R1[e];
    if (tid == 0) { fail_s = 0; err_s = 0ull; }

    // lower tiles of the Gram matrix of the columns of R1, each to put(ti, tj, tile).  lower: the columns are zero above row
    // 16 floor(column / 16) (a triangular factor), so the sum starts there
    auto gram = [&](bool lower, auto put) {
        for (int tile = wave; tile < T16 * (T16 + 1) / 2; tile += nwaves) {    // `wave` is a scalar: a uniform loop
            int ti = 0, tj = tile;
            while (tj > ti) { tj -= ti + 1; ++ti; }
            const int ci = 16 * ti + r16, cj = 16 * tj + r16;
            put(ti, tj, tile_mma(n, ci, cj, kq, [&](int i, int k) { return R1[(size_t)i * lda + k]; },
                                 [&](int k, int c) { return R1[(size_t)c * lda + k]; }, lower ? 16 * ti : 0, n));
        }
    };
    // a symmetric matrix's lower tile to both halves of R2
    auto mirror = [&](int ti, int tj, double4_t acc) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ti + 4 * v + kq, j = 16 * tj + r16;
            if (i < n && j < n) {
                R2[(size_t)i * lda + j] = acc[v];
                R2[(size_t)j * lda + i] = acc[v];
            }
        }
    };

    // ---- 1: A = L^T L ----
    gram(true, mirror);
    for (int i = tid; i < N16; i += nthr) {
        tauv[i] = 0.0;
        if (i >= n) { dd[i] = 4.0; ee[i] = 0.0; }
    }
    __syncthreads();
    // ---- 2: tridiagonalisation.  Lane l holds column o + l (o = n - 64, or 0) and wave w of the first four its rows w, w + 4, ...; the
    //         first o columns sit in lanes of the other four waves, which retire with them.  Step j eliminates column j below its
    //         subdiagonal with u = (column j below row j+1, and g = alpha - beta at row j+1), A <- H A H, H = I - t u u^T.
    //         Row j (x) and row j+1 (ra) are known to every wave at work, so that vectors by columns are formed by each for
    //         itself, and one barrier a step is enough: a wave publishes its rows' share of A x and its candidate for row
    //         j+2 as it is before this step, wave 4 the reflector's scalars g and t, and the two rows the next step starts from follow from
    //             row' = row - u[row] (t p - t^2 (u^T p) u) - p[row] t u,   p = A u.
    //         The scalars' chain (a sum over the wave, a square root, a reciprocal) runs on wave 4 while the others form A x.  u and p
    //         reach the rows' products by row broadcasts from registers that hold 16 of a wave's rows.  Columns up to j go
    //         through the update as well (u is zero there, they keep their norm) and are not read again.  Lanes past the last
    //         column write to places of their own: no branch in a step.
    {
        const int o = n > 64 ? n - 64 : 0, wr = wave & 3;
        constexpr int NT = 4 * NE, NB = (NT + 15) / 16;        // rows a wave; registers of 16 rows
        constexpr int PS = pre_row(N16);
        const int c0 = o + lane, c1 = lane;
        const bool ok0 = c0 < n, ok1 = c1 < o;
        const bool second = wave >= 4;                         // uniform: holds the first o columns
        double* parts = scr;                                   // [2][4][PS] shares of A x by column
        double* row2s = parts + 8 * PS;                        // [2][4][PS]
        double* ub = row2s + 8 * PS;                           // [4][16 NB] u by row, the 16 rows of a register next to each other
        double* pb = ub + 64 * NB;                             // same for p
        double* scal = pb + 64 * NB;                           // [2][2] g, t
        double* dummy = scal + 4;                              // [64 + 1]
        auto slot = [](int r) { return (r & 3) * (16 * NB) + (r >> 2); };
        const int s0 = slot(c0), s1 = ok1 ? slot(c1) : (int)(dummy - ub) + 64;
        const int s1p = ok1 ? slot(c1) : (int)(dummy - pb) + 64;
        const int cown = second ? (ok1 ? c1 : PS - 1) : c0;    // (column PS - 1 is nobody's)
        double a[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
            a[t] = (second ? ok1 : ok0) && 4 * t + wr < n ? R2[(size_t)(4 * t + wr) * lda + cown] : 0.0;
        double x0 = ok0 ? R2[c0] : 0.0, x1 = ok1 ? R2[c1] : 0.0, ra0 = ok0 ? R2[lda + c0] : 0.0, ra1 = ok1 ? R2[lda + c1] : 0.0;
        double d0 = 0.0, d1 = 0.0;                             // the diagonal, of wave 4
        for (int e = tid; e < 128 * NB; e += nthr) ub[e] = 0.0;
        __syncthreads();                                       // the matrix is in registers: the reflectors take its place
        for (int r = tid >> 4; r < o; r += nthr >> 4)          // zeros above the reflectors of the later columns
            for (int c = o + r16; c < n; c += 16) R2[(size_t)r * lda + c] = 0.0;
        auto step = [&](int j, auto ES, auto SETS, auto ROLE) {
            constexpr int es = decltype(ES)::value;            // (j + 2) / 16: rows below 16 es are dead
            constexpr bool two = decltype(SETS)::value == 2;   // columns of the second set are alive
            constexpr int role = decltype(ROLE)::value;        // 0: rows of set 0; 1: rows of set 1; 2: the scalars; 3: both
            constexpr bool rows = role != 2, scalars = role >= 2;
            const int par = j & 1;
            auto at = [&](double v0, double v1, int c) {
                if constexpr (!two) return readlane64(v0, c - o);
                const double l1 = readlane64(v1, min(c, 63)), l0 = readlane64(v0, max(c - o, 0));
                return c >= o ? l0 : l1;
            };
            const double m0 = c0 > j + 1 ? x0 : 0.0, m1 = two && c1 > j + 1 ? x1 : 0.0;
            double u16[NB];
            if constexpr (rows) {
                double q[4] = {0.0, 0.0, 0.0, 0.0};
                ub[s0] = m0;
                if constexpr (two) ub[s1] = m1;
#pragma unroll
                for (int b = es / 4; b < NB; ++b) u16[b] = ub[wr * 16 * NB + 16 * b + r16];
                const int ts = ((j + 2) >> 2) & 3;
                const double lo = ts & 1 ? a[4 * es + 1] : a[4 * es], hi = ts & 1 ? a[4 * es + 3] : a[4 * es + 2];
                row2s[(par * 4 + wr) * PS + cown] = ts & 2 ? hi : lo;
#pragma unroll
                for (int b = es / 4; b < NB; ++b) dpp_settle(u16[b]);
                for_each_block<NT - 4 * es>([&](auto I) {
                    constexpr int t = 4 * es + decltype(I)::value;
                    fmac_row<t % 16>(q[t % 4], u16[t / 16], a[t]);
                });
                parts[(par * 4 + wr) * PS + cown] = (q[0] + q[1]) + (q[2] + q[3]);
            }
            double g, t;
            if constexpr (scalars) {
                // t = -1 / (beta g)
                const double sg = wave_sum(two ? __builtin_fma(m1, m1, m0 * m0) : m0 * m0);
                const double alpha = at(x0, x1, j + 1);
                const bool some = sg > 0.0, pos = alpha >= 0.0;
                const double h = some ? __builtin_fma(alpha, alpha, sg) : 1.0, ri = chol_rsqrt(h), nr = h * ri;
                const double beta = some ? (pos ? -nr : nr) : alpha, rb = pos ? -ri : ri;      // rb = 1 / beta
                const double gg = some ? alpha - beta : 1.0, sc = rcp_nr2(gg);
                g = some ? gg : 0.0;
                t = some ? -(rb * sc) : 0.0;
                scal[2 * par] = g;
                scal[2 * par + 1] = t;
                ee[j] = beta;
                tauv[j] = some ? -(gg * rb) : 0.0;
                // the reflector, zeros down to the diagonal
                const double scale = some ? sc : 0.0;
                (ok0 ? R2 + (size_t)c0 * lda + j : dummy + lane)[0] = (c0 == j + 1 ? g : m0) * scale;
                d0 = c0 == j ? x0 : d0;
                if constexpr (two) {
                    (ok1 ? R2 + (size_t)c1 * lda + j : dummy + lane)[0] = (c1 == j + 1 ? g : m1) * scale;
                    d1 = c1 == j ? x1 : d1;
                }
            }
            __syncthreads();
            {
                const double* pp = parts + par * 4 * PS;
                const double* r2 = row2s + (par * 4 + ((j + 2) & 3)) * PS;
                if constexpr (!scalars) { g = scal[2 * par]; t = scal[2 * par + 1]; }
                const double rb0 = r2[c0];
                const double p0 = __builtin_fma(g, ra0, (pp[c0] + pp[PS + c0]) + (pp[2 * PS + c0] + pp[3 * PS + c0]));
                double p1 = 0.0, rb1 = 0.0;
                if constexpr (two) {
                    rb1 = r2[c1];
                    p1 = __builtin_fma(g, ra1, (pp[c1] + pp[PS + c1]) + (pp[2 * PS + c1] + pp[3 * PS + c1]));
                    if (!ok1) { p1 = 0.0; rb1 = 0.0; }
                }
                double p16[NB];
                if constexpr (rows) {
                    pb[s0] = p0;
                    if constexpr (two) pb[s1p] = p1;
#pragma unroll
                    for (int b = es / 4; b < NB; ++b) p16[b] = pb[wr * 16 * NB + 16 * b + r16];
                }
                const double u0 = c0 == j + 1 ? g : m0, u1 = two && c1 == j + 1 ? g : m1;
                const double ks = wave_sum(two ? __builtin_fma(u1, p1, u0 * p0) : u0 * p0);
                const double pj1 = at(p0, p1, j + 1), pj2 = at(p0, p1, j + 2), uj2 = at(m0, m1, j + 2);
                const double tk = t * t * ks;
                const double al0 = __builtin_fma(-tk, u0, t * p0), be0 = t * u0;
                const double al1 = __builtin_fma(-tk, u1, t * p1), be1 = t * u1;
                x0 = __builtin_fma(-pj1, be0, __builtin_fma(-g, al0, ra0));
                ra0 = __builtin_fma(-pj2, be0, __builtin_fma(-uj2, al0, rb0));
                if constexpr (two) {
                    x1 = __builtin_fma(-pj1, be1, __builtin_fma(-g, al1, ra1));
                    ra1 = __builtin_fma(-pj2, be1, __builtin_fma(-uj2, al1, rb1));
                }
                if constexpr (rows) {
                    const double na = role == 0 ? -al0 : -al1, nb = role == 0 ? -be0 : -be1;
#pragma unroll
                    for (int b = es / 4; b < NB; ++b) dpp_settle(p16[b]);
                    for_each_block<NT - 4 * es>([&](auto I) {
                        constexpr int t = 4 * es + decltype(I)::value;
                        fmac_row<t % 16>(a[t], u16[t / 16], na);
                        fmac_row<t % 16>(a[t], p16[t / 16], nb);
                    });
                }
            }
        };
        auto reduce = [&](auto ROLE1, auto ROLE2) {            // a wave's role while the second set is alive, and after
            for_each_block<NE>([&](auto ES) {
                constexpr int es = decltype(ES)::value;
                const int jlo = es == 0 ? 0 : 16 * es - 2, jhi = min(16 * es + 13, n - 3);
                int j = jlo;
                if constexpr (NE > 4 && 16 * es - 2 < N16 - 64)
                    for (; j <= min(jhi, o - 1); ++j) step(j, ES, std::integral_constant<int, 2>{}, ROLE1);
                for (; j <= jhi; ++j) {
                    if constexpr (decltype(ROLE2)::value < 0) __syncthreads();
                    else step(j, ES, std::integral_constant<int, 1>{}, ROLE2);
                }
            });
        };
        if (wave < 4) reduce(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        else if (wave == 4) reduce(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{});
        else reduce(std::integral_constant<int, 1>{}, std::integral_constant<int, -1>{});
        // what is left: rows n - 2 (x) and n - 1, in set 0
        if (wave == 4) {
            if (c0 == n - 1) { ee[n - 2] = x0; ee[n - 1] = 0.0; }
            d0 = c0 == n - 2 ? x0 : (c0 == n - 1 ? ra0 : d0);
            if (ok0) dd[c0] = d0;
            if (ok1) dd[c1] = d1;
        }
        __syncthreads();
    }
    // ---- 3: eigenvalues of T.  Scale T by a power of two so that |d| + 2|e| <= 1, then multisection ----
    double* tw = scr;                             // [2][N16][2] the twisted factorisation's (d, coupling to the next row), from either end
    {
        if (wave == 0) {
            double g = 0.0;
            for (int i = lane; i < n; i += 64)
                g = fmax(g, fabs(dd[i]) + fabs(ee[i]) + (i ? fabs(ee[i - 1]) : 0.0));
            g = wave_max(g);
            const double s = g > 0.0 ? ldexp(1.0, -ilogb(g) - 1) : 1.0;
            for (int i = lane; i < n; i += 64) { dd[i] *= s; ee[i] *= s; }
        }
        __syncthreads();
        for (int i = tid; i < N16; i += nthr) {
            tw[2 * i] = dd[i];
            tw[2 * i + 1] = ee[i];
            tw[2 * N16 + 2 * i] = dd[N16 - 1 - i];
            tw[2 * N16 + 2 * i + 1] = i < N16 - 1 ? ee[N16 - 2 - i] : 0.0;
        }
        // The eigenvalues are dealt over all waves and the lanes over a wave's eigenvalues: n = 80: 10 and 6, sections of 1/7; n = 64: 8
        // and 8, sections of 1/9.  The coefficients are row broadcasts.
        const int epw = (n + nwaves - 1) / nwaves, G = min(64 / epw, 16);
        const int idx = lane / G, q = lane - G * idx, i = epw * wave + idx;
        const bool mine = idx < epw && i < n;
        double dreg[NE], nereg[NE];
#pragma unroll
        for (int b = 0; b < NE; ++b) {
            const int k = 16 * b + r16;
            const double e = k ? ee[k - 1] : 0.0;
            dreg[b] = dd[k];
            nereg[b] = -(e * e);
        }
        if (epw * wave < n) {                                   // uniform
            const double rs = 1.0 / (double)(G + 1);
            const float bits = __log2f((float)(G + 1));
            const int rounds = (int)ceilf(PRE_BITS / bits), max_rounds = (int)ceilf(PRE_MAX_BITS / bits);
            double lo = -1.0 - 1e-9, hi = 1.0 + 1e-9;       // Gershgorin after scaling
            for (int round = 0; round < max_rounds; ++round) {
                // enough once the interval is below 2^-38 of the spectrum's scale and 1e-9 of the eigenvalue itself
                // (small eigenvalues of a graded matrix keep going); the lanes of a wave leave together
                const bool done = !mine || (round >= rounds && (hi - lo) <= 1e-9 * fmax(fabs(lo), fabs(hi)));
                if (__ballot(!done) == 0ull) break;
                const double w = (hi - lo) * rs;
                const double nmu = -(lo + w * (double)(q + 1));
                // Sturm count: sign changes in the sequence of leading principal minors of T - mu,
                // p_k = (d_k - mu) p_{k-1} - e_{k-1}^2 p_{k-2}; the pair is renormalised, and the signs of the last
                // 8 steps, one bit each, are counted every 8 steps (rows past n change no sign)
                double p2 = 0.0, p1 = 1.0;
                uint32_t signs = 0;
                int cnt = 0;
#pragma unroll
                for (int b = 0; b < NE; ++b) { dpp_settle(dreg[b]); dpp_settle(nereg[b]); }
                for_each_block<N16>([&](auto K) {
                    constexpr int k = decltype(K)::value;
                    double p = nmu * p1;
                    fmac_row<k % 16>(p, dreg[k / 16], p1);
                    fmac_row<k % 16>(p, nereg[k / 16], p2);
                    signs = __builtin_amdgcn_alignbit(signs, (uint32_t)__double2hiint(p), 31);     // signs << 1 | sign(p)
                    p2 = p1; p1 = p;
                    if constexpr (k % 8 == 7) {
                        cnt += __popc((signs ^ (signs >> 1)) & 0xFFu);
                        const int ex = max((__double2hiint(p1) >> 20) & 0x7ff, (__double2hiint(p2) >> 20) & 0x7ff);
                        p1 = ldexp(p1, 1023 - ex);
                        p2 = ldexp(p2, 1023 - ex);
                    }
                });
                // probes at or below lambda_i have cnt <= i; they form a prefix of the group's lanes
                const unsigned long long b = __ballot(cnt <= i);
                const int k0 = __popc((unsigned)(b >> (G * idx)) & ((1u << G) - 1u));
                const double nlo = k0 > 0 ? lo + w * (double)k0 : lo;
                const double nhi = k0 < G ? lo + w * (double)(k0 + 1) : hi;
                lo = nlo; hi = nhi;
            }
            if (q == 0 && mine) lamv[i] = 0.5 * (lo + hi);
        }
        __syncthreads();
        // eigenvalues closer than the accuracy of the vectors that follow (repeated eigenvalues, rank deficiency):
        // those vectors would not come out orthogonal, so the remaining phases are skipped
        if (tid + 1 < n) {
            const double a = lamv[tid], b = lamv[tid + 1], m = fmax(fabs(a), fabs(b));
            if (b - a < 1e-9 * m || m < 1e-14) atomicOr(&fail_s, 1);    // relative: a graded spectrum is fine
        }
        __syncthreads();
    }
    // ---- 4: eigenvectors of T by twisted factorisation into R1 (column-major, lda).  Even lanes factor T - lambda from the top, odd
    //         lanes from the bottom, in the same instructions (t counts rows from the lane's end); what is kept of a row is
    //         m = coupling to the next row / pivot, both the next pivot's correction and the factor of the vector's recurrence.
    //         The twist is where |gamma_k| = |D+_k + D-_k - (d_k - lambda)| is smallest; each lane looks at its own half ----
    const bool early_fail = fail_s != 0;          // uniform: read after a barrier
    constexpr int TW_WAVES = 4;                   // one a SIMD
    if (wave < TW_WAVES && !early_fail) {
        const int i = wave + TW_WAVES * (lane >> 1), side = lane & 1;
        const bool mine = i < n;
        const double lam = lamv[mine ? i : 0], pm = 1e-100;
        const double* co = tw + side * 2 * N16;
        double m[N16];
        {
            double prev = 0.0, ein = 0.0;
#pragma unroll
            for (int t = 0; t < N16; ++t) {
                const double e = co[2 * t + 1];
                double D = __builtin_fma(-ein, prev, co[2 * t] - lam);
                D = fabs(D) < pm ? -pm : D;
                prev = e * rcp_nr(D);
                m[t] = prev;
                ein = e;
                if (t % 8 == 7) __builtin_amdgcn_sched_barrier(0);      // (m takes 2 N16 registers: no load far ahead of its use)
            }
        }
        asm volatile("" ::: "memory");            // (nor the pairs kept from above)
        double best = 1e300;
        int rr = 0;                               // in rows from this lane's end
#pragma unroll
        for (int t = 0; t < N16 / 2; ++t) {
            double gam = co[2 * t] - lam;
            if (t > 0) gam = __builtin_fma(-co[2 * t - 1], m[t > 0 ? t - 1 : 0], gam);
            gam = fabs(__builtin_fma(-co[2 * t + 1], dpp_mov64<0xB1>(m[N16 - 2 - t]), gam));
            const bool less = gam < best;
            best = less ? gam : best;
            rr = less ? t : rr;
            if (t % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
        {
            const double ob = dpp_mov64<0xB1>(best);
            const int orr = __builtin_amdgcn_mov_dpp(rr, 0xB1, 0xF, 0xF, true);
            const bool other = ob < best || (ob == best && side == 1);
            rr = other ? N16 - 1 - orr : rr;
        }
        // z at the twist is 1; from there towards this lane's end z_t = -m_t z_{t+1}
        double zz = 1.0, n0 = 0.0, n1 = 0.0;
#pragma unroll
        for (int t = N16 - 2; t >= 0; --t) {
            zz *= t < rr ? -m[t] : 1.0;
            m[t] = zz;
            if (t & 1) n1 = __builtin_fma(zz, zz, n1); else n0 = __builtin_fma(zz, zz, n0);
        }
        double nrm2 = (n0 + n1) - (double)(N16 - 1 - rr);      // without the ones past the twist
        nrm2 = 1.0 + (nrm2 + dpp_mov64<0xB1>(nrm2));
        if (mine && !(nrm2 < 1e300)) atomicOr(&fail_s, 1);
        const double rn = rsqrt_nr(nrm2);
        // rows from n up sit at the start of the odd lanes' count
        double* z = R1 + (size_t)(mine ? i : 0) * lda + (side ? N16 - 1 : 0);
        const int dir = side ? -1 : 1, t0 = side ? N16 - n : 0;
        const unsigned rows = mine && rr > t0 ? rr - t0 : 0;
#pragma unroll
        for (int t = 0; t < N16 - 1; ++t)
            if ((unsigned)(t - t0) < rows) z[dir * t] = m[t] * rn;
        if (mine && side == 0 && rr < n) z[rr] = rn;
    }
    // ---- 5: P = H_0 H_1 ... H_{n-3} Z.  16 reflectors at a time are I - V T V^T with T upper triangular: T_jj = tau_j and
    //         T_rj = -tau_j sum_{r <= u < j} T_ru v_u^T v_j.  A wave takes 16 columns of Z through all of them in registers: the
    //         accumulators of one product are the right operand of the next (element v of a tile is its contraction chunk v) ----
    {
        double* Tb = scr;                         // [T16][16][17]; the products v_u^T v_j first
        __syncthreads();                          // (the twisted pairs have been read)
        for (int b = wave; b < T16; b += nwaves) {
            const double4_t S = tile_mma(n, 16 * b + r16, 16 * b + r16, kq, [&](int i, int k) { return R2[(size_t)k * lda + i]; },
                                         [&](int k, int c) { return R2[(size_t)k * lda + c]; }, 16 * b, n);
#pragma unroll
            for (int v = 0; v < 4; ++v) Tb[(b * 16 + 4 * v + kq) * 17 + r16] = S[v];
        }
        __syncthreads();
        if (tid < 16 * T16) {
            const int b = tid >> 4, r = tid & 15;
            const double* S = Tb + b * 16 * 17;
            double x[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double tj = tauv[16 * b + j];
                double v = 0.0;
#pragma unroll
                for (int u = 0; u < j; ++u) v = __builtin_fma(x[u], S[u * 17 + j], v);      // (x[u] = 0 for u < r)
                x[j] = j == r ? tj : (j > r ? -tj * v : 0.0);
            }
            // (the block's 16 threads are of one wave: all have read the products before any stores)
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 16; ++j) Tb[(b * 16 + r) * 17 + j] = x[j];
        }
        __syncthreads();
        for (int tc = wave; tc < T16 && !early_fail; tc += nwaves) {
            const int c = min(16 * tc + r16, n - 1);
            double* zc = R1 + (size_t)c * lda;
            double4_t Z[NE];
#pragma unroll
            for (int ti = 0; ti < NE; ++ti)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + 4 * v + kq;
                    Z[ti][v] = i < n ? zc[i] : 0.0;
                }
            for_each_block<NE>([&](auto B) {
                constexpr int b = NE - 1 - decltype(B)::value;
                // columns past n - 3 hold no reflector and their tau is zero, but what they hold has to be finite: it is the matrix
                const int j = min(16 * b + r16, n - 1);
                double4_t Y = {0.0, 0.0, 0.0, 0.0}, Y2 = {0.0, 0.0, 0.0, 0.0};
                asm volatile("" ::: "memory");    // (a block's operands are fetched with the block: all of them do not fit)
                __builtin_amdgcn_sched_barrier(0);
                for_each_block<NE - b>([&](auto I) {
                    constexpr int ti = b + decltype(I)::value;
                    double va[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) va[v] = R2[(size_t)min(16 * ti + 4 * v + kq, n - 1) * lda + j];   // (Z is zero past n)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Y = __builtin_amdgcn_mfma_f64_16x16x4f64(va[v], Z[ti][v], Y, 0, 0, 0);
                });
                double ta[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) ta[v] = -Tb[(b * 16 + r16) * 17 + 4 * v + kq];
#pragma unroll
                for (int v = 0; v < 4; ++v) Y2 = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[v], Y[v], Y2, 0, 0, 0);
                for_each_block<NE - b>([&](auto I) {
                    constexpr int ti = b + decltype(I)::value;
                    const int i = min(16 * ti + r16, n - 1);
                    double va[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) va[v] = R2[(size_t)i * lda + min(16 * b + 4 * v + kq, n - 1)];
#pragma unroll
                    for (int v = 0; v < 4; ++v) Z[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[v], Y2[v], Z[ti], 0, 0, 0);
                    if (16 * ti + 16 > n) {       // rows past n took a copy of the last row's update: they stay zero
#pragma unroll
                        for (int v = 0; v < 4; ++v) Z[ti][v] = 16 * ti + 4 * v + kq < n ? Z[ti][v] : 0.0;
                    }
                });
            });
            if (16 * tc + r16 < n) {
#pragma unroll
                for (int ti = 0; ti < NE; ++ti)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * ti + 4 * v + kq;
                        if (i < n) zc[i] = Z[ti][v];
                    }
            }
        }
    }
    __syncthreads();
    // a product of n x n matrices, tile t of this wave into acc[t]: formed by every wave before any of them stores
    constexpr int TWAVE = (NE * NE + 7) / 8;
    double4_t acc[TWAVE];
    auto product = [&](auto fa, auto fb, bool lower) {      // lower: the left factor is lower triangular
#pragma unroll
        for (int t = 0; t < TWAVE; ++t) {
            const int tile = wave + t * nwaves;
            if (tile >= ntiles) continue;         // (uniform)
            const int ti = tile / T16, tj = tile - ti * T16;
            acc[t] = tile_mma(n, 16 * ti + r16, 16 * tj + r16, kq, fa, fb, 0, lower ? min(16 * ti + 16, n) : n);
        }
    };
    auto each = [&](auto put) {
#pragma unroll
        for (int t = 0; t < TWAVE; ++t) {
            const int tile = wave + t * nwaves;
            if (tile >= ntiles) continue;
            const int ti = tile / T16, tj = tile - ti * T16, j = 16 * tj + r16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * ti + 4 * v + kq;
                if (i < n && j < n) put(i, j, acc[t][v]);
            }
        }
    };
    // ---- 6: orthogonality check and Newton-Schulz polish ----
    bool ok = fail_s == 0;
    for (int it = 0; it < 4 && ok; ++it) {
        double m = 0.0;
        bool bad = false;
        gram(false, [&](int ti, int tj, double4_t E) {       // E = P^T P - I
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * ti + 4 * v + kq, j = 16 * tj + r16;
                if (i == j) E[v] -= 1.0;
                if (i < n && j < n) { m = fmax(m, fabs(E[v])); bad = bad || !(fabs(E[v]) < 0.03); }      // (a NaN is bad)
            }
            mirror(ti, tj, E);
        });
        m = __ballot(bad) ? 1.0 : wave_max(m);
        if (lane == 0) atomicMax(&err_s, (unsigned long long)__double_as_longlong(m));
        __syncthreads();
        const double err = __longlong_as_double((long long)err_s);
        if (!(err < 0.03)) { ok = false; break; }
        if (err < 1e-10) break;
        if (it == 3) { ok = false; break; }
        const bool last = err < 1e-4;             // one step squares the error (to < 1e-8): no need to look again
        // P <- P - P E / 2
        product([&](int i, int k) { return R1[(size_t)k * lda + i]; }, [&](int k, int c) { return R2[(size_t)k * lda + c]; }, false);
        __syncthreads();
        if (tid == 0) err_s = 0ull;
        each([&](int i, int j, double v) { R1[(size_t)j * lda + i] -= 0.5 * v; });
        __syncthreads();
        if (last) break;
    }
    // ---- 7: W0 = L P into R2 (or L itself when the preconditioner was dropped) ----
    if (ok)
        product([&](int i, int k) { return gscr[(size_t)k * lda + i]; },           // L[i][k], k <= i
                [&](int k, int c) { return R1[(size_t)c * lda + k]; }, true);      // P[k][c]
    __syncthreads();                              // P and E have been read: R1 takes a copy of W0 in its own stride for the check below
    for (int c = tid >> 4; c <= ne; c += nthr >> 4)
        for (int i = r16; i < ld; i += 16) {
            const bool in = c < n && i < n;
            if (!in || !ok) R2[(size_t)c * ld + i] = in ? gscr[(size_t)c * lda + i] : 0.0;
        }
    if (ok)
        each([&](int i, int j, double v) {
            R2[(size_t)j * ld + i] = v;
            R1[(size_t)j * lda + i] = v;
        });
    __syncthreads();
    return ok;
}

// One-sided Jacobi on the Cholesky factor of G.  JGL lanes share a pair of columns, NE = ceil(n / JGL)
// elements of each column per lane; the two columns of a group live in registers for a whole sweep.
//
// Ordering: odd-even transposition.  The active columns sit in slots 0 .. m-1; on even steps group g
// rotates slots (2g, 2g+1), on odd steps slots (2g+1, 2g+2), and after every rotation the two
// columns trade slots, so in m steps every pair of columns meets exactly once.  Between steps a
// group keeps one column and passes the other to a neighbour through an LDS mailbox (one column
// written and one read per group and step, one barrier per step).
//
// Deflation: a column that met every partner of a sweep without rotating is orthogonal (to tol)
// to all the others, and rotations among the others keep it so; it leaves the tournament, and
// the later sweeps run over the columns that still move.
// SMALL: n <= 4 (see chol_blocked).
// PRE: the preconditioner runs, for orders of PRE 16-row tiles.  REPAIR: the problems bring CholeskyQR's second pass (JacobiProblem::gram);
// instances of their own: inlined everywhere, its code left 36 bytes of scratch a lane also where it never runs (eigenproblems of order 32
// and 20, us on average: 50.4 without the code, 51.3 with it, 50.6 so; of 64 and more no difference).
template <int NE, int JGL, bool REPAIR, bool SMALL = false, int PRE = 0>
__global__ void __launch_bounds__(NE * JGL <= 64 || PRE ? 512 : 8 * NE * JGL)
k_jacobi_eig(const JacobiBatch batch, int n, int kk) {
    extern __shared__ double sm[];
    const JacobiProblem& prob = batch.p[blockIdx.x];
    const double* G = prob.G;                // (repaired in place, below)
    double* __restrict__ lam = prob.lam;
    double* __restrict__ vec = prob.vec;
    double* __restrict__ tmat = prob.tmat;
    float* __restrict__ sval = prob.sval;
    double* __restrict__ gscr = PRE ? prob.gscr : nullptr;
    const int ne = n + (n & 1);             // even number of columns (a zero column pads odd n)
    // Column stride = 8 (mod 16) doubles spreads the columns that one LDS instruction touches over the banks.
    const int ld = jacobi_ld(n, JGL);
    const size_t rsize = (size_t)(ne + 1) * ld;
    // gscr != nullptr: the eigenvector preconditioner runs and needs a second matrix-sized region
    double* W = sm;                              // column-major: W[p*ld + i] = element i of column p; column ne is a spare zero column
    double* mailn = sm + (gscr ? 2 : 1) * rsize; // [ne/2] squared norm of the column in transit to even slot 2j
    double* nrm = mailn + ne / 2;                // [ne + 1]
    int* order = (int*)(nrm + ne + 1);           // [ne]
    int* colmap = order + ne;                    // [ne + 1] slot -> column of the columns still rotating
    int* rotf = colmap + ne + 1;                 // [ne + 1] column took part in a rotation this sweep
    // [pre_doubles(n)] the preconditioner's vectors, past the int arrays, on an even double index (16-byte loads)
    double* pre_sa = sm + (((gscr ? 2 : 1) * rsize + ne / 2 + ne + 1 + (3 * ne + 4) / 2 + 2) & ~(size_t)1);
    __shared__ int nact_sh, wcnt[2];
    const int tid = threadIdx.x, nthr = blockDim.x, grp = tid / JGL, gl = tid % JGL;

    // the preconditioner works on an odd column stride (and on n columns alone), the sweeps on theirs; only the lower triangle
    // is loaded (G is symmetric: column p of it is the rest of row p), so that L comes out with zeros above its diagonal
    const int ldc = gscr ? n | 1 : ld;
    auto load = [&]() {
        for (int p = tid >> 4; p < (gscr ? n : ne + 1); p += nthr >> 4)
            for (int i = tid & 15; i < ldc; i += 16) W[(size_t)p * ldc + i] = (p < n && i < n && i >= p) ? G[(size_t)p * n + i] : 0.0;
    };
    load();
    // CholeskyQR's second pass, where the first one's factor was not well conditioned: its inverse X, and G <- X G X^T.  (In a
    // launch of its own before this one it cost 4.5 us with nothing to repair; here the flag arrives with G.)
    const bool repair = REPAIR && prob.gram && !(prob.wellcond && *prob.wellcond);
    __shared__ double rinv_sh[SM_MAX_N];
    if constexpr (REPAIR) {
        if (repair) {
            __syncthreads();
            chol_inverse<SMALL>(prob.gram, prob.post, prob.info, nullptr, prob.G, n, sm, rinv_sh);
            __syncthreads();
            load();
        }
    }
    if (tid <= ne) { colmap[tid] = tid; rotf[tid] = 0; nrm[tid] = 0.0; }
    if (tid == 0) { nact_sh = ne; wcnt[0] = 0; wcnt[1] = 0; }
    __syncthreads();
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Precondition: replace G by its Cholesky factor L (G = L L^T, column j of L in column j of W).
    // The columns of L are far closer to orthogonal than those of G (one Cholesky-LR step), the
    // rotations then converge in about half the sweeps, and column j ends as sigma_j u_j with
    // sigma_j^2 = lambda_j, u_j the eigenvector of G.  A pivot at rounding level (semi-definite G)
    // zeroes its column.
    {
        double m = 0.0;                           // every wave finds the largest diagonal entry for itself
        for (int j = lane; j < n; j += 64) m = fmax(m, W[(size_t)j * ldc + j]);
        chol_blocked<true, SMALL>(W, ldc, n, rinv_sh, wave_max(m) * 1e-30, nullptr);
    }
    const double tol2 = 1e-14, floor2 = 1e-28;
    double amax = 0.0;
    // keep the columns that have to rotate (rotf set), in slot order; returns their number
    auto compact = [&](int m) {
        int myc = -1, f = 0;
        __syncthreads();
        if (tid < m) { myc = colmap[tid]; f = rotf[myc]; }
        const unsigned long long bal = __ballot(f);
        if (lane == 0 && wave < 2) wcnt[wave] = __popcll(bal);
        __syncthreads();
        const int total = wcnt[0] + wcnt[1];
        if (f) {
            colmap[__popcll(bal & ((1ull << lane) - 1ull)) + (wave == 1 ? wcnt[0] : 0)] = myc;
            rotf[myc] = 0;
        }
        if (tid == 0) {
            if (total & 1) colmap[total] = ne;
            nact_sh = total + (total & 1);
        }
        __syncthreads();
        return total;
    };
    bool checked = false;
    if constexpr (PRE > 0) {
        W = sm + rsize;
        checked = eig_precondition<PRE>(sm, W, ld, ldc, n, ne, gscr, pre_sa);
    }
    if (checked) {
        // The preconditioned columns are (nearly) orthogonal: which of them still have to rotate is decided on their
        // Gram matrix, all pairs at once on the matrix cores, instead of in a sweep (n = 80: 32 us) that
        // would leave nearly all of them alone.
        const double* C = sm;
        for (int c = tid >> 3; c < n; c += nthr >> 3) {
            double s = 0.0;
            for (int i = tid & 7; i < n; i += 8) s += C[(size_t)c * ldc + i] * C[(size_t)c * ldc + i];
            s = group8_sum(s);
            if ((tid & 7) == 0) nrm[c] = s;
        }
        __syncthreads();
        for (int j = lane; j < n; j += 64) amax = fmax(amax, nrm[j]);
        amax = wave_max(amax);
        const int T16 = (n + 15) / 16;
        for (int tile = wave; tile < T16 * (T16 + 1) / 2; tile += nthr >> 6) {
            int ti = 0, tj = tile;
            while (tj > ti) { tj -= ti + 1; ++ti; }
            const int ci = 16 * ti + (lane & 15), cj = 16 * tj + (lane & 15), kq = lane >> 4;
            const double4_t acc = tile_mma(n, ci, cj, kq, [&](int i, int k) { return C[(size_t)i * ldc + k]; },
                                           [&](int k, int c) { return C[(size_t)c * ldc + k]; }, 0, n);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * ti + 4 * v + kq;
                if (i < n && cj < n && i != cj) {
                    const double a = nrm[i], b = nrm[cj];
                    if (acc[v] * acc[v] > tol2 * a * b + floor2 * amax * (a + b)) { rotf[i] = 1; rotf[cj] = 1; }
                }
            }
        }
        compact(ne);
    }

    // Rotate while gamma^2 > tol^2 alpha beta + (c eps)^2 amax (alpha + beta), tol = 1e-7: the
    // eigenvectors are then accurate to ~1e-7 / (relative gap), far inside the 1e-2 rad the split needs.  The second term is
    // the rounding floor of a dot product of two columns that each carry an absolute error of
    // ~eps * lambda_max (the columns are lambda_j v_j, formed from O(lambda_max) entries): below it
    // a rotation only reshuffles noise and the sweeps would never end.
    double X[NE], Y[NE];
    double nX = 0.0, nY = 0.0;

    // rows n .. JGL*NE-1 of every column are zero padding: no bounds checks
    auto load_col = [&](double* dst, const double* src) {
#pragma unroll
        for (int e = 0; e < NE; ++e) dst[e] = src[gl + JGL * e];
    };
    auto store_col = [&](double* dst, const double* src) {
#pragma unroll
        for (int e = 0; e < NE; ++e) dst[gl + JGL * e] = src[e];
    };
    // orthogonalise the pair in registers: X <- c X - s Y, Y <- s X + c Y.  The squared norms travel with
    // their columns; a set sign bit marks a column that has rotated in this sweep.
    auto rotate = [&]() {
        double g0 = 0.0, g1 = 0.0;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            if (e & 1) g1 += X[e] * Y[e]; else g0 += X[e] * Y[e];
        }
        const double gamma = group_sum<JGL>(g0 + g1);
        const double a = fabs(nX), b = fabs(nY);
        // (a zero column gives gamma = 0 and never passes the test)
        if (gamma * gamma > tol2 * a * b + floor2 * amax * (a + b)) {
            // With tau = beta - alpha and hyp = sqrt(tau^2 + 4 gamma^2) the rotation that zeroes the pair
            // (angle at most 45 degrees) has c^2 = (1 + |tau| / hyp) / 2 and s c = sign(tau) gamma / hyp.
            // The hardware reciprocal square roots are good to ~1e-7, which only steers the angle; the
            // pair (c, s) is then rescaled to unit length to second order (error ~1e-21).
            const double tau = b - a;
            const double hh = tau * tau + 4.0 * gamma * gamma;
            const double rh = __builtin_amdgcn_rsq(hh);
            const double c2 = 0.5 + 0.5 * fabs(tau) * rh;
            const double rc = __builtin_amdgcn_rsq(c2);
            double c = c2 * rc;
            double s = (tau < 0.0 ? -gamma : gamma) * rh * rc;
            const double d = c * c + (s * s - 1.0);
            const double f = 1.0 + d * (0.375 * d - 0.5);
            c *= f;
            s *= f;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const double x = X[e], y = Y[e];
                X[e] = c * x - s * y;
                Y[e] = s * x + c * y;
            }
            // squared norms after the rotation (their sum is preserved), flagged as rotated
            const double na = fabs(a + (s * s) * tau - 2.0 * (c * s) * gamma);
            nX = -na;
            nY = -fabs((a + b) - na);
        }
    };

    for (int sweep = 0; sweep < 40; ++sweep) {
        const int m = nact_sh, gs = m / 2;           // even number of slots, groups this sweep
        if (m == 0) break;
        const bool act = grp < gs, inner = grp < gs - 1;
        int idX = ne, idY = ne;
        if (act) {
            idX = colmap[2 * grp];
            idY = colmap[2 * grp + 1];
            load_col(X, W + (size_t)idX * ld);
            load_col(Y, W + (size_t)idY * ld);
            double sx = 0.0, sy = 0.0;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                sx += X[e] * X[e];
                sy += Y[e] * Y[e];
            }
            nX = group_sum<JGL>(sx);              // exact squared norms at the start of every sweep
            nY = group_sum<JGL>(sy);
        }
        double* const mail_lo = W + (size_t)idX * ld;                                  // mailbox of slot 2g
        double* const mail_hi = W + (size_t)(inner ? colmap[2 * grp + 2] : ne) * ld;   // mailbox of slot 2g + 2
        // a full sweep reverses the slot order: the columns this group ends up with
        const int endX = act ? colmap[m - 1 - 2 * grp] : ne, endY = act ? colmap[m - 2 - 2 * grp] : ne;
        __syncthreads();                          // every column is in registers before the first mailbox write
        if (sweep == 0 && !checked) {
            if (act && gl == 0) { nrm[idX] = nX; nrm[idY] = nY; }
            __syncthreads();
            for (int j = lane; j < ne; j += 64) amax = fmax(amax, nrm[j]);
            amax = wave_max(amax);
        }
        // The loop starts on a cache line of instructions (ten instructions' bytes behind the directive): where it lay by chance, what stands
        // before it in the kernel moved it by up to 2.5 % (96 columns 885 us at 0 bytes past a line, 910 at 24; 48: 278, 282 at 40).
        asm volatile(".p2align 6\n\t.rept 6\n\ts_nop 0\n\t.endr");
        for (int s2 = 0; s2 < gs; ++s2) {
            // even step: slots (2g, 2g+1) are (X, Y); afterwards Y moves down to group g-1
            if (act) {
                rotate();
                store_col(mail_lo, Y);
                mailn[grp] = nY;                  // all lanes of the group write the same value
            }
            __syncthreads();
            if (inner) {
                load_col(Y, mail_hi);
                nY = mailn[grp + 1];
            }
            // odd step: slots (2g+1, 2g+2) are (X, Y); afterwards X moves up to group g+1.  The last
            // group holds the unpaired top slot and only renames it.
            if (inner) {
                rotate();
                store_col(mail_hi, X);
                mailn[grp + 1] = nX;
            } else if (act) {
#pragma unroll
                for (int e = 0; e < NE; ++e) Y[e] = X[e];
                nY = nX;
            }
            __syncthreads();
            if (act) {
                load_col(X, mail_lo);
                nX = mailn[grp];
            }
        }
        __syncthreads();                          // the last mailbox reads are done
        if (act) {
            store_col(W + (size_t)endX * ld, X);
            store_col(W + (size_t)endY * ld, Y);
            if (gl == 0) {
                if (__double2hiint(nX) < 0) rotf[endX] = 1;
                if (__double2hiint(nY) < 0) rotf[endY] = 1;
            }
        }
        if (compact(m) == 0) break;               // keep the columns that rotated
    }
    // column norms = singular values of L = square roots of the eigenvalues
    for (int pp = grp; pp < ne; pp += nthr / JGL) {
        double s = 0.0;
        for (int i = gl; i < n; i += JGL) s += W[(size_t)pp * ld + i] * W[(size_t)pp * ld + i];
        s = group_sum<JGL>(s);
        if (gl == 0) nrm[pp] = (pp < n) ? sqrt(s) : -1.0;
    }
    __syncthreads();
    if (tid < ne) {                          // rank by counting: descending, ties by index
        double me = nrm[tid];
        int r = 0;
        for (int j = 0; j < ne; ++j) r += (nrm[j] > me) || (nrm[j] == me && j < tid);
        order[r] = tid;
    }
    __syncthreads();
    {
        // a thread's columns stay the same for all its rows
        constexpr int NJ = (NE * JGL + 15) / 16;
        int pp[NJ];
        double rl[NJ];
        bool zero[NJ];
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const int j = min((tid & 15) + 16 * q, n - 1);
            pp[q] = order[j];
            const double l = nrm[pp[q]];
            zero[q] = !(l > 0.0);
            rl[q] = zero[q] ? 0.0 : rcp_nr2(l);
        }
        for (int i = tid >> 4; i < n; i += nthr >> 4)
#pragma unroll
            for (int q = 0; q < NJ; ++q) {
                const int j = (tid & 15) + 16 * q;
                if (j >= n) continue;
                const double v = zero[q] ? (i == j ? 1.0 : 0.0) : W[(size_t)pp[q] * ld + i] * rl[q];
                if (vec) vec[(size_t)i * n + j] = v;
                if (tmat && j < kk && !repair) tmat[(size_t)i * kk + j] = v * rl[q];
            }
    }
    // G stood for X F X^T, X lower triangular: what multiplies F's basis is X^T tmat.  (On the matrix cores: as sums of a thread each over X in
    // global memory it was most of the repair.  The batch of a layer's 21 operands, gradients repaired, order 80: 307 -> 226 us.)
    if constexpr (REPAIR) {
        if (repair) {
            const double* X = prob.post;
            const int T16 = (n + 15) / 16, TK = (kk + 15) / 16, r16 = lane & 15, kq = lane >> 4;
            for (int tile = wave; tile < T16 * TK; tile += nthr >> 6) {        // (uniform)
                const int tj = tile / T16, ti = tile - tj * T16, j = 16 * tj + r16, p = order[min(j, n - 1)];
                const double* w = W + (size_t)p * ld;
                const double l = nrm[p], rl = l > 0.0 ? rcp_nr2(l) : 0.0;
                const double4_t acc = tile_mma(n, 16 * ti + r16, j, kq, [&](int i, int k) { return X[(size_t)k * n + i]; },
                                               [&](int k, int) { return w[k]; }, 16 * ti, n);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + 4 * v + kq;
                    if (i < n && j < kk) tmat[(size_t)i * kk + j] = l > 0.0 ? (acc[v] * rl) * rl : 0.0;
                }
            }
        }
    }
    if (tid < n) {
        double l = nrm[order[tid]];              // sigma_j = sqrt(lambda_j)
        lam[tid] = l * l;
        if (sval && tid < kk) sval[tid] = (float)l;
    }
}

int launch_chol_inv_batch(hipStream_t s, const CholProblem* probs, int count, int n) {
    if (n < 1 || n > SM_MAX_CHOL || count < 0) return METIS_UNSUPPORTED;
    size_t lds = 2 * (size_t)n * (n + 1) * sizeof(double);
    auto kern = n <= 4 ? k_chol_inv<true> : k_chol_inv<false>;
    static LdsLimitCache lds_set[2];
    if (!ensure_dyn_lds((const void*)kern, lds, lds_set[n <= 4])) return METIS_HIP_ERROR;
    for (int b0 = 0; b0 < count; b0 += SM_MAX_BATCH) {
        const int nb = count - b0 < SM_MAX_BATCH ? count - b0 : SM_MAX_BATCH;
        CholBatch batch;
        for (int i = 0; i < SM_MAX_BATCH; ++i) batch.p[i] = probs[b0 + (i < nb ? i : 0)];
        hipLaunchKernelGGL(kern, dim3(nb), dim3(CI_THREADS), lds, s, batch, n);
        METIS_LAUNCH_CHECK();
    }
    return METIS_OK;
}

// The orders from which on the preconditioner runs.  (It pays from 32 on: a lone decomposition with eigenproblems of order 36 and 28
// takes 287 us with it and 316 with plain sweeps, of 72 and 56 435 and 616.  A singular vector's sign is the one that the method leaves
// it with.  No sign is promised, and those of orders 72 to 84 may change with this method's code; but below 72, and for the second problem
// of every decomposition, which sets the signs of U and V, it has always been the plain sweeps', and callers keep their factors from one
// build to the next.)
#define PRE_MIN_N 72
int launch_jacobi_eig_batch(hipStream_t s, const JacobiProblem* probs, int count, int n, int kk) {
    if (n < 1 || n > 128 || count < 0) return METIS_UNSUPPORTED;
    const int ne = n + (n & 1);
    auto region = [&](int jgl) { return (size_t)(ne + 1) * jacobi_ld(n, jgl); };
    const size_t small = ((size_t)ne / 2 + ne + 1) * sizeof(double) + (size_t)(3 * ne + 4) * sizeof(int) + 16;
    // the preconditioner needs two matrix-sized regions and its vectors, which fit in the 160 KB of LDS (2 KB of them for static
    // arrays) up to n = 84.  It runs when every problem of the batch brings scratch.
    bool pre = count > 0 && n >= PRE_MIN_N;
    for (int i = 0; i < count; ++i) pre = pre && probs[i].gscr != nullptr;
    const size_t lds_pre = (2 * region(PRE_JGL) + pre_doubles(n) + 2) * sizeof(double) + small;
    pre = pre && lds_pre <= 158 * 1024;
    // one group of jgl lanes per column pair, in whole waves and at least 512 threads (the Cholesky pre-pass, the
    // bookkeeping and the preconditioner use them); no idle waves beyond that: every wave of the workgroup takes part in every
    // barrier.  After the preconditioner few columns still move, and 512 threads leave its phases 256 registers.
    const int jgl = pre ? PRE_JGL : JGL_PLAIN;
    size_t lds = pre ? lds_pre : region(jgl) * sizeof(double) + small;
    bool repair = false;
    for (int i = 0; i < count; ++i) repair = repair || probs[i].gram;
    if (repair && n > SM_MAX_CHOL) return METIS_UNSUPPORTED;
    if (repair) lds = std::max(lds, 2 * (size_t)n * (n + 1) * sizeof(double));
    const int need = (ne / 2 * jgl + 63) / 64 * 64;               // at most 128 ceil(n / 16): the kernel's launch bound
    const int threads = need > 512 ? need : 512;
    for (int b0 = 0; b0 < count; b0 += SM_MAX_BATCH) {
        const int nb = count - b0 < SM_MAX_BATCH ? count - b0 : SM_MAX_BATCH;
        JacobiBatch batch;
        for (int i = 0; i < SM_MAX_BATCH; ++i) batch.p[i] = probs[b0 + (i < nb ? i : 0)];
#define JACOBI_CASE(...)                                                                                          \
    {                                                                                                             \
        static LdsLimitCache lds_set;                                                                             \
        if (!ensure_dyn_lds((const void*)k_jacobi_eig<__VA_ARGS__>, lds, lds_set)) return METIS_HIP_ERROR;        \
        hipLaunchKernelGGL((k_jacobi_eig<__VA_ARGS__>), dim3(nb), dim3(threads), lds, s, batch, n, kk);           \
    }
#define JACOBI_REPAIR(T, ...) if (repair) JACOBI_CASE(T, JGL_PLAIN, true, __VA_ARGS__) else JACOBI_CASE(T, JGL_PLAIN, false, __VA_ARGS__)
#define JACOBI_PRE(T) if (pre) JACOBI_CASE(16 / PRE_JGL * T, PRE_JGL, true, false, T) else JACOBI_REPAIR(T, false)
        switch ((n + 15) / 16) {
            case 1: if (n <= 4) JACOBI_REPAIR(1, true) else JACOBI_REPAIR(1, false) break;
            case 2: JACOBI_REPAIR(2, false) break;
            case 3: JACOBI_REPAIR(3, false) break;
            case 4: JACOBI_REPAIR(4, false) break;
            case 5: JACOBI_PRE(5) break;
            case 6: JACOBI_PRE(6) break;
            case 7: JACOBI_CASE(7, JGL_PLAIN, false) break;
            default: JACOBI_CASE(8, JGL_PLAIN, false) break;
        }
#undef JACOBI_PRE
#undef JACOBI_REPAIR
#undef JACOBI_CASE
        METIS_LAUNCH_CHECK();
    }
    return METIS_OK;
}

size_t jacobi_scratch_doubles(int n) { return (size_t)n * (n | 1); }       // the Cholesky factor while its place is in use
