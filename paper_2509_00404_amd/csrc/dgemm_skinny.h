// The two contractions of the sample stage that read every sampled row of the bf16 input
// (Sec. 3.1): the sketch Z = A_s Omega and the projection B = H^T A_s.  One side of each
// product is skinny (r = k + p <= 128 columns), so a workgroup owns a full-width strip of the
// output, the bf16 input travels HBM -> registers -> LDS in 16-byte row pieces, and the fp64
// matrix cores (v_mfma_f64_16x16x4_f64) do the arithmetic: bf16 values are exact in fp64 and the
// accumulation is fp64 throughout.  The contraction is split over blockIdx.z; chunk z stores its partial
// strip at part z of the output (parts Ms r resp. r N elements apart), and k_sum_parts_batch adds the parts in
// a fixed order afterwards: no atomics, so the result does not depend on the order workgroups finish in.
//
// Bound by the fp64 matrix cores: a register loop of the instruction with the conversions beside it takes 84 cycles each (58
// TFLOP/s; without them 74; nominal 64), these loops 88.  What the rest was spent on, 4096 x 4096 at 80 columns, of 65 us (sketch)
// and 63: clearing LDS for columns that 80 = 5 x 16 does not have 2, SIMDs with four waves beside others with two, and one
// operand read at a time 8: 57 and 63 now; of fp32 weight gradients at rank 64 58 -> 48 and 63 -> 50.  The partial strips (21 MB
// here) and the launch are the other 10.
#pragma once
#include "dgemm.h"
#include <algorithm>

__device__ __forceinline__ double skinny_to_f64(bf16_t h) { return (double)__uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ double skinny_to_f64(float x) { return (double)x; }

// The order of 16 contraction elements' work: a matrix instruction (64 cycles), then two LDS reads of the next 16 and up to four vector
// instructions, so that neither a read's latency nor a conversion ever stands between two matrix instructions.
template <int NT>
__device__ __forceinline__ void skinny_interleave() {
#pragma unroll
    for (int m = 0; m < 4 * NT; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
}

// ---------------------------------------------------------------------------------------
// Sketch: Z[m][j] += sum_k A[rowmap[m]][k] * Om[k][j],  m < Ms, j < r, k in the split's chunk.
//   A   bf16 (or fp32: the weight gradient of the factor gradients), rows of whole 16-byte pieces, 16-byte aligned, K % 8 == 0
//   Om  bf16 [K][r] row-major, r % 8 == 0, base 16-byte aligned
//   Z   fp64 [ksplit][Ms][r] partial products
// one workgroup of 256 per 64 rows and chunk: wave w owns rows 16w..16w+15 and all NT column tiles.
// ---------------------------------------------------------------------------------------
// Waves per SIMD of both kernels.  At 3 and 4 column tiles two and no more: the contraction is cut so that two workgroups share a CU, and
// with room for a third wave some SIMDs get three and others one (48 columns, fp32 14336 x 4096: 250 us, 262 without the limit).  With
// 5 and more the registers see to that.  With 1 and 2 the pass is bound by memory and wants every wave it can get: 14336 x 4096 at
// 16 columns 121 us with the limit and the split of the wide ones, 102 without; 32 columns 185 and 170.
#define SKINNY_NARROW 2
template <int NT> struct SkinnyWaves { static constexpr int MIN = NT == 3 || NT == 4 ? 2 : 1, MAX = NT == 3 || NT == 4 ? 2 : 8; };
#define SK_ROWS 64
#define SK_KS 64                      // unit of the contraction split
template <int NT, typename TA>
struct SketchCfg {
    static constexpr int E = 16 / sizeof(TA);                        // elements per 16-byte piece
    static constexpr int KS = 8 * E;                                 // stage depth: 64 bf16 or 32 fp32, 8 pieces a row
    static constexpr int LDA = KS + E;                               // LDS row of the A stage (144 B: 16-byte aligned, bank-spread)
    // LDS row length of the Omega stage, = 16 (mod 32) so that the four k-rows a B fragment
    // touches fall into disjoint bank ranges
    static constexpr int LDO = NT * 16 + ((NT * 16) % 32 == 16 ? 0 : 16);
    static constexpr int OM_LOADS = (KS * NT * 2 + 255) / 256;    // 16-byte pieces per thread and stage
};

template <typename TA>
struct SketchCall {
    const TA* A;
    int64_t lda;
    const uint32_t* rowmap;
    int64_t Ms, K;
    const bf16_t* Om;
    int r;
    uint32_t wgs, tiles;              // workgroups; of one chunk
    int64_t kchunk;
    double* Z;
};

template <int NT, typename TA>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SkinnyWaves<NT>::MIN, SkinnyWaves<NT>::MAX)))
k_sketch(const CallBatch<SketchCall<TA>> batch) {
    uint32_t local;
    const SketchCall<TA> call = batch_call(batch, local);
    const TA* __restrict__ A = in_global(call.A);
    const uint32_t* __restrict__ rowmap = in_global(call.rowmap);
    const bf16_t* __restrict__ Om = in_global(call.Om);
    const int64_t lda = call.lda, Ms = call.Ms, K = call.K, kchunk = call.kchunk;
    const int r = call.r;
    const uint32_t chunk = local / call.tiles;
    typedef SketchCfg<NT, TA> Cfg;
    constexpr int LDO = Cfg::LDO, OML = Cfg::OM_LOADS, KS = Cfg::KS, LDA = Cfg::LDA;
    __shared__ __align__(16) TA As[2][SK_ROWS * LDA];
    __shared__ __align__(16) uint16_t Os[2][KS * LDO];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m0 = (int64_t)(local - chunk * call.tiles) * SK_ROWS;
    const int64_t kbeg = (int64_t)chunk * kchunk;
    const int64_t kend = kbeg + kchunk < K ? kbeg + kchunk : K;
    double* __restrict__ Z = in_global(call.Z) + (int64_t)chunk * Ms * r;
    if (kbeg >= kend) return;

    // the pad columns r .. 16 NT of the Omega stage, if there are any, stay zero
    if (r < 16 * NT) {
        for (int e = tid; e < KS * LDO / 4; e += 256) reinterpret_cast<uint4*>(&Os[0][0])[e] = make_uint4(0, 0, 0, 0);
        __syncthreads();
    }

    // A pieces: 64 rows x 8 pieces, two per thread
    const TA* arow[2];
    bool aok[2];
    int a_lds[2], a_k[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = tid + 256 * i, row = c >> 3, kc = c & 7;
        const int64_t m = m0 + row;
        aok[i] = m < Ms;
        const int64_t src = aok[i] ? (rowmap ? (int64_t)rowmap[m] : m) : 0;
        arow[i] = A + src * lda;
        a_lds[i] = row * LDA + Cfg::E * kc;
        a_k[i] = Cfg::E * kc;
    }
    // Omega pieces: KS k-rows x r/8 pieces
    const int rc = r >> 3;
    int o_k[OML], o_j[OML];
    bool ook[OML];
#pragma unroll
    for (int i = 0; i < OML; ++i) {
        const int c = tid + 256 * i;
        o_k[i] = c / rc;
        o_j[i] = 8 * (c - o_k[i] * rc);
        ook[i] = o_k[i] < KS;
    }

    uint4 ra[2], ro[OML];
    auto fetch = [&](int64_t kt) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t k = kt + a_k[i];
            ra[i] = (aok[i] && k < kend) ? *reinterpret_cast<const uint4*>(arow[i] + k) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < OML; ++i) {
            const int64_t k = kt + o_k[i];
            ro[i] = (ook[i] && k < kend) ? *reinterpret_cast<const uint4*>(Om + k * r + o_j[i]) : make_uint4(0, 0, 0, 0);
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(&As[buf][a_lds[i]]) = ra[i];
#pragma unroll
        for (int i = 0; i < OML; ++i)
            if (ook[i]) *reinterpret_cast<uint4*>(&Os[buf][o_k[i] * LDO + o_j[i]]) = ro[i];
    };

    double4_t acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = (double4_t){0.0, 0.0, 0.0, 0.0};

    fetch(kbeg);
    stash(0);
    __syncthreads();
    int buf = 0;
    const int arow_l = (wave * 16 + (lane & 15)) * LDA;
    for (int64_t kt = kbeg; kt < kend; kt += KS) {
        const bool more = kt + KS < kend;
        if (more) fetch(kt + KS);
        if constexpr (NT == 1) {           // bound by memory: read where they are used, fewer registers, more waves
#pragma unroll 4
            for (int s = 0; s < KS / 4; ++s) {
                const int kr = 4 * s + (lane >> 4);
                const double a = skinny_to_f64(As[buf][arow_l + kr]);
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, skinny_to_f64(Os[buf][kr * LDO + (lane & 15)]), acc[0], 0, 0, 0);
            }
        } else {
            // 16 elements at a time: the operands of the next 16 are read while these are multiplied (see skinny_interleave)
            constexpr int G = KS / 16;
            TA ar[2][4];
            bf16_t br[2][4][NT];
            auto read = [&](int g, int n) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int kr = 16 * g + 4 * s + (lane >> 4);
                    ar[n][s] = As[buf][arow_l + kr];
#pragma unroll
                    for (int j = 0; j < NT; ++j) br[n][s][j] = Os[buf][kr * LDO + 16 * j + (lane & 15)];
                }
            };
            read(0, 0);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                __builtin_amdgcn_sched_barrier(0);
                if (g + 1 < G) read(g + 1, (g + 1) & 1);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double a = skinny_to_f64(ar[g & 1][s]);
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, skinny_to_f64(br[g & 1][s][j]), acc[j], 0, 0, 0);
                }
                skinny_interleave<NT>();
            }
        }
        if (more) stash(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
    // D layout: lane l, element v -> row 4 v + l / 16, column l % 16
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t m = m0 + wave * 16 + 4 * v + (lane >> 4);
            const int col = 16 * j + (lane & 15);
            if (m < Ms && col < r) Z[m * r + col] = acc[j][v];
        }
}

// ---------------------------------------------------------------------------------------
// Projection: B[j][n] += sum_k H[k][j] * A[rowmap[k]][n],  j < r, n < N, k < Ms in the split's chunk.
//   H   fp64 [Ms][r] row-major, r even
//   A   bf16 as above, N % 8 == 0
//   B   fp64 [ksplit][r][N] partial products
// one workgroup of 256 per 64 columns and chunk: wave w owns columns 16w..16w+15 and all NT row tiles.
// Dynamic LDS: 2 H stages (fp64) + 2 A stages (bf16).
// ---------------------------------------------------------------------------------------
#define PJ_COLS 64
#define PJ_KS 32
#define PJ_LDA 80                     // elements per LDS row of the A stage: = 16 (mod 32)
template <int NT, typename TA>
struct ProjectCfg {
    static constexpr int LDH = NT * 16 + ((NT * 16) % 32 == 16 ? 0 : 16);    // doubles, = 16 (mod 32)
    static constexpr int H_LOADS = (PJ_KS * NT * 8 + 255) / 256;              // double2 pieces per thread and stage
    static constexpr size_t LDS = 2 * (size_t)PJ_KS * LDH * sizeof(double) + 2 * (size_t)PJ_KS * PJ_LDA * sizeof(TA);
};

template <typename TA>
struct ProjectCall {
    const double* H;
    int r;
    uint32_t wgs, tiles;              // workgroups; of one chunk
    const TA* A;
    int64_t lda;
    const uint32_t* rowmap;
    int64_t Ms, N, kchunk;
    double* B;
};

template <int NT, typename TA>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SkinnyWaves<NT>::MIN, SkinnyWaves<NT>::MAX)))
k_project(const CallBatch<ProjectCall<TA>> batch) {
    uint32_t local;
    const ProjectCall<TA> call = batch_call(batch, local);
    const double* __restrict__ H = in_global(call.H);
    const TA* __restrict__ A = in_global(call.A);
    const uint32_t* __restrict__ rowmap = in_global(call.rowmap);
    const int64_t lda = call.lda, Ms = call.Ms, N = call.N, kchunk = call.kchunk;
    const int r = call.r;
    const uint32_t chunk = local / call.tiles;
    constexpr int LDH = ProjectCfg<NT, TA>::LDH;
    constexpr int HL = ProjectCfg<NT, TA>::H_LOADS;
    extern __shared__ __align__(16) unsigned char pj_smem[];
    double* Hs = reinterpret_cast<double*>(pj_smem);                                   // [2][PJ_KS * LDH]
    TA* As = reinterpret_cast<TA*>(pj_smem + 2 * (size_t)PJ_KS * LDH * sizeof(double));   // [2][PJ_KS * PJ_LDA]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n0 = (int64_t)(local - chunk * call.tiles) * PJ_COLS;
    const int64_t kbeg = (int64_t)chunk * kchunk;
    const int64_t kend = kbeg + kchunk < Ms ? kbeg + kchunk : Ms;
    double* __restrict__ B = in_global(call.B) + (int64_t)chunk * r * N;
    if (kbeg >= kend) return;

    if (r < 16 * NT) {                                                 // pad columns r .. 16 NT stay zero
        for (int e = tid; e < PJ_KS * LDH; e += 256) reinterpret_cast<double2*>(Hs)[e] = make_double2(0.0, 0.0);
        __syncthreads();
    }

    // H pieces: 32 k-rows x r/2 pairs of doubles
    const int rc = r >> 1;
    int h_k[HL], h_j[HL];
    bool hok[HL];
#pragma unroll
    for (int i = 0; i < HL; ++i) {
        const int c = tid + 256 * i;
        h_k[i] = c / rc;
        h_j[i] = 2 * (c - h_k[i] * rc);
        hok[i] = h_k[i] < PJ_KS;
    }
    // A pieces: 32 k-rows x 64 columns, one (bf16) or two (fp32) per thread
    constexpr int E = 16 / sizeof(TA), AP = 8 / E;
    int a_kr[AP], a_n[AP];
    bool a_nok[AP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int c = tid + 256 * i;
        a_kr[i] = c / (PJ_COLS / E);
        a_n[i] = E * (c % (PJ_COLS / E));
        a_nok[i] = n0 + a_n[i] < N;
    }

    double2 rh[HL];
    uint4 ra[AP];
    auto fetch = [&](int64_t kt) {
#pragma unroll
        for (int i = 0; i < HL; ++i) {
            const int64_t k = kt + h_k[i];
            rh[i] = (hok[i] && k < kend) ? *reinterpret_cast<const double2*>(H + k * r + h_j[i]) : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int i = 0; i < AP; ++i) {
            const int64_t k = kt + a_kr[i];
            if (a_nok[i] && k < kend) {
                const int64_t src = rowmap ? (int64_t)rowmap[k] : k;
                ra[i] = *reinterpret_cast<const uint4*>(A + src * lda + n0 + a_n[i]);
            } else {
                ra[i] = make_uint4(0, 0, 0, 0);
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < HL; ++i)
            if (hok[i]) *reinterpret_cast<double2*>(&Hs[(size_t)buf * PJ_KS * LDH + h_k[i] * LDH + h_j[i]]) = rh[i];
#pragma unroll
        for (int i = 0; i < AP; ++i) *reinterpret_cast<uint4*>(&As[buf * PJ_KS * PJ_LDA + a_kr[i] * PJ_LDA + a_n[i]]) = ra[i];
    };

    double4_t acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = (double4_t){0.0, 0.0, 0.0, 0.0};

    fetch(kbeg);
    stash(0);
    __syncthreads();
    int buf = 0;
    for (int64_t kt = kbeg; kt < kend; kt += PJ_KS) {
        const bool more = kt + PJ_KS < kend;
        if (more) fetch(kt + PJ_KS);
        const double* hs = Hs + (size_t)buf * PJ_KS * LDH;
        const TA* as = As + buf * PJ_KS * PJ_LDA;
        if constexpr (NT == 1) {           // as in k_sketch
#pragma unroll 4
            for (int s = 0; s < PJ_KS / 4; ++s) {
                const int kr = 4 * s + (lane >> 4);
                const double b = skinny_to_f64(as[kr * PJ_LDA + wave * 16 + (lane & 15)]);
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(hs[kr * LDH + (lane & 15)], b, acc[0], 0, 0, 0);
            }
        } else {
            constexpr int G = PJ_KS / 16;
            constexpr bool AHEAD = NT <= 6;                    // (two sets of operands for more would not fit the registers)
            double ar[AHEAD ? 2 : 1][4][NT];
            TA br[AHEAD ? 2 : 1][4];
            auto read = [&](int g, int n) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int kr = 16 * g + 4 * s + (lane >> 4);
                    br[n][s] = as[kr * PJ_LDA + wave * 16 + (lane & 15)];
#pragma unroll
                    for (int i = 0; i < NT; ++i) ar[n][s][i] = hs[kr * LDH + 16 * i + (lane & 15)];
                }
            };
            if (AHEAD) read(0, 0);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int c = AHEAD ? g & 1 : 0;
                __builtin_amdgcn_sched_barrier(0);
                if (!AHEAD) read(g, 0);
                else if (g + 1 < G) read(g + 1, c ^ 1);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double b = skinny_to_f64(br[c][s]);
#pragma unroll
                    for (int i = 0; i < NT; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[c][s][i], b, acc[i], 0, 0, 0);
                }
                skinny_interleave<NT>();
            }
        }
        if (more) stash(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = 16 * i + 4 * v + (lane >> 4);
            const int64_t n = n0 + wave * 16 + (lane & 15);
            if (j < r && n < N) B[(int64_t)j * N + n] = acc[i][v];
        }
}

// Contraction split.  Up to 32 columns about 768 workgroups.  From 33 on the split with the least estimated time (us): two workgroups
// share a CU (256 of them a constant here: workspace sizes are asked for without a device); a round of them takes 0.067 per
// contraction element and 80 columns (0.045 where CUs have one only), 2 us besides, and every part costs its traffic, written and
// read once, at 4 TB/s.  Few tiles take many parts: sketch and projection of 64 rows x 14336 at 80 columns 28 us with up to 64
// parts, 23 with as many as the estimate asks for (112); 50256 x 256 115 and 105.
static inline int64_t skinny_kchunk(int64_t K, int64_t tiles, int stage, int64_t outputs, int r) {
    if (r <= 16 * SKINNY_NARROW) {
        int64_t ks = ceil_div64(768, tiles);
        const int64_t maxs = ceil_div64(K, stage);
        if (ks > maxs) ks = maxs;
        return ceil_div64(ceil_div64(K, ks), stage) * stage;
    }
    const double per_k = 0.067 / 80.0 * (double)((r + 15) / 16 * 16);
    double best_t = 1e30;
    int64_t best = stage;
    auto consider = [&](int64_t chunk) {
        const int64_t parts = ceil_div64(K, chunk), wgs = tiles * parts, rounds = ceil_div64(wgs, 512);
        const double t = (double)rounds * ((double)chunk * per_k * (wgs <= 256 ? 0.67 : 1.0) + 2.0) +
                         (parts > 1 ? (double)parts : 0.0) * (double)outputs * 16.0 / 4e6;
        if (t < best_t - 1e-9) {
            best_t = t;
            best = chunk;
        }
        return wgs;
    };
    // 1 to 64 parts, then every shorter chunk, up to two rounds of workgroups
    int64_t chunk = 0;
    for (int64_t n = 1; n <= 64 && chunk != stage; ++n) {
        chunk = ceil_div64(ceil_div64(K, n), stage) * stage;
        consider(chunk);
    }
    while (chunk > stage && consider(chunk -= stage) < 1024) {}
    return best;
}

// true when the fast kernels' layout preconditions hold
template <typename TA>
static inline bool skinny_ok(const TA* A, int64_t lda, int64_t N, int r) {
    return r % 8 == 0 && r >= 8 && r <= 128 && N % 8 == 0 && lda % (16 / (int64_t)sizeof(TA)) == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0;
}

// number of partial products the two kernels write
static inline int64_t sketch_kchunk(int64_t Ms, int64_t K, int r) { return skinny_kchunk(K, ceil_div64(Ms, SK_ROWS), SK_KS, Ms * r, r); }
static inline int64_t project_kchunk(int64_t Ms, int64_t N, int r) { return skinny_kchunk(Ms, ceil_div64(N, PJ_COLS), PJ_KS, N * r, r); }
static inline int sketch_parts(int64_t Ms, int64_t K, int r) { return (int)ceil_div64(K, sketch_kchunk(Ms, K, r)); }
static inline int project_parts(int64_t Ms, int64_t N, int r) { return (int)ceil_div64(Ms, project_kchunk(Ms, N, r)); }

// Z = sketch_parts(Ms, K, r) partial products [Ms][r]
template <typename TA>
static inline SketchCall<TA> sketch_call(const TA* A, int64_t lda, const uint32_t* rowmap, int64_t Ms, int64_t K, const bf16_t* Om, int r,
                                         double* Z) {
    const int64_t kchunk = sketch_kchunk(Ms, K, r);
    const uint32_t tiles = (uint32_t)ceil_div64(Ms, SK_ROWS);
    return {A, lda, rowmap, Ms, K, Om, r, tiles * (uint32_t)ceil_div64(K, kchunk), tiles, kchunk, Z};
}
// B = project_parts(Ms, N, r) partial products [r][N]
template <typename TA>
static inline ProjectCall<TA> project_call(const double* H, int r, const TA* A, int64_t lda, const uint32_t* rowmap, int64_t Ms, int64_t N,
                                           double* B) {
    const int64_t kchunk = project_kchunk(Ms, N, r);
    const uint32_t tiles = (uint32_t)ceil_div64(N, PJ_COLS);
    return {H, r, tiles * (uint32_t)ceil_div64(Ms, kchunk), tiles, A, lda, rowmap, Ms, N, kchunk, B};
}

// The calls whose width is NT column tiles, those with the longest workgroups first (the short ones fill the last round).
template <typename Call>
static inline std::vector<Call> skinny_of_width(const std::vector<Call>& calls, int nt) {
    std::vector<Call> g;
    for (const Call& c : calls)
        if ((c.r + 15) / 16 == nt) g.push_back(c);
    std::stable_sort(g.begin(), g.end(), [](const Call& a, const Call& b) { return a.kchunk > b.kchunk; });
    return g;
}

template <int NT, typename TA>
static inline int launch_sketch_width(hipStream_t s, const std::vector<SketchCall<TA>>& calls) {
    const std::vector<SketchCall<TA>> g = skinny_of_width(calls, NT);
    return launch_calls(g.data(), g.size(), [&](const CallBatch<SketchCall<TA>>& b, uint32_t wgs) {
        hipLaunchKernelGGL((k_sketch<NT, TA>), dim3(wgs), dim3(256), 0, s, b);
    });
}
template <int NT, typename TA>
static inline int launch_project_width(hipStream_t s, const std::vector<ProjectCall<TA>>& calls) {
    const std::vector<ProjectCall<TA>> g = skinny_of_width(calls, NT);
    if (g.empty()) return METIS_OK;
    const size_t lds = ProjectCfg<NT, TA>::LDS;
    static LdsLimitCache lds_set;
    if (!ensure_dyn_lds((const void*)k_project<NT, TA>, lds, lds_set)) return METIS_HIP_ERROR;
    return launch_calls(g.data(), g.size(), [&](const CallBatch<ProjectCall<TA>>& b, uint32_t wgs) {
        hipLaunchKernelGGL((k_project<NT, TA>), dim3(wgs), dim3(256), lds, s, b);
    });
}
#define SKINNY_WIDTHS(LAUNCH)                                                                                   \
    for (int nt = 1, st; nt <= 8; ++nt) {                                                                       \
        switch (nt) {                                                                                           \
            case 1: st = LAUNCH<1>(s, calls); break;                                                            \
            case 2: st = LAUNCH<2>(s, calls); break;                                                            \
            case 3: st = LAUNCH<3>(s, calls); break;                                                            \
            case 4: st = LAUNCH<4>(s, calls); break;                                                            \
            case 5: st = LAUNCH<5>(s, calls); break;                                                            \
            case 6: st = LAUNCH<6>(s, calls); break;                                                            \
            case 7: st = LAUNCH<7>(s, calls); break;                                                            \
            default: st = LAUNCH<8>(s, calls); break;                                                           \
        }                                                                                                       \
        if (st != METIS_OK) return st;                                                                          \
    }                                                                                                           \
    return METIS_OK;
// (r <= 128, skinny_ok)
template <typename TA>
static inline int launch_sketch(hipStream_t s, const std::vector<SketchCall<TA>>& calls) { SKINNY_WIDTHS(launch_sketch_width) }
template <typename TA>
static inline int launch_project(hipStream_t s, const std::vector<ProjectCall<TA>>& calls) { SKINNY_WIDTHS(launch_project_width) }

// ---------------------------------------------------------------------------------------
// Gram matrix of a tall skinny matrix given as a sum of partial arrays (the broadcast's per-split
// partial products):  S = sum_p C_p  (M x r, fp32),  G_b = S_b^T S_b  (r x r, fp64) for the rows S_b of workgroup b:
// G holds gram_blocks(M) partial Gram matrices, added in a fixed order afterwards (k_sum_parts_batch).
// The summed matrix is written back as fp32 (sum_out, may alias part 0) for the later U = S T.
//   r % 4 == 0, C 16-byte aligned.
// gram_blocks(M) workgroups of 256; wave w owns row tiles w, w+4 of G and all NT column tiles.
// ---------------------------------------------------------------------------------------
#define GR_KS 32                      // rows per stage
// Rows of C per workgroup: one stage while that leaves at most 256 partial matrices (bound by the latency of the parts'
// loads), two beyond, where the partial matrices' own traffic counts (k = 64: 32 KB each).  4096 rows: 11.5 -> 7.2 us against two.
static inline int gram_rows(int64_t M) { return M <= 256 * GR_KS ? GR_KS : 2 * GR_KS; }
static inline int64_t gram_blocks(int64_t M) { return ceil_div64(M, gram_rows(M)); }
struct GramCall {
    const float* C;
    int r, rows, nparts;
    uint32_t wgs;
    int64_t M, part_stride;
    float* sum_out;
    double* G;
};
template <int NT>
__global__ void __launch_bounds__(256)
k_gram_parts(const CallBatch<GramCall> batch) {
    uint32_t local;
    const GramCall call = batch_call(batch, local);
    const float* C = in_global(call.C);
    float* sum_out = in_global(call.sum_out);
    const int r = call.r, rows = call.rows, nparts = call.nparts;
    const int64_t M = call.M, part_stride = call.part_stride;
    constexpr int LDC = NT * 16 + ((NT * 16) % 32 == 16 ? 0 : 16);      // doubles, = 16 (mod 32)
    constexpr int PIECES = (GR_KS * NT * 4 + 255) / 256;                // float4 pieces per thread and stage
    constexpr int RT = (NT + 3) / 4;                                     // row tiles per wave
    __shared__ double Cs[GR_KS * LDC];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m0 = (int64_t)local * rows;
    double* __restrict__ G = in_global(call.G) + (int64_t)local * r * r;
    const int rc = r >> 2;
    for (int e = tid; e < GR_KS * LDC; e += 256) Cs[e] = 0.0;           // pad columns r .. 16 NT stay zero
    double4_t acc[RT][NT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (double4_t){0.0, 0.0, 0.0, 0.0};
    __syncthreads();
    for (int64_t mt = m0; mt < m0 + rows && mt < M; mt += GR_KS) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int c = tid + 256 * i, row = c / rc, col = 4 * (c - row * rc);
            if (row < GR_KS) {
                const int64_t m = mt + row;
                double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
                if (m < M) {
                    const float* src = C + m * r + col;
                    int p = 0;
                    for (; p + 8 <= nparts; p += 8) {          // eight loads in flight
                        float4 v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(src + (p + u) * part_stride);
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            s0 += (double)v[u].x;
                            s1 += (double)v[u].y;
                            s2 += (double)v[u].z;
                            s3 += (double)v[u].w;
                        }
                    }
                    for (; p < nparts; ++p) {
                        const float4 v = *reinterpret_cast<const float4*>(src + p * part_stride);
                        s0 += (double)v.x;
                        s1 += (double)v.y;
                        s2 += (double)v.z;
                        s3 += (double)v.w;
                    }
                    if (sum_out) {
                        // the Gram matrix is taken of the rounded sums, the same matrix the caller multiplies later
                        const float4 o = make_float4((float)s0, (float)s1, (float)s2, (float)s3);
                        *reinterpret_cast<float4*>(sum_out + m * r + col) = o;
                        s0 = o.x; s1 = o.y; s2 = o.z; s3 = o.w;
                    }
                }
                double* d = &Cs[row * LDC + col];
                d[0] = s0; d[1] = s1; d[2] = s2; d[3] = s3;
            }
        }
        __syncthreads();
#pragma unroll 2
        for (int s = 0; s < GR_KS / 4; ++s) {
            const int kr = 4 * s + (lane >> 4);
            double b[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = Cs[kr * LDC + 16 * j + (lane & 15)];
            // no branch around the matrix instructions: a wave whose row tile does not exist recomputes
            // tile 0 and drops the result in the epilogue
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int it = wave + 4 * i < NT ? wave + 4 * i : 0;
                const double a = Cs[kr * LDC + 16 * it + (lane & 15)];
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int it = wave + 4 * i;
        if (it >= NT) continue;
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int a = 16 * it + 4 * v + (lane >> 4), b = 16 * j + (lane & 15);
                if (a < r && b < r) G[a * r + b] = acc[i][j][v];
            }
    }
}

static inline GramCall gram_call(const float* C, int r, int64_t M, int nparts, int64_t part_stride, float* sum_out, double* G) {
    return {C, r, gram_rows(M), nparts, (uint32_t)gram_blocks(M), M, part_stride, sum_out, G};
}
template <int NT>
static inline int launch_gram_width(hipStream_t s, const std::vector<GramCall>& calls) {
    std::vector<GramCall> g;
    for (const GramCall& c : calls)
        if ((c.r + 15) / 16 == NT) g.push_back(c);
    return launch_calls(g.data(), g.size(), [&](const CallBatch<GramCall>& b, uint32_t wgs) {
        hipLaunchKernelGGL(k_gram_parts<NT>, dim3(wgs), dim3(256), 0, s, b);
    });
}
// (r <= 128)
static inline int launch_gram_parts(hipStream_t s, const std::vector<GramCall>& calls) { SKINNY_WIDTHS(launch_gram_width) }
