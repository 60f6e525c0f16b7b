// FP4 GEMMs on split operands (Sec. 3.2: Eq. 2 fprop, Eq. 3 dgrad, dL/dW_R wgrad).
//
// One NT kernel serves all three: C[M,N] = alpha * deq(A)[M,K] deq(B)[N,K]^T + Aext Bext^T.
// NVFP4 (block 16, E4M3 scale) is not an MX format, so the scaled-MFMA path cannot apply
// the block scales; codes are expanded in registers to fp16 (grid * e4m3 has at most 6
// significant bits: exact) and multiplied on the fp16 matrix cores with fp32 accumulation.
// The low-rank terms of the split enter as extra contraction columns (bf16, same
// accumulators):  Abar Bbar^T = Ra Rb^T + [(Ra Vb + Ua Sa Va^T Vb) Sb] Ub^T + (Ua Sa)(Rb Va)^T.
#include <algorithm>
#include <stdlib.h>
#include "common.h"
#include "gemm_tile.h"
#include "stream_dev.h"

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

namespace {

#define G_KI 128                    // contraction elements per LDS stage
#define G_CROW (G_KI / 2 + 4)       // padded code row in LDS (bytes): dword stride 17, conflict-free
#define G_SROW 20                   // 8 block scales per row and stage as fp16, + pad (dword stride 5: conflict-free)

struct Fp4Operand {
    const uint8_t* codes;           // [rows, K/2]
    const uint8_t* scales;          // [rows, K/16]
    int64_t rows;
};

// Vector loads at any byte address (rows start on 16-byte code and 8-byte scale boundaries only when K % 128 == 0;
// the hardware loads unaligned vectors in one instruction, it only touches one cache line more now and then).
typedef uint32_t uvec4_u __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t uvec2_u __attribute__((ext_vector_type(2), aligned(1)));
__device__ __forceinline__ uint4 load16_any(const uint8_t* p) {
    const uvec4_u v = *reinterpret_cast<const uvec4_u*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 load8_any(const uint8_t* p) {
    const uvec2_u v = *reinterpret_cast<const uvec2_u*>(p);
    return make_uint2(v.x, v.y);
}

// One thread's share of a stage of ROWS rows x 64 B of codes: V = ROWS*4/NT 16-byte code vectors.
// NT = threads per workgroup.
template <int V>
struct StageRegs {
    uint4 c[V];
};

// The 8 scale bytes per row and stage of both operands, dealt over all threads of the workgroup:
// thread t takes rows t, t + NT, ... of the BM + BN staged rows (A's rows first).
template <int V>
struct ScaleRegs {
    uint2 s[V];
};

// `whole`: all 128 contraction elements of the stage exist (uniform; a constant where PART is false); otherwise the
// missing ones read as zero
template <int BM, int BN, int NT>
__device__ __forceinline__ void scale_load(const Fp4Operand& A, const Fp4Operand& B, int64_t m0, int64_t n0, int64_t K,
                                           int64_t k0, bool whole, ScaleRegs<(BM + BN + NT - 1) / NT>& rg, int tid) {
    constexpr int V = (BM + BN + NT - 1) / NT;
    const int64_t sstride = K / 16;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int e = tid + NT * v;
        if ((BM + BN) % NT == 0 || e < BM + BN) {
            const bool isa = e < BM;
            const Fp4Operand& op = isa ? A : B;
            int64_t gr = isa ? m0 + e : n0 + (e - BM);
            if (gr >= op.rows) gr = op.rows - 1;
            const uint8_t* src = op.scales + gr * sstride + k0 / 16;
            if (whole) {
                rg.s[v] = load8_any(src);
            } else {
                // the row's last 8 scales end at its end: load those and shift the missing ones in as zeros
                uint64_t w = 0;
                if (sstride >= 8) {
                    const uint2 x = load8_any(op.scales + (gr + 1) * sstride - 8);
                    w = ((uint64_t)x.y << 32 | x.x) >> (8 * (int)(k0 / 16 + 8 - sstride));
                } else {
                    for (int i = 0; i < (int)sstride; ++i) w |= (uint64_t)src[i] << (8 * i);   // K < 128: one stage
                }
                rg.s[v] = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
            }
        }
    }
}

// E4M3 bytes -> fp16 with the hardware FP8 converter (exact; checked against the format's
// definition for all 256 bytes), 8 scales = 16 bytes per row
template <int BM, int BN, int NT>
__device__ __forceinline__ void scale_store(const ScaleRegs<(BM + BN + NT - 1) / NT>& rg, uint8_t* __restrict__ lsa,
                                            uint8_t* __restrict__ lsb, int tid) {
    constexpr int V = (BM + BN + NT - 1) / NT;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int e = tid + NT * v;
        if ((BM + BN) % NT == 0 || e < BM + BN) {
            uint32_t* dst = reinterpret_cast<uint32_t*>(e < BM ? lsa + e * G_SROW : lsb + (e - BM) * G_SROW);
            dst[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rg.s[v].x, 1.0f, false));
            dst[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rg.s[v].x, 1.0f, true));
            dst[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rg.s[v].y, 1.0f, false));
            dst[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rg.s[v].y, 1.0f, true));
        }
    }
}

template <int ROWS, int NT>
__device__ __forceinline__ void stage_load(const Fp4Operand& op, int64_t r0, int64_t K, int64_t k0, bool whole,
                                           StageRegs<ROWS * 4 / NT>& rg, int tid) {
    constexpr int T = ROWS * 4 / NT;
    const int64_t cstride = K / 2;
#pragma unroll
    for (int v = 0; v < T; ++v) {
        int e = tid + NT * v;
        int row = e >> 2, seg = e & 3;
        int64_t gr = r0 + row;
        if (gr >= op.rows) gr = op.rows - 1;
        const uint8_t* src = op.codes + gr * cstride + k0 / 2 + 16 * seg;
        if (whole) {
            rg.c[v] = load16_any(src);
        } else {
            // K is a multiple of 16: the row ends on an 8-byte boundary of the stage.  (Byte by byte, the last stage of a 1360 x
            // 1232 x 752 training step cost its skinny pre-products 12.3 us a launch against 8.6.)
            const int64_t kb = k0 / 2 + 16 * seg;
            const uint8_t* row_p = op.codes + gr * cstride;
            const uint2 lo = load8_any(kb < cstride ? src : row_p), hi = load8_any(kb + 8 < cstride ? src + 8 : row_p);
            const uint32_t mlo = kb < cstride ? ~0u : 0u, mhi = kb + 8 < cstride ? ~0u : 0u;
            rg.c[v] = make_uint4(lo.x & mlo, lo.y & mlo, hi.x & mhi, hi.y & mhi);
        }
    }
}

template <int ROWS, int NT>
__device__ __forceinline__ void stage_store(const StageRegs<ROWS * 4 / NT>& rg, uint8_t* __restrict__ lc, int tid) {
    constexpr int T = ROWS * 4 / NT;
#pragma unroll
    for (int v = 0; v < T; ++v) {
        int e = tid + NT * v;
        int row = e >> 2, seg = e & 3;
        uint32_t* dst = reinterpret_cast<uint32_t*>(lc + row * G_CROW + 16 * seg);
        dst[0] = rg.c[v].x; dst[1] = rg.c[v].y; dst[2] = rg.c[v].z; dst[3] = rg.c[v].w;
    }
}

// 8 codes (one dword) times one block scale -> 8 fp16.  `spair` holds the fp16 scales of two
// consecutive blocks; `hi` picks the second (the splat folds into the packed multiply's operand select).
__device__ __forceinline__ half8_t dequant8(uint32_t cw, uint32_t spair, bool hi) {
    const half2_t sp = __builtin_bit_cast(half2_t, spair);
    const half2_t s2 = hi ? (half2_t){sp[1], sp[1]} : (half2_t){sp[0], sp[0]};
    const half2_t c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(cw, 1.0f, 0);
    const half2_t c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(cw, 1.0f, 1);
    const half2_t c2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(cw, 1.0f, 2);
    const half2_t c3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(cw, 1.0f, 3);
    half2_t p0 = c0 * s2, p1 = c1 * s2, p2 = c2 * s2, p3 = c3 * s2;
    half8_t r = {p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
    return r;
}

union BFrag {
    uint4 u;
    bf16x8_t v;
};

template <int BM, int BN>
constexpr size_t gemm_lds_bytes() {
    return 2 * ((size_t)BM * (G_CROW + G_SROW) + (size_t)BN * (G_CROW + G_SROW));
}

// The extra contraction columns (bf16, Ke % 16 == 0) are stored in the order the matrix instruction wants them:
// element (row r, column c) at (((r/32 * Ke/16 + c/16) * 2 + (c%16)/8) * 32 + r%32) * 8 + c%8, rows padded to a
// multiple of 32 -- the 64 lanes' 16-byte operands of one 32-row block and 16-column step are 1 KiB of
// consecutive memory (read row-major, one such load touched 32 cache lines and used a quarter of each).
__host__ __device__ __forceinline__ int64_t ext_chunk(int64_t row_block, int step, int half, int li, int nsteps) {
    return (((row_block * nsteps + step) * 2 + half) * 32 + li) * 8;
}

// One output tile by a workgroup of WMW x WNW waves, each wave TM x TN tiles of 32x32 (BM = 32 TM WMW,
// BN = 32 TN WNW), over the contraction stages [it0, niter).
// PART: the last stage may end past K.  (A template parameter: the test costs the wait counts of every stage, 5 % of a
// small product.)
template <int TM, int TN, int WMW, int WNW, bool PART, typename OUT>
__device__ __forceinline__ void
gemm_nt_tile(const Fp4Operand& A, const Fp4Operand& B, int64_t K, const bf16_t* __restrict__ Aext,
             const bf16_t* __restrict__ Bext, int Ke, float alpha, OUT* __restrict__ C, int64_t ldc, int tile_m, int tile_n,
             int64_t it0, int64_t niter) {
    constexpr int BM = 32 * TM * WMW, BN = 32 * TN * WNW, NT = 64 * WMW * WNW;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // LDS: [buffer][codes A | codes B | scales A | scales B]
    constexpr int OFF_CB = BM * G_CROW, OFF_SA = (BM + BN) * G_CROW, OFF_SB = OFF_SA + BM * G_SROW,
                  BUF = OFF_SB + BN * G_SROW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int wm = (wave / WNW) * 32 * TM, wn = (wave % WNW) * 32 * TN;
    const int li = lane & 31, half = lane >> 5;

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // this workgroup's stages of the contraction: [it0, niter)
    StageRegs<BM * 4 / NT> ra;
    StageRegs<BN * 4 / NT> rb;
    ScaleRegs<(BM + BN + NT - 1) / NT> rs;
    auto load = [&](int64_t it) {
        const int64_t k0 = it * G_KI;
        const bool whole = !PART || k0 + G_KI <= K;
        stage_load<BM, NT>(A, m0, K, k0, whole, ra, tid);
        stage_load<BN, NT>(B, n0, K, k0, whole, rb, tid);
        scale_load<BM, BN, NT>(A, B, m0, n0, K, k0, whole, rs, tid);
    };
    load(it0);
    stage_store<BM, NT>(ra, lds, tid);
    stage_store<BN, NT>(rb, lds + OFF_CB, tid);
    scale_store<BM, BN, NT>(rs, lds + OFF_SA, lds + OFF_SB, tid);
    __syncthreads();
    for (int64_t it = it0; it < niter; ++it) {
        const int cur = (int)((it - it0) & 1);
        const bool more = it + 1 < niter;
        if (more) load(it + 1);
        const uint8_t* bufc = lds + cur * BUF;
        uint8_t* bufn = lds + (cur ^ 1) * BUF;
        const uint8_t* ca = bufc + (wm + li) * G_CROW + 4 * half;
        const uint8_t* cb = bufc + OFF_CB + (wn + li) * G_CROW + 4 * half;
        const uint8_t* sa = bufc + OFF_SA + (wm + li) * G_SROW;
        const uint8_t* sb = bufc + OFF_SB + (wn + li) * G_SROW;
#pragma unroll
        for (int s = 0; s < G_KI / 16; ++s) {
            half8_t fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = dequant8(*reinterpret_cast<const uint32_t*>(ca + 32 * i * G_CROW + 8 * s),
                                 *reinterpret_cast<const uint32_t*>(sa + 32 * i * G_SROW + 4 * (s >> 1)), s & 1);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[j] = dequant8(*reinterpret_cast<const uint32_t*>(cb + 32 * j * G_CROW + 8 * s),
                                 *reinterpret_cast<const uint32_t*>(sb + 32 * j * G_SROW + 4 * (s >> 1)), s & 1);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (more) {
            stage_store<BM, NT>(ra, bufn, tid);
            stage_store<BN, NT>(rb, bufn + OFF_CB, tid);
            scale_store<BM, BN, NT>(rs, bufn + OFF_SA, bufn + OFF_SB, tid);
        }
        __syncthreads();
    }
    // low-rank terms: extra contraction columns in bf16, read straight from global memory
    if (Ke > 0) {
        const int nks = Ke >> 4;
        const int64_t rba_max = (A.rows + 31) / 32 - 1, rbb_max = (B.rows + 31) / 32 - 1;
        // (the operands of a step travel while the step before is multiplied)
        auto load_ext = [&](int ks, BFrag (&fa)[TM], BFrag (&fb)[TN]) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                int64_t rb = (m0 + wm) / 32 + i;
                if (rb > rba_max) rb = rba_max;
                fa[i].u = *reinterpret_cast<const uint4*>(Aext + ext_chunk(rb, ks, half, li, nks));
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                int64_t rb = (n0 + wn) / 32 + j;
                if (rb > rbb_max) rb = rbb_max;
                fb[j].u = *reinterpret_cast<const uint4*>(Bext + ext_chunk(rb, ks, half, li, nks));
            }
        };
        BFrag fa[TM], fb[TN];
        load_ext(0, fa, fb);
        for (int ks = 0; ks < nks; ++ks) {
            BFrag na[TM], nb[TN];
            load_ext(ks + 1 < nks ? ks + 1 : ks, na, nb);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].v, fb[j].v, acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = na[i];
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = nb[j];
        }
    }
    // D layout 32x32: lane l, element v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int64_t c = n0 + wn + 32 * j + li;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int64_t r = m0 + wm + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                if (r < A.rows && c < B.rows) store_out<OUT>(C + r * ldc + c, alpha * acc[i][j][v]);
            }
        }
}

// 1-D grid of ceil(M / BM) * ceil(N / BN) workgroups; workgroup -> tile by TileMap; the first niter stages of the
// contraction (all of them, unless the last, partial one is among the extra columns)
template <int TM, int TN, int WMW, int WNW, bool PART, typename OUT>
__global__ void __launch_bounds__(64 * WMW * WNW)
k_fp4_gemm_nt(Fp4Operand A, Fp4Operand B, int64_t K, int64_t niter, const bf16_t* __restrict__ Aext,
              const bf16_t* __restrict__ Bext, int Ke, float alpha, OUT* __restrict__ C, int64_t ldc, TileMap tmap) {
    int tile_m, tile_n;
    tile_coords(tmap, tile_m, tile_n);
    gemm_nt_tile<TM, TN, WMW, WNW, PART, OUT>(A, B, K, Aext, Bext, Ke, alpha, C, ldc, tile_m, tile_n, 0, niter);
}

// The same tiles with the contraction cut into parts of `ips` stages: workgroup b takes part b / tiles of tile b % tiles and
// writes an fp32 tile of P[part] (M x N each, side by side); the low-rank columns enter with part 0.
template <int TM, int TN, int WMW, int WNW, bool PART>
__global__ void __launch_bounds__(64 * WMW * WNW)
k_fp4_gemm_nt_parts(Fp4Operand A, Fp4Operand B, int64_t K, int64_t niter, int ips, const bf16_t* __restrict__ Aext,
                    const bf16_t* __restrict__ Bext, int Ke, float alpha, float* __restrict__ P, int tiles, int tiles_n) {
    const int z = (int)blockIdx.x / tiles, t = (int)blockIdx.x - z * tiles;
    const int64_t it0 = (int64_t)z * ips, it1 = it0 + ips < niter ? it0 + ips : niter;
    gemm_nt_tile<TM, TN, WMW, WNW, PART, float>(A, B, K, Aext, Bext, z == 0 ? Ke : 0, alpha, P + (size_t)z * A.rows * B.rows, B.rows,
                                               t / tiles_n, t % tiles_n, it0, it1);
}

// C = sum of the parts, in ascending order; a thread takes 4 consecutive elements.  They lie in one row, 16-byte aligned in every
// part, when N % 4 == 0; an unsplit right operand may have any number of rows, and then each element finds its own row.
template <typename OUT>
__global__ void __launch_bounds__(256)
k_sum_output_parts(const float* __restrict__ P, int parts, int64_t MN, int64_t N, OUT* __restrict__ C, int64_t ldc) {
    const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= MN) return;
    auto row_of = [&](int64_t x) { return (uint64_t)MN >> 32 ? x / N : (int64_t)((uint32_t)x / (uint32_t)N); };
    if (N % 4 != 0) {                                    // (uniform)
        for (int64_t x = e; x < e + 4 && x < MN; ++x) {
            float acc = P[x];
            for (int p = 1; p < parts; ++p) acc += P[(size_t)p * MN + x];
            const int64_t r = row_of(x);
            store_out<OUT>(C + r * ldc + (x - r * N), acc);
        }
        return;
    }
    float4 acc = *reinterpret_cast<const float4*>(P + e);
#pragma unroll 4
    for (int p = 1; p < parts; ++p) {
        const float4 x = *reinterpret_cast<const float4*>(P + (size_t)p * MN + e);
        acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
    }
    const int64_t r = row_of(e);
    OUT* c = C + r * ldc + (e - r * N);
    store_out<OUT>(c, acc.x); store_out<OUT>(c + 1, acc.y); store_out<OUT>(c + 2, acc.z); store_out<OUT>(c + 3, acc.w);
}

// The block scales of both operands in fp16, in the order k_fp4_gemm_nt_stream reads them: 4 KiB for 256 rows and one unit of 128,
// [64 rows][lane][4] dwords, the dword of lane 16 kg + r and t the scales of row 16 t + r's blocks 2 kg and 2 kg + 1.  (Fetched from the
// rows themselves, 8 bytes from each, a unit's scales cost the address units twice what its codes do: 2922 against 2544 cycles
// for 64 columns of a 256 x 256 tile; and the conversion of 32 pairs a unit is done once instead of in every tile.)
// A thread takes one row and four units; rows past the end get zeros.
#define GS_SCALES 4096                                   // bytes for 256 rows and one unit
struct ScalePlan {
    const uint8_t *scales_a, *scales_b;
    int64_t rows_a, rows_b, sstride;
    uint8_t *plan_a, *plan_b;
    int blocks_a, blocks, niter;                         // of 256 rows: A's, all (an operand may have none to do); units
    int first, count;                                    // workgroups of a shared launch
};
__device__ __forceinline__ void scale_plan_block(const ScalePlan& o, int index) {
    const int by = index / o.blocks, bx = index - by * o.blocks;
    const bool isb = bx >= o.blocks_a;
    const uint8_t* scales = isb ? o.scales_b : o.scales_a;
    uint8_t* plan = isb ? o.plan_b : o.plan_a;
    const int64_t rows = isb ? o.rows_b : o.rows_a;
    const int rb = bx - (isb ? o.blocks_a : 0), lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t row = 256 * (int64_t)rb + 64 * w + 16 * (lane & 3) + (lane >> 2);
    uint2 x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int u = 4 * by + i;
        x[i] = row < rows && u < o.niter ? load8_any(scales + row * o.sstride + 8 * u) : make_uint2(0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int u = 4 * by + i;
        if (u >= o.niter) break;
        uint32_t* p = reinterpret_cast<uint32_t*>(plan + ((int64_t)rb * o.niter + u) * GS_SCALES + 1024 * w) + lane;
        p[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x[i].x, 1.0f, false));
        p[64] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x[i].x, 1.0f, true));
        p[128] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x[i].y, 1.0f, false));
        p[192] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x[i].y, 1.0f, true));
    }
}
__global__ void __launch_bounds__(256)
k_scale_plan(ScalePlan o) { scale_plan_block(o, (int)blockIdx.x); }

// Up to three skinny products in one launch, each cut along the contraction into `splits` parts that are written
// side by side (part z of problem q at P + z rows_a rows_b, plain stores): the consumer adds the parts in a fixed
// order, so the result does not depend on the order in which workgroups finish.  128 x 64 tiles, 4 waves.
struct SkinnyProblem {
    Fp4Operand A, B;         // C = alpha A B^T, [A.rows, B.rows]
    float alpha;
    float* P;
    int tiles_n, tiles;      // tiles along B.rows, tiles in all
    int ips;                 // stages per part
    int first;               // first workgroup of this problem
};
struct SkinnyBatch {
    SkinnyProblem p[3];
    int count;
    ScalePlan plan;          // workgroups plan.first .. (none if count is 0)
};

template <bool PART>
__global__ void __launch_bounds__(256)
k_fp4_skinny_batch(SkinnyBatch batch, int64_t K) {
    if (batch.plan.count > 0 && (int)blockIdx.x >= batch.plan.first) {
        scale_plan_block(batch.plan, (int)blockIdx.x - batch.plan.first);
        return;
    }
    int q = 0;
#pragma unroll
    for (int i = 1; i < 3; ++i)
        if (i < batch.count && (int)blockIdx.x >= batch.p[i].first) q = i;
    SkinnyProblem pr = batch.p[0];
    if (q == 1) pr = batch.p[1];
    if (q == 2) pr = batch.p[2];
    const int local = (int)blockIdx.x - pr.first, z = local / pr.tiles, t = local - z * pr.tiles;
    const int64_t niter_all = (K + G_KI - 1) / G_KI;
    const int64_t it0 = (int64_t)z * pr.ips;
    const int64_t niter = it0 + pr.ips < niter_all ? it0 + pr.ips : niter_all;
    gemm_nt_tile<2, 1, 2, 2, PART, float>(pr.A, pr.B, K, nullptr, nullptr, 0, pr.alpha,
                                         pr.P + (size_t)z * pr.A.rows * pr.B.rows, pr.B.rows, t / pr.tiles_n, t % pr.tiles_n,
                                         it0, niter);
}

// Software-pipelined variant, for large outputs that are too few or too short for k_fp4_gemm_nt_stream, or whose caller brought no
// room for its scale plan: 256 x 256 tile, 4 waves of 128 x 128 (16 accumulator tiles per wave,
// one wave per SIMD).  Half as many code expansions per MFMA as the 8-wave kernel, so the matrix
// cores rather than the vector ALUs bound it -- provided the matrix pipe never drains:
//  * within a stage, the raw codes/scales of contraction step s+2 are read from LDS and step s+1
//    is expanded to fp16 between the 16 MFMAs of step s (register double-buffering, interleaving
//    pinned with sched_group_barrier);
//  * across stages, the next stage's global data is written to the other LDS buffer during steps
//    0-4 (each staging register is refilled with the stage after next right after its write), the
//    workgroup barrier sits at the start of step 6, and steps 6 and 7 already read and expand the
//    next stage's first two steps, so no MFMA waits for a barrier, an LDS round trip or a global load.
// The stage body is branch-free and the same for every stage (the last one stages and expands data
// that nobody uses), which keeps the whole loop one scheduling region.  It covers the K / 128 whole stages; the
// elements past the last whole stage are among the extra columns (see k_assemble_ext).
template <typename OUT>
__global__ void __launch_bounds__(256)
k_fp4_gemm_nt_pipe(Fp4Operand A, Fp4Operand B, int64_t K, const bf16_t* __restrict__ Aext,
                   const bf16_t* __restrict__ Bext, int Ke_all, float alpha, OUT* __restrict__ C, int64_t ldc, TileMap tmap,
                   int total_tiles, int tail_first, int tail_parts, float* __restrict__ partial, int total_items) {
    constexpr int TM = 4, TN = 4, BM = 256, BN = 256, NT = 256, KS = G_KI / 16;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // LDS layout of a stage, chosen so that ONE 16-byte read per lane fetches the raw words of all four row
    // tiles of a wave (a lone wave per SIMD is bound by the number of instructions it issues, so instructions, not bytes, count):
    // codes of an operand: planes (g = row / 128, step s, half) of 32 lanes x 4 tiles dwords,
    //   dword (g, s, half, l, i) = the 8 codes of row 128 g + 32 i + l at contraction 16 s + 8 half;
    // scales: planes (g, pair q of steps) of 32 x 4 dwords, dword (g, q, l, i) = the fp16 scales of blocks 2q, 2q+1.
    // A plane is 512 bytes, padded to 528 (planes of neighbouring 16-byte code segments then start in different banks).
    constexpr int PL = 528, CODES_OP = 2 * KS * 2 * PL, SC_OP = 2 * (KS / 2) * PL;
    constexpr int OFF_CB = CODES_OP, OFF_SA = 2 * CODES_OP, OFF_SB = OFF_SA + SC_OP, BUF = OFF_SB + SC_OP;
    static_assert(2 * BUF <= (int)gemm_lds_bytes<256, 256>(), "two stages fit the allocation");
    // The tiles of the last, partly filled round of workgroups (launch positions tail_first ..) are cut along the
    // contraction into tail_parts workgroups each, which write fp32 partial tiles that a small kernel adds up:
    // the round then takes 1 / tail_parts of a tile's time instead of leaving most CUs idle for a whole one.
    // A workgroup walks the launch positions blockIdx.x, blockIdx.x + gridDim.x, ... itself (one workgroup per CU):
    // the stores of a finished tile drain while the next tile's contraction runs, and no CU waits for a dispatch.
    // (No barrier between tiles is needed: after the barrier in the last stage every LDS read fetches words
    // that are never used, and the next tile's first reads come after the barrier of its own first stage.)
    for (int pos = (int)blockIdx.x; pos < total_items; pos += (int)gridDim.x) {
    // (the thread index passes through an empty asm in every round, so that nothing derived from it counts as
    // loop-invariant: hoisted out of this loop, the per-lane offsets of all phases would be live at once and spill)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    int tile = pos, part = 0, parts = 1;
    if (tile >= tail_first) {
        const int idx = tile - tail_first;
        tile = tail_first + idx / tail_parts;
        part = idx - (tile - tail_first) * tail_parts;
        parts = tail_parts;
    }
    int tile_m, tile_n;
    tile_coords_of(tmap, tile, total_tiles, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int wm = (wave >> 1) * 128, wn = (wave & 1) * 128;
    const int li = lane & 31, half = lane >> 5;

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int niter_all = (int)(K / G_KI);
    const int it_begin = (int)((int64_t)part * niter_all / parts), it_end = (int)((int64_t)(part + 1) * niter_all / parts);
    const int niter = it_end - it_begin;                 // >= 1: the host keeps tail_parts <= K / 128
    const int Ke = part == 0 ? Ke_all : 0;               // the low-rank columns enter once
    // this thread's share of a stage: code vectors v = 0..3 of each operand (row tid/4 + 64 v, 16-byte
    // segment tid%4) and the scale rows tid (A) and tid (B); rows past the operand's end re-read its last row
    const uint8_t* pa[4];
    const uint8_t* pb[4];
    const int64_t cstride = K / 2, sstride = K / 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        int64_t ga = m0 + (tid >> 2) + 64 * v, gb = n0 + (tid >> 2) + 64 * v;
        if (ga >= A.rows) ga = A.rows - 1;
        if (gb >= B.rows) gb = B.rows - 1;
        pa[v] = A.codes + ga * cstride + 16 * (tid & 3) + (int64_t)it_begin * (G_KI / 2);
        pb[v] = B.codes + gb * cstride + 16 * (tid & 3) + (int64_t)it_begin * (G_KI / 2);
    }
    const uint8_t* psa;
    const uint8_t* psb;
    {
        int64_t ga = m0 + tid, gb = n0 + tid;
        if (ga >= A.rows) ga = A.rows - 1;
        if (gb >= B.rows) gb = B.rows - 1;
        psa = A.scales + ga * sstride + (int64_t)it_begin * (G_KI / 16);
        psb = B.scales + gb * sstride + (int64_t)it_begin * (G_KI / 16);
    }
    uint4 ra[4], rb[4];
    uint2 rsa, rsb;
    // st = stage index within this workgroup's range, clamped by the caller
    auto load_codes = [&](int st, int v) {
        ra[v] = load16_any(pa[v] + st * (G_KI / 2));
        rb[v] = load16_any(pb[v] + st * (G_KI / 2));
    };
    auto load_scales = [&](int st) {
        rsa = load8_any(psa + st * (G_KI / 16));
        rsb = load8_any(psb + st * (G_KI / 16));
    };
    auto load_stage = [&](int st) {
#pragma unroll
        for (int v = 0; v < 4; ++v) load_codes(st, v);
        load_scales(st);
    };
    // a 16-byte code vector = two steps (2 seg, 2 seg + 1) x two halves of one row: four dwords to four planes
    auto store_codes = [&](uint8_t* buf, int v) {
        const int e = tid + NT * v, row = e >> 2, seg = e & 3;
        const int off = (((row >> 7) * KS + 2 * seg) * 2) * PL + (row & 31) * 16 + ((row >> 5) & 3) * 4;
        uint8_t* da = buf + off;
        uint8_t* db = buf + OFF_CB + off;
        *reinterpret_cast<uint32_t*>(da) = ra[v].x;
        *reinterpret_cast<uint32_t*>(da + PL) = ra[v].y;
        *reinterpret_cast<uint32_t*>(da + 2 * PL) = ra[v].z;
        *reinterpret_cast<uint32_t*>(da + 3 * PL) = ra[v].w;
        *reinterpret_cast<uint32_t*>(db) = rb[v].x;
        *reinterpret_cast<uint32_t*>(db + PL) = rb[v].y;
        *reinterpret_cast<uint32_t*>(db + 2 * PL) = rb[v].z;
        *reinterpret_cast<uint32_t*>(db + 3 * PL) = rb[v].w;
    };
    auto store_scales = [&](uint8_t* buf) {
        const int off = ((tid >> 7) * (KS / 2)) * PL + (tid & 31) * 16 + ((tid >> 5) & 3) * 4;
        uint8_t* da = buf + OFF_SA + off;
        uint8_t* db = buf + OFF_SB + off;
        *reinterpret_cast<uint32_t*>(da) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsa.x, 1.0f, false));
        *reinterpret_cast<uint32_t*>(da + PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsa.x, 1.0f, true));
        *reinterpret_cast<uint32_t*>(da + 2 * PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsa.y, 1.0f, false));
        *reinterpret_cast<uint32_t*>(da + 3 * PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsa.y, 1.0f, true));
        *reinterpret_cast<uint32_t*>(db) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsb.x, 1.0f, false));
        *reinterpret_cast<uint32_t*>(db + PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsb.x, 1.0f, true));
        *reinterpret_cast<uint32_t*>(db + 2 * PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsb.y, 1.0f, false));
        *reinterpret_cast<uint32_t*>(db + 3 * PL) = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsb.y, 1.0f, true));
    };
    load_stage(0);
#pragma unroll
    for (int v = 0; v < 4; ++v) store_codes(lds, v);
    store_scales(lds);
    __syncthreads();
    // (in the order the stage loop issues and consumes them -- scheduling fences keep it: the wait in front of the
    // loop's first LDS write is computed over both ways into the loop, and with this order reversed here it has to
    // wait for every load in flight instead of the oldest pair)
    {
        const int st1 = niter > 1 ? 1 : 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            load_codes(st1, v);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_scales(st1);
        __builtin_amdgcn_sched_barrier(0);
    }

    // per-lane byte offsets of this wave's planes inside a buffer (step 0 / pair 0)
    typedef uint32_t rawvec_t __attribute__((ext_vector_type(4)));
    const int oca = (((wave >> 1) * KS) * 2 + half) * PL + li * 16, ocb = OFF_CB + (((wave & 1) * KS) * 2 + half) * PL + li * 16;
    const int osa = OFF_SA + ((wave >> 1) * (KS / 2)) * PL + li * 16, osb = OFF_SB + ((wave & 1) * (KS / 2)) * PL + li * 16;
    uint32_t rawc[2][TM + TN], raws[2][TM + TN];
    half8_t frag[2][TM + TN];
    auto read_raw = [&](const uint8_t* buf, int s, int slot) {
        const rawvec_t ca = *reinterpret_cast<const rawvec_t*>(buf + oca + 2 * s * PL);
        const rawvec_t cb = *reinterpret_cast<const rawvec_t*>(buf + ocb + 2 * s * PL);
        const rawvec_t sa = *reinterpret_cast<const rawvec_t*>(buf + osa + (s >> 1) * PL);
        const rawvec_t sb = *reinterpret_cast<const rawvec_t*>(buf + osb + (s >> 1) * PL);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            rawc[slot][i] = ca[i];
            raws[slot][i] = sa[i];
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            rawc[slot][TM + j] = cb[j];
            raws[slot][TM + j] = sb[j];
        }
    };
    read_raw(lds, 0, 0);
    read_raw(lds, 1, 1);
#pragma unroll
    for (int t = 0; t < TM + TN; ++t) frag[0][t] = dequant8(rawc[0][t], raws[0][t], false);

#pragma unroll 1
    for (int it = 0; it < niter; ++it) {
        const uint8_t* bufc = lds + (it & 1) * BUF;
        uint8_t* bufn = lds + ((it & 1) ^ 1) * BUF;
        const int stn = it + 2 < niter ? it + 2 : niter - 1;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int c = s & 1, n = c ^ 1;
            if (s + 2 == KS) __syncthreads();     // next stage is in LDS, this stage's raw words are all read
            // expand step s+1 (its raw words arrived during step s-1), then refill that raw slot with s+2
#pragma unroll
            for (int t = 0; t < TM + TN; ++t) frag[n][t] = dequant8(rawc[n][t], raws[n][t], (s + 1) & 1);
            if (s + 2 < KS) read_raw(bufc, s + 2, c);
            else read_raw(bufn, s + 2 - KS, c);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(frag[c][i], frag[c][TM + j], acc[i][j], 0, 0, 0);
            // a staging register is refilled with the stage after next as soon as it has been written
            // to LDS, which gives every global load a whole stage to arrive
            if (s < 4) {
                store_codes(bufn, s);
                load_codes(stn, s);
            }
            if (s == 4) {
                store_scales(bufn);
                load_scales(stn);
            }
            // one MFMA, then its share of the other work: 4 of the 64 expansion ops (5 early in a staging step: the
            // address arithmetic of the LDS writes and the loads needs slots too, or it drifts to the end of the
            // stage and takes the loads with it), 1 of the 16 LDS reads, and where the step has them an LDS write
            // or a global load.  Four load slots per staging step, right behind its LDS writes: with two, half of
            // the loads were issued a third of a stage later, and a load has to be back one stage after its issue.
#pragma unroll
            for (int m = 0; m < TM * TN; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (s <= 4 && m < 12) __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                else __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (s <= 4) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                if (s <= 4 && m >= 6 && m < 10) {                      // the step's global loads, after its LDS writes
                    __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
            }
        }
    }

    // low-rank terms: extra contraction columns in bf16, read straight from global memory; three steps of
    // fragments in flight, a step's registers are refilled with the step three ahead as soon as it is used
    const int nks = Ke >> 4;
    if (nks > 0) {
        const bf16_t* ea[TM];
        const bf16_t* eb[TN];
        const int64_t rba_max = (A.rows + 31) / 32 - 1, rbb_max = (B.rows + 31) / 32 - 1;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int64_t rb = (m0 + wm) / 32 + i;
            if (rb > rba_max) rb = rba_max;
            ea[i] = Aext + ext_chunk(rb, 0, half, li, nks);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int64_t rb = (n0 + wn) / 32 + j;
            if (rb > rbb_max) rb = rbb_max;
            eb[j] = Bext + ext_chunk(rb, 0, half, li, nks);
        }
        constexpr int EXT_DEPTH = 3;      // four fit the registers only with spills, and run no faster
        BFrag f[EXT_DEPTH][TM + TN];
        auto load_ext = [&](int step, int slot) {
#pragma unroll
            for (int i = 0; i < TM; ++i) f[slot][i].u = *reinterpret_cast<const uint4*>(ea[i] + step * 512);
#pragma unroll
            for (int j = 0; j < TN; ++j) f[slot][TM + j].u = *reinterpret_cast<const uint4*>(eb[j] + step * 512);
        };
#pragma unroll
        for (int u = 0; u < EXT_DEPTH; ++u)
            if (u < nks) load_ext(u, u);
        for (int ks = 0; ks < nks; ks += EXT_DEPTH) {
#pragma unroll
            for (int u = 0; u < EXT_DEPTH; ++u) {
                if (ks + u < nks) {                                   // uniform (kernel argument)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[u][i].v, f[u][TM + j].v, acc[i][j], 0, 0, 0);
                    if (ks + u + EXT_DEPTH < nks) load_ext(ks + u + EXT_DEPTH, u);
                }
            }
        }
    }
    // D layout 32x32: lane l, element v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
    if (parts > 1) {
        // partial tile, fp32, [tail tile][part][256][256]; bounds are applied when the parts are added up
        float* __restrict__ P = partial + ((size_t)(tile - tail_first) * parts + part) * (size_t)(BM * BN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    P[(wm + 32 * i + 4 * half + 8 * (v >> 2) + (v & 3)) * BN + wn + 32 * j + li] = alpha * acc[i][j][v];
        continue;
    }
    const bool interior = m0 + BM <= A.rows && n0 + BN <= B.rows;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t c = n0 + wn + 32 * j + li;
            const int64_t rbase = m0 + wm + 32 * i + 4 * half;
            if (interior) {
                store_tile16<OUT>(C + rbase * ldc + c, ldc, acc[i][j], alpha);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int64_t r = rbase + 8 * (v >> 2) + (v & 3);
                    if (r < A.rows && c < B.rows) store_out<OUT>(C + r * ldc + c, alpha * acc[i][j][v]);
                }
            }
        }
    }
}

// adds the parts of the split tail tiles and writes them to C (see k_fp4_gemm_nt_pipe); one workgroup per 32 rows of a tile
template <typename OUT, typename MAP>
__global__ void __launch_bounds__(256)
k_gemm_tail_sum(const float* __restrict__ partial, int parts, int tail_first, int total_tiles, MAP tmap, int64_t M,
                int64_t N, OUT* __restrict__ C, int64_t ldc) {
    const int tile = tail_first + (int)blockIdx.x / 8, rb = (int)blockIdx.x % 8;
    int tile_m, tile_n;
    tile_coords_of(tmap, tile, total_tiles, tile_m, tile_n);
    const float* __restrict__ P = partial + (size_t)(tile - tail_first) * parts * 65536;
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {          // 32 rows x 64 float4
        const int r = 32 * rb + e / 64, c4 = (e % 64) * 4;
        float4 acc = *reinterpret_cast<const float4*>(P + r * 256 + c4);
        for (int p = 1; p < parts; ++p) {
            const float4 x = *reinterpret_cast<const float4*>(P + (size_t)p * 65536 + r * 256 + c4);
            acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
        }
        const int64_t gr = (int64_t)tile_m * 256 + r, gc = (int64_t)tile_n * 256 + c4;
        if (gr >= M) continue;
        const float v[4] = {acc.x, acc.y, acc.z, acc.w};
        for (int i = 0; i < 4; ++i)
            if (gc + i < N) store_out<OUT>(C + gr * ldc + gc + i, v[i]);
    }
}

// bytes of fp32 partial tiles the pipelined kernel wants for an M x N output (0: no tail split)
static size_t gemm_tail_bytes(int64_t M, int64_t N, int64_t K, int* parts_out = nullptr, int* tail_first_out = nullptr) {
    const int64_t tiles = ceil_div64(M, 256) * ceil_div64(N, 256);
    const int64_t tail = tiles % 256, niter = K / G_KI;
    int parts = tail > 0 ? (int)(256 / tail) : 1;
    if (parts > 4) parts = 4;
    if (parts > niter) parts = (int)niter;
    if (parts_out) *parts_out = parts;
    if (tail_first_out) *tail_first_out = (int)(tiles - tail);
    if (tail == 0 || parts < 2) return 0;
    return (size_t)tail * parts * 65536 * sizeof(float);
}

#include "gemm_stream.h"

template <typename OUT>
int launch_gemm_stream(hipStream_t s, const Fp4Operand& a, const Fp4Operand& b, int64_t K, const uint8_t* plan, const bf16_t* Aext,
                       const bf16_t* Bext, int Ke, float alpha, OUT* C, int64_t ldc, float* partial, size_t partial_bytes) {
    const int64_t tm = ceil_div64(a.rows, 256), tn = ceil_div64(b.rows, 256);
    if (tm * tn > 0x7FFFFFFF) return METIS_UNSUPPORTED;
    const int total = (int)(tm * tn);
    int parts = 1, tail_first = total;
    const size_t want = gemm_tail_bytes(a.rows, b.rows, K, &parts, &tail_first);
    const bool split = want > 0 && partial && partial_bytes >= want;
    if (!split) { parts = 1; tail_first = total; }
    const int tail = total - tail_first;
    const int items = tail_first + tail * parts;
    const int cus = device_cu_count();
    if (cus < 1) return METIS_HIP_ERROR;
    dim3 grid((unsigned)(items < cus ? items : cus));
    auto kern = k_fp4_gemm_nt_stream<OUT>;
    static LdsLimitCache lds_set;
    if (!ensure_dyn_lds((const void*)kern, GS_LDS, lds_set)) return METIS_HIP_ERROR;
    const BandMap tmap = make_band_map(tm, tn, GS_BAND);
    const bool vec = (uintptr_t)C % 16 == 0 && (ldc * sizeof(OUT)) % 16 == 0;
    hipLaunchKernelGGL(kern, grid, dim3(256), GS_LDS, s, a, b, K, plan,
                       plan + (size_t)tm * (K / G_KI) * GS_SCALES, Aext, Bext, Ke, alpha, C, ldc, vec, tmap, total, tail_first, parts,
                       partial, items);
    METIS_LAUNCH_CHECK();
    if (split) {
        hipLaunchKernelGGL((k_gemm_tail_sum<OUT, BandMap>), dim3((unsigned)(tail * 8)), dim3(256), 0, s, partial, parts, tail_first, total,
                           tmap, a.rows, b.rows, C, ldc);
        METIS_LAUNCH_CHECK();
    }
    return METIS_OK;
}

template <typename OUT>
int launch_gemm_pipe(hipStream_t s, const Fp4Operand& a, const Fp4Operand& b, int64_t K, const bf16_t* Aext,
                     const bf16_t* Bext, int Ke, float alpha, OUT* C, int64_t ldc, float* partial, size_t partial_bytes) {
    const int64_t tm = ceil_div64(a.rows, 256), tn = ceil_div64(b.rows, 256);
    if (tm * tn > 0x7FFFFFFF) return METIS_UNSUPPORTED;
    constexpr size_t lds = gemm_lds_bytes<256, 256>();
    const int total = (int)(tm * tn);
    int parts = 1, tail_first = total;
    const size_t want = gemm_tail_bytes(a.rows, b.rows, K, &parts, &tail_first);
    const bool split = want > 0 && partial && partial_bytes >= want;
    if (!split) { parts = 1; tail_first = total; }
    const int tail = total - tail_first;
    const int items = tail_first + tail * parts;
    const int cus = device_cu_count();
    if (cus < 1) return METIS_HIP_ERROR;
    dim3 grid((unsigned)(items < cus ? items : cus));
    auto kern = k_fp4_gemm_nt_pipe<OUT>;
    static LdsLimitCache lds_set;
    if (!ensure_dyn_lds((const void*)kern, lds, lds_set)) return METIS_HIP_ERROR;
    const TileMap tmap = make_tile_map(tm, tn);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, s, a, b, K, Aext, Bext, Ke, alpha, C, ldc, tmap, total, tail_first, parts,
                       partial, items);
    METIS_LAUNCH_CHECK();
    if (split) {
        hipLaunchKernelGGL((k_gemm_tail_sum<OUT, TileMap>), dim3((unsigned)(tail * 8)), dim3(256), 0, s, partial, parts, tail_first, total,
                           tmap, a.rows, b.rows, C, ldc);
        METIS_LAUNCH_CHECK();
    }
    return METIS_OK;
}

template <int TM, int TN, int WMW, int WNW, typename OUT>
int launch_gemm_tile(hipStream_t s, const Fp4Operand& a, const Fp4Operand& b, int64_t K, int64_t niter, const bf16_t* Aext,
                     const bf16_t* Bext, int Ke, float alpha, OUT* C, int64_t ldc) {
    constexpr int BM = 32 * TM * WMW, BN = 32 * TN * WNW, NT = 64 * WMW * WNW;
    static_assert(BM * 4 >= NT && BN * 4 >= NT, "every thread stages at least one code vector");
    const int64_t tm = ceil_div64(a.rows, BM), tn = ceil_div64(b.rows, BN);
    if (tm * tn > 0x7FFFFFFF) return METIS_UNSUPPORTED;
    constexpr size_t lds = gemm_lds_bytes<BM, BN>();
    const bool part = niter * G_KI > K;
    auto kern = part ? k_fp4_gemm_nt<TM, TN, WMW, WNW, true, OUT> : k_fp4_gemm_nt<TM, TN, WMW, WNW, false, OUT>;
    static LdsLimitCache lds_set[2];
    if (!ensure_dyn_lds((const void*)kern, lds, lds_set[part])) return METIS_HIP_ERROR;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tm * tn)), dim3(NT), lds, s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc,
                       make_tile_map(tm, tn));
    METIS_LAUNCH_CHECK();
    return METIS_OK;
}

// How an output of at most 256 tiles of the bounds-checked kernel is produced, by estimates (in us) that were fitted to
// measurements at rank 64 on 256 CUs (a constant here: the workspace's size is asked for without a device, too):
//   - small tiles (128 x 128 for large sides): a 128-deep stage takes 1.4 us (expansion bound, 1.15 per workgroup once a CU holds
//     several; 0.82 to 0.95, and 0.66, for tiles with a side of 64), the rest 8.  Few tiles leave most CUs idle while each walks
//     its whole contraction: the contraction is cut into parts where that costs less than it saves, a launch of 3.5 and 6 bytes of
//     traffic per element and part at ~4 TB/s.  Where the whole call would be one short launch (lone: no extra columns; a side of
//     64) the second one also costs the host 2.5 us (64 x 4096 x 1024: cut 9.4 us in a graph, 11.5 call after call; whole 10.6
//     both);
//   - both sides at least 1024: the pipelined kernel's 256 x 256 tiles, 3.3 per stage of a tile cut into `pipe_parts`, the rest 13,
//     a launch of 3 and the sum of its parts.
// 4096 x 1024: K = 1024 43 -> 20 (small tiles, whole), K = 4096 59 -> 52, K = 14336 stays pipelined (119; small tiles 157);
// 1024 x 1024: K = 4096 45 -> 31, K = 14336 89 -> 53 (4 parts); 1360 x 1232 x 768 35 -> 13.  Whole calls with one side below 1024:
// 256 x 4096 x 4096 56 -> 39, 256 x 4096 x 14336 153 -> 66, 512 x 4096 x 4096 58 -> 48, 512 x 1024 x 4096 55 -> 35.  The rank
// does not enter: it costs every form about the same.  256 x 4096 x 4096 without factors 41 -> 26, at rank 16 53 -> 38, at 128
// 61 -> 42; 512 x 1024 x 4096 41 -> 21, 53 -> 33, 61 -> 37.
struct SmallPlan {
    bool small;              // small tiles (otherwise: too many of them, or the pipelined kernel with its own cut is faster)
    int parts;               // their contraction parts
};
SmallPlan small_plan(int64_t M, int64_t N, int64_t niter, int pipe_parts, bool lone) {
    SmallPlan best = {false, 1};
    const int64_t bm = M <= 64 ? 64 : 128, bn = N <= 64 && M > 64 ? 64 : 128;
    const int64_t tiles = ceil_div64(M, bm) * ceil_div64(N, bn);
    if (tiles > 256) return best;
    const double mn = (double)M * (double)N;
    double best_t = pipe_parts > 0 ? 16.0 + 3.3 * (double)ceil_div64(niter, pipe_parts) + pipe_parts * mn * 1e-6 : 1e30;
    const bool half = bm * bn < 128 * 128;
    const double one = half ? 0.95 : 1.4, many = half ? 0.66 : 1.15, launch = lone && half ? 6.0 : 3.5;
    for (int p = 1; p <= 16 && (p == 1 || 2 * p <= niter); ++p) {
        const int64_t ips = ceil_div64(niter, p);
        if (ceil_div64(niter, ips) != p) continue;                       // no empty part
        const double per_cu = (double)ceil_div64(tiles * p, 256);
        const double t = 8.0 + (double)ips * (per_cu > 1.5 ? many * per_cu : one) + (p > 1 ? launch + p * mn * 1.5e-6 : 0.0);
        if (t < best_t - 1e-9) {
            best_t = t;
            best = {true, p};
        }
    }
    return best;
}

// The plan of an M x N output over `niter` stages; whole: every stage is a whole one; lone: there are no extra columns
SmallPlan gemm_plan(int64_t M, int64_t N, int64_t niter, bool whole, bool lone) {
    int pipe_parts = 0;
    if (M >= 1024 && N >= 1024 && whole && gemm_tail_bytes(M, N, niter * G_KI, &pipe_parts) == 0) pipe_parts = 0;
    return small_plan(M, N, niter, pipe_parts, lone);
}

template <int TM, int TN, int WMW, int WNW, typename OUT>
int launch_gemm_parts(hipStream_t s, const Fp4Operand& a, const Fp4Operand& b, int64_t K, int64_t niter, int parts,
                      const bf16_t* Aext, const bf16_t* Bext, int Ke, float alpha, OUT* C, int64_t ldc, float* partial) {
    constexpr int BM = 32 * TM * WMW, BN = 32 * TN * WNW, NT = 64 * WMW * WNW;
    const int64_t tn = ceil_div64(b.rows, BN), tiles = ceil_div64(a.rows, BM) * tn;
    constexpr size_t lds = gemm_lds_bytes<BM, BN>();
    const bool part = niter * G_KI > K;
    auto kern = part ? k_fp4_gemm_nt_parts<TM, TN, WMW, WNW, true> : k_fp4_gemm_nt_parts<TM, TN, WMW, WNW, false>;
    static LdsLimitCache lds_set[2];
    if (!ensure_dyn_lds((const void*)kern, lds, lds_set[part])) return METIS_HIP_ERROR;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * parts)), dim3(NT), lds, s, a, b, K, niter, (int)ceil_div64(niter, parts), Aext,
                       Bext, Ke, alpha, partial, (int)tiles, (int)tn);
    METIS_LAUNCH_CHECK();
    const int64_t mn = a.rows * b.rows;
    hipLaunchKernelGGL(k_sum_output_parts<OUT>, dim3((unsigned)ceil_div64(mn, 1024)), dim3(256), 0, s, partial, parts, mn, b.rows,
                       C, ldc);
    METIS_LAUNCH_CHECK();
    return METIS_OK;
}

// Shapes whose last, partial contraction stage travels as extra bf16 columns (exact: grid * e4m3 has at most 6
// significant bits) so that the software-pipelined kernel's branch-free stages serve any K: large outputs with K % 128.
// (The byte-wise staging it replaced took 798 us for the 4096 x 4096 weight gradient over 6000 tokens, 2.2 times the
// two aligned products of that step together; the whole step went from 2718 to 2029 us.)
bool tail_as_columns(int64_t M, int64_t N, int64_t K) { return M >= 1024 && N >= 1024 && K > G_KI && K % G_KI != 0; }

// ext_tail: the elements past the last whole stage are among the extra columns
template <typename OUT>
int launch_gemm(hipStream_t s, const metis_fp4& A, const metis_fp4& B, const bf16_t* Aext, const bf16_t* Bext, int Ke,
                bool ext_tail, float alpha, OUT* C, int64_t ldc, float* partial = nullptr, size_t partial_bytes = 0,
                const uint8_t* plan_room = nullptr) {
    const int64_t M = A.rows, N = B.rows, K = A.cols;
    const Fp4Operand a = {A.codes, A.scales, M}, b = {B.codes, B.scales, N};
    const int64_t niter = ext_tail ? K / G_KI : ceil_div64(K, G_KI);
    if (M >= 1024 && N >= 1024) {
        // 256x256 tile, 4 waves of 128x128, software-pipelined (whole 128-deep stages); the tiles of a partly filled
        // last round are cut along the contraction when the caller brought room for the parts
        const bool whole = K % G_KI == 0 || ext_tail;
        const size_t tail_need = gemm_tail_bytes(M, N, K);
        const bool can_split = tail_need > 0 && partial && partial_bytes >= tail_need;
        const int64_t tiles = ceil_div64(M, 256) * ceil_div64(N, 256);
        const SmallPlan plan = gemm_plan(M, N, niter, whole, Ke == 0);
        const bool room = partial && partial_bytes >= (size_t)plan.parts * M * N * sizeof(float);
        // few tiles: small ones, whole or in parts (without the room for those the call works too, on the kernels below)
        if (whole && plan.small && (plan.parts == 1 || room)) {
            if (plan.parts == 1) return launch_gemm_tile<2, 2, 2, 2, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
            return launch_gemm_parts<2, 2, 2, 2, OUT>(s, a, b, K, niter, plan.parts, Aext, Bext, Ke, alpha, C, ldc, partial);
        }
        if (plan_room)
            return launch_gemm_stream<OUT>(s, a, b, K, plan_room, Aext, Bext, Ke, alpha, C, ldc, partial, partial_bytes);
        if (whole && (can_split || tiles > 128))
            return launch_gemm_pipe<OUT>(s, a, b, K, Aext, Bext, Ke, alpha, C, ldc, partial, partial_bytes);
        // an output of at most 128 tiles of 256 x 256 would leave half the CUs without work: 128 x 128 tiles
        // (four times as many workgroups, each less efficient) finish sooner
        if (tiles <= 128) return launch_gemm_tile<2, 2, 2, 2, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
        // a partial stage that could not become extra columns (no workspace): 8 waves of 128x64, bounds-checked staging
        return launch_gemm_tile<4, 2, 2, 4, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
    }
    const int parts = gemm_plan(M, N, niter, false, Ke == 0).parts;
    if (parts > 1 && partial && partial_bytes >= (size_t)parts * M * N * sizeof(float)) {
        if (N > 64 && M > 64)
            return launch_gemm_parts<2, 2, 2, 2, OUT>(s, a, b, K, niter, parts, Aext, Bext, Ke, alpha, C, ldc, partial);
        if (M > 64) return launch_gemm_parts<2, 1, 2, 2, OUT>(s, a, b, K, niter, parts, Aext, Bext, Ke, alpha, C, ldc, partial);
        return launch_gemm_parts<1, 2, 2, 2, OUT>(s, a, b, K, niter, parts, Aext, Bext, Ke, alpha, C, ldc, partial);
    }
    if (N > 64 && M > 64) return launch_gemm_tile<2, 2, 2, 2, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
    if (N <= 64) return launch_gemm_tile<2, 1, 2, 2, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
    return launch_gemm_tile<1, 2, 2, 2, OUT>(s, a, b, K, niter, Aext, Bext, Ke, alpha, C, ldc);
}

// ---- few rows (decode): Y[M <= 64, N] = A Bbar^T with A unsplit, Bbar = U S V^T + R ----
// Two launches.  The first multiplies A with the rows of R_b and, as more columns, with those of V_b (T1 = A V_b^T), cut
// along the contraction into `z` parts so that a few workgroups per CU exist however few columns there are.  A workgroup
// owns 32 columns and all rows; its 4 waves deal the 128-deep stages of the part among themselves, so no stage
// passes through LDS and no wave waits for another: a lane reads the 64 codes (two 16-byte loads) and 4 scales of its row
// and half of the stage and expands them where they are.  The order of the contraction elements inside a stage is the
// lane's own (step s, half h = elements 64 h + 8 s ..), the same for both operands.  The waves' tiles are added in wave
// order through LDS.  The second launch adds the parts in order and Y = alpha A R_b^T + (T1 S_b) U_b^T in fp32.
// Bound by latency: 16 x 4096 x 4096 at rank 64 6.6 + 5.4 us (the general path's three kernels: 8.3 + 4.5 + 31 us), the whole
// call 42 -> 11 us in a graph; 16 x 4096 x 14336 114 -> 20 us, 64 x 4096 x 14336 116 -> 32 us.  At 128 rows a CU spends its
// time on reading and expanding A again for every 32 columns: 128 x 14336 x 4096 60 us against the general path's 47.
// (One launch whose every workgroup forms T1 again was measured too: 32 x 4096 x 4096 at rank 64 16 us, 16 x 4096 x 14336
// 41 us; two thirds of its vector instructions expanded V_b.)
#define DC_MAX_ROWS 64
struct DecodeRaw {
    uint4 c0, c1;
    uint32_t s;
};
typedef uint32_t u32_u __attribute__((aligned(1)));

// the lane's share of a stage: codes and scales of the contraction elements k .. k + 63 of a row (zeros from K on;
// `whole`, uniform: none is missing)
__device__ __forceinline__ DecodeRaw decode_load(const uint8_t* codes, const uint8_t* scales, int64_t k, int64_t K, bool whole) {
    DecodeRaw r;
    if (whole) {
        r.c0 = load16_any(codes + k / 2);
        r.c1 = load16_any(codes + k / 2 + 16);
        r.s = *reinterpret_cast<const u32_u*>(scales + k / 16);
    } else {
        uint2 c[4];
        r.s = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const bool in = k + 16 * b < K;
            c[b] = load8_any(in ? codes + k / 2 + 8 * b : codes);
            const uint32_t sc = in ? scales[k / 16 + b] : 0u;
            r.s |= sc << (8 * b);
            c[b].x = in ? c[b].x : 0u;
            c[b].y = in ? c[b].y : 0u;
        }
        r.c0 = make_uint4(c[0].x, c[0].y, c[1].x, c[1].y);
        r.c1 = make_uint4(c[2].x, c[2].y, c[3].x, c[3].y);
    }
    return r;
}

__device__ __forceinline__ half8_t decode_frag(const DecodeRaw& r, const uint32_t (&sp)[2], int s) {
    const uint32_t w = s == 0 ? r.c0.x : s == 1 ? r.c0.y : s == 2 ? r.c0.z : s == 3 ? r.c0.w
                     : s == 4 ? r.c1.x : s == 5 ? r.c1.y : s == 6 ? r.c1.z : r.c1.w;
    return dequant8(w, sp[s >> 2], (s >> 1) & 1);
}

// column blocks of 32: [0, nb) are R_b's rows, the rest V_b's; P [z][M][ldp], ldp = 32 x all column blocks
template <int TM>
__global__ void __launch_bounds__(256)
k_fp4_decode(Fp4Operand A, Fp4Operand B, Fp4Operand V, int blk0, int nb, int64_t K, int ips, float* __restrict__ P, int64_t ldp) {
    __shared__ float red[4][32][32];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, half = lane >> 5;
    const int64_t cstride = K / 2, sstride = K / 16;
    const int blk = blk0 + (int)blockIdx.x;
    // rows past an operand's end re-read its last row; what they give is not stored, or dropped by the second kernel
    const uint8_t *ca[TM], *sa[TM], *cb, *sb;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int64_t r = 32 * i + li < A.rows ? 32 * i + li : A.rows - 1;
        ca[i] = A.codes + r * cstride;
        sa[i] = A.scales + r * sstride;
    }
    {
        const bool isv = blk >= nb;
        const int64_t rows = isv ? V.rows : B.rows, r0 = 32 * (int64_t)(isv ? blk - nb : blk) + li;
        const int64_t r = r0 < rows ? r0 : rows - 1;
        cb = (isv ? V.codes : B.codes) + r * cstride;
        sb = (isv ? V.scales : B.scales) + r * sstride;
    }
    float16_t acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
    const int nst = (int)((K + G_KI - 1) / G_KI), it0 = (int)blockIdx.y * ips, it1 = it0 + ips < nst ? it0 + ips : nst;
    DecodeRaw a[TM], b;
    auto load = [&](int it) {
        const int64_t k0 = (int64_t)it * G_KI, k = k0 + 64 * half;
        const bool whole = k0 + G_KI <= K;
        b = decode_load(cb, sb, k, K, whole);
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = decode_load(ca[i], sa[i], k, K, whole);
    };
    if (it0 + wave < it1) load(it0 + wave);
    for (int it = it0 + wave; it < it1; it += 4) {
        DecodeRaw a0[TM];
        const DecodeRaw b0 = b;
        uint32_t pa[TM][2], pb[2];
        auto scales2 = [](uint32_t s, uint32_t (&o)[2]) {
            o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(s, 1.0f, false));
            o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(s, 1.0f, true));
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) { a0[i] = a[i]; scales2(a0[i].s, pa[i]); }
        scales2(b0.s, pb);
        if (it + 4 < it1) load(it + 4);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const half8_t fb = decode_frag(b0, pb, s);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(decode_frag(a0[i], pa[i], s), fb, acc[i], 0, 0, 0);
        }
    }
    // D layout 32x32: lane l, element v -> row 8*(v/4) + 4*(l/32) + v%4, column l%32
    const int row = tid >> 5, col = tid & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i > 0) __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][8 * (v >> 2) + 4 * half + (v & 3)][li] = acc[i][v];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = row + 8 * q;
            const float x = ((red[0][r][col] + red[1][r][col]) + red[2][r][col]) + red[3][r][col];
            if (32 * i + r < A.rows) P[((int64_t)blockIdx.y * A.rows + 32 * i + r) * ldp + 32 * (int64_t)blk + col] = x;
        }
    }
}

// Y = alpha sum_z P + (T1 S_b) U_b^T; a workgroup owns 16 rows and 64 columns, a thread 4 columns of one row.  All global
// loads of a thread are issued before the first use (a missing part re-reads the last one with weight 0).  H = 64-column
// halves of the rank.
#define DF_ROWS 16
#define DF_COLS 64
#define DC_MAX_PARTS 4
struct Parts4 {
    float4 x[DC_MAX_PARTS];
};
__device__ __forceinline__ Parts4 load_parts4(const float* __restrict__ p, int64_t zs, int parts) {
    Parts4 r;
#pragma unroll
    for (int u = 0; u < DC_MAX_PARTS; ++u) r.x[u] = *reinterpret_cast<const float4*>(p + (u < parts ? u : parts - 1) * zs);
    return r;
}
__device__ __forceinline__ float4 add_parts4(const Parts4& r, int parts) {
    float4 s = r.x[0];
#pragma unroll
    for (int u = 1; u < DC_MAX_PARTS; ++u) {
        const float w = u < parts ? 1.0f : 0.0f;
        s.x = fmaf(w, r.x[u].x, s.x); s.y = fmaf(w, r.x[u].y, s.y);
        s.z = fmaf(w, r.x[u].z, s.z); s.w = fmaf(w, r.x[u].w, s.w);
    }
    return s;
}

template <int H, typename OUT>
__global__ void __launch_bounds__(256)
k_decode_finish(const float* __restrict__ P, int parts, int M, int64_t N, int64_t ldp, int nb, int kb,
                const uint8_t* __restrict__ ub_codes, const uint8_t* __restrict__ ub_scales, const float* __restrict__ Sb,
                float alpha, float alpha_lr, OUT* __restrict__ C, int64_t ldc) {
    constexpr int KP = 64 * H, LT = KP + 4;
    __shared__ __attribute__((aligned(16))) float t1[H ? DF_ROWS * LT : 4];     // T1 S_b with the tensor scales, [row][j]
    __shared__ __attribute__((aligned(16))) bf16_t ub[H ? DF_COLS * LT : 8];    // U_b without its own (exact), [column][j]
    const int tid = threadIdx.x, r16 = tid >> 4, c4 = tid & 15;
    const int64_t zs = (int64_t)M * ldp;
    const int64_t n0 = (int64_t)blockIdx.x * DF_COLS, n = n0 + 4 * c4;
    const int m = (int)blockIdx.y * DF_ROWS + r16;
    const bool in = n < N && m < M;
    const int64_t mrow = m < M ? m : M - 1;
    Parts4 tp[H ? H : 1];
    float4 sv[H ? H : 1];
    uint32_t uw[H ? 2 * H : 1], us[H ? 2 * H : 1];
    // T1: row r16, columns 64 h + 4 c4 .. + 3 (the padded columns of V_b's last block hold copies of its last row)
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int j = 64 * h + 4 * c4;
        tp[h] = load_parts4(P + mrow * ldp + 32 * nb + (j < kb ? j : 0), zs, parts);
        sv[h] = make_float4(j < kb ? Sb[j] : 0.0f, j + 1 < kb ? Sb[j + 1] : 0.0f, j + 2 < kb ? Sb[j + 2] : 0.0f,
                            j + 3 < kb ? Sb[j + 3] : 0.0f);
    }
#pragma unroll
    for (int i = 0; i < 2 * H; ++i) {
        const int j = (tid >> 3) + 32 * i, c = 8 * (tid & 7);
        uw[i] = us[i] = 0;
        if (j < kb && n0 + c < N) {
            uw[i] = *reinterpret_cast<const u32_u*>(ub_codes + j * (N / 2) + (n0 + c) / 2);
            us[i] = ub_scales[j * (N / 16) + (n0 + c) / 16];
        }
    }
    const Parts4 yp = load_parts4(P + (in ? m * ldp + n : 0), zs, parts);
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const float4 x = add_parts4(tp[h], parts);
        const int j = 64 * h + 4 * c4;
        float4 v;
        v.x = j < kb ? x.x * (sv[h].x * alpha_lr) : 0.0f;
        v.y = j + 1 < kb ? x.y * (sv[h].y * alpha_lr) : 0.0f;
        v.z = j + 2 < kb ? x.z * (sv[h].z * alpha_lr) : 0.0f;
        v.w = j + 3 < kb ? x.w * (sv[h].w * alpha_lr) : 0.0f;
        *reinterpret_cast<float4*>(t1 + r16 * LT + j) = v;
    }
    const float grid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
#pragma unroll
    for (int i = 0; i < 2 * H; ++i) {
        const int j = (tid >> 3) + 32 * i, c = 8 * (tid & 7);
        const float s = e4m3_decode(us[i]);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t nib = (uw[i] >> (4 * q)) & 15u;
            const float x = grid[nib & 7u] * s;
            ub[(c + q) * LT + j] = f32_to_bf16_rne((nib & 8u) ? -x : x);
        }
    }
    const float4 y = add_parts4(yp, parts);
    float o[4] = {alpha * y.x, alpha * y.y, alpha * y.z, alpha * y.w};
    if (H) __syncthreads();
    if (!in) return;
#pragma unroll 4
    for (int q = 0; q < KP; q += 4) {
        const float4 a = *reinterpret_cast<const float4*>(t1 + r16 * LT + q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint2 u = *reinterpret_cast<const uint2*>(ub + (4 * c4 + i) * LT + q);
            o[i] = fmaf(a.x, bf16lo_to_f32(u.x), o[i]);
            o[i] = fmaf(a.y, bf16hi_to_f32(u.x), o[i]);
            o[i] = fmaf(a.z, bf16lo_to_f32(u.y), o[i]);
            o[i] = fmaf(a.w, bf16hi_to_f32(u.y), o[i]);
        }
    }
    // (without factors the right operand may have any number of rows: the last group of a row can be a partial one)
    OUT* c = C + m * ldc + n;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (n + i < N) store_out<OUT>(c + i, o[i]);
}

// Few rows of an unsplit left operand, where the few-row kernels are the faster ones.  Every workgroup of 32 columns expands all of
// A's rows again, in blocks of 32, and the parts of the whole output travel through memory; the general path does neither, but
// has two launches more with factors.  So wide outputs are its own, from fewer elements on when there are two row blocks, when a short
// contraction gives little to gain, and without factors or above rank 64 (a longer second kernel).  us in a graph, few-row against
// general, N x K:
//   rank 64: 64 x 14336 x 4096 33 against 34, 64 x 20480 x 4096 42 against 39, 64 x 12288 x 512 16 against 18, 64 x 50256 x 512 38
//   against 27, 32 x 50256 x 768 25 against 30; rank 16: 32 x 28672 x 4096 35 against 41, x 512 16.5 against 16.4;
//   rank 128: 64 x 8192 x 4096 29 against 34, 64 x 14336 x 4096 41 against 37, 32 x 28672 x 1024 28 against 30;
//   no factors: 64 x 8192 x 4096 17.4 against 17.6, 64 x 16384 x 4096 26 against 23, 17 x 50256 x 4096 37 against 46.
// Up to 16 rows it is cheap at every width (rank 64, 16 x 50256 x 4096 43 against 63).  Without factors the general path is one launch
// when its contraction is short, which saves the host 2.6 us (16 x 4096 x 512 5.1 against 6.5, but 11.2 against 8.7 call after
// call; x 1024 5.3 against 9.8).
bool decode_shape(int64_t Ma, int64_t Nb, int ka, int kb, int64_t Kc) {
    if (ka > 0 || Ma > DC_MAX_ROWS) return false;
    const int64_t niter = ceil_div64(Kc, G_KI);
    if (kb == 0 && niter <= 6) return false;
    if (Ma <= 16) return true;
    const bool low = kb > 0 && kb <= 64;
    int64_t most;                                   // output elements, in units of 2^16
    if (Ma <= 32) most = low ? (niter >= 6 ? 32 : 12) : niter >= (kb > 0 ? 6 : 16) ? 16 : 8;
    else most = low ? (niter >= 12 ? 15 : 12) : 8;
    return Ma * Nb <= most << 16;
}

struct DecodePlan {
    int nb, nv, ips, parts;              // column blocks of 32 of R_b, of V_b; stages per part, parts
    int64_t ldp;
    size_t bytes;
};
DecodePlan decode_plan(int64_t M, int64_t N, int kb, int64_t K) {
    DecodePlan d;
    d.nb = (int)ceil_div64(N, 32);
    d.nv = (kb + 31) / 32;
    d.ldp = 32 * (int64_t)(d.nb + d.nv);
    // about three workgroups per CU, each with a stage for every wave (the rank does not enter: a workspace sized for a larger
    // rank fits a smaller one)
    const int64_t wgs = d.nb + 2, nst = ceil_div64(K, G_KI);
    int64_t want = ceil_div64(768, wgs), most = nst / 4 > 0 ? nst / 4 : 1;
    if (want > most) want = most;
    if (want > DC_MAX_PARTS) want = DC_MAX_PARTS;
    d.ips = (int)ceil_div64(nst, want);
    d.parts = (int)ceil_div64(nst, d.ips);
    d.bytes = (size_t)d.parts * M * d.ldp * sizeof(float);
    return d;
}

// U_b^T (k x N FP4, N % 16 == 0) and S_b as PREPARE leaves them for APPLY, in `keep`: codes, scales, S on a 16-byte boundary
size_t decode_keep_scales(int64_t N, int kb) { return (size_t)kb * N / 2; }
size_t decode_keep_s(int64_t N, int kb) { return align_up(decode_keep_scales(N, kb) + (size_t)kb * N / 16, 16); }
__global__ void __launch_bounds__(256)
k_decode_keep(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales, const float* __restrict__ S, int64_t N, int kb,
              uint8_t* __restrict__ kc, uint8_t* __restrict__ ks, float* __restrict__ kS) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;       // 16 elements: 8 code bytes, one scale
    if (t < kb * N / 16) {
        const uint2 c = load8_any(codes + 8 * t);
        *reinterpret_cast<uint2*>(kc + 8 * t) = c;
        ks[t] = scales[t];
    }
    if (t < kb) kS[t] = S[t];
}

// One phase of the product, or both.  What PREPARE leaves is what depends on the right operand's factors, as on the general path:
// their columns of P (the parts of T1), and U_b and S_b, which the second kernel wants, copied to `keep`.
template <typename OUT>
int launch_decode(hipStream_t s, const metis_fp4& A, const metis_fp4& B, const metis_fp4* Ub, const metis_fp4* Vb, const float* Sb,
                  int kb, float* P, uint8_t* keep, int phase, OUT* C, int64_t ldc) {
    if (phase == METIS_LINEAR_PREPARE && kb == 0) return METIS_OK;
    const Fp4Operand a = {A.codes, A.scales, A.rows}, b = {B.codes, B.scales, B.rows};
    Fp4Operand v = {nullptr, nullptr, 0};
    const uint8_t *uc = nullptr, *us = nullptr;
    float alpha_lr = 0.0f;
    uint8_t* keep_us = keep + decode_keep_scales(B.rows, kb);
    float* keep_s = (float*)(keep + decode_keep_s(B.rows, kb));
    if (kb > 0) {
        v = {Vb->codes, Vb->scales, kb};
        uc = phase == METIS_LINEAR_APPLY ? keep : Ub->codes;
        us = phase == METIS_LINEAR_APPLY ? keep_us : Ub->scales;
        if (phase == METIS_LINEAR_APPLY) Sb = keep_s;
        alpha_lr = A.tscale * Vb->tscale * Ub->tscale;
    }
    const DecodePlan d = decode_plan(A.rows, B.rows, kb, A.cols);
    auto kern = A.rows <= 32 ? k_fp4_decode<1> : k_fp4_decode<2>;
    const int blk0 = phase == METIS_LINEAR_PREPARE ? d.nb : 0, blk1 = phase == METIS_LINEAR_APPLY ? d.nb : d.nb + d.nv;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blk1 - blk0), (unsigned)d.parts), dim3(256), 0, s, a, b, v, blk0, d.nb, A.cols, d.ips, P,
                       d.ldp);
    METIS_LAUNCH_CHECK();
    if (phase == METIS_LINEAR_PREPARE) {
        hipLaunchKernelGGL(k_decode_keep, dim3((unsigned)ceil_div64((int64_t)kb * B.rows / 16, 256)), dim3(256), 0, s, Ub->codes,
                           Ub->scales, Sb, B.rows, kb, keep, keep_us, keep_s);
        METIS_LAUNCH_CHECK();
        return METIS_OK;
    }
    auto finish = kb == 0 ? k_decode_finish<0, OUT> : kb <= 64 ? k_decode_finish<1, OUT> : k_decode_finish<2, OUT>;
    hipLaunchKernelGGL(finish, dim3((unsigned)ceil_div64(B.rows, DF_COLS), (unsigned)ceil_div64(A.rows, DF_ROWS)), dim3(256), 0, s, P,
                       d.parts, (int)A.rows, B.rows, d.ldp, d.nb, kb, uc, us, Sb, A.tscale * B.tscale, alpha_lr, C, ldc);
    METIS_LAUNCH_CHECK();
    return METIS_OK;
}

// value of one FP4 element without the tensor scale: grid[code] * e4m3(scale)
__device__ __forceinline__ float fp4_elem_nog(const uint8_t* codes, const uint8_t* scales, int64_t cols, int64_t r,
                                              int64_t c) {
    uint32_t byte = codes[r * (cols / 2) + c / 2];
    uint32_t nib = (c & 1) ? (byte >> 4) : (byte & 15u);
    const float grid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
    float v = grid[nib & 7u] * e4m3_decode(scales[r * (cols / 16) + c / 16]);
    return (nib & 8u) ? -v : v;
}

// Extra contraction columns for Abar Bbar^T (see file header).  Column layout, Kep = padded kb+ka:
//   Aext[m, 0:kb]     = (T1[m,:] + sum_j Ua[m,j] Sa_j Mk[j,:]) * Sb * gUb / (gRa gRb)
//   Aext[m, kb:kb+ka] = Ua[m,:] without its tensor scale (exact in bf16)
//   Bext[n, 0:kb]     = Ub[n,:] without its tensor scale (exact in bf16)
//   Bext[n, kb:kb+ka] = E2[n,:] * Sa * gUa / (gRa gRb)
//   Aext[m, Kep:Kep+Kt] = Ra[m, K-Kt:K] and Bext[n, Kep:Kep+Kt] = Rb[n, K-Kt:K] without tensor scales (exact in bf16):
//                       the contraction elements past the last whole stage, when they are taken as columns
// T1, E2 and Mk arrive as n1, n2, n3 contraction parts that are added here in ascending order.
// Blocks [0, ceil(Ma/32)) build 32 rows of Aext each: the dequantized factor rows U_a and the small matrix
// Sa Mk sit in LDS; thread (row t/8, column group t%8) owns the columns 64 h + 8 (t%8) + 0..7 of its row.  The
// remaining blocks build 32 rows of Bext each the same way.  The kernel moves little data and is bound by
// load latency: the loads of all parts of a sum are issued before the first use, and four workgroups share a CU.  TRIP: those of T1
// and Mk together (220 registers, two workgroups per CU), for calls whose workgroups fit like that, see assemble_in_one_trip.
#define AX_ROWS 32

// acc[i] += sum over parts p < n <= NP of base[p * pstride + off + i], i < 8, 16-byte aligned: all loads issued, then added in
// ascending order (a missing part re-reads the last one with weight 0)
template <int NP>
struct Parts8 {
    float4 lo[NP], hi[NP];
};
template <int NP>
__device__ __forceinline__ Parts8<NP> load_parts8(const float* __restrict__ base, size_t pstride, int n, size_t off) {
    Parts8<NP> r;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const float* q = base + (size_t)(u < n ? u : n - 1) * pstride + off;
        r.lo[u] = *reinterpret_cast<const float4*>(q);
        r.hi[u] = *reinterpret_cast<const float4*>(q + 4);
    }
    return r;
}
template <int NP>
__device__ __forceinline__ void add_parts8(const Parts8<NP>& r, int n, float (&acc)[8]) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const float w = u < n ? 1.0f : 0.0f;
        acc[0] = fmaf(w, r.lo[u].x, acc[0]); acc[1] = fmaf(w, r.lo[u].y, acc[1]);
        acc[2] = fmaf(w, r.lo[u].z, acc[2]); acc[3] = fmaf(w, r.lo[u].w, acc[3]);
        acc[4] = fmaf(w, r.hi[u].x, acc[4]); acc[5] = fmaf(w, r.hi[u].y, acc[5]);
        acc[6] = fmaf(w, r.hi[u].z, acc[6]); acc[7] = fmaf(w, r.hi[u].w, acc[7]);
    }
}

// acc[i] += sum over parts p < n <= 8 of base[p * pstride + off + i], i < cnt <= 8 (vec: cnt = 8 and 16-byte aligned).
// FOUR: sums of up to four parts load no more than those (a branch that the one-trip form, with eight parts as a rule, goes without)
template <bool FOUR>
__device__ __forceinline__ void sum_parts8(const float* __restrict__ base, size_t pstride, int n, size_t off, int cnt,
                                           bool vec, float (&acc)[8]) {
    if (vec) {
        if (FOUR && n <= 4) add_parts8(load_parts8<4>(base, pstride, n, off), n, acc);       // (uniform)
        else add_parts8(load_parts8<8>(base, pstride, n, off), n, acc);
        return;
    }
    for (int p0 = 0; p0 < n; p0 += 4) {
        float x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = p0 + u < n ? p0 + u : n - 1;
            const float* q = base + (size_t)p * pstride + off;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[u][i] = i < cnt ? q[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float w = p0 + u < n ? 1.0f : 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = fmaf(w, x[u][i], acc[i]);
        }
    }
}

// Rows r0 .. r0 + 31 of a factor stored transposed in FP4 (codes [k, rows], rows % 16 == 0), without the tensor
// scale, into dst[32][k + 1]: a thread decodes 8 consecutive rows of one stored row j (4 code bytes, one scale).
__device__ __forceinline__ void decode_factor_rows(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                                   int64_t rows, int k, int64_t r0, float* dst, int tid) {
    const float grid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
    const int q = tid & 3;
    const int64_t r = r0 + 8 * q;
    for (int j = tid >> 2; j < k; j += 64) {
        uint32_t by[4] = {0, 0, 0, 0};
        float sc = 0.0f;
        if (r < rows) {
            const uint8_t* c = codes + (int64_t)j * (rows / 2) + r / 2;
#pragma unroll
            for (int i = 0; i < 4; ++i) by[i] = c[i];
            sc = e4m3_decode(scales[(int64_t)j * (rows / 16) + r / 16]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t nib = (i & 1) ? (by[i >> 1] >> 4) : (by[i >> 1] & 15u);
            const float v = grid[nib & 7u] * sc;
            dst[(8 * q + i) * (k + 1) + j] = (nib & 8u) ? -v : v;
        }
    }
}

// The last Kt contraction elements of rows r0 .. r0 + 31 of a residual as bf16 columns from column Kep on: thread
// (row rr, column group cg) decodes 8 elements = 4 code bytes and one scale at a time.
__device__ __forceinline__ uint4 pack8_bf16(const float (&v)[8]);
__device__ __forceinline__ void tail_columns(const Fp4Operand& R, int64_t K, int Kt, int64_t row, int rr, int cg, int Kep,
                                             int nsteps, bf16_t* __restrict__ ext) {
    const float grid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
    for (int c0 = 8 * cg; c0 < Kt; c0 += 64) {
        const int64_t k = K - Kt + c0;
        const uint8_t* c = R.codes + row * (K / 2) + k / 2;
        const float sc = e4m3_decode(R.scales[row * (K / 16) + k / 16]);
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t byte = c[i >> 1], nib = (i & 1) ? (byte >> 4) : (byte & 15u);
            const float x = grid[nib & 7u] * sc;
            v[i] = (nib & 8u) ? -x : x;
        }
        const int col = Kep + c0;
        *reinterpret_cast<uint4*>(ext + ext_chunk(row >> 5, col >> 4, (col >> 3) & 1, rr, nsteps)) = pack8_bf16(v);
    }
}

__device__ __forceinline__ uint4 pack8_bf16(const float (&v)[8]) {
    uint4 o;
    o.x = (uint32_t)f32_to_bf16_rne(v[0]) | (uint32_t)f32_to_bf16_rne(v[1]) << 16;
    o.y = (uint32_t)f32_to_bf16_rne(v[2]) | (uint32_t)f32_to_bf16_rne(v[3]) << 16;
    o.z = (uint32_t)f32_to_bf16_rne(v[4]) | (uint32_t)f32_to_bf16_rne(v[5]) << 16;
    o.w = (uint32_t)f32_to_bf16_rne(v[6]) | (uint32_t)f32_to_bf16_rne(v[7]) << 16;
    return o;
}

// NCH = ceil(kb / 64): column groups of a row that hold T1-type columns
template <int NCH, bool TRIP>
__global__ void __launch_bounds__(256)
k_assemble_ext(int64_t Ma, int64_t Nb, int ka, int kb, int Kep, Fp4Operand Ra, Fp4Operand Rb, int64_t K, int Kt,
               const float* __restrict__ T1, int n1, const float* __restrict__ Mk, int n3, const float* __restrict__ E2, int n2,
               const uint8_t* __restrict__ ua_codes, const uint8_t* __restrict__ ua_scales, float g_ua,
               const float* __restrict__ Sa, const uint8_t* __restrict__ ub_codes,
               const uint8_t* __restrict__ ub_scales, float g_ub, const float* __restrict__ Sb,
               float inv_grr, bf16_t* __restrict__ Aext, bf16_t* __restrict__ Bext) {
    extern __shared__ __attribute__((aligned(16))) float ax_sm[];
    const int nblk_a = (int)((Ma + AX_ROWS - 1) / AX_ROWS);
    const int tid = threadIdx.x, rr = tid >> 3, cg = tid & 7, nsteps = (Kep + Kt) >> 4;
    if ((int)blockIdx.x < nblk_a) {
        float* ua = ax_sm;                                          // [AX_ROWS][ka + 1]
        float* mk = ax_sm + (AX_ROWS * (ka + 1) + 3) / 4 * 4;       // [ka][kb] (+ 8 floats of slack)
        const int64_t r0 = (int64_t)blockIdx.x * AX_ROWS, row = r0 + rr;
        const bool in = row < Ma;
        const int64_t lrow = in ? row : Ma - 1;
        const int nmk = ka * kb;
        float t1[NCH][8];
#pragma unroll
        for (int h = 0; h < NCH; ++h)
#pragma unroll
            for (int i = 0; i < 8; ++i) t1[h][i] = 0.0f;
        if constexpr (TRIP) {
            // every group of 8 is whole, aligned and inside one row of Mk
            const int c0 = 8 * cg < kb ? 8 * cg : 0, ea = 8 * tid < nmk ? 8 * tid : 0, eb = 8 * tid + 2048 < nmk ? 8 * tid + 2048 : 0;
            const Parts8<8> pt = load_parts8<8>(T1, (size_t)Ma * kb, n1, (size_t)lrow * kb + c0);
            const Parts8<8> pa = load_parts8<8>(Mk, (size_t)nmk, n3, (size_t)ea);
            const Parts8<8> pb = load_parts8<8>(Mk, (size_t)nmk, n3, (size_t)eb);
            const float fa = g_ua * Sa[ea / kb], fb = g_ua * Sa[eb / kb];
            float ma[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f}, mb[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            add_parts8(pt, n1, t1[0]);
            add_parts8(pa, n3, ma);
            add_parts8(pb, n3, mb);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (8 * tid < nmk) mk[ea + i] = ma[i] * fa;
                if (8 * tid + 2048 < nmk) mk[eb + i] = mb[i] * fb;
            }
        } else {
            // this thread's sums of the T1 parts
#pragma unroll
            for (int h = 0; h < NCH; ++h) {
                const int c0 = 64 * h + 8 * cg;
                if (c0 < kb && n1 > 0) {
                    const int cnt = kb - c0 < 8 ? kb - c0 : 8;
                    sum_parts8<true>(T1, (size_t)Ma * kb, n1, (size_t)lrow * kb + c0, cnt, cnt == 8 && kb % 4 == 0, t1[h]);
                }
            }
            // Sa Mk (with U_a's tensor scale) into LDS, the parts added on the way
            for (int e0 = 8 * tid; e0 < nmk; e0 += 8 * 256) {
                float m[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                const int cnt = nmk - e0 < 8 ? nmk - e0 : 8;
                sum_parts8<true>(Mk, (size_t)nmk, n3, (size_t)e0, cnt, cnt == 8 && nmk % 4 == 0, m);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (i < cnt) mk[e0 + i] = m[i] * g_ua * Sa[(e0 + i) / kb];
            }
        }
        decode_factor_rows(ua_codes, ua_scales, Ma, ka, r0, ua, tid);
        __syncthreads();
        if (!in) return;
        tail_columns(Ra, K, Kt, row, rr, cg, Kep, nsteps, Aext);
        const bool vecmk = kb % 4 == 0;
        const float gs = g_ub * inv_grr;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int c0 = 64 * h + 8 * cg;
            if (c0 >= Kep) continue;
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = c0 + i;
                v[i] = (c >= kb && c < kb + ka) ? ua[rr * (ka + 1) + c - kb] : 0.0f;
            }
            if (h < NCH && c0 < kb) {
                float acc[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] = t1[h < NCH ? h : 0][i];
                for (int j = 0; j < ka; ++j) {
                    const float u = ua[rr * (ka + 1) + j];
                    const float* mrow = mk + j * kb + c0;
                    if (vecmk) {
                        const float4 lo = *reinterpret_cast<const float4*>(mrow), hi = *reinterpret_cast<const float4*>(mrow + 4);
                        acc[0] = fmaf(u, lo.x, acc[0]); acc[1] = fmaf(u, lo.y, acc[1]);
                        acc[2] = fmaf(u, lo.z, acc[2]); acc[3] = fmaf(u, lo.w, acc[3]);
                        acc[4] = fmaf(u, hi.x, acc[4]); acc[5] = fmaf(u, hi.y, acc[5]);
                        acc[6] = fmaf(u, hi.z, acc[6]); acc[7] = fmaf(u, hi.w, acc[7]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) acc[i] = fmaf(u, mrow[i], acc[i]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (c0 + i < kb) v[i] = acc[i] * Sb[c0 + i] * gs;
            }
            *reinterpret_cast<uint4*>(Aext + ext_chunk(row >> 5, c0 >> 4, (c0 >> 3) & 1, rr, nsteps)) = pack8_bf16(v);
        }
        return;
    }
    // Bext rows
    float* ub = ax_sm;                              // [AX_ROWS][kb + 1]
    const int64_t r0 = ((int64_t)blockIdx.x - nblk_a) * AX_ROWS, row = r0 + rr;
    const bool in = row < Nb;
    const int64_t lrow = in ? row : Nb - 1;
    float e2[4][8];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
#pragma unroll
        for (int i = 0; i < 8; ++i) e2[h][i] = 0.0f;
        // the E2-type columns of this group: c in [max(c0, kb), min(c0 + 8, kb + ka)) <-> E2 columns c - kb
        const int c0 = 64 * h + 8 * cg;
        const int lo = c0 > kb ? c0 : kb, hi = c0 + 8 < kb + ka ? c0 + 8 : kb + ka;
        if (lo < hi && n2 > 0) {
            const int cnt = hi - lo;
            sum_parts8<!TRIP>(E2, (size_t)Nb * ka, n2, (size_t)lrow * ka + (lo - kb), cnt,
                       cnt == 8 && ka % 4 == 0 && (lo - kb) % 4 == 0, e2[h]);
        }
    }
    decode_factor_rows(ub_codes, ub_scales, Nb, kb, r0, ub, tid);
    __syncthreads();
    if (!in) return;
    tail_columns(Rb, K, Kt, row, rr, cg, Kep, nsteps, Bext);
    const float gs = g_ua * inv_grr;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int c0 = 64 * h + 8 * cg;
        if (c0 >= Kep) continue;
        const int lo = c0 > kb ? c0 : kb;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = c0 + i;
            float x = 0.0f;
            if (c < kb) x = ub[rr * (kb + 1) + c];
            else if (c < kb + ka) {
                // e2[h] holds the group's E2-type columns from index 0 on
                float t = 0.0f;
#pragma unroll
                for (int z = 0; z < 8; ++z) t = (c - lo == z) ? e2[h][z] : t;
                x = t * Sa[c - kb] * gs;
            }
            v[i] = x;
        }
        *reinterpret_cast<uint4*>(Bext + ext_chunk(row >> 5, c0 >> 4, (c0 >> 3) & 1, rr, nsteps)) = pack8_bf16(v);
    }
}

// The form of k_assemble_ext whose loads are all in flight at once: both operands split, every group of 8 whole, aligned and inside
// one row of Mk, and (nblk) few enough workgroups that two per CU hold them.  In a training step of 4096 x 1024 x 4096 at rank 64
// (160 to 256 workgroups) a launch takes 15.8 us against 16.8; 128 x 50256 x 4096 at rank 64 (1575) whole 141 against 139,
// 16 x 50256 x 4096 at rank 16 107 against 102.
bool assemble_in_one_trip(int ka, int kb, int64_t nblk) {
    return ka > 0 && kb > 0 && kb <= 64 && kb % 8 == 0 && ka * kb <= 2 * 8 * 256 && nblk <= 512;
}

// Products for the streaming kernel (instead of the pipelined one).  It wants a workgroup on every CU, and work enough per CU to pay
// for its start and the scale plan (lone: no extra columns, so that the plan is a launch of its own, ~5 us).  Measured call for call
// against the pipelined kernel, parts of its time.  With factors, at the line of 32 units: 8192 x 4096, K = 2048 0.92; 8192 x 8192,
// K = 1024 0.90; 16384 x 16384, K = 256 0.79 to 0.85; 32768 x 32768, K = 128 0.79; above it 4096 x 4096, K = 4096 0.90.  Without, at 64:
// 4096 x 4096, K = 8192 0.88; 8192 x 8192, K = 2048 0.88; 16384 x 16384, K = 512 0.82.  Below the line it depends on the shape, and the
// pipelined kernel keeps them all: 8192 x 8192, K = 512 0.95 / 0.93 (with factors / without), 4096 x 4096, K = 2048 0.97 / 1.00,
// 8192 x 4096, K = 1024 1.00 / 1.04, 2048 x 14336, K = 2048 0.95 / 1.02.  Fewer than 256 tiles leave CUs idle, and the pipelined kernel
// then has the power to itself: 3072 x 4096, K = 4096 1.00 / 1.06 (with so few that their contractions are cut: not measured).
// (Its offsets within a tile's 256 rows of codes are 32 bits wide: rows of up to 2^32 / 255 bytes, 16.8 MB.)
bool stream_shape(int64_t M, int64_t N, int64_t niter, int64_t row_bytes, bool lone) {
    if (M < 1024 || N < 1024 || row_bytes > 0xFFFFFFFFll / 255) return false;
    const int64_t tiles = ceil_div64(M, 256) * ceil_div64(N, 256);
    return tiles >= 256 && ceil_div64(tiles, 256) * niter >= (lone ? 64 : 32);
}

struct NtOperand {            // one side of Abar Bbar^T: Abar = U diag(S) V^T + R, R [rows, Kc]
    metis_fp4 R, Ut, Vt;      // Ut [k, rows], Vt [k, Kc]
    const float* S;
    int k;
};

struct LinWs {
    size_t off_t1, off_mk, off_e2, off_aext, off_bext, off_tail, tail_bytes, off_plan, plan_bytes, total;
    int Kep;                 // low-rank columns, padded to 16
    int Kt;                  // columns of the last, partial contraction stage (0: none or not taken as columns)
    int s1, s2, s3;          // contraction parts of T1, E2, Mk
    bool decode;             // few rows of an unsplit operand: the tail region holds the parts of both products
};

// Parts of a skinny product with rows x cols outputs: few output tiles, long contraction -> cut it so that about
// 256 workgroups share the work, each with at least two stages.
int skinny_parts(int64_t rows, int64_t cols, int64_t Kc, int64_t cap) {
    const int64_t tiles = ceil_div64(rows, 128) * ceil_div64(cols, 64), iters = ceil_div64(Kc, G_KI);
    int64_t want = ceil_div64(256, tiles);
    const int64_t maxs = iters / 2 > 0 ? iters / 2 : 1;
    if (want > maxs) want = maxs;
    if (want > cap) want = cap;
    const int64_t ips = ceil_div64(iters, want);
    return (int)ceil_div64(iters, ips);           // no empty part
}

LinWs lin_layout(int64_t Ma, int64_t Nb, int ka, int kb, int64_t Kc) {
    LinWs w;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    w.Kt = tail_as_columns(Ma, Nb, Kc) ? (int)(Kc % G_KI) : 0;
    const bool large = Ma >= 1024 && Nb >= 1024, whole = Kc % G_KI == 0 || w.Kt > 0;
    const int64_t niter = w.Kt > 0 ? Kc / G_KI : ceil_div64(Kc, G_KI);
    const SmallPlan plan = gemm_plan(Ma, Nb, niter, whole, ka + kb + w.Kt == 0);
    w.Kep = (ka + kb + 15) / 16 * 16;
    bool stream = whole && !plan.small && stream_shape(Ma, Nb, niter, Kc / 2, ka + kb + w.Kt == 0);
    if (stream && (w.Kep + w.Kt) % 32 != 0) {
        if (w.Kep + 16 <= 256) w.Kep += 16;               // (the assembly kernel clears up to 256 columns)
        else stream = false;
    }
    // (the assembly kernel adds the parts up, two rounds of four loads at most)
    w.s1 = kb > 0 ? skinny_parts(Ma, kb, Kc, 8) : 1;
    w.s2 = ka > 0 ? skinny_parts(Nb, ka, Kc, 8) : 1;
    w.s3 = ka > 0 && kb > 0 ? skinny_parts(ka, kb, Kc, 8) : 1;
    w.off_t1 = take((size_t)w.s1 * Ma * (kb > 0 ? kb : 1) * 4);
    w.off_mk = take((size_t)w.s3 * (ka > 0 ? ka : 1) * (kb > 0 ? kb : 1) * 4);
    w.off_e2 = take((size_t)w.s2 * Nb * (ka > 0 ? ka : 1) * 4);
    const int ext = w.Kep + w.Kt > 0 ? w.Kep + w.Kt : 16;
    w.off_aext = take((size_t)((Ma + 31) / 32 * 32) * ext * 2);       // rows padded to whole 32-row blocks
    w.off_bext = take((size_t)((Nb + 31) / 32 * 32) * ext * 2);
    w.decode = decode_shape(Ma, Nb, ka, kb, Kc);
    const size_t parts_bytes = plan.parts > 1 ? (size_t)plan.parts * Ma * Nb * sizeof(float) : 0;
    if (w.decode) w.tail_bytes = decode_plan(Ma, Nb, kb, Kc).bytes;
    else if (large) w.tail_bytes = !whole ? 0 : plan.small ? parts_bytes : gemm_tail_bytes(Ma, Nb, Kc);
    else w.tail_bytes = parts_bytes;
    w.off_tail = take(w.tail_bytes);
    w.plan_bytes = stream ? (size_t)(ceil_div64(Ma, 256) + ceil_div64(Nb, 256)) * niter * GS_SCALES : 0;
    w.off_plan = take(w.plan_bytes);
    w.total = o;
    return w;
}

bool fp4_valid(const metis_fp4& f) { return f.codes && f.scales && f.rows > 0 && f.cols > 0 && f.cols % 16 == 0; }

// phase: METIS_LINEAR_ALL, or only the pre-pass (PREPARE: fills the workspace) / only the main kernel (APPLY)
int linear_nt(hipStream_t s, const NtOperand& a, const NtOperand& b, metis_mat* out, void* workspace,
              size_t workspace_bytes, int phase = METIS_LINEAR_ALL) {
    const bool do_pre = phase != METIS_LINEAR_APPLY, do_main = phase != METIS_LINEAR_PREPARE;
    if (do_main && (!out || !out->ptr)) return METIS_INVALID_ARG;
    if (!fp4_valid(a.R) || !fp4_valid(b.R) || a.R.cols != b.R.cols) return METIS_BAD_SHAPE;
    const int64_t Ma = a.R.rows, Nb = b.R.rows, Kc = a.R.cols;
    if (do_main) {
        if (out->rows != Ma || out->cols != Nb || out->ld < Nb) return METIS_BAD_SHAPE;
        if (out->dtype != METIS_BF16 && out->dtype != METIS_F32) return METIS_INVALID_ARG;
    }
    const int ka = a.k, kb = b.k;
    if (ka < 0 || kb < 0 || ka > 128 || kb > 128) return METIS_UNSUPPORTED;
    if (ka > 0 && (!a.S || !fp4_valid(a.Ut) || !fp4_valid(a.Vt) || a.Ut.rows != ka || a.Ut.cols != Ma ||
                   a.Vt.rows != ka || a.Vt.cols != Kc)) return METIS_BAD_SHAPE;
    if (kb > 0 && (!b.S || !fp4_valid(b.Ut) || !fp4_valid(b.Vt) || b.Ut.rows != kb || b.Ut.cols != Nb ||
                   b.Vt.rows != kb || b.Vt.cols != Kc)) return METIS_BAD_SHAPE;
    const float grr = a.R.tscale * b.R.tscale;
    int Ke = 0;
    const bf16_t *Aext = nullptr, *Bext = nullptr;
    bool ext_tail = false;
    int st;
    const LinWs w = lin_layout(Ma, Nb, ka, kb, Kc);
    const bool ws_fits = workspace && workspace_bytes >= w.off_tail;                        // the tail region is optional
    const bool ws_aligned = reinterpret_cast<uintptr_t>(workspace) % 16 == 0;
    if (ka > 0 || kb > 0) {
        if (!ws_fits) return METIS_WORKSPACE_TOO_SMALL;
        if (!ws_aligned) return METIS_INVALID_ARG;
    }
    if (w.decode && workspace && workspace_bytes >= w.off_plan && ws_aligned) {
        float* P = (float*)((char*)workspace + w.off_tail);
        // the kept factors, 9/16 byte per element of U_b and 4 per singular value, take the place of Bext: 2 bytes per element
        uint8_t* keep = (uint8_t*)workspace + w.off_bext;
        if (!do_main) return launch_decode<float>(s, a.R, b.R, &b.Ut, &b.Vt, b.S, kb, P, keep, phase, (float*)nullptr, 0);
        const int pi = metis_prof_begin(METIS_PROF_GEMM, s);
        if (out->dtype == METIS_BF16)
            st = launch_decode<bf16_t>(s, a.R, b.R, &b.Ut, &b.Vt, b.S, kb, P, keep, phase, (bf16_t*)out->ptr, out->ld);
        else
            st = launch_decode<float>(s, a.R, b.R, &b.Ut, &b.Vt, b.S, kb, P, keep, phase, (float*)out->ptr, out->ld);
        metis_prof_end(METIS_PROF_GEMM, pi, s);
        return st;
    }
    // Room for the streaming kernel's scale plan, when the workspace has it (and the codes start on 16 bytes).  PREPARE may lay out the
    // scales of a residual that it reads anyway (the other side's factors multiply it, or its last columns are among the extra ones);
    // the other residual need not be there, or be the last one, before APPLY, which then lays it out in a launch of its own.
    uint8_t* plan = nullptr;
    ScalePlan sp{};
    if (w.plan_bytes > 0 && workspace && workspace_bytes >= w.total && ws_aligned && (uintptr_t)a.R.codes % 16 == 0 &&
        (uintptr_t)b.R.codes % 16 == 0) {
        plan = (uint8_t*)workspace + w.off_plan;
        const bool early_a = kb > 0 || w.Kt > 0, early_b = ka > 0 || w.Kt > 0;
        const bool lay_a = early_a ? do_pre : do_main, lay_b = early_b ? do_pre : do_main;
        const int blocks_a = (int)ceil_div64(Ma, 256);
        sp.niter = (int)(Kc / G_KI);
        sp.blocks_a = lay_a ? blocks_a : 0;
        sp.blocks = sp.blocks_a + (lay_b ? (int)ceil_div64(Nb, 256) : 0);
        sp.scales_a = a.R.scales; sp.scales_b = b.R.scales;
        sp.rows_a = Ma; sp.rows_b = Nb; sp.sstride = Kc / 16;
        sp.plan_a = plan;
        sp.plan_b = plan + (size_t)blocks_a * sp.niter * GS_SCALES;
        sp.count = sp.blocks * (int)ceil_div64(sp.niter, 4);
    }
    // (two unsplit operands work without a workspace: a partial last stage then takes the bounds-checked kernel)
    if (ka > 0 || kb > 0 || (w.Kt > 0 && ws_fits && ws_aligned)) {
        char* ws = (char*)workspace;
        float* T1 = (float*)(ws + w.off_t1);
        float* Mk = (float*)(ws + w.off_mk);
        float* E2 = (float*)(ws + w.off_e2);
        bf16_t* ae = (bf16_t*)(ws + w.off_aext);
        bf16_t* be = (bf16_t*)(ws + w.off_bext);
        if (do_pre) {
            // the skinny products T1 = R_a V_b^T, E2 = R_b V_a^T and Mk = V_a V_b^T in one launch, cut along the contraction
            // (Mk is a single output tile: alone, one workgroup would walk the whole contraction, ~100 us at 14336 columns)
            SkinnyBatch sb;
            sb.count = 0;
            int wgs = 0;
            const int64_t iters = ceil_div64(Kc, G_KI);
            auto add = [&](const metis_fp4& X, const metis_fp4& Y, float* P, int parts) {
                SkinnyProblem& q = sb.p[sb.count++];
                q.A = {X.codes, X.scales, X.rows};
                q.B = {Y.codes, Y.scales, Y.rows};
                q.alpha = X.tscale * Y.tscale;
                q.P = P;
                q.tiles_n = (int)ceil_div64(Y.rows, 64);
                q.tiles = (int)ceil_div64(X.rows, 128) * q.tiles_n;
                q.ips = (int)ceil_div64(iters, parts);
                q.first = wgs;
                wgs += q.tiles * parts;
            };
            if (ceil_div64(Ma, 128) * 64 * w.s1 + ceil_div64(Nb, 128) * 64 * w.s2 > 0x3FFFFFFF) return METIS_UNSUPPORTED;
            if (kb > 0) add(a.R, b.Vt, T1, w.s1);
            if (ka > 0) add(b.R, a.Vt, E2, w.s2);
            if (ka > 0 && kb > 0) add(a.Vt, b.Vt, Mk, w.s3);
            for (int i = sb.count; i < 3; ++i) sb.p[i] = sb.count ? sb.p[0] : SkinnyProblem{};
            sb.plan = sp;
            sb.plan.first = wgs;
            if (sb.count > 0) {
                wgs += sp.count;
                sp.count = 0;                                // on its way
                constexpr size_t lds = gemm_lds_bytes<128, 64>();
                const bool part = Kc % G_KI != 0;
                auto skinny = part ? k_fp4_skinny_batch<true> : k_fp4_skinny_batch<false>;
                static LdsLimitCache lds_set[2];
                if (!ensure_dyn_lds((const void*)skinny, lds, lds_set[part])) return METIS_HIP_ERROR;
                hipLaunchKernelGGL(skinny, dim3((unsigned)wgs), dim3(256), lds, s, sb, Kc);
                METIS_LAUNCH_CHECK();
            }
            const int64_t nblk = ceil_div64(Ma, AX_ROWS) + ceil_div64(Nb, AX_ROWS);
            const size_t ax_lds = ((size_t)(AX_ROWS * ((ka > kb ? ka : kb) + 1) + 3) / 4 * 4 + (size_t)ka * kb + 8) * sizeof(float);
            const int form = assemble_in_one_trip(ka, kb, nblk) ? 2 : kb > 64 ? 1 : 0;
            auto assemble = form == 2 ? k_assemble_ext<1, true> : form == 1 ? k_assemble_ext<2, false> : k_assemble_ext<1, false>;
            static LdsLimitCache ax_set[3];
            if (ax_lds > 48 * 1024 && !ensure_dyn_lds((const void*)assemble, ax_lds, ax_set[form])) return METIS_HIP_ERROR;
            hipLaunchKernelGGL(assemble, dim3((unsigned)nblk), dim3(256), ax_lds, s, Ma, Nb, ka, kb, w.Kep,
                               Fp4Operand{a.R.codes, a.R.scales, Ma}, Fp4Operand{b.R.codes, b.R.scales, Nb}, Kc, w.Kt, T1,
                               w.s1, Mk, w.s3, E2, w.s2, a.Ut.codes, a.Ut.scales, ka > 0 ? a.Ut.tscale : 1.0f, a.S, b.Ut.codes,
                               b.Ut.scales, kb > 0 ? b.Ut.tscale : 1.0f, b.S, 1.0f / grr, ae, be);
            METIS_LAUNCH_CHECK();
        }
        Ke = w.Kep + w.Kt;
        ext_tail = w.Kt > 0;
        Aext = ae;
        Bext = be;
    }
    if (sp.count > 0) {                                      // no skinny products in this phase, no launch to share
        hipLaunchKernelGGL(k_scale_plan, dim3((unsigned)sp.count), dim3(256), 0, s, sp);
        METIS_LAUNCH_CHECK();
    }
    // room for the partial tiles of a split last round, when the workspace has it
    float* partial = nullptr;
    size_t partial_bytes = 0;
    if (w.tail_bytes > 0 && !w.decode && workspace && workspace_bytes >= w.off_plan && ws_aligned) {
        partial = (float*)((char*)workspace + w.off_tail);
        partial_bytes = w.tail_bytes;
    }
    if (!do_main) return METIS_OK;
    const int pi = metis_prof_begin(METIS_PROF_GEMM, s);
    if (out->dtype == METIS_BF16)
        st = launch_gemm<bf16_t>(s, a.R, b.R, Aext, Bext, Ke, ext_tail, grr, (bf16_t*)out->ptr, out->ld, partial, partial_bytes, plan);
    else
        st = launch_gemm<float>(s, a.R, b.R, Aext, Bext, Ke, ext_tail, grr, (float*)out->ptr, out->ld, partial, partial_bytes, plan);
    metis_prof_end(METIS_PROF_GEMM, pi, s);
    return st;
}

NtOperand nt(const metis_fp4& R, const metis_fp4& Ut, const metis_fp4& Vt, const float* S, int k) {
    NtOperand o;
    o.R = R; o.Ut = Ut; o.Vt = Vt; o.S = S; o.k = k;
    return o;
}

}  // namespace

extern "C" size_t metis_linear_workspace_bytes(int64_t L, int64_t N, int64_t K, int k) {
    if (L < 1 || N < 1 || K < 1 || k < 0) return 0;
    // The operands' ranks may be any two up to k.  A layout without the streaming kernel's scale plan grows with each of them, except
    // that a skinny product of up to 64 columns is cut into more parts than one of 65 to 128, and that unsplit operands take other
    // kernels: the largest is at one of these.  The plan, the same for all ranks, may be there for some and not for others.
    const int ranks[3] = {0, k < 64 ? k : 64, k};
    const int64_t shapes[3][3] = {{L, N, K}, {L, K, N}, {N, K, L}};
    size_t most = 0;
    for (const auto& p : shapes) {
        size_t rest = 0, plan = 0;
        for (int ka : ranks)
            for (int kb : ranks) {
                const LinWs w = lin_layout(p[0], p[1], ka, kb, p[2]);
                rest = std::max(rest, w.off_plan);
                plan = std::max(plan, w.total - w.off_plan);
            }
        most = std::max(most, rest + plan);
    }
    return most;
}

// Y[L,N] = Xbar Wbar^T: contraction over K
extern "C" int metis_fp4_linear_fwd(void* stream, const metis_split* X, const metis_split* W, metis_mat* Y,
                                    void* workspace, size_t workspace_bytes) {
    if (!X || !W) return METIS_INVALID_ARG;
    return linear_nt((hipStream_t)stream, nt(X->R, X->Ut, X->Vt, X->S, X->k), nt(W->R, W->Ut, W->Vt, W->S, W->k), Y,
                     workspace, workspace_bytes);
}

// dX[L,K] = Gbar Wbar: contraction over N; Wbar^T [K,N] = Vw Sw Uw^T + Rw^T
extern "C" int metis_fp4_linear_dgrad(void* stream, const metis_split* G, const metis_split* W, metis_mat* dX,
                                      void* workspace, size_t workspace_bytes) {
    if (!G || !W) return METIS_INVALID_ARG;
    return linear_nt((hipStream_t)stream, nt(G->R, G->Ut, G->Vt, G->S, G->k), nt(W->Rt, W->Vt, W->Ut, W->S, W->k), dX,
                     workspace, workspace_bytes);
}

// dW[N,K] = Gbar^T Xbar: contraction over L; Gbar^T [N,L] = Vg Sg Ug^T + Rg^T, Xbar^T [K,L] likewise
extern "C" int metis_fp4_linear_wgrad(void* stream, const metis_split* G, const metis_split* X, metis_mat* dW,
                                      void* workspace, size_t workspace_bytes) {
    if (!G || !X) return METIS_INVALID_ARG;
    return linear_nt((hipStream_t)stream, nt(G->Rt, G->Vt, G->Ut, G->S, G->k), nt(X->Rt, X->Vt, X->Ut, X->S, X->k), dW,
                     workspace, workspace_bytes);
}

extern "C" int metis_fp4_linear_phase(void* stream, int product, int phase, const metis_split* a, const metis_split* b,
                                      metis_mat* out, void* workspace, size_t workspace_bytes) {
    if (!a || !b || phase < METIS_LINEAR_ALL || phase > METIS_LINEAR_APPLY) return METIS_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    switch (product) {
        case METIS_LINEAR_FWD:        // a = X, b = W
            return linear_nt(s, nt(a->R, a->Ut, a->Vt, a->S, a->k), nt(b->R, b->Ut, b->Vt, b->S, b->k), out, workspace,
                             workspace_bytes, phase);
        case METIS_LINEAR_DGRAD:      // a = G, b = W
            return linear_nt(s, nt(a->R, a->Ut, a->Vt, a->S, a->k), nt(b->Rt, b->Vt, b->Ut, b->S, b->k), out, workspace,
                             workspace_bytes, phase);
        case METIS_LINEAR_WGRAD:      // a = G, b = X
            return linear_nt(s, nt(a->Rt, a->Vt, a->Ut, a->S, a->k), nt(b->Rt, b->Vt, b->Ut, b->S, b->k), out, workspace,
                             workspace_bytes, phase);
        default: return METIS_INVALID_ARG;
    }
}
