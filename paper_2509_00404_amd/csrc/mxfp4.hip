// MXFP4 variant of the block-FP4 GEMM: the microscaling format that Sec. 2.3 names next to NVFP4
// (OCP MX v1.0: blocks of 32, one power-of-two E8M0 scale per block, E2M1 elements).  Its scales are
// exactly what gfx950's block-scaled matrix instruction applies in hardware, so the codes go from
// LDS straight into v_mfma_scale_f32_32x32x64_f8f6f4 with no expansion in the vector ALUs: this is
// the chip's FP4 rate, against which the NVFP4 path (E4M3 scales per 16, expanded to fp16) can be read.
#include <type_traits>
#include "common.h"
#include "gemm_tile.h"
#include "stream_dev.h"
#include "../../include/metis.h"

typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef uint32_t uvec4_t __attribute__((ext_vector_type(4)));   // a native vector: copies stay in registers
typedef uint32_t uvec2_t __attribute__((ext_vector_type(2)));

namespace {

// ---- quantizer: one lane per block of 32 consecutive elements of a row ----
// X = 2^(floor(log2 amax) - 2); elements round to the nearest E2M1 value of e / X, ties to the even code,
// magnitudes above 6 saturate (the packed converter does the rounding, saturation and nibble packing).
template <typename T>
__global__ void __launch_bounds__(256)
k_quantize_mx(const T* __restrict__ A, int64_t ld, int64_t M, int64_t nblk /* cols / 32 */, uint8_t* __restrict__ codes,
              uint8_t* __restrict__ scales) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= M * nblk) return;
    const int64_t row = t / nblk, bc = t - row * nblk;
    float v[32];
    if constexpr (sizeof(T) == 2) {
        const uint4* src = reinterpret_cast<const uint4*>(A + row * ld + bc * 32);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 a = src[i];
            const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[8 * i + 2 * j] = bf16lo_to_f32(w[j]);
                v[8 * i + 2 * j + 1] = bf16hi_to_f32(w[j]);
            }
        }
    } else {
        const float4* src = reinterpret_cast<const float4*>(A + row * ld + bc * 32);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 a = src[i];
            v[4 * i] = a.x; v[4 * i + 1] = a.y; v[4 * i + 2] = a.z; v[4 * i + 3] = a.w;
        }
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) amax = fmaxf(amax, fabsf(v[i]));
    int sh = -127;
    if (amax > 0.0f) {
        sh = ilogbf(amax) - 2;
        sh = sh < -127 ? -127 : (sh > 127 ? 127 : sh);
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float y0 = ldexpf(v[8 * i + 2 * j], -sh), y1 = ldexpf(v[8 * i + 2 * j + 1], -sh);   // exact
            switch (j) {
                case 0: w[i] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[i], y0, y1, 1.0f, 0); break;
                case 1: w[i] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[i], y0, y1, 1.0f, 1); break;
                case 2: w[i] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[i], y0, y1, 1.0f, 2); break;
                default: w[i] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[i], y0, y1, 1.0f, 3); break;
            }
        }
    }
    *reinterpret_cast<uint4*>(codes + t * 16) = make_uint4(w[0], w[1], w[2], w[3]);     // [M, cols/2] contiguous
    scales[t] = (uint8_t)(sh + 127);
}

// ---- GEMM C[M,N] = A[M,K] B[N,K]^T ----
// Large outputs of whole units of 256 go to the streaming kernel (mx_stream.h, rule at launch_mx_tile); this one takes the rest.
// 256 x 256 tile, 8 waves of 128 x 64 (4 x 2 accumulator tiles of 32 x 32, two waves per SIMD); for few tiles 128 x 128, 8 waves of 64 x
// 32 and two workgroups a CU (BT, see launch_mx_gemm).  A lane's operand of
// one matrix instruction is the 32 codes (16 bytes) of row lane % 32, contraction half lane / 32, and the E8M0 byte
// of exactly that block of 32.  With no expansion work the kernel lives on operand delivery:
//  * a stage is 256 contraction elements = 128 bytes of every row = whole cache lines (with 64-byte stages every
//    line crossed L2 -> L1 twice, which was the limit), four matrix instructions deep;
//  * the next stage's global data sits in registers for one stage before it is written to the other LDS buffer;
//  * fragments are double-buffered in registers: step s+1 is read from LDS while step s multiplies;
//  * a wave issues in order and a matrix instruction holds its pipe for 32 cycles, so memory instructions of one
//    wave leave the pipe idle while they issue: the second wave on the SIMD fills those gaps (four waves of
//    128 x 128 need fewer LDS bytes per flop but reach 10 % less);
//  * the tiles an XCD has in work share few panels of both operands (mx_order);
//  * bf16 accumulator tiles are transposed (B's fragment first): a lane then holds runs of four columns of one row, which go to whole
//    lines by way of the finished stage's LDS, 16 bytes a lane (as 2-byte stores, half a line of two rows each, a tile took 128
//    store instructions a wave instead of 16).  An fp32 row of 32 is a whole line as it is: by way of LDS 16384 x 14336 x 512 takes 197
//    us instead of 188, 6144 x 6144 x 1024 47 for 45, 4352 x 4352 x 512 23.8 for 22.5 (128 x 128 tiles, where it makes no difference,
//    use the one path).
// The stage body is branch-free (stage indices are clamped; the last stage loads and stores data nobody uses).
#define MX_KI 256
#define MX_CROW (MX_KI / 2 + 16)      // padded code row in LDS: 144 bytes, 16-byte reads of 8 consecutive rows hit 8 bank groups
#define MX_SROW 8                     // the row's eight scale bytes of a stage
#define MX_BAND 4                     // tiles side by side in a band: an XCD has 4 of B's panels and 8 of A's in work

struct MxOrder {
    TileMap regions;
    BandMap bands;                    // bands.group == 0: regions
};

struct MxOperand {
    const uint8_t* codes;             // [rows, K/2]
    const uint8_t* scales;            // [rows, K/32]
    int64_t rows;
};

// four neighbouring outputs of a row
__device__ __forceinline__ void mx_put4(bf16_t* p, float x, float y, float z, float w) {
    typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    const f2_t lo = {x, y}, hi = {z, w};
    *reinterpret_cast<uvec2_t*>(p) = uvec2_t{__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf2_t)),
                                             __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf2_t))};
}
__device__ __forceinline__ void mx_put4(float* p, float x, float y, float z, float w) {
    *reinterpret_cast<float4*>(p) = make_float4(x, y, z, w);
}

// A wave's TM x TN accumulator tiles to memory.  LINES: 32 rows of its columns at a time are staged at sm (mx_wave_rows bytes), else
// straight from the registers.  whole: the workgroup's tile is stored without looking at each element (mx_whole).
template <typename OUT, int TN>
constexpr int mx_wave_rows() { return 32 * (32 * TN * (int)sizeof(OUT) + 16); }
// A tile inside the matrix; by way of LDS C has to allow 16-byte stores too, as vec says.  (Straight from the registers it has not: asked
// for it all the same, fp32 rows off 16 bytes took 151 us for 8192 x 14336 x 512 and 353 for x 4096, 131 and 332 without.)
template <bool LINES>
__device__ __forceinline__ bool mx_whole(bool inside, bool vec) { return inside && (!LINES || vec); }
template <typename OUT, bool LINES, int TM, int TN>
__device__ __forceinline__ void mx_store_wave(const float16_t (&acc)[TM][TN], uint8_t* sm, OUT* __restrict__ C, int64_t ldc, int64_t m0,
                                              int64_t n0, int64_t M, int64_t N, bool vec, bool whole, int lane) {
    const int li = lane & 31, half = lane >> 5;
    if constexpr (!LINES) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t c = n0 + 32 * j + li;
                const int64_t rbase = m0 + 32 * i + 4 * half;
                if (whole) {
                    store_tile16<OUT>(C + rbase * ldc + c, ldc, acc[i][j], 1.0f);
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int64_t r = rbase + 8 * (v >> 2) + (v & 3);
                        if (r < M && c < N) store_out<OUT>(C + r * ldc + c, acc[i][j][v]);
                    }
                }
            }
    } else {
        constexpr int E = 16 / (int)sizeof(OUT), LROW = 32 * TN * (int)sizeof(OUT) + 16, UNITS = 32 * TN / E, ROWS = 64 / UNITS;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; v += 4)
                    mx_put4(reinterpret_cast<OUT*>(sm + li * LROW) + 32 * j + 2 * v + 4 * half, acc[i][j][v], acc[i][j][v + 1],
                            acc[i][j][v + 2], acc[i][j][v + 3]);
            gs_wave_order();
#pragma unroll
            for (int t = 0; t < 32 / ROWS; ++t) {
                const int row = ROWS * t + lane / UNITS, unit = lane % UNITS;
                const uint8_t* q = sm + row * LROW + 16 * unit;
                const uvec4_t w = *reinterpret_cast<const uvec4_t*>(q);
                const int64_t r = m0 + 32 * i + row, c = n0 + E * unit;
                OUT* p = C + r * ldc + c;
                if (whole) {
                    *reinterpret_cast<uvec4_t*>(p) = w;
                } else if (r < M) {
                    const int64_t left = N - c;
                    if (vec && left >= E) {
                        *reinterpret_cast<uvec4_t*>(p) = w;
                    } else {
#pragma unroll 1
                        for (int e = 0; e < E && e < left; ++e) p[e] = reinterpret_cast<const OUT*>(q)[e];
                    }
                }
            }
            gs_wave_order();
        }
    }
}

// MODE: MX_WHOLE for K a multiple of the 256-deep stage.  Else the last stage exists only in part, and its missing blocks of 32 enter as
// zero codes under a unit scale.  MX_TAIL: what is missing is put in on the way to LDS, where the data has arrived, so that
// nothing waits for a load when it is issued; scale rows are not 8-byte aligned and are fetched 8 bytes at a time all the same, from
// up to 7 bytes before where that would cross the operand's end.  MX_SHORT: K < 256, one stage and perhaps fewer than 8
// scale bytes in all, fetched one by one.
// (With the zeros and the scale bytes put together behind the load, in one kernel for both, 240 registers were spilled and a stage had no
// load in flight; quantizers included: 8192 x 4096 x 4064 915 -> 118 us, where 4096 takes 117; 1000 x 1008 x 1248 187 -> 20.6.)
typedef uint32_t mx_uvec2_any __attribute__((ext_vector_type(2), aligned(1)));
enum { MX_WHOLE, MX_TAIL, MX_SHORT };
template <typename OUT, int MODE, int BT>
__global__ void __launch_bounds__(512, BT == 256 ? 2 : 4)
k_mxfp4_gemm_nt(MxOperand A, MxOperand B, int64_t K, OUT* __restrict__ C, int64_t ldc, bool vec, MxOrder order) {
    constexpr bool LINES = sizeof(OUT) == 2 || BT == 128;              // outputs by way of LDS, accumulator tiles transposed
    constexpr int TM = BT / 64, TN = BT / 128, BM = BT, BN = BT, NV = BT / 64;   // NV: 16-byte code vectors per thread, operand and stage
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int OFF_CB = BM * MX_CROW, OFF_SA = (BM + BN) * MX_CROW, OFF_SB = OFF_SA + BM * MX_SROW,
                  BUF = OFF_SB + BN * MX_SROW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int tile_m, tile_n;
    if (order.bands.group > 0) tile_coords(order.bands, tile_m, tile_n);
    else tile_coords(order.regions, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int wm = (wave >> 2) * (BT / 2), wn = (wave & 3) * (BT / 4);
    const int li = lane & 31, half = lane >> 5;

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int niter = (int)((K + MX_KI - 1) / MX_KI);
    // this thread's share of a stage: code vectors v of each operand (row tid/8 + 64 v, 16-byte segment
    // tid % 8: a row's 128 bytes are read by 8 consecutive lanes) and the 8 scale bytes of one row;
    // rows past the operand's end re-read its last row.  Byte offsets fit 32 bits (checked by the host).
    uint32_t oa[NV], ob[NV], osga, osgb;
    const uint32_t cstride = (uint32_t)(K / 2), sstride = (uint32_t)(K / 32);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        int64_t ga = m0 + (tid >> 3) + 64 * v, gb = n0 + (tid >> 3) + 64 * v;
        if (ga >= A.rows) ga = A.rows - 1;
        if (gb >= B.rows) gb = B.rows - 1;
        oa[v] = (uint32_t)ga * cstride + 16u * (tid & 7);
        ob[v] = (uint32_t)gb * cstride + 16u * (tid & 7);
    }
    {
        int64_t ga = m0 + (tid & (BT - 1)), gb = n0 + (tid & (BT - 1));
        if (ga >= A.rows) ga = A.rows - 1;
        if (gb >= B.rows) gb = B.rows - 1;
        osga = (uint32_t)ga * sstride;
        osgb = (uint32_t)gb * sstride;
    }
    // the first BT threads carry A's scale rows, the next BT B's (and with BT = 128 the other half the same once more)
    const int srow = tid & (2 * BT - 1);
    const bool sc_a = srow < BT;
    uvec4_t ra[NV], rb[NV];
    uvec2_t rs;
    auto clampst = [&](int st) { return st < niter ? st : niter - 1; };
    auto seg_exists = [&](int st) __attribute__((always_inline)) { return 8u * st + (tid & 7) < sstride; };
    // where the 8 scale bytes are fetched (K > 256: an operand has more than 8)
    const uint32_t slast = (uint32_t)(sc_a ? A.rows : B.rows) * sstride - 8u;
    auto scale_offset = [&](int st) __attribute__((always_inline)) {
        const uint32_t o = (sc_a ? osga : osgb) + 8u * st;
        return o < slast ? o : slast;
    };
    auto load_stage = [&](int st) __attribute__((always_inline)) {
        const uint8_t* ca = A.codes + (size_t)st * (MX_KI / 2);
        const uint8_t* cb = B.codes + (size_t)st * (MX_KI / 2);
        if (MODE == MX_WHOLE) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                ra[v] = *reinterpret_cast<const uvec4_t*>(ca + oa[v]);
                rb[v] = *reinterpret_cast<const uvec4_t*>(cb + ob[v]);
            }
            rs = *reinterpret_cast<const uvec2_t*>((sc_a ? A.scales + osga : B.scales + osgb) + (size_t)st * (MX_KI / 32));
        } else {
            // this lane's 16-byte segment is one block of 32 contraction elements: if it does not exist the row's first is read
            const uint32_t d = seg_exists(st) ? (uint32_t)st * (MX_KI / 2) : 0u - 16u * (tid & 7);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                ra[v] = *reinterpret_cast<const uvec4_t*>(A.codes + (uint32_t)(oa[v] + d));
                rb[v] = *reinterpret_cast<const uvec4_t*>(B.codes + (uint32_t)(ob[v] + d));
            }
            const uint8_t* sp = sc_a ? A.scales : B.scales;
            if (MODE == MX_TAIL) {
                rs = *reinterpret_cast<const mx_uvec2_any*>(sp + scale_offset(st));
            } else {
                const uint32_t o = sc_a ? osga : osgb;
                uint32_t w[2] = {0u, 0u};
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i >> 2] |= (uint32_t)sp[o + (i < (int)sstride ? i : 0)] << (8 * (i & 3));
                rs.x = w[0];
                rs.y = w[1];
            }
        }
    };
    auto store_stage = [&](uint8_t* buf, int st) __attribute__((always_inline)) {       // st: the stage that the registers hold
        if (MODE != MX_WHOLE) {
            const bool ok = seg_exists(st);
            const uvec4_t zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                ra[v] = ok ? ra[v] : zero4;
                rb[v] = ok ? rb[v] : zero4;
            }
            uint64_t w = (uint64_t)rs.y << 32 | rs.x;
            if (MODE == MX_TAIL) w >>= 8 * ((sc_a ? osga : osgb) + 8u * st - scale_offset(st));
            const int have = (int)sstride - 8 * st;                                     // >= 1; 127 = scale 1 for an absent block
            const uint64_t absent = have < 8 ? ~0ull << (8 * have) : 0ull;
            w = (w & ~absent) | (0x7F7F7F7F7F7F7F7Full & absent);
            rs.x = (uint32_t)w;
            rs.y = (uint32_t)(w >> 32);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int row = (tid >> 3) + 64 * v, seg = tid & 7;
            *reinterpret_cast<uvec4_t*>(buf + row * MX_CROW + 16 * seg) = ra[v];
            *reinterpret_cast<uvec4_t*>(buf + OFF_CB + row * MX_CROW + 16 * seg) = rb[v];
        }
        *reinterpret_cast<uvec2_t*>(buf + OFF_SA + srow * MX_SROW) = rs;          // B's scale rows follow A's
    };

    // per-lane byte offsets of this wave's fragment rows inside a buffer
    const int oca = (wm + li) * MX_CROW + 16 * half, ocb = OFF_CB + (wn + li) * MX_CROW + 16 * half;
    const int osa = OFF_SA + (wm + li) * MX_SROW, osb = OFF_SB + (wn + li) * MX_SROW;
    uvec4_t fa[2][TM], fb[2][TN];     // code fragments, two slots
    uint32_t sa[2][TM], sb[2][TN];    // the rows' two scale words of the stage, shifted so that byte 0 / byte 2 are this lane's blocks
    auto read_codes = [&](const uint8_t* buf, int ks, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[slot][i] = *reinterpret_cast<const uvec4_t*>(buf + oca + 32 * i * MX_CROW + 32 * ks);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[slot][j] = *reinterpret_cast<const uvec4_t*>(buf + ocb + 32 * j * MX_CROW + 32 * ks);
    };
    auto read_scales = [&](const uint8_t* buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uvec2_t w = *reinterpret_cast<const uvec2_t*>(buf + osa + 32 * i * MX_SROW);
            sa[0][i] = w.x >> (8 * half);
            sa[1][i] = w.y >> (8 * half);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const uvec2_t w = *reinterpret_cast<const uvec2_t*>(buf + osb + 32 * j * MX_SROW);
            sb[0][j] = w.x >> (8 * half);
            sb[1][j] = w.y >> (8 * half);
        }
    };
    auto mma = [&](auto KSC) __attribute__((always_inline)) {
        constexpr int ks = decltype(KSC)::value, slot = ks & 1, word = ks >> 1, sel = 2 * (ks & 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int8v_t a = {(int)fa[slot][i].x, (int)fa[slot][i].y, (int)fa[slot][i].z, (int)fa[slot][i].w, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int8v_t b = {(int)fb[slot][j].x, (int)fb[slot][j].y, (int)fb[slot][j].z, (int)fb[slot][j].w, 0, 0, 0, 0};
                // formats 4 = FP4 (E2M1) for both operands; the scale byte is byte `sel` of the shifted word
                if constexpr (LINES)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b, a, acc[i][j], 4, 4, sel, (int)sb[word][j],
                                                                                 sel, (int)sa[word][i]);
                else
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 4, 4, sel, (int)sa[word][i],
                                                                                 sel, (int)sb[word][j]);
            }
        }
    };

    load_stage(0);
    store_stage(lds, 0);
    __syncthreads();
    load_stage(clampst(1));
    read_codes(lds, 0, 0);
    read_scales(lds);

#pragma unroll 1
    for (int it = 0; it < niter; ++it) {
        const uint8_t* bufc = lds + (it & 1) * BUF;
        uint8_t* bufn = lds + ((it & 1) ^ 1) * BUF;
        read_codes(bufc, 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(std::integral_constant<int, 0>{});
        store_stage(bufn, clampst(it + 1));                        // stage it + 1 (loaded one stage ago) to the other buffer ...
        load_stage(clampst(it + 2));              // ... and its registers take stage it + 2
        __builtin_amdgcn_sched_barrier(0);
        read_codes(bufc, 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        mma(std::integral_constant<int, 1>{});
        __builtin_amdgcn_sched_barrier(0);
        read_codes(bufc, 3, 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(std::integral_constant<int, 2>{});
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();                          // next stage is in LDS; this stage's codes are all in registers
        read_codes(bufn, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        mma(std::integral_constant<int, 3>{});
        __builtin_amdgcn_sched_barrier(0);
        read_scales(bufn);
    }

    if constexpr (LINES) static_assert(8 * mx_wave_rows<OUT, TN>() <= BUF, "the staged rows fit one buffer");
    // The last stage's buffer is free: its codes and scales were in registers before the last meeting, and that stage stored to the
    // other one.
    const bool inside = m0 + BM <= A.rows && n0 + BN <= B.rows;
    mx_store_wave<OUT, LINES, TM, TN>(acc, lds + ((niter - 1) & 1) * BUF + wave * mx_wave_rows<OUT, TN>(), C, ldc, m0 + wm, n0 + wn, A.rows,
                                      B.rows, vec, mx_whole<LINES>(inside, vec), lane);
}

#include "mx_stream.h"

// Regions or bands.  An XCD's tiles in work should share few panels: a region near square sees to that and writes longer runs of
// C's rows, which counts while a tile's contraction is short; bands see to it whatever the grid, and over many tiles of a long contraction
// share better than a wide region walked by rows.  Multiplication alone, us, regions / bands: 16384 x 14336 x 4096 597 / 569, x 2048
// 329 / 313, x 1056 255 / 241, x 1024 fp32 256 / 260, x 512 fp32 196 / 205; 8192 x 14336 x 512 fp32 100 / 107; 16384 x 4096 x 512
// 39.0 / 40.9, x 4096 162 / 160; no region (8448 x 8448 x 2048) 112 / 100; one of 47 x 7 (12000 x 14336 x 4096) 438 / 432.  128 x 128
// tiles are all in work at once: regions where there are any, 512 x 7168 x 4096 15.6 / 17.3, 2048 x 3584 x 14336 95.9 / 97.6.
MxOrder mx_order(int64_t tiles_m, int64_t tiles_n, int64_t K, int bt) {
    MxOrder o = {make_tile_map(tiles_m, tiles_n), {0, 0, 0}};
    const int rm = o.regions.rm, rn = o.regions.rn;
    const bool near_square = rm > 0 && rm <= 4 * rn && rn <= 4 * rm;
    if (bt == 256 ? !near_square || (K > 1024 && tiles_m * tiles_n >= 1536) : rm == 0) o.bands = make_band_map(tiles_m, tiles_n, MX_BAND);
    return o;
}

template <typename OUT, int BT>
int launch_mx_tile(hipStream_t s, const MxOperand& a, const MxOperand& b, int64_t K, OUT* C, int64_t ldc) {
    constexpr size_t LDS = 2 * (size_t)(2 * BT) * (MX_CROW + MX_SROW);
    const int64_t tm = ceil_div64(a.rows, BT), tn = ceil_div64(b.rows, BT);
    if (tm * tn > 0x7FFFFFFF) return METIS_UNSUPPORTED;
    const MxOrder order = mx_order(tm, tn, K, BT);
    const bool vec = (uintptr_t)C % 16 == 0 && (ldc * sizeof(OUT)) % 16 == 0;
    auto launch = [&](auto kern, LdsLimitCache& lds_set) {
        if (!ensure_dyn_lds((const void*)kern, LDS, lds_set)) return false;
        hipLaunchKernelGGL(kern, dim3((unsigned)(tm * tn)), dim3(512), LDS, s, a, b, K, C, ldc, vec, order);
        return true;
    };
    // The streaming kernel: whole units, two at least (its transfers are two ahead of the products), and several tiles a CU or a long
    // contraction.  A lone tile a CU gains nothing from a stream that crosses tiles: us, the kernel above / streaming, 4096 x 4096 x
    // 512 13.0 / 13.2, x 1024 15.4 / 15.7, x 4096 (with quantizers) 56.6 / 55.9; 4352 x 4352 x 512 17.7 / 17.0, 8192 x 8192 x 512 39.6 / 35.5.
    const int cus = device_cu_count();
    if (cus < 1) return METIS_HIP_ERROR;
    if (BT == 256 && K % MX_KI == 0 && K >= 2 * MX_KI && (tm * tn > cus || K >= 8 * MX_KI)) {
        auto kern = k_mxfp4_gemm_nt_stream<OUT>;
        static LdsLimitCache stream_set;
        if (!ensure_dyn_lds((const void*)kern, MXS_LDS, stream_set)) return METIS_HIP_ERROR;
        hipLaunchKernelGGL(kern, dim3((unsigned)(tm * tn < cus ? tm * tn : cus)), dim3(512), MXS_LDS, s, a, b, K, C, ldc, vec, order,
                           (int)(tm * tn));
        METIS_LAUNCH_CHECK();
        return METIS_OK;
    }
    static LdsLimitCache lds_set[3];
    const bool ok = K % MX_KI == 0 ? launch(k_mxfp4_gemm_nt<OUT, MX_WHOLE, BT>, lds_set[0])
                    : K > MX_KI    ? launch(k_mxfp4_gemm_nt<OUT, MX_TAIL, BT>, lds_set[1])
                                   : launch(k_mxfp4_gemm_nt<OUT, MX_SHORT, BT>, lds_set[2]);
    if (!ok) return METIS_HIP_ERROR;
    METIS_LAUNCH_CHECK();
    return METIS_OK;
}

// 128 x 128 tiles while two workgroups a CU hold them all, with an eighth of the places to spare: the chip is fuller and a stage
// shorter.  With the quantizers, against 256 x 256 tiles, K = 4096: 27 of them 37.1 -> 22.6 us, 128 41.4 -> 26.6, 256 41.0 -> 27.0, 384
// 43.1 -> 40.1.  448, multiplication alone: K = 4096 32.3 -> 30.4, 14336 96.1 -> 95.9.  With the quantizers, 512 would take 44.6 for 45.1
// at K = 4096 but 139.1 for 137.6 at K = 14336, 640 57.5 for 47.2.
template <typename OUT>
int launch_mx_gemm(hipStream_t s, const MxOperand& a, const MxOperand& b, int64_t K, OUT* C, int64_t ldc) {
    const int cus = device_cu_count();
    if (cus < 1) return METIS_HIP_ERROR;
    if (ceil_div64(a.rows, 128) * ceil_div64(b.rows, 128) <= 7 * (int64_t)cus / 4) return launch_mx_tile<OUT, 128>(s, a, b, K, C, ldc);
    return launch_mx_tile<OUT, 256>(s, a, b, K, C, ldc);
}

bool mx_ok(const metis_mxfp4* t) { return t && t->codes && t->scales && t->rows >= 1 && t->cols >= 32 && t->cols % 32 == 0; }

}  // namespace

extern "C" int metis_quantize_mx(void* stream, const metis_mat* A, metis_mxfp4* out) {
    if (!A || !A->ptr || !mx_ok(out)) return METIS_INVALID_ARG;
    if (A->dtype != METIS_BF16 && A->dtype != METIS_F32) return METIS_INVALID_ARG;
    if (A->rows != out->rows || A->cols != out->cols || A->ld < A->cols) return METIS_BAD_SHAPE;
    const int64_t esz = A->dtype == METIS_BF16 ? 2 : 4;
    if ((A->ld * esz) % 16 || reinterpret_cast<uintptr_t>(A->ptr) % 16 || reinterpret_cast<uintptr_t>(out->codes) % 16)
        return METIS_BAD_SHAPE;                                       // 16-byte row loads and code stores
    const int64_t nblk = A->cols / 32, total = A->rows * nblk;
    hipStream_t s = (hipStream_t)stream;
    if (A->dtype == METIS_BF16)
        hipLaunchKernelGGL(k_quantize_mx<bf16_t>, dim3((unsigned)ceil_div64(total, 256)), dim3(256), 0, s,
                           (const bf16_t*)A->ptr, A->ld, A->rows, nblk, out->codes, out->scales);
    else
        hipLaunchKernelGGL(k_quantize_mx<float>, dim3((unsigned)ceil_div64(total, 256)), dim3(256), 0, s,
                           (const float*)A->ptr, A->ld, A->rows, nblk, out->codes, out->scales);
    METIS_LAUNCH_CHECK();
    return METIS_OK;
}

extern "C" int metis_mxfp4_gemm_nt(void* stream, const metis_mxfp4* A, const metis_mxfp4* B, metis_mat* C) {
    if (!mx_ok(A) || !mx_ok(B) || !C || !C->ptr) return METIS_INVALID_ARG;
    if (C->dtype != METIS_BF16 && C->dtype != METIS_F32) return METIS_INVALID_ARG;
    if (A->cols != B->cols || C->rows != A->rows || C->cols != B->rows || C->ld < C->cols) return METIS_BAD_SHAPE;
    const int64_t K = A->cols;
    if (A->rows * (K / 2) > 0xFFFFFFFFll || B->rows * (K / 2) > 0xFFFFFFFFll) return METIS_UNSUPPORTED;   // 32-bit byte offsets
    if (reinterpret_cast<uintptr_t>(A->codes) % 16 || reinterpret_cast<uintptr_t>(B->codes) % 16 ||
        (K % MX_KI == 0 && (reinterpret_cast<uintptr_t>(A->scales) % 8 || reinterpret_cast<uintptr_t>(B->scales) % 8)))
        return METIS_BAD_SHAPE;
    const MxOperand a = {A->codes, A->scales, A->rows}, b = {B->codes, B->scales, B->rows};
    hipStream_t s = (hipStream_t)stream;
    if (C->dtype == METIS_F32) return launch_mx_gemm<float>(s, a, b, K, (float*)C->ptr, C->ld);
    return launch_mx_gemm<bf16_t>(s, a, b, K, (bf16_t*)C->ptr, C->ld);
}
