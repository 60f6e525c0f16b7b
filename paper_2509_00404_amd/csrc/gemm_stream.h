// The main FP4 GEMM kernel for large outputs (included by gemm.hip, inside its namespace).
#pragma once

typedef uint32_t gs_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t gs_u32x2 __attribute__((ext_vector_type(2)));
typedef float gs_acc_t __attribute__((ext_vector_type(4)));

// acc += X Y^T, 16 x 16 over 32 columns, the accumulator in place in the accumulation registers (left to itself the compiler keeps
// it in vector registers, moves it about and runs out of them; the instruction is also 40 % slower on those: 3375 cycles
// against 2060 for 64 x 2).  The hazards that the compiler then does not see: X or Y written by a vector instruction
// fewer than two instructions before (the expansions are at least three matrix instructions ahead), and an accumulator written
// by a vector instruction just before or read by one soon after (gs_settle).
__device__ __forceinline__ void gs_mfma_f16(gs_acc_t& acc, const gs_u32x4& x, const gs_u32x4& y) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(x), "v"(y));
}
__device__ __forceinline__ void gs_mfma_bf16(gs_acc_t& acc, const gs_u32x4& x, const gs_u32x4& y) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(x), "v"(y));
}
// Two codes (byte K of the word) to fp16, and their block's scale (the pair's upper or lower half) onto them.  In asm for their
// place alone: the order of the volatile ones is the order of the source, and the matrix instructions between them are what hides
// them (as ordinary code they sink to just before their use).  A conversion's result may not be read by the very next
// vector instruction: in the source another one always lies between.
template <int K>
__device__ __forceinline__ uint32_t gs_convert(uint32_t w) {
    uint32_t d;
    if constexpr (K == 0) asm volatile("v_cvt_scalef32_pk_f16_fp4 %0, %1, 1.0" : "=v"(d) : "v"(w));
    if constexpr (K == 1) asm volatile("v_cvt_scalef32_pk_f16_fp4 %0, %1, 1.0 op_sel:[1,0,0]" : "=v"(d) : "v"(w));
    if constexpr (K == 2) asm volatile("v_cvt_scalef32_pk_f16_fp4 %0, %1, 1.0 op_sel:[0,1,0]" : "=v"(d) : "v"(w));
    if constexpr (K == 3) asm volatile("v_cvt_scalef32_pk_f16_fp4 %0, %1, 1.0 op_sel:[1,1,0]" : "=v"(d) : "v"(w));
    return d;
}
template <bool HI>
__device__ __forceinline__ uint32_t gs_scale(uint32_t v, uint32_t pair) {
    uint32_t d;
    if constexpr (HI) asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel:[0,1]" : "=v"(d) : "v"(v), "v"(pair));
    else asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(d) : "v"(v), "v"(pair));
    return d;
}
template <int N>
__device__ __forceinline__ void gs_settle(gs_acc_t (&a)[8]) {
    asm volatile("s_nop %8\n\ts_nop %8" : "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3]), "+a"(a[4]), "+a"(a[5]), "+a"(a[6]), "+a"(a[7])
                 : "n"(N));
}
// LDS: four buffers of one unit: the codes of A's and of B's 256 rows, 128 elements each, then the block scales of both as
// k_scale_plan lays them out.  The stores use the buffer of the unit just finished.
#define GS_BAND 4                                        // tiles side by side that an XCD has in work, see make_band_map
#define GS_CODES 16384
#define GS_UNIT (2 * GS_CODES + 2 * GS_SCALES)
#define GS_LDS (4 * GS_UNIT)

// A wave's 16 x 16 accumulator tiles, transposed (lane l: row l % 16, element v: column 4 (l / 16) + v), to row-major memory by
// way of 2 KiB of LDS, 128 bytes of 16 rows at a time, so that a store instruction writes eight whole lines.
template <typename OUT> struct GsStage;
template <> struct GsStage<bf16_t> {
    static constexpr int TILES = 4;                      // tiles side by side in 128 bytes
    __device__ static __forceinline__ void put(uint8_t* sm, int row, int kg, int z, const gs_acc_t& a, float alpha) {
        typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
        typedef float f2_t __attribute__((ext_vector_type(2)));
        const f2_t x = {alpha * a[0], alpha * a[1]}, y = {alpha * a[2], alpha * a[3]};
        const gs_u32x2 w = {__builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf2_t)),
                            __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf2_t))};
        *reinterpret_cast<gs_u32x2*>(sm + row * 128 + (((2 * z + (kg >> 1)) ^ (row >> 1)) * 16) + 8 * (kg & 1)) = w;
    }
};
template <> struct GsStage<float> {
    static constexpr int TILES = 2;
    __device__ static __forceinline__ void put(uint8_t* sm, int row, int kg, int z, const gs_acc_t& a, float alpha) {
        const float4 w = make_float4(alpha * a[0], alpha * a[1], alpha * a[2], alpha * a[3]);
        *reinterpret_cast<float4*>(sm + row * 128 + (((4 * z + kg) ^ (row >> 1)) * 16)) = w;
    }
};
// the 16 staged rows to C (first row r0, first column c0); whole: inside the matrix and 16-byte aligned
template <typename OUT>
__device__ __forceinline__ void gs_store_rows(const uint8_t* sm, OUT* C, int64_t ldc, int64_t r0, int64_t c0, int64_t M, int64_t N,
                                              bool whole, bool vec, int lane) {
    constexpr int E = 16 / (int)sizeof(OUT);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int row = 8 * it + (lane >> 3), unit = lane & 7;
        const uint8_t* q = sm + row * 128 + ((unit ^ (row >> 1)) * 16);
        const gs_u32x4 w = *reinterpret_cast<const gs_u32x4*>(q);
        // (uniform part and the lane's 32-bit offset apart)
        OUT* p = reinterpret_cast<OUT*>(reinterpret_cast<uint8_t*>(C + (r0 + 8 * it) * ldc + c0) +
                                        ((uint32_t)(lane >> 3) * (uint32_t)ldc + (uint32_t)(E * unit)) * (uint32_t)sizeof(OUT));
        if (whole) {
            *reinterpret_cast<gs_u32x4*>(p) = w;
        } else if (r0 + row < M) {
            const int64_t left = N - (c0 + E * unit);
            if (vec && left >= E) {
                *reinterpret_cast<gs_u32x4*>(p) = w;
            } else {
#pragma unroll 1
                for (int e = 0; e < E && e < left; ++e) p[e] = reinterpret_cast<const OUT*>(q)[e];
            }
        }
    }
}
template <typename OUT>
__device__ __forceinline__ void gs_store_tile(uint8_t* sm, const gs_acc_t (&acc)[8][8], float alpha, OUT* C, int64_t ldc, int64_t r0,
                                              int64_t c0, int64_t M, int64_t N, bool whole, bool vec, int lane) {
    // (16 rows are staged while the 16 before travel through the other half)
    constexpr int Z = GsStage<OUT>::TILES, CT = 8 / Z, CHUNKS = 8 * CT;
    const int row = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int z = 0; z < Z; ++z) GsStage<OUT>::put(sm, row, kg, z, acc[0][z], alpha);
    gs_wave_order();
#pragma unroll
    for (int q = 0; q < CHUNKS; ++q) {
        const int n = q + 1;
        if (n < CHUNKS) {
#pragma unroll
            for (int z = 0; z < Z; ++z) GsStage<OUT>::put(sm + (n & 1) * 2048, row, kg, z, acc[n / CT][(n % CT) * Z + z], alpha);
        }
        gs_store_rows<OUT>(sm + (q & 1) * 2048, C, ldc, r0 + 16 * (q / CT), c0 + 16 * Z * (q % CT), M, N, whole, vec, lane);
        gs_wave_order();                                 // both for the rows staged above and for the half just read
    }
}

// C = alpha deq(A) deq(B)^T + Aext Bext^T in 256 x 256 tiles, 4 waves of 128 x 128, one per SIMD.
// What bounds it: the issue of a lone wave per SIMD.  64 contraction elements of a tile are 128 matrix instructions of 16 cycles
// and 256 expansion instructions a wave; in the order M V V they take 2227 cycles where the matrix instructions alone take
// 2060 (a register loop of the same), with the reads of the codes 2311, with the transfers 2544 (a transfer costs the wave ~45
// cycles, whatever its place), and a tile's 4 units of extra columns, its stores and its start another 17000: 180500 cycles
// for K = 4096 + 128 against a matrix core's 135200.  (With all that is below, by the counter of wave cycles over products of 4096
// and 14336 elements at rank 64 on both sides: 2486 for 64 elements, 28600 for the rest of a tile.  57 of a unit's 920 instructions
// are s_nops that the compiler puts between a matrix instruction and a multiplication of two asm statements.)  Why so:
//  * 16 x 16 x 32 matrix instructions, not 32 x 32 x 16: an accumulator is read and written half as often, and in long runs,
//    where the card holds its power and not its clock, the same loop on random codes runs at 1.97 PFLOP/s instead of 1.78;
//  * accumulators in the accumulation registers, everything that is ordered in volatile asm (above);
//  * transfers straight into LDS, three units (of 128) ahead through four buffers, one meeting of the workgroup per unit: no
//    registers, and the wait for memory is gone from the loop.  The units of a workgroup's tiles are one stream: the next tile's
//    first ones travel while this tile's last are multiplied, and its first step is expanded there too;
//  * the block scales ready in fp16 and in order (k_scale_plan);
//  * both operands' codes expanded in the loop.  The smaller operand expanded ahead to fp16 (half the expansions, 8 waves of
//    128 x 64) is no faster: its panel is four times the bytes to move through L2 and LDS, 2680 cycles, and the expansion ahead
//    costs 8 to 30 us a product.
// Where it stands against the pipelined kernel it took these products from (fp32 partial sums in the same order, so mostly the same
// bits), alone: 16384 x 4096 x 4096 430 -> 372 us, 16384 x 14336 x 4096 1505 -> 1270, 16384 x 4096 x 14336 1386 -> 1210, 2048 x 14336 x
// 4096 200 -> 179.  (What was tried before: M V V with the expansions as ordinary code, which the compiler sinks to where they are
// used, 3215 cycles; the block scales fetched from the rows; a wave-dependent delay behind the meeting, no effect.)
// The tiles of a last round that fills few CUs are cut along the contraction (tail_first, tail_parts), as there.
template <typename OUT>
__global__ void __launch_bounds__(256)
k_fp4_gemm_nt_stream(Fp4Operand A, Fp4Operand B, int64_t K, const uint8_t* __restrict__ Aplan,
                     const uint8_t* __restrict__ Bplan, const bf16_t* __restrict__ Aext, const bf16_t* __restrict__ Bext,
                     int Ke_all, float alpha, OUT* __restrict__ C, int64_t ldc, bool vec, BandMap tmap, int total_tiles,
                     int tail_first, int tail_parts, float* __restrict__ partial, int total_items) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int niter_all = (int)(K / G_KI), e_all = Ke_all >> 5;
    const uint32_t cstride = (uint32_t)(K / 2);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wa = wave >> 1, wb = wave & 1;
    constexpr int STORES = 64 / GsStage<OUT>::TILES * 2;

    // what a launch position stands for: a tile, or a part of one
    struct Item {
        int m0, n0, it_begin, niter, e;      // first row and column, units of 128, units of 32 extra columns
        int cut;                             // < 0: a whole tile, else the index of its partial tile
    };
    auto item_of = [&](int pos) GS_INLINE {
        Item w;
        int tile = pos, part = 0, parts = 1;
        w.cut = -1;
        // (opaque: else the reciprocals of these divisions are kept in registers through the whole kernel)
        BandMap map = tmap;
        int cuts = tail_parts;
        asm volatile("" : "+s"(map.tiles_m), "+s"(map.tiles_n), "+s"(cuts));
        if (tile >= tail_first) {
            w.cut = tile - tail_first;
            const int t = w.cut / cuts;
            tile = tail_first + t;
            part = w.cut - t * cuts;
            parts = cuts;
        }
        int tile_m, tile_n;
        tile_coords_of(map, tile, total_tiles, tile_m, tile_n);
        w.m0 = tile_m * 256;
        w.n0 = tile_n * 256;
        w.it_begin = part * niter_all / parts;
        w.niter = (part + 1) * niter_all / parts - w.it_begin;
        w.e = part == 0 ? e_all : 0;
        return w;
    };

    const int lane = (int)threadIdx.x & 63;
    const uint32_t vlane = 16u * (uint32_t)lane;

    // ---- transfers.  The units of a workgroup's tiles form one stream, fetched three units ahead of the products
    const uint8_t *qa, *qb, *qsa, *qsb;      // the next unit's codes and scales, or extra columns
    int lpos = (int)blockIdx.x, lcnt, lext, lm, ln;   // item being fetched; units left, extra-column units behind them (< 0: these are they)
    int qstep, sstep;                        // from unit to unit
    uint32_t va[4], vb[4];                   // the lane's offsets
    auto enter = [&]() GS_INLINE {
        const Item w = item_of(lpos < total_items ? lpos : total_items - 1);   // (past the end: fetched again, unused)
        lm = w.m0;
        ln = w.n0;
        lcnt = w.niter;
        lext = w.e;
        qstep = 64;
        sstep = GS_SCALES;
        qa = A.codes + (int64_t)lm * cstride + (int64_t)w.it_begin * 64;
        qb = B.codes + (int64_t)ln * cstride + (int64_t)w.it_begin * 64;
        qsa = Aplan + ((int64_t)(lm / 256) * niter_all + w.it_begin) * GS_SCALES + 1024 * wave;
        qsb = Bplan + ((int64_t)(ln / 256) * niter_all + w.it_begin) * GS_SCALES + 1024 * wave;
        const int ta = (int)(A.rows - lm < 256 ? A.rows - lm : 256) - 1, tb = (int)(B.rows - ln < 256 ? B.rows - ln : 256) - 1;
        const int l = gs_fresh_lane();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 64 * wave + 16 * v + (l & 15);
            va[v] = (uint32_t)(row < ta ? row : ta) * cstride + (uint32_t)(l >> 4) * 16;
            vb[v] = (uint32_t)(row < tb ? row : tb) * cstride + (uint32_t)(l >> 4) * 16;
        }
    };
    // extra columns: a wave brings two 32-row blocks of each operand as 1 KiB chunks [column group of 8][row of 16][8]
    auto enter_ext = [&]() GS_INLINE {
        const int am = (int)((A.rows + 31) / 32) - 1, bm = (int)((B.rows + 31) / 32) - 1;
        const int l = gs_fresh_lane();
        const uint32_t vx = (uint32_t)(((l >> 5) * 1024) + ((l >> 4) & 1) * 512 + 16 * (l & 15));
        qa = (const uint8_t*)Aext;
        qb = (const uint8_t*)Bext;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int ra = lm / 32 + 2 * wave + (v >> 1), rb = ln / 32 + 2 * wave + (v >> 1);
            if (ra > am) ra = am;
            if (rb > bm) rb = bm;
            va[v] = (uint32_t)((v & 1) * 256) + vx;
            vb[v] = va[v];
            // (a block's columns lie together; 64-bit base for the first block, the second one's distance in the offset)
            if (v == 0) {
                qa += (int64_t)ra * e_all * 2048;
                qb += (int64_t)rb * e_all * 2048;
            } else if (v >= 2) {
                const int r2a = lm / 32 + 2 * wave < am ? lm / 32 + 2 * wave : am, r2b = ln / 32 + 2 * wave < bm ? ln / 32 + 2 * wave : bm;
                va[v] += (uint32_t)((ra - r2a) * e_all * 2048);
                vb[v] += (uint32_t)((rb - r2b) * e_all * 2048);
            }
        }
        lcnt = lext;
        lext = -1;
        qstep = 2048;
        sstep = 0;
        qsa -= GS_SCALES;
        qsb -= GS_SCALES;
    };
    // before the first transfer of a unit
    auto advance = [&]() GS_INLINE {
        if (lcnt == 0) {
            if (lext > 0) {
                enter_ext();
            } else {
                lpos += (int)gridDim.x;
                enter();
            }
        }
        --lcnt;
        qa = gs_uniform(qa);
        qb = gs_uniform(qb);
        qsa = gs_uniform(qsa);
        qsb = gs_uniform(qsb);
    };
    // transfer k (0 .. 9) of the next unit into buffer `buf` (extra columns have no scales: 8 and 9 bring those of the unit before
    // again, unused, where leaving them out would cost a branch)
    auto issue = [&](uint32_t buf, auto kc) GS_INLINE {
        constexpr int k = decltype(kc)::value;
        const uint32_t dc = lds0 + buf + 4096u * wave, ds = lds0 + buf + 1024u * wave;
        if constexpr (k < 4) gs_dma16<1024 * k>(dc, va[k], qa);
        else if constexpr (k < 8) gs_dma16<GS_CODES + 1024 * (k - 4)>(dc, vb[k - 4], qb);
        else if constexpr (k == 8) gs_dma16<2 * GS_CODES>(ds, vlane, qsa);
        else gs_dma16<2 * GS_CODES + GS_SCALES>(ds, vlane, qsb);
        if constexpr (k == 7) {
            qa += qstep;
            qb += qstep;
        }
        if constexpr (k == 9) {
            qsa += sstep;
            qsb += sstep;
        }
    };

    int pos = (int)blockIdx.x;
    if (pos >= total_items) return;
    uint32_t b0 = 0;                          // buffer of the unit in work; the next ones follow cyclically
    auto buf = [&](uint32_t ahead) GS_INLINE { uint32_t x = b0 + ahead * GS_UNIT; return x >= 4 * GS_UNIT ? x - 4 * GS_UNIT : x; };
    enter();
    advance();
    gs_for<10>([&](auto k) GS_INLINE { issue(0, k); });
    advance();
    gs_for<10>([&](auto k) GS_INLINE { issue(GS_UNIT, k); });
    advance();
    gs_for<10>([&](auto k) GS_INLINE { issue(2 * GS_UNIT, k); });

    gs_acc_t acc[8][8];
    // fragments 0 .. 7: the wave's 128 rows of A, 8 .. 15: of B
    gs_u32x4 f[2][16], raw[16], sc[4];       // sc: block scales of fragments 4 x .. 4 x + 3, a pair each
    const uint32_t ra0 = wa * 8192 + vlane, rb0 = GS_CODES + wb * 8192 + vlane;
    const uint32_t sa0 = 2 * GS_CODES + wa * 2048 + vlane, sb0 = 2 * GS_CODES + GS_SCALES + wb * 2048 + vlane;
    auto read_raw = [&](uint32_t bu, int i) GS_INLINE {
        raw[i] = *reinterpret_cast<const gs_u32x4*>(lds + bu + (i < 8 ? ra0 : rb0) + (i & 7) * 1024);
    };
    auto read_sc = [&](uint32_t bu, int x) GS_INLINE {
        sc[x] = *reinterpret_cast<const gs_u32x4*>(lds + bu + (x < 2 ? sa0 : sb0) + (x & 1) * 1024);
    };
    // two codes (pair k of 4) of fragment i for step s: the conversion, then the multiplication by the block's scale
    auto convert = [&](int s, int i, int n, auto kc) GS_INLINE {
        constexpr int k = decltype(kc)::value;
        f[n][i][k] = gs_convert<k>(raw[i][s]);
    };
    auto scale = [&](int s, int i, int n, auto kc) GS_INLINE {
        constexpr int k = decltype(kc)::value;
        f[n][i][k] = s >> 1 ? gs_scale<true>(f[n][i][k], sc[i >> 2][i & 3]) : gs_scale<false>(f[n][i][k], sc[i >> 2][i & 3]);
    };
    // a quarter (x of 4) of fragment i's expansion for step s
    auto expand = [&](int s, int i, int n, auto xc) GS_INLINE {
        constexpr int x = decltype(xc)::value;
        if constexpr (x < 2) {
            convert(s, i, n, std::integral_constant<int, 2 * x>{});
            convert(s, i, n, std::integral_constant<int, 2 * x + 1>{});
        } else {
            scale(s, i, n, std::integral_constant<int, 2 * x - 4>{});
            scale(s, i, n, std::integral_constant<int, 2 * x - 3>{});
        }
    };
    gs_meet<20>();
#pragma unroll
    for (int i = 0; i < 16; ++i) read_raw(0, i);
    gs_for<16>([&](auto ic) GS_INLINE {
        constexpr int i = decltype(ic)::value;
        if constexpr (i % 4 == 0) read_sc(0, i / 4);
        gs_for<4>([&](auto x) GS_INLINE { expand(0, i, 0, x); });
    });

    bool stored = false;                     // exactly STORES stores of the tile before may still be on their way
    for (;;) {
        const Item cur = item_of(pos);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = (gs_acc_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < 8; ++i) gs_settle<0>(acc[i]);

#pragma unroll 1
        for (int u = 0; u < cur.niter; ++u) {
            const uint32_t b1 = buf(1), b3 = buf(3);
            gs_for<4>([&](auto sc_) GS_INLINE {
                constexpr int s = decltype(sc_)::value, c = s & 1, n = c ^ 1;
                if constexpr (s == 2) {
                    // the next unit is there.  (Stores are counted with the transfers, in order: those of the tile before are
                    // younger than what its first meeting waits for.)
                    if (u > 0 || !stored) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                    gs_meet<(STORES + 8 < 63 ? STORES + 8 : 63)>();
                    advance();
                }
                gs_for<64>([&](auto mc) GS_INLINE {
                    constexpr int m = decltype(mc)::value, j = m >> 3, i = m & 7, fr = m >> 2, x = m & 3;
                    // a fragment's codes of the next unit are read as soon as the present ones are expanded
                    if constexpr (s == 2 && x == 0 && fr > 0) read_raw(b1, fr - 1);
                    if constexpr (s == 3 && m == 0) read_raw(b1, 15);
                    if constexpr (s == 2 && m % 16 == 2 && m > 2) read_sc(b1, m / 16 - 1);
                    if constexpr (s == 3 && m == 2) read_sc(b1, 3);
                    if constexpr (s >= 2 && m % 12 == 9 && m < 60) issue(b3, std::integral_constant<int, 5 * (s - 2) + m / 12>{});
                    gs_mfma_f16(acc[i][j], f[c][8 + j], f[c][i]);
                    expand((s + 1) & 3, fr, n, std::integral_constant<int, x>{});
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            b0 = b1;
        }
        // low-rank columns: units of 32, both operands in bf16; the fragments alternate between f[0] and f[1] so that the last unit's
        // are in f[1], and beside its products the next tile's first step is expanded into f[0]
        if (cur.e > 0) {
            auto read_ext = [&](uint32_t bu, int i, int n) GS_INLINE {
                f[n][i] = *reinterpret_cast<const gs_u32x4*>(lds + bu + (i < 8 ? ra0 : rb0) + (i & 7) * 1024);
            };
            auto unit = [&](auto slot_, auto final_) GS_INLINE {
                constexpr int slot = decltype(slot_)::value;
                constexpr bool final = decltype(final_)::value;
                const uint32_t b1 = buf(1), b3 = buf(3);
                gs_meet<8>();
                advance();
                gs_for<64>([&](auto mc) GS_INLINE {
                    constexpr int m = decltype(mc)::value, j = m >> 3, i = m & 7;
                    if constexpr (m % 6 == 2 && m / 6 < 8) issue(b3, std::integral_constant<int, m / 6>{});
                    if constexpr (m % 6 == 2 && (m / 6 == 8 || m / 6 == 9)) {
                        if (lext >= 0) issue(b3, std::integral_constant<int, m / 6>{});
                    }
                    if constexpr (!final && m % 3 == 0 && m < 48) read_ext(b1, m / 3, slot ^ 1);
                    if constexpr (final && m < 16) read_raw(b1, m);
                    if constexpr (final && m < 16 && m % 4 == 3) read_sc(b1, m / 4);
                    gs_mfma_bf16(acc[i][j], f[slot][8 + j], f[slot][i]);
                    if constexpr (final && m >= 16) {
                        constexpr int fr = (m - 16) / 3, x = (m - 16) % 3;
                        if constexpr (x < 2) expand(0, fr, 0, std::integral_constant<int, x>{});
                        if constexpr (x == 2) {
                            expand(0, fr, 0, std::integral_constant<int, 2>{});
                            expand(0, fr, 0, std::integral_constant<int, 3>{});
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                b0 = b1;
            };
            constexpr std::integral_constant<int, 0> zero{};
            constexpr std::integral_constant<int, 1> one{};
            int left = cur.e;
            if (left & 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) read_ext(b0, i, 1);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) read_ext(b0, i, 0);
                unit(zero, std::false_type{});
                --left;
            }
#pragma unroll 1
            for (; left > 1; left -= 2) {
                unit(one, std::false_type{});
                unit(zero, std::false_type{});
            }
            unit(one, std::true_type{});
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) gs_settle<15>(acc[i]);
        const int slane = gs_fresh_lane();
        uint8_t* sm = lds + buf(3) + 4096 * wave;               // (read by nobody any more, fetched into after the next meeting)
        stored = false;
        if (cur.cut >= 0) {
            gs_store_tile<float>(sm, acc, alpha, partial + (size_t)cur.cut * 65536, 256, 128 * wa, 128 * wb, 256, 256, true, true, slane);
        } else if (vec && cur.m0 + 256 <= A.rows && cur.n0 + 256 <= B.rows) {
            gs_store_tile<OUT>(sm, acc, alpha, C, ldc, cur.m0 + 128 * wa, cur.n0 + 128 * wb, A.rows, B.rows, true, true, slane);
            stored = true;
        } else {
            gs_store_tile<OUT>(sm, acc, alpha, C, ldc, cur.m0 + 128 * wa, cur.n0 + 128 * wb, A.rows, B.rows, false, vec, slane);
        }
        pos += (int)gridDim.x;
        if (pos >= total_items) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // no transfer may outlive the workgroup's LDS
}
