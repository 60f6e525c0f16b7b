// The MXFP4 GEMM for large outputs (included by mxfp4.hip, inside its namespace).
#pragma once

// acc (+)= X Y^T, 32 x 32 over 64 columns, block scales in byte 0 (HI: 2) of xs and ys; the accumulator in the accumulation registers.
// In asm for its place and its registers.  What the compiler then does not see: an accumulator read by a vector
// instruction soon after (mxs_settle); operands come from LDS, scales are shifted a step ahead.
template <bool FIRST, bool HI>
__device__ __forceinline__ void mxs_mfma(float16_t& acc, const uvec4_t& x, const uvec4_t& y, uint32_t xs, uint32_t ys) {
    if constexpr (FIRST)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, 0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                     : "=a"(acc) : "v"(x), "v"(y), "v"(xs), "v"(ys));
    else if constexpr (HI)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[1,1,0] cbsz:4 blgp:4"
                     : "+a"(acc) : "v"(x), "v"(y), "v"(xs), "v"(ys));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4"
                     : "+a"(acc) : "v"(x), "v"(y), "v"(xs), "v"(ys));
}
__device__ __forceinline__ void mxs_settle(float16_t (&a)[2]) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(a[0]), "+a"(a[1]));
}
// between a vector instruction's result and the matrix instruction that reads it
__device__ __forceinline__ void mxs_settle_scales(uint32_t (&x)[6]) {
    asm volatile("s_nop 1" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]));
}

// 256 x 256 tiles, 8 waves of 128 x 64, two per SIMD; a unit is 256 contraction elements, 128 bytes of every row = whole cache lines.
// What it changed against the kernel above, which it took these products from: codes and scales go straight into LDS (no registers, no
// LDS stores, and the waits leave the loop), the accumulators stay in the accumulation registers, the next tile's first unit travels
// and its first fragments are read while this tile's last unit is multiplied, and a tile's first step needs no cleared accumulator.
// Product alone, us, 8192 x 14336 x 2048 / 4096 / 8192: 184 / 297 / 505 -> 168 / 267 / 459; with the quantizers 16384 x 4096 x 512 48.8
// -> 44.5, 6000 x 6000 x 4096 130 -> 118, 5000 x 5000 x 14336 286 -> 267, 16384 x 14336 x 512 fp32 205 -> 196.
// What bounds it: a unit's 256 matrix instructions take 2048 cycles of its ~3200, LDS reads and transfers run beside them (without the
// transfers the 267 are 219, without waiting for them 261, without the fragments' reads 262), and a tile's rows on their way
// out take 5 us, the staging 3 (without both 245: the card then holds a lower clock).  Tried: 4 waves of 128 x 128, which
// read a third less from LDS but leave the pipe idle whenever a transfer is issued (45 cycles each), 287; a unit's fragments read
// two steps ahead and its buffer given back a step earlier, the transfers' offsets then formed where they are issued, 277; starts of the
// workgroups staggered by 0.5 to 2 us, stores past the caches: no difference.
// LDS: two buffers of a unit: A's and B's codes row by row, 128 bytes a row, its 16-byte segments permuted by their number xor row / 2 %
// 8 (a transfer's lanes land side by side, and this is what spreads sixteen rows' reads of one segment over the banks), then 8 scale
// bytes of every row of both.
#define MXS_CODES 32768
#define MXS_SCALES 2048
#define MXS_UNIT (2 * MXS_CODES + 2 * MXS_SCALES)
#define MXS_LDS (2 * MXS_UNIT)
#define MXS_DMA 10                                       // transfers a wave makes for a unit
template <typename OUT>
__global__ void __launch_bounds__(512, 2)
k_mxfp4_gemm_nt_stream(MxOperand A, MxOperand B, int64_t K, OUT* __restrict__ C, int64_t ldc, bool vec, MxOrder order, int total) {
    constexpr bool LINES = sizeof(OUT) == 2;             // outputs by way of LDS, accumulator tiles transposed
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int niter = (int)(K / MX_KI);                  // at least 2
    const uint32_t cstride = (uint32_t)(K / 2), sstride = (uint32_t)(K / 32);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wa = wave >> 2, wb = wave & 3;
    const int lane = (int)threadIdx.x & 63, li = lane & 31, half = lane >> 5;
    auto tile_of = [&](int pos, int& m0, int& n0) GS_INLINE {
        int tm, tn;
        if (order.bands.group > 0) tile_coords_of(order.bands, pos, total, tm, tn);
        else tile_coords_of(order.regions, pos, total, tm, tn);
        m0 = 256 * tm;
        n0 = 256 * tn;
    };

    // ---- transfers.  The units of a workgroup's tiles form one stream, fetched two units ahead of the products
    const uint8_t *qa, *qb, *qsa, *qsb;                  // the next unit's codes and scales
    int lpos = (int)blockIdx.x, lcnt;                    // tile being fetched, units left of it
    uint32_t va[4], vb[4], wsa, wsb;               // the lane's offsets
    auto enter = [&]() GS_INLINE {
        int m0, n0;
        tile_of(lpos < total ? lpos : total - 1, m0, n0);         // (past the end: fetched again, unused)
        lcnt = niter;
        qa = A.codes + (int64_t)m0 * cstride;
        qb = B.codes + (int64_t)n0 * cstride;
        qsa = A.scales + (int64_t)m0 * sstride;
        qsb = B.scales + (int64_t)n0 * sstride;
        const int ta = (int)(A.rows - m0 < 256 ? A.rows - m0 : 256) - 1, tb = (int)(B.rows - n0 < 256 ? B.rows - n0 : 256) - 1;
        const int l = gs_fresh_lane();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 32 * wave + 8 * v + (l >> 3);         // rows past the operand's end: its last row
            const uint32_t seg = (uint32_t)((l & 7) ^ (l >> 4) ^ (4 * (v & 1))) * 16;
            va[v] = (uint32_t)(row < ta ? row : ta) * cstride + seg;
            vb[v] = (uint32_t)(row < tb ? row : tb) * cstride + seg;
        }
        const int row = 32 * wave + (l >> 1);
        wsa = (uint32_t)(row < ta ? row : ta) * sstride + 4u * (l & 1);
        wsb = (uint32_t)(row < tb ? row : tb) * sstride + 4u * (l & 1);
    };
    auto advance = [&]() GS_INLINE {                     // before the first transfer of a unit
        if (lcnt == 0) {
            lpos += (int)gridDim.x;
            enter();
        }
        --lcnt;
        qa = gs_uniform(qa);
        qb = gs_uniform(qb);
        qsa = gs_uniform(qsa);
        qsb = gs_uniform(qsb);
    };
    auto issue = [&](uint32_t buf, auto kc) GS_INLINE {
        constexpr int k = decltype(kc)::value;
        const uint32_t dc = lds0 + buf + 4096u * wave, ds = lds0 + buf + 256u * wave;
        if constexpr (k < 4) gs_dma16<1024 * k>(dc, va[k], qa);
        else if constexpr (k < 8) gs_dma16<MXS_CODES + 1024 * (k - 4)>(dc, vb[k - 4], qb);
        else if constexpr (k == 8) gs_dma4<2 * MXS_CODES>(ds, wsa, qsa);
        else gs_dma4<2 * MXS_CODES + MXS_SCALES>(ds, wsb, qsb);
        if constexpr (k == MXS_DMA - 1) {
            qa += MX_KI / 2;
            qb += MX_KI / 2;
            qsa += MX_KI / 32;
            qsb += MX_KI / 32;
        }
    };

    int pos = (int)blockIdx.x;
    if (pos >= total) return;
    enter();
    advance();
    gs_for<MXS_DMA>([&](auto k) GS_INLINE { issue(0, k); });
    advance();
    gs_for<MXS_DMA>([&](auto k) GS_INLINE { issue(MXS_UNIT, k); });

    float16_t acc[4][2];
    uvec4_t f[2][6];                                     // fragments of a step: 0 .. 3 of A's rows, 4 and 5 of B's
    uvec2_t raw[6];                                      // their rows' scale bytes of a unit
    uint32_t sx[6], sy[6];                               // steps 0 and 1, 2 and 3: bytes 0 and 2 are this lane's blocks
    uint32_t ad[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) ad[s] = 128u * li + 16u * (uint32_t)((2 * s + half) ^ (li >> 1 & 7));
    auto read_frag = [&](uint32_t bu, int s, int n, int x) GS_INLINE {
        const uint32_t at = (x < 4 ? 16384u * wa : MXS_CODES + 8192u * wb) + 4096u * (x & 3);
        f[n][x] = *reinterpret_cast<const uvec4_t*>(lds + bu + at + ad[s]);
    };
    auto read_scale = [&](uint32_t bu, int x) GS_INLINE {
        const uint32_t at = 2 * MXS_CODES + (x < 4 ? 1024u * wa : MXS_SCALES + 512u * wb) + 256u * (x & 3);
        raw[x] = *reinterpret_cast<const uvec2_t*>(lds + bu + at + 8u * li);
    };
    gs_meet<MXS_DMA>();
#pragma unroll
    for (int x = 0; x < 6; ++x) {
        read_frag(0, 0, 0, x);
        read_scale(0, x);
    }
#pragma unroll
    for (int x = 0; x < 6; ++x) sx[x] = raw[x].x >> (8 * half);
    mxs_settle_scales(sx);

    uint32_t b0 = 0;                                     // buffer of the unit in work
    auto unit = [&](auto first_, auto last_) GS_INLINE {
        constexpr bool first = decltype(first_)::value, last = decltype(last_)::value;
        const uint32_t b1 = MXS_UNIT - b0;
        gs_for<4>([&](auto sc_) GS_INLINE {
            constexpr int s = decltype(sc_)::value, n = s & 1;
            gs_for<8>([&](auto mc) GS_INLINE {
                constexpr int m = decltype(mc)::value, i = m & 3, j = m >> 2;
                if constexpr (s == 0 && m < 6) sy[m] = raw[m].y >> (8 * half);
                if constexpr (s < 3 && m < 6) read_frag(b0, s + 1, n ^ 1, m);
                if constexpr (s == 3) {
                    // the next unit is there, and this one's buffer has been read by all
                    if constexpr (m == 1) {
                        gs_meet<0>();
                        if constexpr (!last) advance();
                    }
                    if constexpr (m >= 1 && m < 7) {
                        read_frag(b1, 0, 0, m - 1);
                        read_scale(b1, m - 1);
                    }
                    if constexpr (!last && m >= 1) {
                        issue(b0, std::integral_constant<int, m - 1>{});
                        if constexpr (m >= 5) issue(b0, std::integral_constant<int, m + 2>{});
                    }
                }
                const uint32_t as = s < 2 ? sx[i] : sy[i], bs = s < 2 ? sx[4 + j] : sy[4 + j];
                if constexpr (LINES) mxs_mfma<first && s == 0, n == 1>(acc[i][j], f[n][4 + j], f[n][i], bs, as);
                else mxs_mfma<first && s == 0, n == 1>(acc[i][j], f[n][i], f[n][4 + j], as, bs);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
#pragma unroll
        for (int x = 0; x < 6; ++x) sx[x] = raw[x].x >> (8 * half);
        mxs_settle_scales(sx);
        b0 = b1;
    };
    for (;;) {
        unit(std::true_type{}, std::false_type{});
#pragma unroll 1
        for (int u = 2; u < niter; ++u) unit(std::false_type{}, std::false_type{});
        unit(std::false_type{}, std::true_type{});
#pragma unroll
        for (int i = 0; i < 4; ++i) mxs_settle(acc[i]);
        const uint32_t bl = MXS_UNIT - b0;               // the last unit's buffer
        int m0, n0;
        tile_of(pos, m0, n0);
        mx_store_wave<OUT, LINES, 4, 2>(acc, lds + bl + wave * mx_wave_rows<OUT, 2>(), C, ldc, m0 + 128 * wa, n0 + 64 * wb, A.rows, B.rows,
                                        vec, mx_whole<LINES>(m0 + 256 <= A.rows && n0 + 256 <= B.rows, vec), gs_fresh_lane());
        pos += (int)gridDim.x;
        if (pos >= total) break;
        // every wave has its rows out of the buffer before any transfers into it
        gs_meet<63>();
        advance();
        gs_for<MXS_DMA>([&](auto k) GS_INLINE { issue(bl, k); });
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no transfer may outlive the workgroup's LDS
}
