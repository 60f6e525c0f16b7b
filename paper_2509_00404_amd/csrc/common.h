// Shared device/host helpers of the HIP path (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/metis.h"

#define METIS_WAVE 64

#define METIS_LAUNCH_CHECK()                                   \
    do {                                                       \
        if (hipGetLastError() != hipSuccess) return METIS_HIP_ERROR; \
    } while (0)

typedef uint16_t bf16_t;   // raw bfloat16 bits

// ---- optional event bracketing of the hot kernels (see metis_profile_events) ----
enum { METIS_PROF_GEMM = 0, METIS_PROF_BROADCAST = 1, METIS_PROF_RESIDUAL_QUANT = 2, METIS_PROF_QUANTIZE = 3,
       METIS_PROF_COUNT = 4 };
struct MetisProfSlot {
    hipEvent_t* start;
    hipEvent_t* stop;
    int n, next;
};
extern MetisProfSlot g_metis_prof[METIS_PROF_COUNT];
static inline int metis_prof_begin(int id, hipStream_t s) {
    MetisProfSlot& p = g_metis_prof[id];
    if (p.n <= 0) return -1;
    int i = p.next % p.n;
    (void)hipEventRecord(p.start[i], s);
    return i;
}
static inline void metis_prof_end(int id, int i, hipStream_t s) {
    if (i < 0) return;
    MetisProfSlot& p = g_metis_prof[id];
    (void)hipEventRecord(p.stop[i], s);
    p.next++;
}

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
// low / high half of a dword holding two bf16
__device__ __forceinline__ float bf16lo_to_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp32 -> bf16, round to nearest even (finite inputs)
__device__ __forceinline__ bf16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// Raising a kernel's dynamic LDS limit is a driver call of tens of microseconds: remember, per device, the largest
// value already set for that kernel (one zero-initialised cache per call site).  Races only repeat the call.
struct LdsLimitCache { int bytes[16]; };
static inline bool ensure_dyn_lds(const void* fn, size_t bytes, LdsLimitCache& c) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const bool slot = dev >= 0 && dev < 16;
    if (slot && c.bytes[dev] >= (int)bytes) return true;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    if (slot) c.bytes[dev] = (int)bytes;
    return true;
}

// compute units of the current device (cached per device), 0 on error
static inline int device_cu_count() {
    static int cached[16];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const bool slot = dev >= 0 && dev < 16;
    if (slot && cached[dev] > 0) return cached[dev];
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (slot) cached[dev] = n;
    return n;
}

static inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// How many ways to cut the second grid dimension (1 .. max_split) when `blocks` workgroups exist along the first and
// the GPU runs `slots` workgroups at a time: the cut whose last round of workgroups is fullest, among those that
// reach at least one full round when possible; ties go to the fewest cuts (longer runs per workgroup).
static inline int64_t balanced_split(int64_t blocks, int64_t max_split, int64_t slots) {
    if (max_split < 1) max_split = 1;
    int64_t best = 1;
    double best_eff = -1.0;
    for (int64_t s = 1; s <= max_split; ++s) {
        const int64_t wgs = blocks * s, rounds = ceil_div64(wgs, slots);
        const double eff = (double)wgs / (double)(rounds * slots);
        if (eff > best_eff + 1e-9) { best_eff = eff; best = s; }
    }
    return best;
}
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// The same step of several independent problems in one launch.  A launch that waits for the one before it takes 4.5 us here
// however little it does, and the small steps of a decomposition do little, so what can go out together does.  The calls travel by
// value in the kernel arguments; call c owns the workgroups [off[c], off[c + 1]) of a one-dimensional grid.
#define MAX_CALLS 16
template <typename Call>
struct CallBatch {
    int n;
    uint32_t off[MAX_CALLS + 1];
    Call c[MAX_CALLS];
};
// The call that a workgroup belongs to, and its number there.  The first call's words are fetched together with the offsets, and the
// empty asm, which changes nothing and writes no memory, keeps them so (the compiler would choose between the calls' addresses first,
// and a lone call would wait for one trip to the arguments after the other, 0.5 us a launch).
template <typename Call>
__device__ __forceinline__ Call batch_call(const CallBatch<Call>& b, uint32_t& local) {
    constexpr int W = sizeof(Call) / 4;
    static_assert(sizeof(Call) % 4 == 0, "whole words");
    uint32_t w[W];
    const uint32_t* first = reinterpret_cast<const uint32_t*>(&b.c[0]);
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = first[i];
    const uint32_t end = b.off[1];
#pragma unroll
    for (int i = 0; i < W; ++i) asm("" : "+s"(w[i]));
    local = blockIdx.x;
    if (local >= end) {
        int c = 1;
        while (c + 1 < b.n && local >= b.off[c + 1]) ++c;
        const uint32_t* other = reinterpret_cast<const uint32_t*>(&b.c[c]);
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = other[i];
        local -= b.off[c];
    }
    Call call;
    __builtin_memcpy(&call, w, sizeof(Call));
    return call;
}
// A pointer that came through batch_call is global memory's again: put together from words, it would be reached by flat instructions,
// which count as LDS accesses too, so that every wait for LDS and every counted wait for loads became one for everything in flight
// (k_broadcast of a lone 14336 x 4096 41.4 us, so 39.6, with arguments of its own 38.2; of 4096 x 4096 23.8, 22.8, 22.3).
template <typename T>
__device__ __forceinline__ T* in_global(T* p) { return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p; }
// n calls of one kernel instance, call.wgs workgroups each, in as few launches as hold them: launch(batch, workgroups)
template <typename Call, typename F>
[[nodiscard]] static inline int launch_calls(const Call* calls, size_t n, F launch) {
    CallBatch<Call> b;
    b.n = 0;
    b.off[0] = 0;
    for (size_t i = 0; i <= n; ++i) {
        if (b.n > 0 && (i == n || b.n == MAX_CALLS || (uint64_t)b.off[b.n] + calls[i].wgs > 0x7FFFFFFFu)) {
            for (int t = b.n; t < MAX_CALLS; ++t) { b.c[t] = b.c[0]; b.off[t + 1] = b.off[b.n]; }
            launch(b, b.off[b.n]);
            METIS_LAUNCH_CHECK();
            b.n = 0;
        }
        if (i == n) break;
        b.c[b.n] = calls[i];
        b.off[b.n + 1] = b.off[b.n] + calls[i].wgs;
        ++b.n;
    }
    return METIS_OK;
}

// ---- Philox4x32-10 (Salmon et al., SC'11), written from the published round function ----
struct u32x4 { uint32_t x, y, z, w; };

__host__ __device__ __forceinline__ u32x4 philox4x32_10(u32x4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32 x 32 -> 64 bit product per multiplier (a single v_mad_u64_u32) instead of separate high and low halves
        // (every vector instruction here, integer multiplies included, costs ~4.5 cycles of issue: their number counts)
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c.x, p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c.z;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        u32x4 n;
        n.x = hi1 ^ c.y ^ k0;
        n.y = lo1;
        n.z = hi0 ^ c.w ^ k1;
        n.w = lo0;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// The four Philox blocks of 16 consecutive words, blk % 4 == 0, under `seed` and `stream` (what quantizing one block of
// 16 elements draws).  Same words as philox_block; written so that a round is four instructions, two
// v_mad_u64_u32 and two three-input v_bitop3_b32, and that the first two rounds only pay for what differs between the
// four counters: the third counter word is the same for all lanes (its products are scalar) and the second one, the
// high half of a block number that is a multiple of four, is the same for the four blocks of a lane.  41 instructions
// per block instead of 62 (the plain rounds compile to 40 xors and 20 products per block).
__device__ __forceinline__ void philox_4blocks(uint64_t seed, uint32_t stream, uint64_t blk, uint32_t (&w)[16]) {
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
    const uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32);
    const uint64_t p1s = (uint64_t)M1 * stream;                               // first round, third counter word
    const uint32_t x1 = (uint32_t)(p1s >> 32) ^ (uint32_t)(blk >> 32) ^ key0;  // after the first round: counter word 0 ...
    const uint32_t y1 = (uint32_t)p1s;                                        // ... and 1, the same for the four blocks
    const uint64_t p0r2 = (uint64_t)M0 * x1;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        // first round: M0 (blk + b), the low word of blk + b never carries
        const uint64_t p0r1 = (uint64_t)M0 * ((uint32_t)blk + b);
        uint32_t z = (uint32_t)(p0r1 >> 32) ^ key1, q = (uint32_t)p0r1;
        // second round
        const uint64_t p1r2 = (uint64_t)M1 * z;
        uint32_t x = __builtin_amdgcn_bitop3_b32((uint32_t)(p1r2 >> 32), y1, key0 + W0, 0x96);
        uint32_t y = (uint32_t)p1r2;
        z = __builtin_amdgcn_bitop3_b32((uint32_t)(p0r2 >> 32), q, key1 + W1, 0x96);
        q = (uint32_t)p0r2;
#pragma unroll
        for (uint32_t r = 2; r < 10; ++r) {
            const uint64_t p0 = (uint64_t)M0 * x, p1 = (uint64_t)M1 * z;
            x = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), y, key0 + r * W0, 0x96);
            z = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), q, key1 + r * W1, 0x96);
            y = (uint32_t)p1;
            q = (uint32_t)p0;
        }
        w[4 * b] = x; w[4 * b + 1] = y; w[4 * b + 2] = z; w[4 * b + 3] = q;
    }
}

// word `w` of stream `t` under `seed`: lane w%4 of block w/4, counter (blk lo, blk hi, t, 0)
__host__ __device__ __forceinline__ u32x4 philox_block(uint64_t seed, uint32_t stream, uint64_t blk) {
    u32x4 c = {(uint32_t)blk, (uint32_t)(blk >> 32), stream, 0u};
    return philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ---- FP8 E4M3 (bias 7, no inf, max 448) for non-negative block scales ----
__device__ __forceinline__ float e4m3_decode(uint32_t b) {
    return b >= 8u ? __uint_as_float((b + (120u << 3)) << 20) : (float)b * 0.001953125f;
}
