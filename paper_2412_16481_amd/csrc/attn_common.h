// Device helpers shared by the forward (attn.hip) and backward (attn_bwd.hip) attention kernels: the MFMA
// fragment types, the scope -> row-segment arithmetic (Section 4.2; Appendix "Bucket-Swin") and bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn.h"

namespace f3d {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;

#define F3D_SB() __builtin_amdgcn_sched_barrier(0)

constexpr int MAXSEG = 16;

union U4 {
    uint4 u;
    bf16x8 b;
    f16x8 f;
    uint16_t h[8];
};

// x / d with the divisor's Divide, which the host worked out (make_divide)
__device__ __forceinline__ int divide(int x, int d, const Divide& by)
{
    if (by.shift >= 0) return (int)((uint32_t)x >> by.shift);
    if (by.magic) return (int)__umulhi((uint32_t)x, by.magic);
    return (int)((uint32_t)x / (uint32_t)d);
}

// Position inside a scope -> bucket-major row. A scope is up to m runs of rows (one per bucket).
struct SegMap {
    int nseg, d0, d1, d2, d3, p1, p2, p3;
};

__device__ __forceinline__ int seg_row_of(const SegMap sm, const int* seg_pre, const int* seg_row0, int x)
{
    if (sm.nseg == 1) return sm.d0 + x;
    if (sm.nseg <= 4) {
        int d = sm.d0;
        d = x >= sm.p1 ? sm.d1 : d;
        d = x >= sm.p2 ? sm.d2 : d;
        d = x >= sm.p3 ? sm.d3 : d;
        return x + d;
    }
    int s = 0;
    while (s + 1 < sm.nseg && x >= seg_pre[s + 1]) ++s;   // the last of several that begin here: the others are empty
    return seg_row0[s] + (x - seg_pre[s]);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 x = {lo, hi};
    bf16x2 y = __builtin_convertvector(x, bf16x2);  // v_cvt_pk_bf16_f32, round to nearest even
    return *reinterpret_cast<uint32_t*>(&y);
}

// bf16 fragment times a power of two: exact
__device__ __forceinline__ U4 scale_pow2(const U4& x, float p2)
{
    U4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t w2 = (&x.u.x)[e];
        (&y.u.x)[e] = pack_bf16(__uint_as_float(w2 << 16) * p2, __uint_as_float(w2 & 0xFFFF0000u) * p2);
    }
    return y;
}

// One 16-byte global -> LDS load per lane: lane i of the wave fills bytes [16 i, 16 i + 16) of the 1 KB block at the
// LDS byte address `lds` (wave-uniform; it travels in M0). Written as assembly so that the compiler does not count
// it among its own memory operations: it would otherwise wait for ALL loads in flight before every LDS read that
// follows, and the loads issued here are meant to stay in flight for a whole stage. The kernel waits for them itself
// (s_waitcnt vmcnt(0) before the barrier that hands a stage over). M0 written by the scalar unit is safe to read one wait
// state later; the compiler does not look for such hazards inside assembly, so the s_nop is written out.
__device__ __forceinline__ void lds_dma16(const void* g, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(g) : "memory", "m0");
}

__device__ __forceinline__ uint2 lds_read_tr(uint32_t addr)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr);
    return *reinterpret_cast<const uint2*>(&v);
}

__device__ __forceinline__ uint4 lds_read16(uint32_t addr)
{
    const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)addr;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Inclusive sums over the 16 lanes of a row, by moves between lanes.
__device__ __forceinline__ int row_sums(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1, zeros from outside the row
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    return v;
}

// The rows of scope slot `slot`: `ng` of them in `sm.nseg` runs, one for plain and shifted scopes, up to m (one bucket each)
// for strided ones. False if the slot has none. Every wave works this out for itself, from two groups of loads the second of
// which depends on the first. Where the addresses are the same for all lanes and few (one scan, up to four runs) they are scalar
// loads, which come back sooner than a lane's; else lane i looks at scan i, then at run i.
// Bound: those two waits, in front of everything else a workgroup does. us with one thread walking through scans and buckets and a
// barrier behind it / a lane per scan and run always / now, 8 heads x 32: 200000 points, scope 256, strided 127 / 131 / 124; scope
// 128, backward 138 / 145 / 134; 100000 + 3000 points, 12 runs of 16, strided 133 / 117 / 117; 64 scans of 1000, strided 48.2 / 44.1 / 43.7.
// `row0` and `pre` (MAXSEG and MAXSEG + 1 words of LDS, the wave's own) are written for more than four runs only.
__device__ __forceinline__ bool scope_of_slot(const AttnArgs& a, int slot, int* row0, int* pre, int& ng, SegMap& sm)
{
    const int lane = threadIdx.x & 63;
    int kb0, K, g;
    if (a.n_scans == 1) {
        const int end = a.sbs[1];
        kb0 = a.sbs[0];
        if (end <= 0) return false;                   // as below: flagged, or no buckets
        K = end - kb0;
        g = slot - divide(kb0, a.m, a.by_m);
    } else if (a.n_scans < 64) {
        // scans own disjoint slot ranges starting at sbs[b]/m + extra*b
        const int first = a.sbs[min(lane, a.n_scans)];
        const int start = divide(first, a.m, a.by_m) + a.extra * lane;
        if (__builtin_amdgcn_readlane(first, a.n_scans) <= 0) return false;
        const int b = max(__popcll(__builtin_amdgcn_ballot_w64(lane < a.n_scans && start <= slot)) - 1, 0);
        kb0 = __builtin_amdgcn_readlane(first, b);
        K = __builtin_amdgcn_readlane(first, b + 1) - kb0;
        g = slot - __builtin_amdgcn_readlane(start, b);
    } else {
        if (a.sbs[a.n_scans] <= 0) return false;
        int b = 0, hi = a.n_scans;
        while (hi - b > 1) {
            const int mid = (b + hi) >> 1;
            if (divide(a.sbs[mid], a.m, a.by_m) + a.extra * mid <= slot) b = mid; else hi = mid;
        }
        kb0 = a.sbs[b];
        K = a.sbs[b + 1] - kb0;
        g = slot - (divide(kb0, a.m, a.by_m) + a.extra * b);
    }
    if (K <= 0) return false;
    constexpr int BIG = 0x7FFFFFFF;
    sm.p1 = sm.p2 = sm.p3 = BIG;
    sm.d1 = sm.d2 = sm.d3 = 0;
    if (a.mode != 2) {
        const int j0 = a.mode == 1 ? (g == 0 ? 0 : a.shift + (g - 1) * a.m) : g * a.m;
        const int j1 = min(a.mode == 1 && g == 0 ? a.shift : j0 + a.m, K);
        if (j0 >= K) return false;
        sm.nseg = 1;
        sm.d0 = a.offsets[kb0 + j0];
        ng = a.offsets[kb0 + j1] - sm.d0;
        return ng > 0;
    }
    const int t = a.stride, mt = a.m * t;
    const int full = divide(K, mt, a.by_mt), rem = K - full * mt;
    if (g >= full * t + min(rem, t)) return false;
    const int blk = divide(g, t, a.by_t), j0 = blk * mt + (g - blk * t);
    if (a.m <= 4) {                                   // the usual scope of four buckets
        int r0[4], r1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {                 // all under way together
            const int* const at = a.offsets + kb0 + min(j0 + min(i, a.m - 1) * t, K - 1);
            r0[i] = at[0];
            r1[i] = at[1];
        }
        int before[5] = {};
        sm.nseg = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool has = i < a.m && j0 + i * t < K;
            sm.nseg += has ? 1 : 0;
            before[i + 1] = before[i] + (has ? max(r1[i] - r0[i], 0) : 0);
        }
        ng = before[4];
        sm.d0 = r0[0];
        if (sm.nseg > 1) { sm.p1 = before[1]; sm.d1 = r0[1] - before[1]; }
        if (sm.nseg > 2) { sm.p2 = before[2]; sm.d2 = r0[2] - before[2]; }
        if (sm.nseg > 3) { sm.p3 = before[3]; sm.d3 = r0[3] - before[3]; }
        return ng > 0;
    }
    const int j = j0 + lane * t;
    const bool has = lane < a.m && j < K;
    int r0 = 0, len = 0;
    if (has) {
        r0 = a.offsets[kb0 + j];
        len = max(a.offsets[kb0 + j + 1] - r0, 0);
    }
    const int sum = row_sums(len), before = sum - len, to_row = r0 - before;
    sm.nseg = __popcll(__builtin_amdgcn_ballot_w64(has));
    ng = __builtin_amdgcn_readlane(sum, 15);          // m is 16 at most
    sm.d0 = __builtin_amdgcn_readlane(to_row, 0);
    if (sm.nseg > 1) {
        sm.p1 = __builtin_amdgcn_readlane(before, 1);
        sm.d1 = __builtin_amdgcn_readlane(to_row, 1);
    }
    if (sm.nseg > 2) {
        sm.p2 = __builtin_amdgcn_readlane(before, 2);
        sm.d2 = __builtin_amdgcn_readlane(to_row, 2);
    }
    if (sm.nseg > 3) {
        sm.p3 = __builtin_amdgcn_readlane(before, 3);
        sm.d3 = __builtin_amdgcn_readlane(to_row, 3);
    }
    if (sm.nseg > 4) {
        if (has) {
            row0[lane] = r0;
            pre[lane] = before;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    }
    return ng > 0;
}

// Which (slot, head, block of rows) is this workgroup: consecutive ids stay on one XCD
__device__ __forceinline__ void block_of_grid(const AttnArgs& a, int blocks, int& slot, int& head, int& blk)
{
    const int total = gridDim.x;  // multiple of 8
    const int w = blockIdx.x;
    const int u = (w & 7) * (total >> 3) + (w >> 3);
    const int x = divide(u, blocks, a.by_blocks);
    blk = u - x * blocks;
    slot = divide(x, a.H, a.by_h);
    head = x - slot * a.H;
}

}  // namespace

}  // namespace f3d
