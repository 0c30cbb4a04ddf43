// Device helpers shared by the backward kernels (attn_bwd.hip, attn_bwd_one.hip): operand splits, the transposing reads of a
// row-major tile, the store of a gradient row.
#pragma once
#include "attn_common.h"

namespace f3d {

namespace {

constexpr float LOG2E = 1.4426950408889634f;

// bf16 fragment times a scalar, split into a bf16 head and a bf16 remainder (x*c = hi + lo up to 2^-17 relative)
__device__ __forceinline__ void scale_split(const U4& x, float c, U4& hi, U4& lo)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t w2 = (&x.u.x)[e];
        const float x0 = __uint_as_float(w2 << 16) * c, x1 = __uint_as_float(w2 & 0xFFFF0000u) * c;
        const uint32_t h = pack_bf16(x0, x1);
        const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xFFFF0000u);
        (&hi.u.x)[e] = h;
        (&lo.u.x)[e] = pack_bf16(r0, r1);
    }
}

// A row's log-sum-exp (in the units of the staged scores) and D as bf16 head + remainder pairs: {L_hi, L_lo}, {D_hi, D_lo}. One more MFMA
// whose other operand holds -1 at the matching two positions subtracts them from a whole score tile (error 2^-17
// relative), which is cheaper than 16 subtractions per lane and tile on the vector ALU.
__device__ __forceinline__ uint2 split_pairs(float l2, float dsum)
{
    const uint32_t lh = pack_bf16(l2, dsum);   // heads: l2 in the low half, dsum in the high half
    const float lr = l2 - __uint_as_float(lh << 16), dr = dsum - __uint_as_float(lh & 0xFFFF0000u);
    const uint32_t lo = pack_bf16(lr, dr);
    // regroup to {L_hi, L_lo} and {D_hi, D_lo}
    return make_uint2((lh & 0xFFFFu) | (lo << 16), (lh >> 16) | (lo & 0xFFFF0000u));
}

template <int D>
__device__ __forceinline__ void store_grad_rows(uint16_t* dst_base, const int32_t* out_perm, int row, int C, size_t hoff, int hf,
                                                const f32x16& acc, float mul)
{
    if (row < 0) return;
    const size_t drow = out_perm ? (size_t)out_perm[row] : (size_t)row;
    uint16_t* dst = dst_base + drow * C + hoff;
#pragma unroll
    for (int blk = 0; blk < D / 8; ++blk) {
        uint2 pk;
        pk.x = pack_bf16(acc[4 * blk] * mul, acc[4 * blk + 1] * mul);
        pk.y = pack_bf16(acc[4 * blk + 2] * mul, acc[4 * blk + 3] * mul);
        *reinterpret_cast<uint2*>(dst + 8 * blk + 4 * hf) = pk;
    }
}

template <int D>
struct BLay {
    static constexpr int NC = D / 8;                 // 16-byte pieces of one head in a row
    static constexpr int ROWB = D * 2;               // bytes of a row
    static constexpr int TILE = 32 * ROWB;           // from one 32-row tile to the next
    static constexpr int ROWS = 128;                 // rows per stage
    static constexpr int BUF = ROWS * ROWB;          // one operand of a stage
    static constexpr int NBUF = 3;
    static constexpr int LPW = ROWS * NC / 256;      // global -> LDS loads per lane, stage and operand
};

// byte offsets inside a tile of the transposing read that delivers X^T as an A operand (rows = dims, k = the tile's rows
// in the order of the score registers): lane 4j + c of a group of 16 hands in the address of dims 4c .. 4c+3 of row
// 4*hf + j (+ 8 s for the s-th read). The pieces of a row are swizzled by the row, which alternates with s. At
// head_dim 16 the second group of 16 lanes repeats the first: the 16 result rows it feeds are never read.
template <int D>
__device__ __forceinline__ void tr_offsets(int lane, uint32_t& even, uint32_t& odd)
{
    const int i16 = lane & 15, j = i16 >> 2, c = i16 & 3, g16 = (lane >> 4) & 1, hf = lane >> 5;
    const int row = 4 * hf + j;
    if (D == 32) {
        even = row * 64 + (((2 * g16 + (c >> 1)) ^ hf) * 16) + (c & 1) * 8;
        odd = even ^ 32;                             // rows 8 further on: swizzle hf + 2
    } else {
        even = row * 32 + (c >> 1) * 16 + (c & 1) * 8;
        odd = even ^ 16;
    }
}

template <int D>
__device__ __forceinline__ void read_tr(U4& x0, U4& x1, uint32_t even, uint32_t odd)
{
    constexpr int STEP = 8 * BLay<D>::ROWB;
    const uint2 a0 = lds_read_tr(even), a1 = lds_read_tr(odd + STEP), a2 = lds_read_tr(even + 2 * STEP), a3 = lds_read_tr(odd + 3 * STEP);
    x0.u = make_uint4(a0.x, a0.y, a1.x, a1.y);
    x1.u = make_uint4(a2.x, a2.y, a3.x, a3.y);
}

__device__ __forceinline__ f32x16 mfma_bf16(const U4& x, const U4& y, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.b, y.b, c, 0, 0, 0);
}

}  // namespace

}  // namespace f3d
