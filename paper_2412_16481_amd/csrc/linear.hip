// The point-wise glue of a transformer block around the attention (Section 4.2, block equations; Section 4.1 "Stage
// Orchestration": the bucket-major array "suits point-wise MLPs and LayerNorm"): LayerNorm + linear map in one pass,
// with the row gather that puts q, k, v into bucket-major order (so that the attention reads contiguous rows) and the
// row scatter + residual that brings a block's output back.
//
//   y[p] = LN(x[row_in[p]]) W^T + bias;   out[row_out[p]] = y[p] + residual[row_out[p]]
//
// One workgroup = 4 waves = 128 rows; a wave owns 32 rows and keeps them in registers for the whole kernel, in the
// layout of the B operand of v_mfma_f32_32x32x16_bf16 (a lane holds half of one row), normalised there and rounded
// to bf16. The weight matrix (resident in L2) streams through LDS in double-buffered tiles of 16 KB filled by
// global -> LDS loads a tile ahead, and is the A operand of the TRANSPOSED product Y^T = W X^T: a lane then owns one row of Y and, with
// the rows of W fetched in a suitable order, 16 consecutive columns of it: 16-byte stores, no shuffles. The bias is the
// accumulator the product starts from.
//
// No wait inside the tile loop may drain the stores: the memory counter retires in order, so the one wait per tile (for
// the next tile's loads, and the next residual) allows the stores issued behind them to stay in flight.
//
// Bound: HBM, mostly the writes. The workgroups of an XCD keep more output rows open (6 MB at 256 channels) than its L2
// holds, so a line that is written in two halves a tile apart leaves L2 half full: pairs of 32-column blocks are stored
// together, whole lines per instruction (914601 rows, 256 -> 3 x 256: WRITE_SIZE 1.60 -> 1.37 GB = what there is to write).
// Results of 4 MB and more are stored non-temporally: kept in L2 their lines only push out x, W and the residual (both maps of a layer,
// us: 100000 rows of 128 channels 53.5 -> 41.0, 400000 of 64 77.5 -> 62.5, 200000 of 256 214 -> 194, 914601 of 256 847 -> 820).
// Smaller ones are still in L2 when the attention reads them. The q, k, v map with the attention behind it, ordinary / non-temporal
// stores, us: 3 MB of results (8000 rows of 64, 4000 of 128, 2000 of 256) 11.0 / 11.2, 12.5 / 13.0, 15.8 / 16.0; 6 MB (16000,
// 8000, 4000) 13.3 / 13.4, 16.3 / 15.4, 20.5 / 19.6; 19 MB (50000 of 64) 28.9 / 27.3; 300 MB (200000 of 256) 238 / 232. Between
// 40 and 160 MB the pair alone takes 1 to 6 % longer (100000 rows of 256 113 / 120), the whole layer with its output map
// 3 % less to 1 % more. Loads of x or the residual marked the same way cost 14 and 8 % more: both are read 16 bytes of a line at a time.
// Measured at 900000 rows with ordinary stores, LayerNorm + q, k, v map / output map with residual: 256 channels 636 -> 530 / 292 -> 242 us, 128
// 253 -> 213 / 133 -> 111, 64 128 -> 89 / 46 -> 43. A third resident tile and 256 rows per workgroup were no faster.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_common.h"
#include "launch.h"
#include "linear.h"

namespace f3d {

namespace {

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// lds_dma16 (see there for the s_nop) with a scalar base and a 32-bit byte offset per lane
__device__ __forceinline__ void lds_dma16_from(const void* base, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}

// s_waitcnt operand that waits for the memory counter alone
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

constexpr int LNW = 4;          // waves per workgroup; a wave owns 32 rows
constexpr int LTH = LNW * 64;
constexpr int LBM = LNW * 32;   // rows per workgroup

// W tiles in LDS: 32 * TCB output columns x CI inputs: 16 KB and 16 MFMAs per wave and barrier at 128 and 256 inputs, 8 KB at
// 64 (c_out is a multiple of 64, so every tile is whole). Row-major, the pieces of a row xor-swizzled so that 16
// consecutive rows read at one column fall on different banks.
template <int CI>
struct Tile {
    static constexpr int TCB = CI == 256 ? 1 : 2;   // 32-column blocks per tile
    static constexpr int TROWS = 32 * TCB;          // rows of W (output columns) per tile
    static constexpr int CPR = CI / 8;              // 16-byte pieces per row of W
    static constexpr int BYTES = TROWS * CI * 2;
    static constexpr int PPT = TROWS * CPR / LTH;   // pieces per thread and tile
    static_assert(TROWS * CPR % LTH == 0 && BYTES % 1024 == 0, "a W tile is a whole number of pieces per thread");
    static __device__ __forceinline__ int swizzle(int row) { return CPR >= 16 ? (row & 15) : ((row >> 1) & 7); }
};

// LN: LayerNorm in front of the map; RES: a residual is added behind it
template <int CI, bool LN, bool RES, bool STREAMED>   // STREAMED: results past the caches
__global__ __launch_bounds__(LTH, 3) void k_ln_linear(LinearArgs a)
{
    using T = Tile<CI>;
    constexpr int KS = CI / 16;                     // MFMA k-steps
    constexpr int TCB = T::TCB, TROWS = T::TROWS, CPR = T::CPR, PPT = T::PPT;
    __shared__ __attribute__((aligned(1024))) unsigned char sw[2 * T::BYTES];
    __shared__ uint4 sy[LNW][256];                  // 32 x 64 results per wave, on their way from one row per lane to whole lines
    float* sgamma = reinterpret_cast<float*>(sy);   // first: LayerNorm scale and shift
    float* sbeta = sgamma + CI;
    extern __shared__ __attribute__((aligned(16))) float sbias[];   // [c_out], zeros without a bias; then the column table
    // where the 16 columns from 16 g on go: their output tensor's address advanced to the first of them
    uint16_t** stab = reinterpret_cast<uint16_t**>(sbias + a.c_out);
    const uint32_t lds_w = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)sw;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long p = (long long)blockIdx.x * LBM + wave * 32 + l32;   // this lane's row of Y
    const bool ok = p < a.n;
    const bool stores = (long long)blockIdx.x * LBM + wave * 32 + 24 < a.n;   // every store instruction of this wave has a row
    const int n_tiles = (a.c_out >> 5) / TCB;
    // few rows: the columns are split over the grid's second dimension
    constexpr int UT = 2 / TCB;                     // tiles of a pair of blocks, which is stored together
    const int units = n_tiles / UT;
    const int t_begin = units * (int)blockIdx.y / (int)gridDim.y * UT, t_end = units * ((int)blockIdx.y + 1) / (int)gridDim.y * UT;

    // ---- staging of W tiles. Load i of this lane fills piece (wave*PPT + i)*64 + lane of the tile: slot = piece / CPR, with
    //      the piece of its row the swizzle puts there. Slot i of a 32-row block holds output column
    //      16*((i>>2)&1) + 4*(i>>3) + (i&3): with this order the 16 accumulator registers of a lane are 16 CONSECUTIVE
    //      columns of its row (two 16-byte stores; the two half-waves of a row write 64 contiguous bytes).
    uint32_t woff[PPT];               // bytes from the first row of a tile
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        const int q = (wave * PPT + i) * 64 + lane;
        const int slot = q / CPR, c = (q % CPR) ^ T::swizzle(slot);
        const int s32 = slot & 31;
        const int col = (slot & ~31) + 16 * ((s32 >> 2) & 1) + 4 * (s32 >> 3) + (s32 & 3);
        woff[i] = (uint32_t)(col * CI * 2 + c * 16);
    }
    auto dma_tile = [&](int t, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            lds_dma16_from(a.w, (uint32_t)(t * T::BYTES) + woff[i], lds_w + buf * T::BYTES + (wave * PPT + i) * 1024);
        }
    };
    // Everything the prologue reads from memory is requested before anything waits.
    const size_t src = ok ? (size_t)(a.row_in ? a.row_in[p] : p) : 0;
    const size_t drow = ok ? (size_t)(a.row_out ? a.row_out[p] : p) : 0;   // a valid row also past the end
    dma_tile(t_begin, 0);
    float gv = 0.f, bev = 0.f;
    if (LN) {
        gv = a.gamma[min(tid, CI - 1)];
        if (a.beta) bev = a.beta[min(tid, CI - 1)];
    }
    // this lane's part of its row: elements 16*ks + 8*hf .. +7 for every k-step, i.e. the B operand of the MFMAs
    U4 xf[KS];
    {
        const uint16_t* xr = a.x + src * CI + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) xf[ks].u = *reinterpret_cast<const uint4*>(xr + 16 * ks);   // rows past the end read row 0 and are never stored
    }
    const int per_out = a.c_out / a.n_outs;
    // the results in LDS: eight 16-byte pieces per row, xor-swizzled by the row; of a pair of blocks this lane puts pieces
    // 4 (block & 1) + 2 hf and + 1 of row l32, and stores piece lane & 7 of rows 8 k + (lane >> 3)
    const int yput = l32 * 8 + ((2 * hf) ^ (l32 & 7)), yget = (lane >> 3) * 8 + ((lane & 7) ^ (lane >> 3));
    int yrow[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) yrow[k] = __shfl(ok ? (int)drow : -1, 8 * k + (lane >> 3), 64);
    for (int i = tid; i < a.c_out; i += LTH) sbias[i] = a.bias ? a.bias[i] : 0.f;
    for (int g = tid; g < a.c_out / 16; g += LTH) {
        const int to = 16 * g / per_out;
        uint16_t* const o = to == 0 ? a.outs[0] : to == 1 ? a.outs[1] : to == 2 ? a.outs[2] : a.outs[3];
        stab[g] = o + (16 * g - to * per_out);
    }
    if (LN && tid < CI) {
        sgamma[tid] = gv;
        sbeta[tid] = bev;
    }
    uint4 rn[2] = {make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)};   // residual of the next 32-column block
    auto fetch_residual = [&](int block) __attribute__((always_inline)) {
        const uint4* rp = reinterpret_cast<const uint4*>(a.residual + drow * a.c_out + block * 32 + 16 * hf);
        rn[0] = rp[0];
        rn[1] = rp[1];
    };
    if (RES) fetch_residual(t_begin * TCB);
    __syncthreads();   // the vectors are in LDS
    if (LN) {   // the two half-waves hold the two halves of a row
        // Between the three passes the packed words are made opaque, so that each pass unpacks them again instead of
        // keeping the whole row alive as binary32 values.
        const auto opaque = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(xf[ks].u.x), "+v"(xf[ks].u.y), "+v"(xf[ks].u.z), "+v"(xf[ks].u.w));
        };
        float sum = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t w4[4] = {xf[ks].u.x, xf[ks].u.y, xf[ks].u.z, xf[ks].u.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += lo16(w4[e]) + hi16(w4[e]);
        }
        sum += __shfl_xor(sum, 32, 64);
        const float mu = sum * (1.0f / CI);
        opaque();
        float sq = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t w4[4] = {xf[ks].u.x, xf[ks].u.y, xf[ks].u.z, xf[ks].u.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d0 = lo16(w4[e]) - mu, d1 = hi16(w4[e]) - mu;
                sq += d0 * d0 + d1 * d1;
            }
        }
        sq += __shfl_xor(sq, 32, 64);
        const float rstd = rsqrtf(sq * (1.0f / CI) + a.eps);
        opaque();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const float4* g4 = reinterpret_cast<const float4*>(sgamma + 16 * ks + 8 * hf);
            const float4 ga = g4[0], gb = g4[1];
            const float4* b4 = reinterpret_cast<const float4*>(sbeta + 16 * ks + 8 * hf);
            const float4 ba = b4[0], bb = b4[1];
            const float gg[8] = {ga.x, ga.y, ga.z, ga.w, gb.x, gb.y, gb.z, gb.w};
            const float bt[8] = {ba.x, ba.y, ba.z, ba.w, bb.x, bb.y, bb.z, bb.w};
            const uint32_t w4[4] = {xf[ks].u.x, xf[ks].u.y, xf[ks].u.z, xf[ks].u.w};
            uint32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = pack_bf16((lo16(w4[e]) - mu) * rstd * gg[2 * e] + bt[2 * e], (hi16(w4[e]) - mu) * rstd * gg[2 * e + 1] + bt[2 * e + 1]);
            xf[ks].u = make_uint4(o[0], o[1], o[2], o[3]);
            // the step's result is wanted here (its inputs would otherwise be kept until the product), and at most two steps
            // of scale/shift reads are in flight
            asm volatile("" : "+v"(xf[ks].u.x), "+v"(xf[ks].u.y), "+v"(xf[ks].u.z), "+v"(xf[ks].u.w));
            if ((ks & 1) == 1) asm volatile("" ::: "memory");
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // the rows, the first W tiles and the first residual are here
    __syncthreads();

    // ---- Y^T = W X^T tile by tile: the A operand (32 rows of W) comes from LDS, the B operand is the wave's rows
    // piece hf of slot l32, swizzled; piece 2 ks + hf is a flip of the bits 32 ks away (slots 32 further on have the same
    // swizzle, pieces 16 further on lie 256 bytes on)
    const uint32_t foff = lds_w + l32 * (CI * 2) + ((hf ^ T::swizzle(l32)) << 4);
    int buf = 0;
    for (int t = t_begin; t < t_end; ++t) {
        // the other buffer is free: every wave passed the barrier at the end of the last iteration, after its last read of it
        if (t + 1 < t_end) dma_tile(t + 1, buf ^ 1);
#pragma unroll
        for (int cb = 0; cb < TCB; ++cb) {
            const int col0 = (t * TCB + cb) << 5;
            const uint4 rv[2] = {rn[0], rn[1]};
            if (RES && (cb + 1 < TCB || t + 1 < t_end)) fetch_residual(t * TCB + cb + 1);
            const int col = col0 + 16 * hf;                      // first of this lane's 16 columns
            f32x16 acc;
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float4 bv = *reinterpret_cast<const float4*>(sbias + col + 4 * q4);
                acc[4 * q4] = bv.x;
                acc[4 * q4 + 1] = bv.y;
                acc[4 * q4 + 2] = bv.z;
                acc[4 * q4 + 3] = bv.w;
            }
            // W fragments some k-steps at a time, one group ahead of the MFMAs that use them
            constexpr int G = 4, NG = KS / G;
            U4 wf[2][G];
            const uint32_t wt = foff + buf * T::BYTES + cb * 32 * CI * 2;
            const auto read_w = [&](int ks) __attribute__((always_inline)) { return lds_read16((wt ^ (32 * (ks & 7))) + (ks >> 3) * 256); };
#pragma unroll
            for (int i = 0; i < G; ++i) wf[0][i].u = read_w(i);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g + 1 < NG) {
#pragma unroll
                    for (int i = 0; i < G; ++i) wf[(g + 1) & 1][i].u = read_w((g + 1) * G + i);
                }
#pragma unroll
                for (int i = 0; i < G; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[g & 1][i].b, xf[g * G + i].b, acc, 0, 0, 0);
                F3D_SB();
            }
            if (RES) {
#pragma unroll
                for (int h8 = 0; h8 < 2; ++h8) {
                    const uint32_t w4[4] = {rv[h8].x, rv[h8].y, rv[h8].z, rv[h8].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[8 * h8 + 2 * e] += lo16(w4[e]);
                        acc[8 * h8 + 2 * e + 1] += hi16(w4[e]);
                    }
                }
            }
            // A lane holds 16 columns of its row. Stored from here, an instruction would write 16 bytes here and there in
            // every row, and lines would leave L2 half written: the workgroups' open rows do not fit there. Through LDS
            // eight lanes write 128 bytes, a whole line, of one row.
            const int odd = (t * TCB + cb) & 1;
#pragma unroll
            for (int h8 = 0; h8 < 2; ++h8)
                sy[wave][(yput ^ h8) ^ (4 * odd)] = make_uint4(pack_bf16(acc[8 * h8], acc[8 * h8 + 1]), pack_bf16(acc[8 * h8 + 2], acc[8 * h8 + 3]),
                                                               pack_bf16(acc[8 * h8 + 4], acc[8 * h8 + 5]), pack_bf16(acc[8 * h8 + 6], acc[8 * h8 + 7]));
            if (odd) {
                uint16_t* const ob = stab[(col0 >> 4) - 2 + ((lane & 7) >> 1)] + (lane & 1) * 8;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint4 y = sy[wave][yget + 64 * k];
                    const u32x4 yv = {y.x, y.y, y.z, y.w};
                    if (yrow[k] >= 0) {
                        u32x4* const to = reinterpret_cast<u32x4*>(ob + (size_t)yrow[k] * per_out);
                        if (STREAMED) __builtin_nontemporal_store(yv, to);
                        else *to = yv;
                    }
                }
            }
        }
        if (t + 1 == t_end) break;
        // The next tile has landed for this wave once only memory operations younger than its loads are outstanding: the
        // tile's own stores (with residual loads between them: the last four), or the residual loads of a tile that stores
        // nothing yet. A wave with rows missing leaves out stores.
        if (TCB == 1 && !(t & 1)) __builtin_amdgcn_s_waitcnt(vmcnt_imm(RES ? 2 : 0));
        else if (stores) __builtin_amdgcn_s_waitcnt(vmcnt_imm(RES || TCB == 1 ? 4 : 2 * TCB));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        buf ^= 1;
        __syncthreads();
    }
}

// Results of this size and more are stored past the caches (see above)
constexpr size_t STREAMED_BYTES = (size_t)4 << 20;

// an output tensor shares memory with x
bool in_place(const LinearArgs& a)
{
    const uintptr_t x0 = (uintptr_t)a.x, x1 = x0 + (size_t)a.n * a.c_in * 2;
    for (int t = 0; t < a.n_outs; ++t) {
        const uintptr_t o0 = (uintptr_t)a.outs[t], o1 = o0 + (size_t)a.n * (a.c_out / a.n_outs) * 2;
        if (o0 < x1 && x0 < o1) return true;
    }
    return false;
}

constexpr size_t linear_lds_bytes(int c_out) { return (size_t)c_out * 4 + (size_t)c_out / 16 * sizeof(uint16_t*); }

template <int CI, bool LN, bool RES, bool STREAMED>
hipError_t launch_form(const LinearArgs& a, hipStream_t stream)
{
    const unsigned blocks = (unsigned)((a.n + LBM - 1) / LBM);
    if (blocks == 0) return hipSuccess;
    // Few rows leave compute units idle while a workgroup walks all of W alone: then the columns are split until there are
    // about two workgroups per compute unit (every part reads and normalises its rows again): 1500 rows, 256 -> 3 x 256:
    // 28 -> 17 us, from 512 workgroups on one part. One part also where an output overwrites x: the workgroup that owns the
    // rows holds them in registers before its first store, a second one would read what the first has stored.
    const unsigned units = (unsigned)(a.c_out / 64);
    const unsigned split = blocks >= 512 || in_place(a) ? 1u : (512u / blocks < units ? 512u / blocks : units);
    const size_t lds = linear_lds_bytes(a.c_out);
    // tiles and results in static LDS, 32 or 48 KB: from 3000 columns or so on the sum passes what a kernel gets unasked
    if (2 * Tile<CI>::BYTES + LNW * 4096 + lds > 60000) {
        const hipError_t e = allow_lds((const void*)k_ln_linear<CI, LN, RES, STREAMED>, linear_lds_bytes(LIN_MAX_COLUMNS));
        if (e != hipSuccess) return e;
    }
    k_ln_linear<CI, LN, RES, STREAMED><<<dim3(blocks, split), LTH, lds, stream>>>(a);
    return hipGetLastError();
}

template <int CI, bool LN, bool RES>
hipError_t launch_one(const LinearArgs& a, hipStream_t stream)
{
    return (size_t)a.n * a.c_out * 2 >= STREAMED_BYTES ? launch_form<CI, LN, RES, true>(a, stream) : launch_form<CI, LN, RES, false>(a, stream);
}

template <int CI>
hipError_t launch_ci(const LinearArgs& a, hipStream_t stream)
{
    if (a.gamma) return a.residual ? launch_one<CI, true, true>(a, stream) : launch_one<CI, true, false>(a, stream);
    return a.residual ? launch_one<CI, false, true>(a, stream) : launch_one<CI, false, false>(a, stream);
}

}  // namespace

hipError_t linear_launch(const LinearArgs& a, hipStream_t stream)
{
    switch (a.c_in) {
        case 64: return launch_ci<64>(a, stream);
        case 128: return launch_ci<128>(a, stream);
        case 256: return launch_ci<256>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace f3d
