// Backward of the Bucket-and-Swin attention in one kernel: every score is computed once and serves all three gradients. (The
// definitions, and the two kernels that compute each score twice and take the launches this one does not, are in attn_bwd.hip.)
//
// One workgroup of eight waves per compute unit takes a task, a scope of one head, at a time. A wave owns 64 keys, 512 the workgroup;
// the scope's queries pass by in tiles of 32, staged in LDS as in attn_bwd.hip. Scores are queries x keys, so P and dS, packed to bf16, are
// the B operands of dV^T += dO^T P and dK^T += Q^T dS straight from the registers. For dQ^T += K^T dS^T the dS tile goes through LDS: written
// as it lies, read back by the transposing read a query tile later. The eight waves' dQ of a tile, binary32, meet in LDS and are added
// in the order of the waves; scopes of more than 512 rows take several passes, whose sums wait in the workspace for the thread that goes on
// with them. So nothing depends on timing, and P and D carry binary32 through: log-sum-exp and D are three bf16 terms each, which an
// MFMA of four k positions multiplies by -1.
//
// Bound: per 32 x 32 scores 11.5 MFMAs of 32 cycles and 320 cycles of the vector ALU (16 exponentials, 32 multiplies, 16 packs), which hide
// each other only in part with two waves per SIMD (all 256 registers are in use): 800 cycles measured, where the two kernels take 462 + 612.
// What comes per step (32 queries) beside it is spread so that of a SIMD's two waves one goes on computing: the upper half of the waves
// loads the stages in the middle of a step, the lower half adds up dQ behind its barrier (both behind the barrier: 914601 points x 8 heads x 32
// 5.30 ms for the whole training pass instead of 5.11). MFMAs stand about 28 cycles of vector work apart (in the compiler's order 5.14 ms
// instead of 4.99; each pair from one card, cards differ by 5 %).
// Backward pass, us, two kernels / this one, scopes of 1024: 200000 points x 4 heads x 16 378 / 326, x 16 heads 1453 / 1184; 401111 x 8 x 16
// 1442 / 1172 (scopes of 512 833 / 740, of 2048 2711 / 2428); 300000 x 8 x 32 1385 / 1186, 60000 x 8 x 32 277 / 243. Workgroups of four
// waves, two per compute unit, at head_dim 16: 1181 for the 1172, 3135 for the 2439 of scopes of 2048 (twice the passes).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn.h"
#include "attn_bwd_common.h"
#include "launch.h"

namespace f3d {

namespace {

constexpr int W = ATTN_BWD_ONE_WAVES;

template <int D>
struct OLay {
    static constexpr int NC = D / 8;                  // 16-byte pieces of one head in a row
    static constexpr int ROWB = D * 2;                // bytes of a row
    static constexpr int TILE = 32 * ROWB;            // from one 32-row tile to the next
    static constexpr int ROWS = 64;                   // query rows per stage
    static constexpr int BUF = ROWS * ROWB;           // one operand of a stage
    static constexpr int NBUF = 3;
    static constexpr int NBLK = 2 * BUF / 1024;       // 1 KB blocks of a stage: Q, then dO
    static constexpr int LPW = NBLK / (W / 2);        // of which a wave of the upper half loads so many
    static constexpr int KB = 64 * W;                 // keys per pass over the queries
    // One wave's share of the dQ of a query tile: binary32, rows 16 bytes apart from each other's banks (the last needs no gap). Of the writes,
    // a piece of every row, no two lanes meet; of the reads in add_up, whole rows, the first and the last row of sixteen lanes meet in one piece.
    static constexpr int PROW = D * 4 + 16, PART = 32 * PROW - 16;
    static constexpr int DS = 2 * 2048;               // a wave's two dS tiles
    static constexpr int AT_G = NBUF * BUF, AT_PART = 2 * NBUF * BUF, AT_DS = AT_PART + 2 * W * PART, AT_X = AT_DS + W * DS;
};

__device__ __forceinline__ void lds_write8(uint32_t addr, uint32_t x, uint32_t y)
{
    *(__attribute__((address_space(3))) u32x2*)(uintptr_t)addr = u32x2{x, y};
}

__device__ __forceinline__ void lds_write16(uint32_t addr, uint32_t x, uint32_t y, uint32_t z, uint32_t w)
{
    *(__attribute__((address_space(3))) u32x4*)(uintptr_t)addr = u32x4{x, y, z, w};
}

__device__ __forceinline__ u32x2 lds_read8(uint32_t addr)
{
    return *(const __attribute__((address_space(3))) u32x2*)(uintptr_t)addr;
}

// binary32 as three bf16 terms {hi, mid}, {lo, 0}: exact but for the last bit
__device__ __forceinline__ u32x2 split_three(float x)
{
    const uint32_t h = pack_bf16(x, 0.f);
    const float r = x - __uint_as_float(h << 16);
    const uint32_t m = pack_bf16(r, 0.f);
    return u32x2{h | (m << 16), pack_bf16(r - __uint_as_float(m << 16), 0.f)};
}

// The lane's number, worked out where it is used: kept in a register over the loops it would push out what they work on.
__device__ __forceinline__ int lane_here()
{
    int x;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
    return x;
}

__device__ __forceinline__ f32x16 mfma_k8(u32x2 x, u32x2 y, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(*reinterpret_cast<s16x4*>(&x), *reinterpret_cast<s16x4*>(&y), c, 0, 0, 0);
}

template <int D>
__global__ __launch_bounds__(64 * W, 2) void k_attn_bwd_one(AttnBwdArgs b)
{
    using L = OLay<D>;
    constexpr bool SPLIT = D == 16;
    constexpr int NC = L::NC, KS = D / 16, SR = L::ROWS;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int seg_row0[MAXSEG], seg_pre[MAXSEG + 1];     // the same from every wave
    const AttnArgs& a = b.f;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool loads = wave >= W / 2;                 // the upper half of the waves loads the stages, the lower adds up dQ
    const uint32_t row_bytes = (uint32_t)a.C * 2u;
    const uint32_t sQ = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
    const uint32_t sG = sQ + L::AT_G, sP = sQ + L::AT_PART, sD = sQ + L::AT_DS + wave * L::DS, sX = sQ + L::AT_X;

    int cexp = 0;
    const float cres = SPLIT ? 1.0f : 2.0f * frexpf(a.c_log2, &cexp);   // c_log2 = cres * 2^(cexp - 1), 1 <= |cres| < 2
    const float cpow = SPLIT ? 1.0f : ldexpf(1.0f, cexp - 1), lmul = LOG2E / cres;

    for (int task = blockIdx.x; task < 8 * b.done; task += gridDim.x) {
        const int u = (task & 7) * (b.tasks >> 3) + (task >> 3);   // consecutive ones stay on one XCD
        const int slot = divide(u, a.H, a.by_h), head = u - slot * a.H;
        int ng;
        SegMap sm;
        __syncthreads();                              // everybody is done with the task before
        if (slot >= a.n_slots || !scope_of_slot(a, slot, seg_row0, seg_pre, ng, sm)) continue;
        ng = __builtin_amdgcn_readfirstlane(min(ng, b.cap));
        for (int* f : {&sm.nseg, &sm.d0, &sm.d1, &sm.d2, &sm.d3, &sm.p1, &sm.p2, &sm.p3}) *f = __builtin_amdgcn_readfirstlane(*f);
        const size_t hoff = (size_t)head * D;
        const int nst = (ng + SR - 1) / SR, ntile = (ng + 31) >> 5, npass = (ng + L::KB - 1) / L::KB;
        // ---- staging: block bi of a stage is 64 16-byte pieces of Q or dO rows, the piece of the row that the swizzle puts there.
        //      q rows go through the permutation, dO rows are bucket-major; positions past the end fetch the scope's last row again.
        uint32_t row_next[L::LPW];
        auto fetch_rows = [&](int st) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < L::LPW; ++i) {
                const int bi = (wave - W / 2) * L::LPW + i;
                const int kk = ((bi % (L::NBLK / 2)) * 64 + lane_here()) / NC;
                const uint32_t r = (uint32_t)seg_row_of(sm, seg_pre, seg_row0, min(st * SR + kk, ng - 1));
                row_next[i] = bi < L::NBLK / 2 && a.perm ? (uint32_t)a.perm[r] : r;
            }
        };
        auto dma_stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < L::LPW; ++i) {
                const int bi = (wave - W / 2) * L::LPW + i;
                const int half = bi % (L::NBLK / 2), p = half * 64 + lane_here(), kk = p / NC, cs = p % NC;
                const int c = (NC == 4) ? (cs ^ ((kk >> 2) & 3)) : (cs ^ ((kk >> 3) & 1));
                const bool isq = bi < L::NBLK / 2;
                const char* base = reinterpret_cast<const char*>((isq ? a.q : b.dout) + hoff + c * 8);
                lds_dma16(base + (uint64_t)row_next[i] * row_bytes, (isq ? sQ : sG) + buf * L::BUF + half * 1024);
            }
        };

        if (loads) {
            fetch_rows(0);
            dma_stage(0);
            if (nst > 1) {
                fetch_rows(1);
                dma_stage(1);
            }
        }
        // ---- this lane's keys of a pass: rows l32 of two tiles; past the end: a valid row, never stored
        U4 kraw[2][KS], vfr[2][KS];
        int krow[2];
        auto key_rows = [&](int pass) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                krow[j] = seg_row_of(sm, seg_pre, seg_row0, min(pass * L::KB + wave * 64 + j * 32 + (lane_here() & 31), ng - 1));
                if (a.perm) krow[j] = a.perm[krow[j]];
            }
        };
        auto load_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const size_t at = (size_t)krow[j] * a.C + hoff + (lane_here() >> 5) * 8;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    kraw[j][ks].u = *reinterpret_cast<const uint4*>(a.k + at + ks * 16);
                    vfr[j][ks].u = *reinterpret_cast<const uint4*>(a.v + at + ks * 16);
                }
            }
        };
        key_rows(0);
        load_keys();

        // ---- log-sum-exp and D of every row; past the end: probabilities exactly zero
        constexpr int XB = 2 * NC;                    // 1024 rows in one go
        for (int i0 = (wave * 64 + lane_here()); i0 < nst * SR * NC; i0 += 64 * W * XB) {
            uint4 o[XB], g[XB];
            float l[XB];
#pragma unroll
            for (int t = 0; t < XB; ++t) {
                const int i = i0 + t * 64 * W, x = min(i / NC, ng - 1);
                const size_t r = (size_t)seg_row_of(sm, seg_pre, seg_row0, x), at = r * a.C + hoff + (i % NC) * 8;
                o[t] = *reinterpret_cast<const uint4*>(a.out + at);
                g[t] = *reinterpret_cast<const uint4*>(b.dout + at);
                l[t] = a.lse[r * a.H + head];
            }
#pragma unroll
            for (int t = 0; t < XB; ++t) {
                const int i = i0 + t * 64 * W, x = i / NC;
                float dot = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t p = (&o[t].x)[e], y = (&g[t].x)[e];
                    dot += __uint_as_float(p << 16) * __uint_as_float(y << 16);
                    dot += __uint_as_float(p & 0xFFFF0000u) * __uint_as_float(y & 0xFFFF0000u);
                }
                dot += __shfl_xor(dot, 1, 64);
                if (NC == 4) dot += __shfl_xor(dot, 2, 64);
                if (i % NC == 0 && x < nst * SR) {
                    const u32x2 ls = split_three(x < ng ? l[t] * lmul : 1e30f), ds = split_three(x < ng ? dot : 0.f);
                    lds_write8(sX + x * 16, ls.x, ls.y);
                    lds_write8(sX + x * 16 + 8, ds.x, ds.y);
                }
            }
        }

        int buf = 0;                                  // of the stage at hand; the stages of one pass follow those of the one before
        for (int pass = 0; pass < npass; ++pass) {
            const int key0 = pass * L::KB + wave * 64;
            const bool active = key0 < ng, last = pass + 1 == npass;
            const int nact = min(W, (ng - pass * L::KB + 63) / 64);   // waves with keys
            const int ln = lane_here(), l32 = ln & 31, hf = ln >> 5, i16 = ln & 15, g16 = (ln >> 4) & 1;
            // ---- this lane's places in LDS
            uint32_t foff[KS];                        // row l32 of a query tile, dims 16*ks + 8*hf ..
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int c = 2 * ks + hf;
                foff[ks] = sQ + (l32 * NC + ((NC == 4) ? (c ^ ((l32 >> 2) & 3)) : (c ^ ((l32 >> 3) & 1)))) * 16;
            }
            uint32_t tre, tro;
            tr_offsets<D>(ln, tre, tro);
            tre += sQ;
            tro += sQ;
            // A dS tile: row = key, its 32 queries in the order of the score registers (queries 8g + 4h .. as 8-byte piece 4h + g), in
            // 16-byte units swizzled by the key. This lane writes row l32, reads, transposed, keys 16m + 8hf + 4i + 0..3 of the sixteen
            // queries 16*g16 .. (unit 2h + (g >> 1) of piece c = 2(g & 1) + h there).
            uint32_t dsw[2], dsr[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                dsw[i] = sD + l32 * 64 + (((hf * 2 + i) ^ (l32 >> 2)) & 3) * 16;
                dsr[i] = sD + (8 * hf + 4 * i + (i16 >> 2)) * 64 + (((i16 & 1) * 2 + g16) ^ (2 * hf + i)) * 16 + ((i16 >> 1) & 1) * 8;
            }
            auto read_ds = [&](U4& x0, U4& x1, int j) __attribute__((always_inline)) {
                const uint2 a0 = lds_read_tr(dsr[0] + j * 2048), a1 = lds_read_tr(dsr[1] + j * 2048);
                const uint2 a2 = lds_read_tr(dsr[0] + j * 2048 + 1024), a3 = lds_read_tr(dsr[1] + j * 2048 + 1024);
                x0.u = make_uint4(a0.x, a0.y, a1.x, a1.y);
                x1.u = make_uint4(a2.x, a2.y, a3.x, a3.y);
            };
            // dQ of a tile: written pieces 2*blk + hf of row l32; read, when the waves' shares are added, piece rp of row rq
            constexpr int PQ = D / 4;
            const uint32_t pw = sP + wave * L::PART + l32 * L::PROW + hf * 16;
            const int rq = (wave * 64 + lane_here()) / PQ, rp = (wave * 64 + lane_here()) % PQ;
            const bool adds = rq < 32;
            const uint32_t pr = sP + rq * L::PROW + rp * 16;
            // S's log-sum-exp and dP's D: three terms each, in the k positions of the lower and the upper half-wave
            const uint32_t neg1 = 0xBF80BF80u;
            const u32x2 negS = {hf == 0 ? neg1 : 0u, hf == 0 ? neg1 : 0u}, negD = {hf == 1 ? neg1 : 0u, hf == 1 ? neg1 : 0u};
            const uint32_t xoff = sX + l32 * 16 + hf * 8;

            // ---- k (scaled), and K^T through the place of the dS tiles, zeros past the end
            U4 khi[2][KS], klo[2][KS], kt[2][2];
            f32x16 dk[2], dv[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    U4 kf = kraw[j][ks];
                    if (SPLIT) scale_split(kf, a.c_log2, khi[j][ks], klo[j][ks]);
                    else khi[j][ks] = scale_pow2(kf, cpow);
                    if (key0 + j * 32 + l32 >= ng) kf.u = make_uint4(0, 0, 0, 0);
                    const uint32_t at = sD + j * 2048 + l32 * 64 + hf * 8;
                    const auto unit = [&](int u) __attribute__((always_inline)) { return at + (u ^ ((l32 >> 2) & 3)) * 16; };
                    lds_write8(unit(ks), kf.u.x, kf.u.y);
                    lds_write8(unit(2 + ks), kf.u.z, kf.u.w);
                    if (KS == 1) {                    // rows 16 .. 31 of the product: never read
                        lds_write8(unit(1), 0u, 0u);
                        lds_write8(unit(3), 0u, 0u);
                    }
                }
                read_ds(kt[j][0], kt[j][1], j);
                dk[j] = f32x16{0};
                dv[j] = f32x16{0};
            }
            if (pass == 0) {
                __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): stages 0 and 1 have landed for every wave
                __syncthreads();
            }

            U4 q[KS], g[KS];                          // the A operands of a query tile's score products
            u32x2 xs, xd;                             // its rows' log-sum-exp and D
            uint32_t fat[KS], tre_at, tro_at;         // foff, tre, tro in the buffer of the stage at hand
            f32x16 s, acc;                            // the scores of the next tile; dQ^T of the query tile before over this wave's keys
            U4 qt0, qt1, gt0, gt1;                    // Q^T and dO^T of the query tile at hand
            auto write_part = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
                for (int blk = 0; blk < D / 8; ++blk)
                    lds_write16(pw + slot * (W * L::PART) + blk * 32, __float_as_uint(acc[4 * blk]), __float_as_uint(acc[4 * blk + 1]),
                                __float_as_uint(acc[4 * blk + 2]), __float_as_uint(acc[4 * blk + 3]));
            };
            // One unit of the pipeline: P = 2^s, dP, dS = P o dP of the current tile (key tile j) and its dV^T, dK^T products; the
            // scores of the NEXT tile and the dQ^T product of the SAME key tile one query tile ago in between, whose dS went through
            // LDS. j == 1: the next tile is the next query tile's, at byte `at` of the stage buffers, with entries `x`.
            auto unit = [&](auto jtag, const uint32_t* nat, uint32_t at, uint32_t x) __attribute__((always_inline)) {
                constexpr int j = decltype(jtag)::value, jn = 1 - j;
                U4 pb, db, d0, d1;
                f32x16 dp, sn;
                const auto probs = [&](int r0, int r1) __attribute__((always_inline)) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (r >= r0 && r < r1) s[r] = __builtin_amdgcn_exp2f(SPLIT ? s[r] : s[r] * cres);
                };
                const auto times = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
                    for (int r = r0; r < r0 + 4; ++r) dp[r] *= s[r];
                };
                const auto packs = [&](U4& to, const f32x16& x, int e0, int e1, int r0) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e >= e0 && e < e1) (&to.u.x)[e] = pack_bf16(x[r0 + 2 * e], x[r0 + 2 * e + 1]);
                };
                read_ds(d0, d1, j);                   // of the query tile before
                F3D_SB();
                dp = mfma_k8(xd, negD, f32x16{0});
                F3D_SB();
                probs(0, 4);
                F3D_SB();
                dp = mfma_bf16(g[0], vfr[j][0], dp);
                if (j == 1) {                         // behind the last use of the rows of the query tile at hand
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) q[ks].u = lds_read16(nat[ks] + at);
                    xs = lds_read8(x);
                }
                F3D_SB();
                probs(4, 7);
                F3D_SB();
                if (KS == 2) dp = mfma_bf16(g[KS - 1], vfr[j][KS - 1], dp);
                F3D_SB();
                probs(7, 8);
                packs(pb, s, 0, 4, 0);
                F3D_SB();
                dv[j] = mfma_bf16(gt0, pb, dv[j]);
                F3D_SB();
                probs(8, 11);
                F3D_SB();
                acc = mfma_bf16(kt[j][0], d0, j == 0 ? f32x16{0} : acc);
                F3D_SB();
                probs(11, 14);
                F3D_SB();
                acc = mfma_bf16(kt[j][1], d1, acc);
                F3D_SB();
                probs(14, 16);
                packs(pb, s, 0, 2, 8);
                F3D_SB();
                sn = mfma_k8(xs, negS, f32x16{0});
                F3D_SB();
                packs(pb, s, 2, 4, 8);
                times(0);
                F3D_SB();
                dv[j] = mfma_bf16(gt1, pb, dv[j]);
                F3D_SB();
                times(4);
                packs(db, dp, 0, 2, 0);
                F3D_SB();
                sn = mfma_bf16(q[0], khi[jn][0], sn);
                F3D_SB();
                packs(db, dp, 2, 4, 0);
                times(8);
                F3D_SB();
                dk[j] = mfma_bf16(qt0, db, dk[j]);
                lds_write16(dsw[0] + j * 2048, db.u.x, db.u.y, db.u.z, db.u.w);
                F3D_SB();
                times(12);
                packs(db, dp, 0, 2, 8);
                F3D_SB();
                sn = SPLIT ? mfma_bf16(q[0], klo[jn][0], sn) : mfma_bf16(q[KS - 1], khi[jn][KS - 1], sn);
                F3D_SB();
                packs(db, dp, 2, 4, 8);
                F3D_SB();
                dk[j] = mfma_bf16(qt1, db, dk[j]);
                lds_write16(dsw[1] + j * 2048, db.u.x, db.u.y, db.u.z, db.u.w);
                if (j == 1) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) g[ks].u = lds_read16(nat[ks] + at + L::AT_G);
                    xd = xs;
                }
                F3D_SB();
                s = sn;
            };
            // The waves' shares of the dQ of tile t, added in the order of the waves by the lower half of them; the sum over the passes so
            // far is kept in the workspace by the thread that goes on with it.
            const uint32_t keep = (uint32_t)((blockIdx.x * b.cap + rq) * D + 4 * rp);
            float4 before = {0.f, 0.f, 0.f, 0.f};
            int to = 0;                               // the row its dQ goes to
            auto prefetch = [&](int t) __attribute__((always_inline)) {
                if (t < 0 || !adds) return;
                if (last) {
                    to = seg_row_of(sm, seg_pre, seg_row0, min(t * 32 + rq, ng - 1));
                    if (a.out_perm) to = a.out_perm[to];
                }
                if (pass > 0) before = *reinterpret_cast<const float4*>(b.scratch + (keep + (uint32_t)((min(t * 32 + rq, ng - 1) - rq) * D)));
            };
            auto add_up = [&](int t, int slot) __attribute__((always_inline)) {
                if (t < 0 || !adds) return;
                const int x = t * 32 + rq;
                const uint32_t at = pr + slot * (W * L::PART);
                float4 sum = before;
                const auto add = [&](const uint4& v) __attribute__((always_inline)) {
                    sum.x += __uint_as_float(v.x);
                    sum.y += __uint_as_float(v.y);
                    sum.z += __uint_as_float(v.z);
                    sum.w += __uint_as_float(v.w);
                };
                if (nact == W) {
#pragma unroll
                    for (int w = 0; w < W; w += 4) {
                        uint4 v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = lds_read16(at + (w + e) * L::PART);
#pragma unroll
                        for (int e = 0; e < 4; ++e) add(v[e]);
                    }
                } else {
                    for (int w = 0; w < nact; ++w) add(lds_read16(at + w * L::PART));
                }
                if (x >= ng) return;
                if (!last) {
                    *reinterpret_cast<float4*>(b.scratch + (keep + (uint32_t)(t * 32 * D))) = sum;
                } else {
                    *reinterpret_cast<uint2*>(b.dq + (size_t)to * a.C + hoff + 4 * rp) =
                        make_uint2(pack_bf16(sum.x * b.scale, sum.y * b.scale), pack_bf16(sum.z * b.scale, sum.w * b.scale));
                }
            };

            if (active) {
                const uint32_t on = (uint32_t)(buf * L::BUF);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    fat[ks] = foff[ks] + on;
                    q[ks].u = lds_read16(fat[ks]);
                    g[ks].u = lds_read16(fat[ks] + L::AT_G);
                }
                tre_at = tre + on;
                tro_at = tro + on;
                xd = xs = lds_read8(xoff);
                s = mfma_k8(xs, negS, f32x16{0});
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    s = mfma_bf16(q[ks], khi[0][ks], s);
                    if (SPLIT) s = mfma_bf16(q[ks], klo[0][ks], s);
                }
            }
            // One query tile, the first (H == 0) or second of its stage. The tile behind the last is some rows in a buffer: its scores are never used.
            auto step = [&](auto htag, int t) __attribute__((always_inline)) {
                constexpr int H = decltype(htag)::value;
                prefetch(t - 1);
                if (active) {
                    read_tr<D>(gt0, gt1, tre_at + H * L::TILE + L::AT_G, tro_at + H * L::TILE + L::AT_G);
                    read_tr<D>(qt0, qt1, tre_at + H * L::TILE, tro_at + H * L::TILE);
                    unit(std::integral_constant<int, 0>{}, fat, 0, 0);
                }
                // The loading waves' part comes here, the adding waves' behind the barrier: of the two waves of a SIMD one goes on computing.
                if (loads && ((t >> 1) + 2 < nst || !last)) {
                    if (H == 0) fetch_rows((t >> 1) + 2 < nst ? (t >> 1) + 2 : (t >> 1) + 2 - nst);
                    else dma_stage(buf == 0 ? L::NBUF - 1 : buf - 1);   // everybody has left the stage before this one
                }
                if (active) {
                    const uint32_t x = xoff + (uint32_t)(min(t + 1, ntile - 1) * 512);
                    if (H == 1) {
                        const uint32_t on = (uint32_t)((buf + 1 == L::NBUF ? 0 : buf + 1) * L::BUF);
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) fat[ks] = foff[ks] + on;
                        tre_at = tre + on;
                        tro_at = tro + on;
                    }
                    unit(std::integral_constant<int, 1>{}, fat, H == 0 ? L::TILE : 0, x);
                    if (t > 0) write_part(1 - H);
                }
                if (loads && H == 0) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the next stage, requested a stage ago
                __syncthreads();
                add_up(t - 1, 1 - H);
            };
            for (int t = 0; t < ntile; t += 2) {
                step(std::integral_constant<int, 0>{}, t);
                if (t + 1 < ntile) step(std::integral_constant<int, 1>{}, t + 1);
                buf = buf + 1 == L::NBUF ? 0 : buf + 1;
            }
            if (loads && !last && (ntile & 1)) dma_stage(buf >= 2 ? buf - 2 : buf + 1);   // the second tile of the last stage would have
            prefetch(ntile - 1);
            if (!last) key_rows(pass + 1);
            // ---- where the gradients of this lane's rows go: 16-byte piece lc of rows lr, lr + 64 / NC .. of every tile
            constexpr int RL = 64 / NC, NR = 32 / RL;
            const int lr = ln / NC, lc = ln % NC;
            int drow[2][NR];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    const int x = key0 + j * 32 + lr + i * RL;
                    drow[j][i] = x < ng ? seg_row_of(sm, seg_pre, seg_row0, x) : -1;
                    if (x < ng && a.out_perm) drow[j][i] = a.out_perm[drow[j][i]];
                }
            }
            if (active) {
                acc = f32x16{0};
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    U4 d0, d1;
                    read_ds(d0, d1, j);
                    acc = mfma_bf16(kt[j][0], d0, acc);
                    acc = mfma_bf16(kt[j][1], d1, acc);
                }
                write_part((ntile - 1) & 1);
            }
            __syncthreads();
            add_up(ntile - 1, (ntile - 1) & 1);
            if (!last) load_keys();
            if (active) {                             // through the place of the dS tiles, so that a row's pieces are stored together
                auto store = [&](uint16_t* to_base, const f32x16& v, float mul, int place, const int* rows) __attribute__((always_inline)) {
                    const uint32_t at = sD + place * 2048;
                    const auto piece = [&](int row, int u) __attribute__((always_inline)) { return at + row * L::ROWB + (NC == 4 ? u ^ ((row >> 2) & 3) : u) * 16; };
#pragma unroll
                    for (int blk = 0; blk < D / 8; ++blk)
                        lds_write8(piece(l32, blk) + hf * 8, pack_bf16(v[4 * blk] * mul, v[4 * blk + 1] * mul), pack_bf16(v[4 * blk + 2] * mul, v[4 * blk + 3] * mul));
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        const uint4 x = lds_read16(piece(lr + i * RL, lc));
                        if (rows[i] >= 0) *reinterpret_cast<uint4*>(to_base + (size_t)rows[i] * a.C + hoff + lc * 8) = x;
                    }
                };
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    store(b.dk, dk[j], b.scale, 0, drow[j]);
                    store(b.dv, dv[j], 1.0f, 1, drow[j]);
                }
            }
        }
    }
}

template <int D>
size_t lds_of(int cap)
{
    return (size_t)OLay<D>::AT_X + (size_t)(cap + 63) / 64 * 64 * 16;
}

template <int D>
hipError_t launch_one(const AttnBwdArgs& b, int grid, hipStream_t stream)
{
    const hipError_t e = allow_lds((const void*)k_attn_bwd_one<D>, lds_of<D>(ATTN_BWD_ONE_ROWS));
    if (e != hipSuccess) return e;
    k_attn_bwd_one<D><<<(unsigned)grid, 64 * W, lds_of<D>(b.cap), stream>>>(b);
    return hipGetLastError();
}

}  // namespace

hipError_t attn_bwd_one_launch(const AttnBwdArgs& b, int head_dim, int grid, hipStream_t stream)
{
    return head_dim == 16 ? launch_one<16>(b, grid, stream) : launch_one<32>(b, grid, stream);
}

}  // namespace f3d
