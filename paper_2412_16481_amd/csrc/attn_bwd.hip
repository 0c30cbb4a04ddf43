// Backward of the Bucket-and-Swin attention (Section 4.2; the experiments report training latency) for gfx950.
//
//   S = scale Q K^T,  P = exp(S - lse),  dP = dO V^T,  D_i = sum_c dO_ic O_ic,  dS = P o (dP - D),
//   dQ = scale dS K,  dK = scale dS^T Q,  dV = P^T dO
// inside every scope, with the same scope -> row arithmetic as the forward kernel. P is recomputed from the
// forward's log-sum-exp; nothing of size n_g^2 ever leaves the registers.
//
// Two kernels, neither needs atomics; in both a wave owns 32 or 64 rows and the scope's other rows stream through LDS in
// row-major stages filled by global -> LDS loads (as in the forward kernel), from which the transposing LDS read
// delivers the transposed operands:
//   k_attn_bwd_dq    owns query rows, streams K and V, works out D on the way. Scores are computed transposed (keys x
//                    queries), so a lane owns 16 keys of ONE query: lse and D are per-lane scalars, and dS^T, packed to
//                    bf16, is directly the B operand of dQ^T += K^T dS^T.
//   k_attn_bwd_dkdv  owns key rows, streams Q and dO (after the first kernel: it reads D). Scores are queries x keys, so
//                    a lane owns 16 queries of ONE key: P and dS, packed to bf16, are the B operands of
//                    dV^T += dO^T P and dK^T += Q^T dS.
// Both recompute the exponentials. k_attn_bwd_one (attn_bwd_one.hip) computes each score once and takes most launches of long scopes;
// these two take short scopes, small launches, scopes of more than 2048 rows, gradients at other rows of the forward output, what that
// kernel leaves of a last round of tasks, and the launches that they are faster at (the rule and its figures: f3d_bucket_swin_attn_bwd).
//
// Bound: power and issue. On 914601 points x 8 heads x 32 (scopes of 1024) the dK/dV kernel kept the matrix core busy
// 61 % and the vector ALU 58 % of the cycles while the clock fell to 1.69 GHz, and ran 1.1 PFLOP/s of MFMAs (an 8192^3
// bf16 matrix product reaches 1.2 here); two MFMAs fewer per tile for 16 multiplies more then took it from 2.6 to 2.5 ms.
// Measured per pass on that input: dQ and D 2.57 -> 1.87 ms, dK/dV 3.19 -> 2.51 ms against staging through registers with
// a transposed copy written by 2-byte LDS stores (bank conflicts in every one of them), a separate pass for D and no
// overlap of one tile's products with another's exponentials; on 200000 points x 4 heads x 16: 0.199 -> 0.175 and
// 0.251 -> 0.232 ms. One row tile per wave at three waves per SIMD (dQ 2.06, dK/dV 3.30 ms) is slower there. In scopes of a
// few tiles latency is the bound instead, and a form of each kernel without the overlap, in fewer registers, puts three
// workgroups on a compute unit (the rule and its figures: f3d_bucket_swin_attn_bwd).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn.h"
#include "attn_bwd_common.h"

namespace f3d {

namespace {

// scope of a workgroup, shared by both kernels
struct ScopeCtx {
    int head, blk, ng;
    SegMap sm;
};

// REST: behind the tasks that one kernel has done already, the same number in the eighth of every XCD. A form of its own: reckoned with in every
// launch it made the two kernels 0.3 to 0.9 % slower (0.5 us of 60, 2.5 of 500).
template <int BM, bool REST>
__device__ __forceinline__ bool scope_of_block(const AttnBwdArgs& b, int blocks_per_scope, int* seg_row0, int* seg_pre, ScopeCtx& c)
{
    const AttnArgs& a = b.f;
    int slot;
    if (REST) {
        const int xcd = blockIdx.x & 7, u = xcd * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // as in block_of_grid
        int x = divide(u, blocks_per_scope, a.by_blocks);
        c.blk = u - x * blocks_per_scope;
        x += (xcd + 1) * b.done;
        slot = divide(x, a.H, a.by_h);
        c.head = x - slot * a.H;
    } else {
        block_of_grid(a, blocks_per_scope, slot, c.head, c.blk);
    }
    return slot < a.n_slots && scope_of_slot(a, slot, seg_row0, seg_pre, c.ng, c.sm) && c.blk * BM < c.ng;
}

// ------------------------------------------------------------------------------------------------
// D by itself, one row and head per thread, for calls whose dQ takes the place of the forward output and is stored at
// permuted rows: there a workgroup of the dQ kernel would read output rows that another has overwritten.
template <int D>
__global__ __launch_bounds__(256) void k_attn_bwd_d(AttnBwdArgs b)
{
    const AttnArgs& a = b.f;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long long)a.n * a.H) return;
    const size_t at = (size_t)(i / a.H) * a.C + (size_t)(i % a.H) * D;
    float dot = 0.f;
#pragma unroll
    for (int c = 0; c < D; c += 8) {
        const uint4 x = *reinterpret_cast<const uint4*>(a.out + at + c), y = *reinterpret_cast<const uint4*>(b.dout + at + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t p = (&x.x)[e], g = (&y.x)[e];
            dot += __uint_as_float(p << 16) * __uint_as_float(g << 16);
            dot += __uint_as_float(p & 0xFFFF0000u) * __uint_as_float(g & 0xFFFF0000u);
        }
    }
    b.dsum[i] = dot;
}

// ------------------------------------------------------------------------------------------------
// dQ, and on the way D, which the other kernel reads. A wave owns QT tiles of 32 query rows; K and V stream through LDS in
// stages of 128 key rows, three resident, as in the forward kernel. Scores are transposed (keys x queries), so a lane
// owns 16 keys of ONE query, its log-sum-exp is a scalar, and dS^T, packed to bf16, is the B operand of
// dQ^T += K^T dS^T, whose A operand comes from the row-major K through the transposing read.
// -D is the accumulator the dP product starts from, so dP - D costs nothing. The scaled score minus the log-sum-exp is
//   head_dim 32: one fused multiply-add per element on the product q k^T (6 MFMAs per tile), with as much of the factor in
//                q as is a power of two. The two more MFMAs the remainder of the scaled query would take cost the same issue
//                time, more registers and more power;
//   head_dim 16: the two-term query of the forward kernel with -lse as the starting accumulator (5 MFMAs per tile): there
//                the remainder is one MFMA, half the issue time of 16 multiply-adds.
// DF: D is there already (k_attn_bwd_d). AHEAD: the score products run a tile ahead; without, the form for short scopes
template <int D, int QT, bool DF, bool AHEAD, bool REST = false>
__global__ __launch_bounds__(256, AHEAD ? 2 : 3) void k_attn_bwd_dq(AttnBwdArgs b)
{
    using L = BLay<D>;
    constexpr bool SPLIT = D == 16;
    constexpr int NC = L::NC, KS = D / 16, LPW = L::LPW, SR = L::ROWS;
    constexpr int BM = 128 * QT;                      // query rows per workgroup
    __shared__ __attribute__((aligned(1024))) unsigned char smem[L::NBUF * 2 * L::BUF];   // K stages, then V stages
    __shared__ int s_row0[4][MAXSEG], s_pre[4][MAXSEG + 1];                               // of each wave
    const AttnArgs& a = b.f;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* const seg_row0 = s_row0[wave];
    int* const seg_pre = s_pre[wave];
    ScopeCtx sc;
    if (!scope_of_block<BM, REST>(b, a.qblocks, seg_row0, seg_pre, sc)) return;
    const int ng = sc.ng, head = sc.head;
    const SegMap sm = sc.sm;
    const int l32 = lane & 31, hf = lane >> 5;
    const size_t hoff = (size_t)head * D;
    const uint32_t row_bytes = (uint32_t)a.C * 2u;
    const uint32_t sK = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
    const uint32_t sV = sK + L::NBUF * L::BUF;

    // ---- staging of K and V rows (see the forward kernel); positions past the end fetch the scope's last row again
    uint32_t rows_next[LPW];
    const char* kthr[LPW];
    const char* vthr[LPW];
    int srow[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int p = (wave * LPW + i) * 64 + lane;
        const int kk = p / NC, cs = p % NC;
        const int c = (NC == 4) ? (cs ^ ((kk >> 2) & 3)) : (cs ^ ((kk >> 3) & 1));
        srow[i] = kk;
        kthr[i] = reinterpret_cast<const char*>(a.k + hoff + c * 8);
        vthr[i] = reinterpret_cast<const char*>(a.v + hoff + c * 8);
    }
    auto fetch_rows = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const uint32_t r = (uint32_t)seg_row_of(sm, seg_pre, seg_row0, min(st * SR + srow[i], ng - 1));
            rows_next[i] = a.perm ? (uint32_t)a.perm[r] : r;
        }
    };
    auto dma_stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const uint64_t at = (uint64_t)rows_next[i] * row_bytes;
            const int blk = wave * LPW + i;
            lds_dma16(kthr[i] + at, sK + buf * L::BUF + blk * 1024);
            lds_dma16(vthr[i] + at, sV + buf * L::BUF + blk * 1024);
        }
    };
    const int nst = (ng + SR - 1) / SR, ntile = (ng + 31) >> 5;
    int orow[QT];
    size_t qrd[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const int xq = sc.blk * BM + (wave * QT + t) * 32 + l32;
        orow[t] = xq < ng ? seg_row_of(sm, seg_pre, seg_row0, xq) : -1;
        const int r = max(orow[t], 0);                // past the end: some valid row, never stored
        qrd[t] = (size_t)(a.perm ? a.perm[r] : r);
    }
    fetch_rows(0);
    dma_stage(0);
    if (nst > 1) {
        fetch_rows(1);
        dma_stage(1);
    }

    // ---- this lane's queries: q and dO fragments, the log-sum-exp, and D = sum over the head's channels of dO * O
    U4 qhi[QT][KS], qlo[QT][KS], dof[QT][KS];
    f32x16 iS[QT], iD[QT], acc[QT];                   // starting accumulators: -lse (log2 units), -D
    float nl[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const size_t orw = (size_t)max(orow[t], 0);
        float dot = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            U4 qf, of;
            qf.u = *reinterpret_cast<const uint4*>(a.q + qrd[t] * a.C + hoff + ks * 16 + hf * 8);
            dof[t][ks].u = *reinterpret_cast<const uint4*>(b.dout + orw * a.C + hoff + ks * 16 + hf * 8);
            if (!DF) of.u = *reinterpret_cast<const uint4*>(a.out + orw * a.C + hoff + ks * 16 + hf * 8);
#pragma unroll
            for (int e = 0; e < 4 && !DF; ++e) {
                const uint32_t x = (&of.u.x)[e], y = (&dof[t][ks].u.x)[e];
                dot += __uint_as_float(x << 16) * __uint_as_float(y << 16);
                dot += __uint_as_float(x & 0xFFFF0000u) * __uint_as_float(y & 0xFFFF0000u);
            }
            if (SPLIT) scale_split(qf, a.c_log2, qhi[t][ks], qlo[t][ks]);
            else qhi[t][ks] = scale_pow2(qf, a.q_pow2);
        }
        dot += __shfl_xor(dot, 32, 64);               // the two half-waves hold the two halves of a row
        if (DF) dot = b.dsum[orw * a.H + head];
        else if (orow[t] >= 0 && hf == 0) b.dsum[orw * a.H + head] = dot;
        // past the end: probabilities exactly zero
        nl[t] = orow[t] >= 0 ? -LOG2E * a.lse[orw * a.H + head] : -1e30f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            iS[t][r] = nl[t];
            iD[t][r] = -dot;
        }
        acc[t] = f32x16{0};
    }

    uint32_t foff[KS];                                // row l32 of a tile, dims 16*ks + 8*hf ..
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int c = 2 * ks + hf;
        foff[ks] = (l32 * NC + ((NC == 4) ? (c ^ ((l32 >> 2) & 3)) : (c ^ ((l32 >> 3) & 1)))) * 16;
    }
    uint32_t tre, tro;
    tr_offsets<D>(lane, tre, tro);
    const float smul = a.s_mul;

    struct Rows { U4 k[KS], v[KS]; };                 // the A operands of one key tile's score products
    auto read_rows = [&](Rows& f, uint32_t at) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            f.k[ks].u = lds_read16(sK + at + foff[ks]);
            f.v[ks].u = lds_read16(sV + at + foff[ks]);
        }
    };
    // One unit of the pipeline: dS^T = P^T o (dP^T - D) of the current tile (query tile t, keys from kbase on) and its dQ^T
    // product, with the score products of the NEXT tile (rows f, query tile tn) issued in between.
    auto unit = [&](f32x16& s, f32x16& dp, int t, int kbase, const U4& kt0, const U4& kt1, f32x16& sn, f32x16& dpn, const Rows& f, int tn)
        __attribute__((always_inline)) {
        const auto prob = [&](int r) __attribute__((always_inline)) {
            s[r] = __builtin_amdgcn_exp2f(SPLIT ? s[r] : __builtin_fmaf(s[r], smul, nl[t]));
        };
        if (kbase + 32 > ng) {                        // keys past the end repeat a key of the scope: their dS is dropped here
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kbase + 8 * (r >> 2) + 4 * hf + (r & 3);
                if (key >= ng) dp[r] = 0.f;
            }
        }
        U4 pb;
        F3D_SB();
#pragma unroll
        for (int r = 0; r < 4; ++r) prob(r);
        F3D_SB();
        sn = mfma_bf16(f.k[0], qhi[tn][0], SPLIT ? iS[tn] : f32x16{0});
        F3D_SB();
#pragma unroll
        for (int r = 4; r < 8; ++r) prob(r);
        F3D_SB();
        sn = SPLIT ? mfma_bf16(f.k[0], qlo[tn][0], sn) : mfma_bf16(f.k[KS - 1], qhi[tn][KS - 1], sn);
        F3D_SB();
#pragma unroll
        for (int r = 0; r < 8; ++r) dp[r] *= s[r];
#pragma unroll
        for (int e = 0; e < 4; ++e) (&pb.u.x)[e] = pack_bf16(dp[2 * e], dp[2 * e + 1]);
        F3D_SB();
        acc[t] = mfma_bf16(kt0, pb, acc[t]);
        F3D_SB();
#pragma unroll
        for (int r = 8; r < 12; ++r) prob(r);
        F3D_SB();
        dpn = mfma_bf16(f.v[0], dof[tn][0], iD[tn]);
        F3D_SB();
#pragma unroll
        for (int r = 12; r < 16; ++r) prob(r);
        F3D_SB();
        if (KS == 2) dpn = mfma_bf16(f.v[KS - 1], dof[tn][KS - 1], dpn);
        F3D_SB();
#pragma unroll
        for (int r = 8; r < 16; ++r) dp[r] *= s[r];
#pragma unroll
        for (int e = 0; e < 4; ++e) (&pb.u.x)[e] = pack_bf16(dp[8 + 2 * e], dp[8 + 2 * e + 1]);
        F3D_SB();
        acc[t] = mfma_bf16(kt1, pb, acc[t]);
        F3D_SB();
    };
    auto handover = [&](int st) __attribute__((always_inline)) {      // as in the forward kernel
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
        if (st + 2 < nst) {
            dma_stage((st + 2) % L::NBUF);
            if (st + 3 < nst) fetch_rows(st + 3);
        }
    };

    __builtin_amdgcn_s_waitcnt(0x0F70);       // stages 0 and 1 have landed for every wave
    __syncthreads();
    if (nst > 2) fetch_rows(2);

    if (!AHEAD) {
        static_assert(AHEAD || QT == 1, "one tile per wave");
        for (int st = 0, buf = 0; st < nst; ++st, buf = buf + 1 == L::NBUF ? 0 : buf + 1) {
#pragma unroll 1
            for (int t4 = 0; t4 < 4 && 4 * st + t4 < ntile; ++t4) {
                const uint32_t at = buf * L::BUF + t4 * L::TILE;
                const int kbase = st * SR + t4 * 32;
                Rows f;
                read_rows(f, at);
                U4 kt0, kt1, p0, p1;
                read_tr<D>(kt0, kt1, sK + at + tre, sK + at + tro);
                f32x16 s = SPLIT ? iS[0] : f32x16{0}, dp = iD[0];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    s = mfma_bf16(f.k[ks], qhi[0][ks], s);
                    if (SPLIT) s = mfma_bf16(f.k[ks], qlo[0][ks], s);
                    dp = mfma_bf16(f.v[ks], dof[0][ks], dp);
                }
                if (kbase + 32 > ng) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (kbase + 8 * (r >> 2) + 4 * hf + (r & 3) >= ng) dp[r] = 0.f;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) dp[r] *= __builtin_amdgcn_exp2f(SPLIT ? s[r] : __builtin_fmaf(s[r], smul, nl[0]));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    (&p0.u.x)[e] = pack_bf16(dp[2 * e], dp[2 * e + 1]);
                    (&p1.u.x)[e] = pack_bf16(dp[8 + 2 * e], dp[8 + 2 * e + 1]);
                }
                acc[0] = mfma_bf16(kt0, p0, acc[0]);
                acc[0] = mfma_bf16(kt1, p1, acc[0]);
                if (t4 == 1) handover(st);
            }
        }
        store_grad_rows<D>(b.dq, a.out_perm, orow[0], a.C, hoff, hf, acc[0], b.scale);
        return;
    }
    f32x16 sa, sb, da, db;
    Rows f;
    read_rows(f, 0);
    sa = SPLIT ? iS[0] : f32x16{0};
    da = iD[0];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        sa = mfma_bf16(f.k[ks], qhi[0][ks], sa);
        if (SPLIT) sa = mfma_bf16(f.k[ks], qlo[0][ks], sa);
        da = mfma_bf16(f.v[ks], dof[0][ks], da);
    }
    if (QT == 1) read_rows(f, L::TILE);
    int bufi = 0;
    for (int st = 0; st < nst; ++st) {
        const int bufn = bufi + 1 == L::NBUF ? 0 : bufi + 1;
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            if (4 * st + t4 >= ntile) break;          // the products computed ahead of the last tile are never used
            const uint32_t at = bufi * L::BUF + t4 * L::TILE;
            const int kbase = st * SR + t4 * 32;
            U4 kt0, kt1;
            read_tr<D>(kt0, kt1, sK + at + tre, sK + at + tro);
            if (QT == 1) {                            // the score registers alternate from one key tile to the next
                Rows fn;
                read_rows(fn, t4 < 2 ? at + 2 * L::TILE : bufn * L::BUF + (t4 - 2) * L::TILE);
                if ((t4 & 1) == 0) unit(sa, da, 0, kbase, kt0, kt1, sb, db, f, 0);
                else unit(sb, db, 0, kbase, kt0, kt1, sa, da, f, 0);
                f = fn;
            } else {                                  // a is query tile 0, b query tile 1 of the same key tile
                unit(sa, da, 0, kbase, kt0, kt1, sb, db, f, QT - 1);
                read_rows(f, t4 < 3 ? at + L::TILE : bufn * L::BUF);
                unit(sb, db, QT - 1, kbase, kt0, kt1, sa, da, f, 0);
            }
            if (t4 == 1) handover(st);
        }
        bufi = bufn;
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) store_grad_rows<D>(b.dq, a.out_perm, orow[t], a.C, hoff, hf, acc[t], b.scale);
}

// ------------------------------------------------------------------------------------------------
// dK and dV. A wave owns KTW tiles of 32 key rows; the scope's query rows stream through LDS in stages of 128, three
// of them resident, filled by global -> LDS loads two stages ahead exactly as the forward kernel fills its K and V.
// Q and dO are kept once, row-major: the rows of the score products come from 16-byte reads (pieces of a row
// xor-swizzled by the row, free of bank conflicts), and Q^T, dO^T, the A operands of dK^T += Q^T dS and
// dV^T += dO^T P, from the transposing read, which follows the same swizzle.
// The vector ALU (16 exponentials, 16 or 32 multiplies and 16 packs per tile and lane) and the matrix core (10 MFMAs at
// head_dim 32) are both busy, so the loop runs one score tile ahead: the products of the next tile are issued between
// the exponentials, multiplies and packs of the current one.
template <int D, int KTW, bool AHEAD, bool REST = false>
__global__ __launch_bounds__(256, AHEAD ? 2 : 3) void k_attn_bwd_dkdv(AttnBwdArgs b)
{
    using L = BLay<D>;
    constexpr bool SPLIT = D == 16;
    constexpr int NC = L::NC, KS = D / 16, LPW = L::LPW, SR = L::ROWS;
    constexpr int BM = 128 * KTW;                     // key rows per workgroup
    __shared__ __attribute__((aligned(1024))) unsigned char smem[L::NBUF * 2 * L::BUF];   // Q stages, then dO stages
    __shared__ uint2 sx[L::NBUF * SR];                // per staged row {lse hi, lo, D hi, lo}, see split_pairs
    __shared__ int s_row0[4][MAXSEG], s_pre[4][MAXSEG + 1];                               // of each wave
    const AttnArgs& a = b.f;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* const seg_row0 = s_row0[wave];
    int* const seg_pre = s_pre[wave];
    ScopeCtx sc;
    if (!scope_of_block<BM, REST>(b, b.kblocks, seg_row0, seg_pre, sc)) return;
    const int ng = sc.ng, head = sc.head;
    const SegMap sm = sc.sm;
    const int l32 = lane & 31, hf = lane >> 5;
    const size_t hoff = (size_t)head * D;
    const uint32_t row_bytes = (uint32_t)a.C * 2u;
    const uint32_t sQ = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
    const uint32_t sG = sQ + L::NBUF * L::BUF;
    const uint32_t sX = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)sx;

    // ---- staging: load i of this lane fills piece (wave*LPW + i)*64 + lane of a stage (row = piece / NC), with the piece
    //      of that row the swizzle puts there. q rows go through the permutation, dO rows are bucket-major. Positions past
    //      the end of the scope fetch its last row again: finite, and their probabilities are exactly zero (lse = 1e30).
    uint32_t qrow_next[LPW], grow_next[LPW];
    const char* qthr[LPW];
    const char* gthr[LPW];
    int srow[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int p = (wave * LPW + i) * 64 + lane;
        const int kk = p / NC, cs = p % NC;
        const int c = (NC == 4) ? (cs ^ ((kk >> 2) & 3)) : (cs ^ ((kk >> 3) & 1));
        srow[i] = kk;
        qthr[i] = reinterpret_cast<const char*>(a.q + hoff + c * 8);
        gthr[i] = reinterpret_cast<const char*>(b.dout + hoff + c * 8);
    }
    int cexp = 0;
    const float cres = SPLIT ? 1.0f : 2.0f * frexpf(a.c_log2, &cexp);   // c_log2 = cres * 2^(cexp - 1), 1 <= |cres| < 2
    const float cpow = SPLIT ? 1.0f : ldexpf(1.0f, cexp - 1), lmul = LOG2E / cres;
    float lreg = 0.f, dreg = 0.f;                     // log-sum-exp and D of row `tid` of the stage fetched last
    auto fetch_rows = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int x = min(st * SR + srow[i], ng - 1);
            const uint32_t r = (uint32_t)seg_row_of(sm, seg_pre, seg_row0, x);
            grow_next[i] = r;
            qrow_next[i] = a.perm ? (uint32_t)a.perm[r] : r;
        }
        if (tid < SR) {
            const int x = st * SR + tid;
            const size_t at = (size_t)seg_row_of(sm, seg_pre, seg_row0, min(x, ng - 1)) * a.H + head;
            const float l = a.lse[at], d = b.dsum[at];
            lreg = x < ng ? l : 1e30f;
            dreg = x < ng ? d : 0.f;
        }
    };
    auto dma_stage = [&](int buf) __attribute__((always_inline)) {   // the rows fetched last -> LDS buffer `buf`
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int blk = wave * LPW + i;
            lds_dma16(qthr[i] + (uint64_t)qrow_next[i] * row_bytes, sQ + buf * L::BUF + blk * 1024);
            lds_dma16(gthr[i] + (uint64_t)grow_next[i] * row_bytes, sG + buf * L::BUF + blk * 1024);
        }
        if (tid < SR) sx[buf * SR + tid] = split_pairs(lreg * lmul, dreg);
    };
    const int nst = (ng + SR - 1) / SR, ntile = (ng + 31) >> 5;
    int krow[KTW];
    size_t krd[KTW];
#pragma unroll
    for (int j = 0; j < KTW; ++j) {
        const int xk = sc.blk * BM + (wave * KTW + j) * 32 + l32;
        krow[j] = xk < ng ? seg_row_of(sm, seg_pre, seg_row0, xk) : -1;
        const int r = max(krow[j], 0);                // past the end: some valid row, never stored
        krd[j] = (size_t)(a.perm ? a.perm[r] : r);
    }
    fetch_rows(0);
    dma_stage(0);
    if (nst > 1) {
        fetch_rows(1);
        dma_stage(1);
    }
    if (nst > 2) fetch_rows(2);

    // ---- this lane's keys: k (scaled, split) and v fragments
    // head_dim 32: k times the power of two below the factor (exact), and what is left of the factor, 1 <= cres < 2, is a
    // multiply behind the product; the staged log-sum-exp is divided by it
    U4 khi[KTW][KS], klo[KTW][KS], vfr[KTW][KS];
    U4 negS, negD;   // B operands with -1 at the positions of a staged row's log-sum-exp pair / D pair
    negS.u = make_uint4(hf == 0 ? 0xBF80BF80u : 0u, 0, 0, 0);
    negD.u = make_uint4(0, hf == 0 ? 0xBF80BF80u : 0u, 0, 0);
#pragma unroll
    for (int j = 0; j < KTW; ++j) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            U4 kf;
            kf.u = *reinterpret_cast<const uint4*>(a.k + krd[j] * a.C + hoff + ks * 16 + hf * 8);
            vfr[j][ks].u = *reinterpret_cast<const uint4*>(a.v + krd[j] * a.C + hoff + ks * 16 + hf * 8);
            if (SPLIT) scale_split(kf, a.c_log2, khi[j][ks], klo[j][ks]);
            else khi[j][ks] = scale_pow2(kf, cpow);
        }
    }

    // ---- this lane's fragment addresses inside a buffer
    uint32_t foff[KS];                                // row l32 of a tile, dims 16*ks + 8*hf ..
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int c = 2 * ks + hf;
        foff[ks] = (l32 * NC + ((NC == 4) ? (c ^ ((l32 >> 2) & 3)) : (c ^ ((l32 >> 3) & 1)))) * 16;
    }
    uint32_t tre, tro;
    tr_offsets<D>(lane, tre, tro);

    f32x16 dk[KTW], dv[KTW];
#pragma unroll
    for (int j = 0; j < KTW; ++j) {
        dk[j] = f32x16{0};
        dv[j] = f32x16{0};
    }

    struct Rows { U4 q[KS], g[KS], x; };              // the A operands of one query tile's score products
    auto read_rows = [&](Rows& f, uint32_t at, uint32_t xat) __attribute__((always_inline)) {   // tile at byte `at`, entries at `xat`
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            f.q[ks].u = lds_read16(sQ + at + foff[ks]);
            f.g[ks].u = lds_read16(sG + at + foff[ks]);
        }
        const u32x2 e = *(const __attribute__((address_space(3))) u32x2*)(uintptr_t)(sX + xat + l32 * 8);
        f.x.u = make_uint4(e.x, e.y, 0, 0);
    };
    // One unit of the pipeline: P = 2^s, dS = P o dp of the current tile (key tile j) and its dV^T, dK^T products, with
    // the products of the NEXT tile (rows f, key tile jn) issued in between.
    auto unit = [&](f32x16& s, f32x16& dp, int j, const U4& qt0, const U4& qt1, const U4& gt0, const U4& gt1, f32x16& sn, f32x16& dpn,
                    const Rows& f, int jn) __attribute__((always_inline)) {
        U4 pb, db;
        const auto prob = [&](int r) __attribute__((always_inline)) { s[r] = __builtin_amdgcn_exp2f(SPLIT ? s[r] : s[r] * cres); };
        F3D_SB();
#pragma unroll
        for (int r = 0; r < 4; ++r) prob(r);
        F3D_SB();
        sn = mfma_bf16(f.x, negS, f32x16{0});
        F3D_SB();
#pragma unroll
        for (int r = 4; r < 8; ++r) prob(r);
        F3D_SB();
        sn = mfma_bf16(f.q[0], khi[jn][0], sn);
        F3D_SB();
#pragma unroll
        for (int e = 0; e < 4; ++e) (&pb.u.x)[e] = pack_bf16(s[2 * e], s[2 * e + 1]);
#pragma unroll
        for (int r = 8; r < 10; ++r) prob(r);
        F3D_SB();
        dv[j] = mfma_bf16(gt0, pb, dv[j]);
        F3D_SB();
#pragma unroll
        for (int r = 10; r < 12; ++r) prob(r);
#pragma unroll
        for (int r = 0; r < 4; ++r) dp[r] *= s[r];
        F3D_SB();
        if (SPLIT) sn = mfma_bf16(f.q[0], klo[jn][0], sn);
        else sn = mfma_bf16(f.q[KS - 1], khi[jn][KS - 1], sn);
        F3D_SB();
#pragma unroll
        for (int r = 4; r < 8; ++r) dp[r] *= s[r];
        prob(12);
        F3D_SB();
        dpn = mfma_bf16(f.x, negD, f32x16{0});
        F3D_SB();
#pragma unroll
        for (int e = 0; e < 4; ++e) (&db.u.x)[e] = pack_bf16(dp[2 * e], dp[2 * e + 1]);
        F3D_SB();
        dk[j] = mfma_bf16(qt0, db, dk[j]);
        F3D_SB();
#pragma unroll
        for (int r = 13; r < 16; ++r) prob(r);
        F3D_SB();
        if (KS == 2) dpn = mfma_bf16(f.g[0], vfr[jn][0], dpn);
        F3D_SB();
#pragma unroll
        for (int e = 0; e < 4; ++e) (&pb.u.x)[e] = pack_bf16(s[8 + 2 * e], s[8 + 2 * e + 1]);
        F3D_SB();
        dv[j] = mfma_bf16(gt1, pb, dv[j]);
        F3D_SB();
#pragma unroll
        for (int r = 8; r < 12; ++r) dp[r] *= s[r];
        F3D_SB();
#pragma unroll
        for (int r = 12; r < 16; ++r) dp[r] *= s[r];
        F3D_SB();
        dpn = mfma_bf16(f.g[KS - 1], vfr[jn][KS - 1], dpn);
        F3D_SB();
#pragma unroll
        for (int e = 0; e < 4; ++e) (&db.u.x)[e] = pack_bf16(dp[8 + 2 * e], dp[8 + 2 * e + 1]);
        F3D_SB();
        dk[j] = mfma_bf16(qt1, db, dk[j]);
        F3D_SB();
    };
    // Hands stage st+1 over to the readers and refills the buffer of stage st-1 with stage st+2: every wave waits for its
    // own loads of stage st+1 (issued a stage ago) and meets the others; whoever arrives has read the last of stage st-1.
    // The rows' log-sum-exp and D are written behind the barrier, one whole stage before they are read.
    auto handover = [&](int st) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
        if (st + 2 < nst) {
            dma_stage((st + 2) % L::NBUF);
            if (st + 3 < nst) fetch_rows(st + 3);
        }
    };

    __builtin_amdgcn_s_waitcnt(0x0F70);       // stages 0 and 1 have landed for every wave
    __syncthreads();

    if (!AHEAD) {
        static_assert(AHEAD || KTW == 1, "one tile per wave");
        for (int st = 0, buf = 0; st < nst; ++st, buf = buf + 1 == L::NBUF ? 0 : buf + 1) {
#pragma unroll 1
            for (int t4 = 0; t4 < 4 && 4 * st + t4 < ntile; ++t4) {
                const uint32_t at = buf * L::BUF + t4 * L::TILE;
                Rows f;
                read_rows(f, at, (buf * SR + t4 * 32) * 8);
                U4 qt0, qt1, gt0, gt1, p0, p1, d0, d1;
                f32x16 s = mfma_bf16(f.x, negS, f32x16{0}), dp = mfma_bf16(f.x, negD, f32x16{0});
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    s = mfma_bf16(f.q[ks], khi[0][ks], s);
                    if (SPLIT) s = mfma_bf16(f.q[ks], klo[0][ks], s);
                    dp = mfma_bf16(f.g[ks], vfr[0][ks], dp);
                }
                read_tr<D>(gt0, gt1, sG + at + tre, sG + at + tro);
                read_tr<D>(qt0, qt1, sQ + at + tre, sQ + at + tro);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    s[r] = __builtin_amdgcn_exp2f(SPLIT ? s[r] : s[r] * cres);
                    dp[r] *= s[r];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    (&p0.u.x)[e] = pack_bf16(s[2 * e], s[2 * e + 1]);
                    (&p1.u.x)[e] = pack_bf16(s[8 + 2 * e], s[8 + 2 * e + 1]);
                    (&d0.u.x)[e] = pack_bf16(dp[2 * e], dp[2 * e + 1]);
                    (&d1.u.x)[e] = pack_bf16(dp[8 + 2 * e], dp[8 + 2 * e + 1]);
                }
                dv[0] = mfma_bf16(gt0, p0, dv[0]);
                dv[0] = mfma_bf16(gt1, p1, dv[0]);
                dk[0] = mfma_bf16(qt0, d0, dk[0]);
                dk[0] = mfma_bf16(qt1, d1, dk[0]);
                if (t4 == 1) handover(st);
            }
        }
        store_grad_rows<D>(b.dk, a.out_perm, krow[0], a.C, hoff, hf, dk[0], b.scale);
        store_grad_rows<D>(b.dv, a.out_perm, krow[0], a.C, hoff, hf, dv[0], 1.0f);
        return;
    }
    f32x16 sa, sb, da, db;
    Rows f;
    read_rows(f, 0, 0);
    sa = mfma_bf16(f.x, negS, f32x16{0});
    da = mfma_bf16(f.x, negD, f32x16{0});
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        sa = mfma_bf16(f.q[ks], khi[0][ks], sa);
        if (SPLIT) sa = mfma_bf16(f.q[ks], klo[0][ks], sa);
        da = mfma_bf16(f.g[ks], vfr[0][ks], da);
    }
    if (KTW == 1) read_rows(f, L::TILE, 32 * 8);
    int bufi = 0;
    for (int st = 0; st < nst; ++st) {
        const int bufn = bufi + 1 == L::NBUF ? 0 : bufi + 1;
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            if (4 * st + t4 >= ntile) break;          // the products computed ahead of the last tile are never used
            const uint32_t at = bufi * L::BUF + t4 * L::TILE;
            U4 qt0, qt1, gt0, gt1;
            read_tr<D>(gt0, gt1, sG + at + tre, sG + at + tro);
            read_tr<D>(qt0, qt1, sQ + at + tre, sQ + at + tro);
            if (KTW == 1) {                           // the score registers alternate from one query tile to the next
                Rows fn;
                read_rows(fn, t4 < 2 ? at + 2 * L::TILE : bufn * L::BUF + (t4 - 2) * L::TILE,
                          (t4 < 2 ? bufi * SR + (t4 + 2) * 32 : bufn * SR + (t4 - 2) * 32) * 8);
                if ((t4 & 1) == 0) unit(sa, da, 0, qt0, qt1, gt0, gt1, sb, db, f, 0);
                else unit(sb, db, 0, qt0, qt1, gt0, gt1, sa, da, f, 0);
                f = fn;
            } else {                                  // a is key tile 0, b key tile 1 of the same query tile
                unit(sa, da, 0, qt0, qt1, gt0, gt1, sb, db, f, KTW - 1);
                read_rows(f, t4 < 3 ? at + L::TILE : bufn * L::BUF, (t4 < 3 ? bufi * SR + (t4 + 1) * 32 : bufn * SR) * 8);
                unit(sb, db, KTW - 1, qt0, qt1, gt0, gt1, sa, da, f, 0);
            }
            if (t4 == 1) handover(st);
        }
        bufi = bufn;
    }
#pragma unroll
    for (int j = 0; j < KTW; ++j) {
        store_grad_rows<D>(b.dk, a.out_perm, krow[j], a.C, hoff, hf, dk[j], b.scale);
        store_grad_rows<D>(b.dv, a.out_perm, krow[j], a.C, hoff, hf, dv[j], 1.0f);
    }
}

template <int D>
hipError_t launch_d(const AttnBwdArgs& b, hipStream_t stream)
{
    const AttnArgs& a = b.f;
    // with tasks done already: whole ones, the same number on every XCD, of long scopes (one tile per wave, D not in front)
    const long long left = b.done ? b.tasks - 8ll * b.done : (long long)a.n_slots * a.H;
    long long total = left * a.qblocks;
    total = (total + 7) / 8 * 8;
    if (total > 0 && b.d_first) {
        k_attn_bwd_d<D><<<(unsigned)(((long long)a.n * a.H + 255) / 256), 256, 0, stream>>>(b);
        if (b.tiles == 2) k_attn_bwd_dq<D, 2, true, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else k_attn_bwd_dq<D, 1, true, true><<<(unsigned)total, 256, 0, stream>>>(b);
    } else if (total > 0) {
        if (b.done) k_attn_bwd_dq<D, 1, false, true, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else if (b.tiles == 2) k_attn_bwd_dq<D, 2, false, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else if (b.ahead) k_attn_bwd_dq<D, 1, false, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else k_attn_bwd_dq<D, 1, false, false><<<(unsigned)total, 256, 0, stream>>>(b);
    }
    total = left * b.kblocks;
    total = (total + 7) / 8 * 8;
    if (total > 0) {
        if (b.done) k_attn_bwd_dkdv<D, 1, true, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else if (b.tiles == 2) k_attn_bwd_dkdv<D, 2, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else if (b.ahead) k_attn_bwd_dkdv<D, 1, true><<<(unsigned)total, 256, 0, stream>>>(b);
        else k_attn_bwd_dkdv<D, 1, false><<<(unsigned)total, 256, 0, stream>>>(b);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t attn_bwd_launch(const AttnBwdArgs& b, int head_dim, hipStream_t stream)
{
    return head_dim == 16 ? launch_d<16>(b, stream) : launch_d<32>(b, stream);
}

}  // namespace f3d
