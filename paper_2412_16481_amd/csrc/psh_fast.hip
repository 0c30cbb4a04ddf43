// PSH bucketing, short-latency path for scans whose [chunk][bucket] count matrix is small (all of the
// paper's operating range: ~1e5 points per scan, a few hundred buckets).
//
// Same schedule and same results as psh.hip (Algorithms 1 and 2 in lock step, index-ordered), but one
// launch per step instead of two: a workgroup ranks a chunk of 2048 (1024) points, writes one row of 16-bit
// counts, and in the NEXT launch every workgroup sums the rows it needs by itself (rows of earlier
// chunks rebase its local ranks, all rows give the new fill levels), so no separate scan kernel and no
// second round trip through the launch queue.
//
// At these sizes the kernels are bound by memory LATENCY and launch boundaries, not bandwidth: every
// kernel is written as "one load that tells the workgroup what to do, then all other loads at once,
// then arithmetic".
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "launch.h"
#include "psh_common.h"

namespace f3d {

namespace {

// Points per workgroup, CH in the kernels below: FCH, and SCH for batches that are small in every way (psh_fast_chunk).
constexpr int FCH = 2048;
constexpr int SCH = 1024;
constexpr int FTH = 512;     // threads per workgroup of the set-up kernels
constexpr int FW = FTH / 64; // waves
constexpr int FKMAX = 2048;           // most buckets per scan on this path
constexpr long long FMATMAX = 131072; // most (chunks of a scan) x (buckets of a scan)
constexpr int SCHUNKS = 256;          // most chunks of SCH points
constexpr uint32_t KEY_WAIT = KEY_PLACED - 1;   // no contender's: a key ends below 2^(11 + LR_BITS)
constexpr int CFGW = (int)(sizeof(ScanCfg) / 4);
static_assert(sizeof(ScanCfg) <= 128 && sizeof(ScanCfg) % 4 == 0, "the workspace reserves 128 bytes per scan");

struct ChunkInfo {
    int b, lc, nc, begin, end, kb0, K, c0;
};
__device__ __forceinline__ ChunkInfo load_chunk(const PshArgs& a, int chunk)
{
    const int4 u = a.chunk_info[2 * chunk], v = a.chunk_info[2 * chunk + 1];
    return ChunkInfo{u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
}

// row pitch of the count matrix in 32-bit words (two 16-bit counts per word), rows 16-byte aligned
__host__ __device__ inline int row_pitch(int kcap) { return (((kcap + 1) >> 1) + 3) & ~3; }

// Words per column group of the sums in LDS: bucket k lies at (k & 7) * pitch + (k >> 3), so that threads of neighbouring column
// groups (eight buckets each) add to neighbouring words, and with 8 modulo 64 neighbouring buckets lie in banks of their own too.
__host__ __device__ inline int group_pitch(int kcap) { return ((((kcap + 7) >> 3) + 55) & ~63) + 8; }

// ------------------------------------------------------------------------------------------------
// per-scan bounding box
__global__ __launch_bounds__(FTH) void k_pshf_minmax(PshArgs a)
{
    constexpr int FPPT = FCH / FTH;
    const ChunkInfo ci = load_chunk(a, blockIdx.x);
    if (ci.b < 0 || a.status[0]) return;
    const int b = ci.b;
    uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
    const float* src = a.coords + (size_t)ci.begin * 3;
    const int nf = (ci.end - ci.begin) * 3;
    float v[3 * FPPT];
#pragma unroll
    for (int j = 0; j < 3 * FPPT; ++j) {   // all twelve loads in flight together
        const int f = threadIdx.x + j * FTH;
        v[j] = f < nf ? src[f] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 3 * FPPT; ++j) {
        const int f = threadIdx.x + j * FTH;
        if (f < nf) {
            const uint32_t o = f2ord(v[j]);
            const int ax = f % 3;
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (ax == t) { mn[t] = min(mn[t], o); mx[t] = max(mx[t], o); }
        }
    }
    __shared__ uint32_t red[8];
    if (threadIdx.x < 3) { red[threadIdx.x] = 0xFFFFFFFFu; red[4 + threadIdx.x] = 0u; }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        uint32_t lo = mn[t], hi = mx[t];
        lo = wave_min(lo);
        hi = wave_max(hi);
        if ((threadIdx.x & 63) == 0) { atomicMin(&red[t], lo); atomicMax(&red[4 + t], hi); }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        atomicMin(&a.mm[b * 8 + threadIdx.x], red[threadIdx.x]);
        atomicMax(&a.mm[b * 8 + 4 + threadIdx.x], red[4 + threadIdx.x]);
    }
}

// ------------------------------------------------------------------------------------------------
// Set-up and bounding boxes in ONE launch, for batches of at most 64 scans. The scan tables (first point, first bucket,
// first chunk of every scan) are a closed form of batch_offsets and S: every workgroup works them out itself (one
// wave, a prefix over the scans), finds its chunk and writes the chunk's own box, without atomics, so nothing has to
// be initialised by an earlier launch; step 0 joins the boxes of a scan's chunks. Workgroup 0 also writes the tables
// the later kernels read.
constexpr int SETUP_MAX_SCANS = 64;

template <int CH>
__global__ __launch_bounds__(FTH) void k_pshf_setup(PshArgs a)
{
    constexpr int FPPT = CH / FTH;
    __shared__ int s_p0[SETUP_MAX_SCANS + 1], s_kb0[SETUP_MAX_SCANS + 1], s_c0[SETUP_MAX_SCANS + 1];
    __shared__ int s_bad;
    __shared__ uint32_t red[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ns = a.n_scans;
    if (wave == 0) {
        int p0 = 0, K = 0, c = 0;
        bool ok = true;
        if (lane < ns) {
            p0 = batch_off(a, lane);
            const int p1 = batch_off(a, lane + 1);
            const long long nb = (long long)p1 - p0;
            ok = nb >= 0 && nb <= a.max_scan_points && p0 >= 0 && p1 <= a.n;
            if (lane == 0 && p0 != 0) ok = false;
            if (lane == ns - 1 && p1 != a.n) ok = false;
            if (ok) {
                K = (int)((nb + a.S - 1) / a.S);
                c = (int)((nb + CH - 1) / CH);
            }
        }
        const bool bad = __builtin_amdgcn_ballot_w64(!ok) != 0ull;
        const int kin = wave_incl_scan(K), cin = wave_incl_scan(c);
        if (lane < ns) {
            s_p0[lane] = p0;
            s_kb0[lane] = kin - K;
            s_c0[lane] = cin - c;
        }
        if (lane == ns - 1) {
            s_p0[ns] = a.n;
            s_kb0[ns] = kin;
            s_c0[ns] = cin;
        }
        if (lane == 0) s_bad = bad ? 1 : 0;
    }
    __syncthreads();
    const int isbad = s_bad, ktot = s_kb0[ns], ctot = s_c0[ns];
    if (blockIdx.x == 0) {   // the tables of the later kernels
        if (tid < ns) {
            a.sbs[tid] = s_kb0[tid];
            a.scan_c0[tid] = s_c0[tid];
            a.scan_p0[tid] = s_p0[tid];
            a.done[tid] = 0;
        }
        if (tid == 0) {
            a.sbs[ns] = isbad ? -1 : ktot;
            a.scan_c0[ns] = isbad ? 0 : ctot;
            a.scan_p0[ns] = a.n;
            a.status[0] = isbad;
        }
        if (tid < 8) a.round_count[tid] = 0;
        if (!isbad) {
            // first row of every bucket (buckets are full except the last of a scan); a wave takes a scan
            for (int b = wave; b < ns; b += FW) {
                const int p0 = s_p0[b], nb = s_p0[b + 1] - p0, kb0 = s_kb0[b], K = s_kb0[b + 1] - kb0;
                for (int j = lane; j < K; j += 64) {
                    a.offsets[kb0 + j] = p0 + min(j * a.S, nb);
                    a.cnt[kb0 + j] = 0;
                }
            }
            for (int j = ktot + tid; j <= a.max_buckets; j += FTH) a.offsets[j] = a.n;
        }
    }
    const int chunk = blockIdx.x;
    if (isbad || chunk >= ctot) {
        if (tid == 0) a.chunk_info[2 * chunk] = make_int4(-1, 0, 0, 0);
        return;
    }
    // the chunk's scan: the last one that starts at or before it (scans without points have no chunks)
    const int b = __popcll(__builtin_amdgcn_ballot_w64(lane < ns && s_c0[lane] <= chunk)) - 1;
    const int p0 = s_p0[b], p1 = s_p0[b + 1], c0 = s_c0[b], lc = chunk - c0;
    const int begin = p0 + lc * CH, end = min(begin + CH, p1);
    if (tid == 0) {
        a.chunk_info[2 * chunk] = make_int4(b, lc, s_c0[b + 1] - c0, begin);
        a.chunk_info[2 * chunk + 1] = make_int4(end, s_kb0[b], s_kb0[b + 1] - s_kb0[b], c0);
    }
    uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
    const float* src = a.coords + (size_t)begin * 3;
    const int nf = (end - begin) * 3;
    float v[3 * FPPT];
#pragma unroll
    for (int j = 0; j < 3 * FPPT; ++j) {   // all twelve loads in flight together
        const int f = tid + j * FTH;
        v[j] = f < nf ? src[f] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 3 * FPPT; ++j) {
        const int f = tid + j * FTH;
        if (f < nf) {
            const uint32_t o = f2ord(v[j]);
            const int ax = f % 3;
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (ax == t) { mn[t] = min(mn[t], o); mx[t] = max(mx[t], o); }
        }
    }
    if (tid < 3) { red[tid] = 0xFFFFFFFFu; red[4 + tid] = 0u; }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        uint32_t lo = mn[t], hi = mx[t];
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0) { atomicMin(&red[t], lo); atomicMax(&red[4 + t], hi); }
    }
    __syncthreads();
    if (tid < 3) {
        a.mmpart[chunk * 8 + tid] = red[tid];
        a.mmpart[chunk * 8 + 4 + tid] = red[4 + tid];
    }
}

// ------------------------------------------------------------------------------------------------
// step r: settle step r-1 from the count rows of that step, then rank the contenders of step r
// dynamic LDS: tot[8][gp] + pre[8][gp] ints + NW x kwp words of packed 16-bit counters.
// TH threads rank the CH points of a chunk: 512 and 2048 (four points each, two workgroups per CU) when the grid is
// larger than the GPU, 1024 threads (two points each: every phase of the step is half as long) when it is not, 1024 and 1024
// (one point each) when the count rows stay few enough.
// A point whose probe meets a full bucket is no contender: it waits for the next step (KEY_WAIT) unranked, and groups of 64
// without a contender, most of them on surfaces, go past the ranks. (The bucketing of 914601 points in eight scans took 122 us
// without that and takes 114, of 457295 in four 92 and 89.)
// LAST (r = n_probes + 1) settles the last probe and recycles in the same launch: the r-th leftover of a scan takes the r-th
// free slot (buckets ascending, slots ascending). The count rows that settle a step also say how many of the earlier chunks'
// contenders it turns away, and with those that waited all along (`left`) that is every leftover before this chunk, so nobody has
// to count them in a launch of its own (a forward pass over a room of 200000 points 334 -> 322 us, the canonical order of
// 457295 points 250 -> 239).
template <int CH, int TH, bool LAST>
__global__ __launch_bounds__(TH) void k_pshf_step(PshArgs a, int r, const uint32_t* __restrict__ mat_prev,
                                                   uint32_t* __restrict__ mat_cur)
{
    constexpr int NW = TH / 64, PPT = CH / TH, KPT_ = FKMAX / TH;
    extern __shared__ int smem[];
    __shared__ ScanCfg cfg;
    __shared__ int placed_ct, recycled_ct, left_before;
    __shared__ int lds17[17];
    const int chunk = blockIdx.x;
    // One scan: its chunks follow from what the launch knows, and nothing waits for the table (a scan's points are all n, so its buckets are
    // kcap; where the offsets say otherwise the status does too, which is looked at behind the loads; a bound below n is refused in any case,
    // and n then says nothing about how many rows there are to sum). us per bucketing, with the table and the
    // status waited for in front: 20000 points 60 -> 56, 130000 72.7 -> 68, 200000 89.8 -> 86.6; 457295 in four scans 78.6 -> 77.
    const ChunkInfo ci = a.n_scans == 1 && a.max_scan_points >= a.n ? ChunkInfo{chunk * CH < a.n ? 0 : -1, chunk, (a.n + CH - 1) / CH, chunk * CH, min(chunk * CH + CH, a.n), 0, a.kcap, 0}
                                        : load_chunk(a, chunk);
    const int bad = a.status[0];                    // looked at behind the loads: in a flagged call the table names no chunk
    if (ci.b < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int K = ci.K, kb0 = ci.kb0, lc = ci.lc, nc = ci.nc;
    const int kwp = row_pitch(a.kcap);
    const int gp = group_pitch(a.kcap);
    int* tot = smem;                                // contenders of step r-1 per bucket, all chunks
    int* pre = smem + 8 * gp;                       // ... of earlier chunks; then rebased fill level
    uint32_t* wh = (uint32_t*)(smem + 16 * gp);     // [NW][kwp]
    const auto of = [gp](int k) { return (k & 7) * gp + (k >> 3); };   // place of bucket k in tot and pre

    // ---- every global load of this kernel is issued here, before anything waits
    uint32_t box[8];
    uint32_t cfgw = 0;
    if (r == 0) {
        if (a.mmpart) {   // the boxes of the scan's chunks, joined by the first wave
            if (wave == 0) {
                uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
                for (int t = lane; t < ci.nc; t += 64) {
                    const uint32_t* pb = a.mmpart + (size_t)(ci.c0 + t) * 8;
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) { lo[ax] = min(lo[ax], pb[ax]); hi[ax] = max(hi[ax], pb[4 + ax]); }
                }
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    lo[ax] = wave_min(lo[ax]);
                    hi[ax] = wave_max(hi[ax]);
                    box[ax] = lo[ax];
                    box[4 + ax] = hi[ax];
                }
            }
        } else if (tid == 0) {
            for (int i = 0; i < 8; ++i) box[i] = a.mm[ci.b * 8 + i];
        }
    } else if (tid < CFGW) {
        cfgw = reinterpret_cast<const uint32_t*>(reinterpret_cast<const ScanCfg*>(a.cfg) + ci.b)[tid];
    }
    uint32_t kwv[PPT];
    float cx[PPT], cy[PPT], cz[PPT];
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int i = ci.begin + wave * (CH / NW) + s * 64 + lane;
        kwv[s] = KEY_PLACED;
        cx[s] = cy[s] = cz[s] = 0.f;
        if (i < ci.end) {
            kwv[s] = r > 0 ? a.key[i] : 0u;
            if (!LAST) {
                const float* c = a.coords + (size_t)i * 3;
                cx[s] = c[0]; cy[s] = c[1]; cz[s] = c[2];
            }
        }
    }
    // Count rows of step r-1, 16 bytes (8 buckets) per load: thread (g, seg) sums column group g over
    // rows seg, seg+nseg, ... in registers; the row segments are joined in LDS afterwards.
    // This was the longest part of a step: counts unpacked one by one (28 instructions a load, 12 now) and joined in words eight
    // apart, sixteen lanes to a bank. The whole bucketing of 200000 points in one scan 103 -> 94 us, of 457295 in four 102 -> 91. With twelve
    // rows a thread whatever there are, most threads added up zeros: as many as are likely to be there, and threads without a row out
    // of the joining, 200000 points 89.3 -> 88.2 us, 457295 83 -> 77.5, 914601 in eight 108 -> 106, one scan of 9000 58.5 -> 54.8 (joining
    // without a branch per word, but by all threads: 73.9). Eleven and twelve rows in two goes of ten are no faster than with twelve for
    // all: 215000 points 97.9 us, 93.9 in one go.
    const int G = (((K + 1) >> 1) + 3) >> 2;        // column groups in use (<= 256)
    const int nseg = TH / G, seg = tid / G, g = tid - seg * G;
    int tl[8], pl[8], cntv[KPT_], waited = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) { tl[e] = 0; pl[e] = 0; }
    if (r > 0) {
        // LB rows of a thread in flight: a row fetch costs a trip to the HBM-side cache
        auto sum_rows = [&](auto most) __attribute__((always_inline)) {
            const uint4* col = reinterpret_cast<const uint4*>(mat_prev + (size_t)ci.c0 * kwp) + g;
            const int pitch4 = kwp >> 2;
            constexpr int LB = decltype(most)::value;
            for (int c = seg; c < nc; c += LB * nseg) {
                static_assert(LB * CH < 65536, "sums of packed counts");
                uint4 v[LB];
                uint32_t t2[4] = {0u, 0u, 0u, 0u}, p2[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < LB; ++j) {
                    const int cj = c + j * nseg;
                    v[j] = cj < nc ? col[(size_t)cj * pitch4] : make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < LB; ++j) {
                    const uint32_t before = (c + j * nseg) < lc ? ~0u : 0u;
                    const uint32_t w4[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {   // two counts per word: a count is at most 2048 and LB of them stay below 2^16
                        t2[e] += w4[e];
                        p2[e] += w4[e] & before;
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    tl[2 * e] += (int)(t2[e] & 0xFFFFu);
                    tl[2 * e + 1] += (int)(t2[e] >> 16);
                    pl[2 * e] += (int)(p2[e] & 0xFFFFu);
                    pl[2 * e + 1] += (int)(p2[e] >> 16);
                }
            }
        };
        if (seg < min(nseg, nc)) {
            if (nc <= 4 * nseg) sum_rows(std::integral_constant<int, 4>{});
            else if (nc <= 7 * nseg) sum_rows(std::integral_constant<int, 7>{});
            else if (nc > 10 * nseg && nc <= 12 * nseg) sum_rows(std::integral_constant<int, 12>{});
            else sum_rows(std::integral_constant<int, 10>{});
        }
#pragma unroll
        for (int j = 0; j < KPT_; ++j) cntv[j] = (tid + j * TH < K) ? a.cnt[kb0 + tid + j * TH] : 0;
        if (LAST)
            for (int c = tid; c < lc; c += TH) waited += a.left[ci.c0 + c];
    }

    if (bad) return;
    // ---- LDS set-up while the loads fly
    for (int w = (r > 0 ? 0 : 4 * gp) + tid; w < 4 * gp + NW * (kwp >> 2); w += TH) reinterpret_cast<int4*>(smem)[w] = make_int4(0, 0, 0, 0);
    if (tid == 0) placed_ct = recycled_ct = left_before = 0;
    if (r == 0) {
        if (tid == 0) {
            compute_cfg(a, ci.b, box, cfg);   // a hundred-odd instructions on one lane
            if (lc == 0) reinterpret_cast<ScanCfg*>(a.cfg)[ci.b] = cfg;   // later steps load it
        }
    } else if (tid < CFGW) {
        reinterpret_cast<uint32_t*>(&cfg)[tid] = cfgw;
    }
    __syncthreads();
    if (r > 0) {
        if (seg < min(nseg, nc)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // counts past the last bucket are zero
                atomicAdd(&tot[e * gp + g], tl[e]);
                atomicAdd(&pre[e * gp + g], pl[e]);
            }
        }
        __syncthreads();
        // fill level before step r-1 plus earlier chunks' contenders = first rank of this chunk's contenders;
        // chunk 0 of the scan also publishes the fill level after step r-1
#pragma unroll
        for (int j = 0; j < KPT_; ++j) {
            const int k = tid + j * TH;
            if (k < K) {
                const int base = cntv[j];
                if (!LAST) {
                    const int cap = k == K - 1 ? cfg.lastcap : a.S, filled = min(base + tot[of(k)], cap);
                    if (lc == 0) a.cnt_next[kb0 + k] = filled;
                    tot[of(k)] = cap - filled;      // the room for step r
                    pre[of(k)] += base;
                }
            }
        }
        __syncthreads();
    }

    if constexpr (LAST) {
        // per bucket: the fill level when the probes are through, the free slots before it in the scan; and the contenders of
        // earlier chunks that found no room
        int* const fill = reinterpret_cast<int*>(wh);
        int* const freepre = tot;
        int carry = 0, turned = waited;
#pragma unroll
        for (int j = 0; j < KPT_; ++j) {
            if (j * TH < K) {
                const int k = tid + j * TH;
                int v = 0;
                if (k < K) {
                    const int room = (k == K - 1 ? cfg.lastcap : a.S) - cntv[j];
                    const int taken = min(tot[of(k)], room);
                    v = room - taken;
                    fill[k] = cntv[j] + taken;
                    turned += max(pre[of(k)] - room, 0);
                    pre[of(k)] += cntv[j];
                }
                int t2;
                const int before = block_excl_scan(v, &t2, lds17);
                if (k < K) freepre[of(k)] = carry + before;
                carry += t2;
            }
        }
        turned = wave_sum(turned);
        if (lane == 0 && turned) atomicAdd(&left_before, turned);
        __syncthreads();
        unsigned long long rest[PPT];
        int nplaced = 0, nrest = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const int i = ci.begin + wave * (CH / NW) + s * 64 + lane;
            bool left = i < ci.end && kwv[s] != KEY_PLACED;
            if (left && kwv[s] != KEY_WAIT) {
                const int hp = (int)(kwv[s] >> LR_BITS);
                const int rank = pre[of(hp)] + (int)(kwv[s] & ((1u << LR_BITS) - 1));
                if (rank < (hp == K - 1 ? cfg.lastcap : a.S)) {
                    const int dst = cfg.p0 + hp * a.S + rank;
                    a.inv_perm[i] = dst;
                    a.perm[dst] = i;
                    left = false;
                    ++nplaced;
                }
            }
            rest[s] = __builtin_amdgcn_ballot_w64(left);
            nrest += __popcll(rest[s]);
        }
        if (lane == 0) lds17[wave] = nrest;
        __syncthreads();
        int at = left_before;
        for (int v = 0; v < wave; ++v) at += lds17[v];
        int nrec = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const int i = ci.begin + wave * (CH / NW) + s * 64 + lane;
            if ((rest[s] >> lane) & 1ull) {
                const int rank = at + bits_below(rest[s]);
                int lo = 0, hi = K;  // largest j with freepre[j] <= rank
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (freepre[of(mid)] <= rank) lo = mid; else hi = mid;
                }
                const int off = lo * a.S + fill[lo] + (rank - freepre[of(lo)]);
                if (off >= 0 && off < cfg.nb) {   // always, while capacities add up to the scan size
                    a.inv_perm[i] = cfg.p0 + off;
                    a.perm[cfg.p0 + off] = i;
                    ++nrec;
                }
            }
            at += __popcll(rest[s]);
        }
        // one atomic per workgroup: hundreds of waves adding to the same counter queue up behind each other
        nplaced = wave_sum(nplaced);
        nrec = wave_sum(nrec);
        if (lane == 0 && nplaced) atomicAdd(&placed_ct, nplaced);
        if (lane == 0 && nrec) atomicAdd(&recycled_ct, nrec);
        __syncthreads();
        if (tid == 0 && placed_ct) atomicAdd(&a.round_count[r - 1], placed_ct);
        if (tid == 0 && recycled_ct) atomicAdd(&a.round_count[r], recycled_ct);
        return;
    }

    const int keybits = max(1, 32 - __clz(max(K - 1, 1)));
    int hh[PPT], wl[PPT];
    bool act[PPT];
    int nplaced = 0, nwait = 0;
    // accept what fits from step r-1, hash what is left for step r
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int i = ci.begin + wave * (CH / NW) + s * 64 + lane;
        bool active = i < ci.end;
        int h = 0;
        if (active && r > 0) {
            const uint32_t kv = kwv[s];
            if (kv == KEY_PLACED) {
                active = false;
            } else if (kv != KEY_WAIT) {
                const int hp = (int)(kv >> LR_BITS), lr = (int)(kv & ((1u << LR_BITS) - 1));
                const int rank = pre[of(hp)] + lr;
                const int cap = (hp == K - 1) ? cfg.lastcap : a.S;
                if (rank < cap) {
                    const int dst = cfg.p0 + hp * a.S + rank;
                    a.inv_perm[i] = dst;
                    a.perm[dst] = i;
                    a.key[i] = KEY_PLACED;
                    active = false;
                    ++nplaced;
                }
            }
        }
        if (active) {
            int x = voxel_of(cx[s], cfg.mn[0], a.inv_voxel);
            int y = voxel_of(cy[s], cfg.mn[1], a.inv_voxel);
            int z = voxel_of(cz[s], cfg.mn[2], a.inv_voxel);
            if (r > 0) probe_voxel(a, r, cfg, x, y, z);
            h = hash_bucket(a.hash, x, y, z, cfg);
            if (r > 0 && tot[of(h)] == 0) {
                if (kwv[s] != KEY_WAIT) a.key[i] = KEY_WAIT;
                active = false;
                ++nwait;
            }
        }
        act[s] = active;
        hh[s] = h;
    }
    // rank inside the chunk: ballots inside the wave, per-wave LDS counters across the wave's four steps
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int h = hh[s];
        const bool active = act[s];
        int old = 0;
        if (__builtin_amdgcn_ballot_w64(active) == 0ull) {
            hh[s] = -1;
            continue;
        }
        const unsigned long long m = match_key(h, active, keybits);
        // every lane reads its bucket's counter (half a word), the first of each bucket advances it (see wave_ranks for the barriers):
        // one trip to LDS, not an add that returns and a shuffle behind it (200000 points 90.4 -> 89.3 us)
        uint16_t* const counter = reinterpret_cast<uint16_t*>(wh + wave * kwp) + h;
        const int before = bits_below(m);
        old = (int)*counter + before;
        __builtin_amdgcn_wave_barrier();
        if (active && before == 0) *counter = (uint16_t)(old + __popcll(m));
        __builtin_amdgcn_wave_barrier();
        if (!active) hh[s] = -1;
        wl[s] = old;
    }
    __syncthreads();
    // join the waves: exclusive prefix over the waves per bucket; the total is this chunk's row
    for (int w = tid; w < kwp; w += TH) {
        uint32_t run = 0, t[NW];
        if (2 * w < K) {
#pragma unroll
            for (int v = 0; v < NW; ++v) t[v] = wh[v * kwp + w];
#pragma unroll
            for (int v = 0; v < NW; ++v) {
                wh[v * kwp + w] = run;
                run += t[v];  // halves cannot carry into each other: a chunk has at most 2048 points
            }
        }
        mat_cur[(size_t)chunk * kwp + w] = run;   // padding words of the row are written as zero
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int i = ci.begin + wave * (CH / NW) + s * 64 + lane;
        if (hh[s] >= 0) {
            const int h = hh[s];
            const int base = (int)((wh[wave * kwp + (h >> 1)] >> ((h & 1) * 16)) & 0xFFFFu);
            a.key[i] = ((uint32_t)h << LR_BITS) | (uint32_t)(base + wl[s]);
        }
    }
    if (r > 0) {
        int n2 = nplaced | (nwait << 16);     // a chunk has at most 2048 points
        n2 = wave_sum(n2);
        if (lane == 0 && n2) atomicAdd(&placed_ct, n2);
        __syncthreads();
        if (tid == 0 && (placed_ct & 0xFFFF)) atomicAdd(&a.round_count[r - 1], placed_ct & 0xFFFF);
    }
    if (r == a.n_probes && tid == 0) a.left[chunk] = placed_ct >> 16;
}

}  // namespace

bool psh_fast_eligible(long long max_scan_points, int kcap)
{
    const long long nc = (max_scan_points + FCH - 1) / FCH;
    return kcap <= FKMAX && nc * kcap <= FMATMAX;
}

// A step of a small batch is instruction issue on the workgroups there are and two round trips to memory: with half the points per
// workgroup the hash, the rank and the accept of a step take half as long, while the GPU has compute units to spare.
// Against that every workgroup sums twice as many count rows, hence the limit on rows times buckets. us per bucketing with 2048 /
// 1024 points: 9000 points 76 / 63, 60000 84 / 72, 130000 (64000 counts) 87 / 78, 2 x 100000 87 / 76; 100000 points in buckets
// of 64 (153000 counts) 98 / 97, 200000 points (153000 counts) 94 / 100, 4 x 114000 (448 chunks) 91 / 99.
int psh_fast_chunk(long long n, int n_scans, long long max_scan_points, int kcap, bool half)
{
    const long long nc = (max_scan_points + SCH - 1) / SCH;
    return half && kcap <= FKMAX && n_scans <= SETUP_MAX_SCANS && n / SCH + n_scans <= SCHUNKS && nc * kcap <= FMATMAX ? SCH : FCH;
}

// Rows of the chunk tables and of a count matrix. Whether a batch takes chunks of 1024 points depends on n, the scans and the
// buckets, and one point more can halve its chunks: rows for the chunks of the batch itself would make a workspace that holds
// for n points too small for fewer. There are rows for the most chunks any batch of up to so many points and scans takes.
long long psh_fast_chunks(long long n, int n_scans) { return n / FCH + n_scans; }
long long psh_fast_most_chunks(long long n, int n_scans)
{
    const long long full = psh_fast_chunks(n, n_scans), halves = n / SCH + n_scans, bounded = halves < SCHUNKS ? halves : SCHUNKS;
    return full > bounded ? full : bounded;
}

size_t psh_fast_matrix_bytes(long long chunks, int kcap)
{
    return (size_t)2 * (size_t)chunks * row_pitch(kcap) * 4;
}

namespace {

inline size_t step_lds_bytes(int threads, int kcap) { return (size_t)group_pitch(kcap) * 64 + (size_t)(threads / 64) * row_pitch(kcap) * 4; }

template <int CH, int TH>
hipError_t launch_steps(PshArgs a, int chunks, hipStream_t stream)
{
    const int kwp = row_pitch(a.kcap);
    const size_t lds = step_lds_bytes(TH, a.kcap);
    if (lds > 60000) {
        for (const void* fn : {(const void*)k_pshf_step<CH, TH, false>, (const void*)k_pshf_step<CH, TH, true>}) {
            const hipError_t e = allow_lds(fn, step_lds_bytes(TH, FKMAX));
            if (e != hipSuccess) return e;
        }
    }
    uint32_t* mat[2] = {reinterpret_cast<uint32_t*>(a.hist), reinterpret_cast<uint32_t*>(a.hist) + (size_t)chunks * kwp};
    int32_t* c0 = a.cnt;
    int32_t* c1 = a.cnt_next;
    for (int r = 0; r <= a.n_probes; ++r) {
        a.cnt = c0;
        a.cnt_next = c1;
        k_pshf_step<CH, TH, false><<<chunks, TH, lds, stream>>>(a, r, mat[(r + 1) & 1], mat[r & 1]);
        if (r > 0) { int32_t* t = c0; c0 = c1; c1 = t; }  // step r wrote the fill levels after step r-1
    }
    a.cnt = c0;
    const int r = a.n_probes + 1;
    k_pshf_step<CH, TH, true><<<chunks, TH, lds, stream>>>(a, r, mat[(r + 1) & 1], nullptr);
    return hipGetLastError();
}

}  // namespace

hipError_t psh_fast_launch(const PshArgs& args, hipStream_t stream)   // args.chunk: psh_fast_chunk
{
    PshArgs a = args;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    if (a.chunk == SCH && a.n / SCH + a.n_scans > cus) a.chunk = FCH;
    const int chunks = (int)(a.n / a.chunk) + a.n_scans;  // upper bound, surplus workgroups exit
    a.n_chunks_ub = chunks;
    if (a.n_scans <= SETUP_MAX_SCANS && a.n > 0) {
        if (a.chunk == SCH) k_pshf_setup<SCH><<<chunks, FTH, 0, stream>>>(a);
        else k_pshf_setup<FCH><<<chunks, FTH, 0, stream>>>(a);
    } else {
        a.mmpart = nullptr;
        k_psh_meta<<<1, 1024, 0, stream>>>(a);
        if (a.n == 0) return hipGetLastError();
        k_pshf_minmax<<<chunks, FTH, 0, stream>>>(a);
    }
    if (a.chunk == SCH) return launch_steps<SCH, 1024>(a, chunks, stream);
    return chunks <= cus ? launch_steps<FCH, 1024>(a, chunks, stream) : launch_steps<FCH, 512>(a, chunks, stream);
}

}  // namespace f3d
