// PSH bucketing, small scans: ONE workgroup per scan with every point of the scan in registers.
//
// Same schedule and same results as the other paths (lock step, contenders served by input index). A scan of at most
// 4096 points (four per thread) fits a workgroup of 1024 threads with its points' packed voxels in registers for all steps, so a step is
// a hash, a rank and an accept without a read or write of global memory and without a launch boundary; the one
// read of the coordinates also gives the bounding box, and with a single scan the tables and bucket offsets are written
// here too, so that the whole bucketing is one launch.
//
// A wave owns up to 64*PPT consecutive points and visits them in index order, 64 at a time: rank inside the 64 from
// ballots over the key bits, contenders before them in the wave from per-wave LDS counters (packed two per word),
// contenders in earlier waves from a prefix over the waves per bucket. The counters and the fill levels are
// double-buffered, the idle copy is cleared between two barriers of a step. When fewer groups of 64 would hold what a step
// leaves, the points left are closed up through LDS in index order, so later steps visit only what is left.
//
// Bound: instruction issue and the chain of hash, ballots, LDS atomics and three barriers per step on ONE compute unit
// (about 300 instructions per visit of 64 points), not memory. That is also where the line to the other paths
// lies: at 4096 points a scan takes 33-43 us here (buckets of 256 and 32 rows) against 77-82 us with one launch per step
// and 49-55 us in psh_scan.hip, 1500 points 26-29 against 70-75 and 40-42, 600 scans of 4096 points 106-136 against
// 295-323 and 141-160. The crossing with one launch per step lies beyond: with eight points per thread and most of them left to
// the recycle step, where nothing is closed up, 8192 points took 82-96 us against 80-84. The sizes between are not
// served here.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "psh_common.h"

namespace f3d {

namespace {

constexpr int MTH = 1024;          // threads per workgroup
constexpr int MNW = MTH / 64;      // waves
constexpr int PPT = 4;             // points per thread at most

// dynamic LDS, in 32-bit words: fill[2][K] wh[2][MNW][kw] list[3][MTH * PPT], with kw = (K + 1) / 2
__global__ __launch_bounds__(MTH) void k_pshs_small(PshArgs a)
{
    extern __shared__ int smem[];
    __shared__ ScanCfg cfg;
    __shared__ uint32_t red[8];
    __shared__ int s_round[8];
    __shared__ int s_left[2][MNW];
    __shared__ int lds17[17];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x;
    const bool single = a.n_scans == 1;
    int p0, nb, kb0, K;
    if (single) {                      // no set-up launch: the checks and tables of k_psh_meta for one scan
        p0 = batch_off(a, 0);
        const int p1 = batch_off(a, 1);
        const bool bad = p0 != 0 || p1 != a.n || (long long)a.n > a.max_scan_points;
        nb = bad ? 0 : a.n;
        kb0 = 0;
        K = (nb + a.S - 1) / a.S;
        if (tid == 0) {
            a.sbs[0] = 0;
            a.sbs[1] = bad ? -1 : K;
            a.status[0] = bad ? 1 : 0;
        }
        if (bad) {
            if (tid < 8) a.round_count[tid] = 0;
            return;
        }
        for (int j = tid; j <= a.max_buckets; j += MTH) a.offsets[j] = j < K ? j * a.S : a.n;
    } else {
        if (a.status[0]) return;       // inconsistent batch offsets: flagged by the set-up kernel, nothing to do
        p0 = a.scan_p0[b];
        nb = a.scan_p0[b + 1] - p0;
        kb0 = a.sbs[b];
        K = a.sbs[b + 1] - kb0;
        if (nb <= 0 || K <= 0) return;
        for (int j = tid; j < K; j += MTH) a.offsets[kb0 + j] = p0 + min(j * a.S, nb);
    }
    const int kw = (K + 1) >> 1;
    int* fillb = smem;
    uint32_t* whb = reinterpret_cast<uint32_t*>(smem + 2 * K);
    uint32_t* list = whb + 2 * MNW * kw;              // index, voxel low, voxel high

    // ---- the points, the bounding box. A wave owns 64*grp consecutive ones.
    int grp = (nb + MTH - 1) / MTH;
    const int i0 = wave * (64 * grp) + lane;          // this lane's points: i0, i0 + 64, ..
    float cx[PPT], cy[PPT], cz[PPT];
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const float* c = a.coords + (size_t)(p0 + min(i0 + 64 * s, nb - 1)) * 3;   // past the end: the last point again
        cx[s] = c[0];
        cy[s] = c[1];
        cz[s] = c[2];
    }
    if (tid < 8) {
        red[tid] = tid < 4 ? 0xFFFFFFFFu : 0u;
        s_round[tid] = 0;
    }
    for (int k = tid; k < K; k += MTH) fillb[k] = 0;
    for (int w = tid; w < MNW * kw; w += MTH) whb[w] = 0u;
    __syncthreads();
    {
        uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const uint32_t o[3] = {f2ord(cx[s]), f2ord(cy[s]), f2ord(cz[s])};
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                mn[t] = min(mn[t], o[t]);
                mx[t] = max(mx[t], o[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            for (int d = 32; d >= 1; d >>= 1) {
                mn[t] = min(mn[t], (uint32_t)__shfl_xor((int)mn[t], d, 64));
                mx[t] = max(mx[t], (uint32_t)__shfl_xor((int)mx[t], d, 64));
            }
            if (lane == 0) {
                atomicMin(&red[t], mn[t]);
                atomicMax(&red[4 + t], mx[t]);
            }
        }
    }
    __syncthreads();
    if (tid == 0) compute_cfg_of(a, p0, nb, kb0, K, red, cfg);
    __syncthreads();

    int idx[PPT];                                     // index inside the scan
    uint32_t vlo[PPT], vhi[PPT];                      // packed voxel: x | y << 21 | z << 42
    uint32_t left = 0;                                // bit s: point s is not placed yet
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const unsigned long long v = (unsigned long long)(uint32_t)voxel_of(cx[s], cfg.mn[0], a.inv_voxel) |
                                     ((unsigned long long)(uint32_t)voxel_of(cy[s], cfg.mn[1], a.inv_voxel) << 21) |
                                     ((unsigned long long)(uint32_t)voxel_of(cz[s], cfg.mn[2], a.inv_voxel) << 42);
        vlo[s] = (uint32_t)v;
        vhi[s] = (uint32_t)(v >> 32);
        idx[s] = i0 + 64 * s;
        if (s < grp && idx[s] < nb) left |= 1u << s;
    }

    const int keybits = max(1, 32 - __clz(max(K - 1, 1)));
    int cur = 0, rest = nb;                           // rest: points not placed yet
    for (int r = 0; r <= a.n_probes; ++r) {
        uint32_t* wh = whb + cur * MNW * kw;
        uint32_t* mine = wh + wave * kw;
        int hk[PPT];                                  // bucket | rank among the wave's contenders << 16
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const bool act = (left >> s) & 1u;
            hk[s] = 0;
            if (__builtin_amdgcn_ballot_w64(act) == 0ull) continue;
            const unsigned long long v = (unsigned long long)vlo[s] | ((unsigned long long)vhi[s] << 32);
            int x = (int)(v & 0x1FFFFFull), y = (int)((v >> 21) & 0x1FFFFFull), z = (int)(v >> 42);
            if (r > 0) probe_voxel(a, r, cfg, x, y, z);
            const int h = hash_bucket(a.hash, x, y, z, cfg);
            const unsigned long long m = match_key(h, act, keybits);
            if (act) {
                const int leader = __ffsll((long long)m) - 1;
                int old = 0;
                if (lane == leader) {
                    const int sh = (h & 1) * 16;
                    old = (int)((atomicAdd(&mine[h >> 1], (uint32_t)__popcll(m) << sh) >> sh) & 0xFFFFu);
                }
                old = __shfl(old, leader, 64) + bits_below(m);
                hk[s] = h | (old << 16);
            }
        }
        __syncthreads();
        // ---- contenders in earlier waves (in place), fill levels after this step; the other counters are cleared
        const int* fill = fillb + cur * K;
        int* fill_next = fillb + (cur ^ 1) * K;
        uint32_t* wh_next = whb + (cur ^ 1) * MNW * kw;
        for (int w = tid; w < kw; w += MTH) {
            uint32_t run = 0;
#pragma unroll
            for (int v = 0; v < MNW; ++v) {
                const uint32_t t = wh[v * kw + w];
                wh[v * kw + w] = run;
                wh_next[v * kw + w] = 0u;
                run += t;                             // halves cannot carry into each other: at most 4096 points
            }
            const int k0 = 2 * w, k1 = 2 * w + 1;
            fill_next[k0] = min(fill[k0] + (int)(run & 0xFFFFu), k0 == K - 1 ? cfg.lastcap : a.S);
            if (k1 < K) fill_next[k1] = min(fill[k1] + (int)(run >> 16), k1 == K - 1 ? cfg.lastcap : a.S);
        }
        __syncthreads();
        // ---- accept while the bucket has room
        int placed = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const bool act = (left >> s) & 1u;
            if (__builtin_amdgcn_ballot_w64(act) == 0ull) continue;
            bool ok = false;
            if (act) {
                const int h = hk[s] & 0xFFFF;
                const int rank = (int)((mine[h >> 1] >> ((h & 1) * 16)) & 0xFFFFu) + (hk[s] >> 16);
                const int f = fill[h];
                if (rank < (h == K - 1 ? cfg.lastcap : a.S) - f) {
                    const int i = p0 + idx[s], dst = p0 + h * a.S + f + rank;
                    a.inv_perm[i] = dst;
                    a.perm[dst] = i;
                    left &= ~(1u << s);
                    ok = true;
                }
            }
            placed += __popcll(__builtin_amdgcn_ballot_w64(ok));
        }
        int n_left = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) n_left += __popcll(__builtin_amdgcn_ballot_w64((left >> s) & 1u));
        if (lane == 0) {
            s_left[r & 1][wave] = n_left;
            if (placed) atomicAdd(&s_round[r], placed);
        }
        cur ^= 1;
        __syncthreads();
        int before = 0;
        rest = 0;
#pragma unroll
        for (int w = 0; w < MNW; ++w) {
            const int c = s_left[r & 1][w];
            before += w < wave ? c : 0;
            rest += c;
        }
        if (rest == 0) break;                         // uniform
        if ((rest + MTH - 1) / MTH < grp) {           // fewer groups of 64 hold what is left: close the gaps, in index order
            grp = (rest + MTH - 1) / MTH;
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                const bool act = (left >> s) & 1u;
                const unsigned long long m = __builtin_amdgcn_ballot_w64(act);
                if (act) {
                    const int e = before + bits_below(m);
                    list[e] = (uint32_t)idx[s];
                    list[MTH * PPT + e] = vlo[s];
                    list[2 * MTH * PPT + e] = vhi[s];
                }
                before += __popcll(m);
            }
            __syncthreads();
            left = 0;
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                const int e = wave * (64 * grp) + 64 * s + lane;
                if (s < grp && e < rest) {
                    left |= 1u << s;
                    idx[s] = (int)list[e];
                    vlo[s] = list[MTH * PPT + e];
                    vhi[s] = list[2 * MTH * PPT + e];
                }
            }
        }
    }

    // ---- recycle: the j-th point left (by index) takes the j-th free slot (buckets ascending, slots ascending)
    if (rest > 0) {
        int n_left = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) n_left += __popcll(__builtin_amdgcn_ballot_w64((left >> s) & 1u));
        if (lane == 0) s_left[(a.n_probes + 1) & 1][wave] = n_left;
        const int* fill = fillb + cur * K;
        int* freepre = fillb + (cur ^ 1) * K;         // last read before the barrier at the end of the last step
        const int own = tid < K ? ((tid == K - 1) ? cfg.lastcap : a.S) - fill[tid] : 0;   // K <= 1024
        int tot;
        const int pre = block_excl_scan(own, &tot, lds17);
        if (tid < K) freepre[tid] = pre;
        __syncthreads();
        int at = 0;
        for (int w = 0; w < wave; ++w) at += s_left[(a.n_probes + 1) & 1][w];
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const bool act = (left >> s) & 1u;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(act);
            if (act) {
                const int j = at + bits_below(m);
                int lo = 0, hi = K;                   // largest k with freepre[k] <= j
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (freepre[mid] <= j) lo = mid; else hi = mid;
                }
                const int dst = p0 + lo * a.S + fill[lo] + (j - freepre[lo]);
                if (dst < p0 + nb) {                  // always, while capacities add up to the scan size
                    a.inv_perm[p0 + idx[s]] = dst;
                    a.perm[dst] = p0 + idx[s];
                }
            }
            at += __popcll(m);
        }
        if (tid == 0) s_round[a.n_probes + 1] = rest;
    }
    __syncthreads();
    if (tid < 8) {
        if (single) a.round_count[tid] = s_round[tid];
        else if (s_round[tid]) atomicAdd(&a.round_count[tid], s_round[tid]);
    }
}

}  // namespace

bool psh_small_eligible(long long n, long long max_scan_points, int kcap)
{
    return n > 0 && max_scan_points <= MTH * PPT && kcap <= MTH;
}

hipError_t psh_small_launch(const PshArgs& args, hipStream_t stream)
{
    PshArgs a = args;
    if (a.n_scans > 1) {
        a.chunk = MTH * PPT;
        a.chunk_info = nullptr;
        a.meta_light = 1;   // the scan's own workgroup writes its bucket offsets
        k_psh_meta<<<1, 1024, 0, stream>>>(a);
    }
    const size_t lds = ((size_t)2 * a.kcap + (size_t)2 * MNW * ((a.kcap + 1) / 2) + (size_t)3 * MTH * PPT) * 4;
    const hipError_t e = hipFuncSetAttribute((const void*)k_pshs_small, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    k_pshs_small<<<a.n_scans, MTH, lds, stream>>>(a);
    return hipGetLastError();
}

}  // namespace f3d
