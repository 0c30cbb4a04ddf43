// PSH bucketing, small scans: ONE workgroup per scan with every point of the scan in registers.
//
// Same schedule and same results as the other paths (lock step, contenders served by input index). A scan of at most
// 8192 points (up to eight per thread) fits a workgroup of 1024 threads with its points in registers for all steps, so a
// step needs no read or write of global memory but the placements and no launch boundary; the one read of the coordinates also
// gives the bounding box, and with a single scan the tables and bucket offsets are written here too, so that the whole
// bucketing is one launch.
//
// A wave owns up to 64*PPT consecutive points. A step ranks the wave's contenders per bucket, joins the waves (prefix per
// bucket) and then accepts in index order (psh_block.h). After the direct step the probes of all points left are looked up at
// once in the room the buckets have then, as in psh_scan.hip: a point that finds none waits for the recycle step, the others
// carry their six bucket numbers (ten bits each), and the probe steps, which end when the last of these is placed, visit nothing
// else. Where few points are left (a small scan, a hash that spreads well) a wave that looked up its own six probes one after the
// other would be a serial chain beside idle waves: these are closed up over the workgroup and each wave takes 64 points and one
// probe. (600 scans of 300 points, Z-order-mod: 43 us when every point left was walked in every step until none was left, 60 with
// six probes looked up per wave and six steps always, 40 now; 4096 points, XOR-mod: 27, 32 and 22.)
//
// Bound: instruction issue and two barriers per step on ONE compute unit, not memory: 4 ns per point of a cube to 8 of a sensor
// sweep. us per scan (cube, room, sweep; scope 512), every point left walked in every step and now: 300 points 22 and 18, 4096
// 41, 49, 59 and 30, 30, 38. Where the line to the launch-per-step path lies: see psh_small_eligible.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "launch.h"
#include "psh_block.h"

namespace f3d {

namespace {

constexpr int MKMAX = 1024;        // most buckets per scan on this path (ten bits; one thread per bucket in the recycle step)

// dynamic LDS, in 32-bit words: cnt[SNW][K] room[2][K] placed[PPT * STH / 32] list[PPT * STH]
template <int PPT>
__global__ __launch_bounds__(STH) void k_pshs_small(PshArgs a)
{
    extern __shared__ int smem[];
    __shared__ ScanCfg cfg;
    __shared__ ZProbe zps[NPROBE];
    __shared__ uint32_t red[8];
    __shared__ int s_round[8];
    __shared__ int s_left[SNW];
    __shared__ int s_full, s_live;
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
        for (int j = tid; j <= a.max_buckets; j += STH) a.offsets[j] = j < K ? j * a.S : a.n;
    } else {
        if (a.status[0]) return;       // inconsistent batch offsets: flagged by the set-up kernel, nothing to do
        p0 = a.scan_p0[b];
        nb = a.scan_p0[b + 1] - p0;
        kb0 = a.sbs[b];
        K = a.sbs[b + 1] - kb0;
        if (nb <= 0 || K <= 0) return;
        for (int j = tid; j < K; j += STH) a.offsets[kb0 + j] = p0 + min(j * a.S, nb);
    }
    uint32_t* cnt = reinterpret_cast<uint32_t*>(smem);
    uint32_t* mine = cnt + wave * K;
    int* roomb[2] = {smem + SNW * K, smem + (SNW + 1) * K};
    uint32_t* placed = reinterpret_cast<uint32_t*>(smem + (SNW + 2) * K);
    uint32_t* list = placed + PPT * STH / 32 + wave * (64 * PPT);   // the wave's own stretch

    // ---- the points, the bounding box. A wave owns 64*grp consecutive ones.
    const int grp = (nb + STH - 1) / STH;
    const int w0 = wave * (64 * grp), i0 = w0 + lane; // this lane's points: i0, i0 + 64, ..
    Point3 c[PPT];
#pragma unroll
    for (int s = 0; s < PPT; ++s)                     // past the end: the last point again
        c[s] = reinterpret_cast<const Point3*>(a.coords)[(uint32_t)(p0 + min(i0 + 64 * (s < grp ? s : 0), nb - 1))];
    if (tid < 8) {
        red[tid] = tid < 4 ? 0xFFFFFFFFu : 0u;
        s_round[tid] = 0;
    }
    if (tid == 0) s_live = 0;
    for (int w = tid; w < SNW * K; w += STH) cnt[w] = 0u;
    for (int w = tid; w < PPT * STH / 32; w += STH) placed[w] = 0u;
    __syncthreads();
    {
        uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const uint32_t o[3] = {f2ord(c[s].x), f2ord(c[s].y), f2ord(c[s].z)};
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                mn[t] = min(mn[t], o[t]);
                mx[t] = max(mx[t], o[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            mn[t] = wave_min(mn[t]);
            mx[t] = wave_max(mx[t]);
            if (lane == 0) {
                atomicMin(&red[t], mn[t]);
                atomicMax(&red[4 + t], mx[t]);
            }
        }
    }
    __syncthreads();
    if (tid == 0) compute_cfg_of(a, p0, nb, kb0, K, red, cfg);
    __syncthreads();
    for (int k = tid; k < K; k += STH) roomb[0][k] = k == K - 1 ? cfg.lastcap : a.S;

    const int keybits = max(1, 32 - __clz(max(K - 1, 1)));
    // The voxel is kept as its Z-order code where the hash and the probes work on that, else packed.
    const bool zc = a.hash == 3 && a.probe_mode == 0;
    if (zc && tid < a.n_probes) zps[tid] = zprobe_of(cfg, tid + 1);
    const bool narrow = zc && max(max(cfg.vmax[0], cfg.vmax[1]), cfg.vmax[2]) < 1024;   // the code fits 30 bits
    unsigned long long vox[PPT];                      // behind the direct step: the bucket numbers of the probes
    int hh[PPT];
    uint32_t left = 0;                                // bit s: point s is not placed by the direct step
    // ---- direct step
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        hh[s] = 0;
        vox[s] = 0ull;
        if (s >= grp || w0 + 64 * s >= nb) continue;  // uniform in the wave
        const int x = voxel_of(c[s].x, cfg.mn[0], a.inv_voxel), y = voxel_of(c[s].y, cfg.mn[1], a.inv_voxel),
                  z = voxel_of(c[s].z, cfg.mn[2], a.inv_voxel);
        if (narrow) {
            vox[s] = (uint32_t)morton3_low(x, y, z);
            hh[s] = zdiv30((uint32_t)vox[s], cfg);
        } else if (zc) {
            vox[s] = cfg.wide ? morton3(x, y, z) : morton3_low(x, y, z);
            hh[s] = hash_code(3, vox[s], cfg);
        } else {
            vox[s] = pack_voxel(x, y, z);
            hh[s] = hash_bucket(a.hash, x, y, z, cfg);
        }
    }
    auto rank_groups = [&](auto groups, int s0) __attribute__((always_inline)) {   // hh: bucket | rank among the wave's contenders << 16
        constexpr int G = decltype(groups)::value;
        int h[G], rank[G];
        bool act[G];
#pragma unroll
        for (int s = 0; s < G; ++s) {
            h[s] = hh[s0 + s];
            act[s] = s0 + s < grp && i0 + 64 * (s0 + s) < nb;
        }
        wave_ranks<G>(h, act, keybits, mine, rank);
#pragma unroll
        for (int s = 0; s < G; ++s) hh[s0 + s] |= rank[s] << 16;
    };
    if (PPT == 4 && grp == 4) {
        // Counted by adds, and ranked behind the join: with all four groups full the ranks wait less there (a forward pass over 4096
        // points 43.7 -> 43.0 us). With fewer groups the ranks go before the join (600 scans of 300 points 42 -> 39).
#pragma unroll
        for (int s = 0; s < PPT; ++s)
            if (i0 + 64 * s < nb) atomicAdd(&mine[hh[s]], 1u);
        __syncthreads();
        join_waves<true>(tid, K, cnt, roomb[0], roomb[1]);
        __syncthreads();
        int h[PPT], rank[PPT];
        bool act[PPT];
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            h[s] = hh[s];
            act[s] = i0 + 64 * s < nb;
        }
        wave_ranks<PPT>(h, act, keybits, mine, rank);
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const bool fits = rank[s] < (h[s] == K - 1 ? cfg.lastcap : a.S);
            if (act[s] && fits) {
                const int i = p0 + i0 + 64 * s, dst = p0 + h[s] * a.S + rank[s];
                a.inv_perm[(uint32_t)i] = dst;
                a.perm[(uint32_t)dst] = i;
            }
            left |= act[s] && !fits ? 1u << s : 0u;
        }
    } else {
        if (w0 < nb) {
            // no more groups than there are: a scan of up to 1024 points has one
            if (grp == 1) rank_groups(std::integral_constant<int, 1>{}, 0);
            else if (grp == 2) rank_groups(std::integral_constant<int, 2>{}, 0);
            else if (grp == 3) rank_groups(std::integral_constant<int, 3>{}, 0);
            else rank_groups(std::integral_constant<int, 4>{}, 0);
            if constexpr (PPT > 4) {
                if (grp == 5) rank_groups(std::integral_constant<int, 1>{}, 4);
                else if (grp == 6) rank_groups(std::integral_constant<int, 2>{}, 4);
            }
            if constexpr (PPT > 6) {
                if (grp == 7) rank_groups(std::integral_constant<int, 3>{}, 4);
                else if (grp == 8) rank_groups(std::integral_constant<int, 4>{}, 4);
            }
        }
        __syncthreads();
        join_waves<true>(tid, K, cnt, roomb[0], roomb[1]);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            if (s >= grp || w0 + 64 * s >= nb) continue;
            const int h = hh[s] & 0xFFFF, rank = (int)mine[h] + (hh[s] >> 16);
            const bool act = i0 + 64 * s < nb, fits = rank < (h == K - 1 ? cfg.lastcap : a.S);
            if (act && fits) {
                const int i = p0 + i0 + 64 * s, dst = p0 + h * a.S + rank;
                a.inv_perm[(uint32_t)i] = dst;
                a.perm[(uint32_t)dst] = i;
            }
            left |= act && !fits ? 1u << s : 0u;
        }
    }
    for (int k = lane; k < K; k += 64) mine[k] = 0u;
    int n_left = 0;                                   // points of this wave that are not placed
#pragma unroll
    for (int s = 0; s < PPT; ++s) n_left += __popcll(__builtin_amdgcn_ballot_w64((left >> s) & 1u));
    if (lane == 0) s_left[wave] = n_left;
    if (tid < K && roomb[1][tid] == 0) s_full = tid;  // some full bucket (there is one if a point is left); any will do
    __syncthreads();
    int rest = 0, before = 0;                         // points not placed: in all, in earlier waves
#pragma unroll
    for (int w = 0; w < SNW; ++w) {
        const int n = s_left[w];
        rest += n;
        before += w < wave ? n : 0;
    }
    rest = __builtin_amdgcn_readfirstlane(rest);
    before = __builtin_amdgcn_readfirstlane(before);
    if (tid == 0) s_round[0] = nb - rest;
    int cur = 1;                                      // roomb[cur]: the room the buckets have now

    int hopeless = rest;                              // points left that no probe can place
    bool walked = false;
    if (rest > 0 && a.n_probes > 0) {
        // ---- all probes of the points left, against the room after the direct step
        const int full = s_full;
        const int* const room0 = roomb[cur];
        // the bucket that probe r of a point looks up if it has room, else `full`
        auto probe = [&](unsigned long long v, int r) __attribute__((always_inline)) -> int {
            int h;
            if (narrow) {
                const ZProbe& z = zps[r - 1];
                h = zdiv30(zprobe30((uint32_t)v, (uint32_t)z.mask, (uint32_t)z.step, (uint32_t)z.lim, (uint32_t)z.vmax, (r - 1) & 1), cfg);
            } else if (zc) {
                h = hash_code(3, zprobe(v, zps[r - 1]), cfg);
            } else {
                int x = (int)(v & 0x1FFFFFull), y = (int)((v >> 21) & 0x1FFFFFull), z = (int)(v >> 42);
                probe_voxel(a, r, cfg, x, y, z);
                h = hash_bucket(a.hash, x, y, z, cfg);
            }
            return room0[h] > 0 ? h : full;
        };
        int idx[PPT];                                 // index inside the scan
        int held = 0;                                 // points this wave goes on with lie in the first so many places
        uint32_t live = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) idx[s] = 0;
        if (NPROBE * rest <= PPT * STH) {          // three words and six halves of one per point fit the list
            // Few are left (a small scan, or a hash that spreads well): one probe after the other in the waves that hold them would be
            // a serial chain beside idle waves. They are closed up over the workgroup, 64 of them and one probe are a wave's
            // task, and the bucket numbers come back through LDS.
            uint32_t* all = placed + PPT * STH / 32;  // number, voxel (low, high) [rest] each; then buckets [n_probes][rest], 16 bits
            uint16_t* bucket = reinterpret_cast<uint16_t*>(all + 3 * rest);
            int at = before;
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                const bool on = (left >> s) & 1u;
                const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
                if (on) {
                    const int e = at + bits_below(m);
                    all[e] = (uint32_t)(i0 + 64 * s);
                    all[rest + e] = (uint32_t)vox[s];
                    all[2 * rest + e] = (uint32_t)(vox[s] >> 32);
                }
                at += __popcll(m);
            }
            __syncthreads();
            const int groups = (rest + 63) >> 6;
            int r = 1, g = wave;                      // group g of probe r
            for (;; g += SNW) {
                while (g >= groups) { g -= groups; ++r; }
                if (r > a.n_probes) break;
                const int e = min(64 * g + lane, rest - 1);
                const unsigned long long v = (unsigned long long)all[rest + e] | ((unsigned long long)all[2 * rest + e] << 32);
                bucket[(r - 1) * rest + e] = (uint16_t)probe(v, r);
            }
            __syncthreads();
            const int per = (rest + STH - 1) / STH, e0 = wave * 64 * per;
            held = min(max(rest - e0, 0), 64 * per);
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                if (64 * s >= held) continue;         // uniform in the wave
                const int e = e0 + min(64 * s + lane, held - 1);
                idx[s] = (int)all[e];
                unsigned long long hs = 0ull;
                bool any = false;
                for (int t = 0; t < a.n_probes; ++t) {
                    const int h = bucket[t * rest + e];
                    any |= h != full;
                    hs |= (unsigned long long)(unsigned int)h << (10 * t);
                }
                vox[s] = hs;
                live |= any && 64 * s + lane < held ? 1u << s : 0u;
            }
        } else {
            // closed up inside the wave, one word of every entry at a time through the wave's stretch of LDS, in index order: where that
            // spares a group before the probes, and those with a hit behind them
            auto exchange = [&](uint32_t from, int n, auto get, auto put) __attribute__((always_inline)) {
                int at = 0;
#pragma unroll
                for (int s = 0; s < PPT; ++s) {
                    const bool on = (from >> s) & 1u;
                    const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
                    if (on) list[at + bits_below(m)] = get(s);
                    at += __popcll(m);
                }
                wave_lds_sync();
#pragma unroll
                for (int s = 0; s < PPT; ++s)
                    if (64 * s < n) put(s, list[min(64 * s + lane, n - 1)]);
                wave_lds_sync();
            };
            auto close_up = [&](uint32_t from, int n) __attribute__((always_inline)) -> uint32_t {
                uint32_t lo[PPT], to = 0;
                exchange(from, n, [&](int s) { return (uint32_t)idx[s]; }, [&](int s, uint32_t v) { idx[s] = (int)v; });
#pragma unroll
                for (int s = 0; s < PPT; ++s) lo[s] = 0u;
                exchange(from, n, [&](int s) { return (uint32_t)vox[s]; }, [&](int s, uint32_t v) { lo[s] = v; });
                exchange(from, n, [&](int s) { return (uint32_t)(vox[s] >> 32); }, [&](int s, uint32_t v) { hh[s] = (int)v; });
#pragma unroll
                for (int s = 0; s < PPT; ++s) {
                    vox[s] = ((unsigned long long)(uint32_t)hh[s] << 32) | lo[s];
                    to |= 64 * s + lane < n ? 1u << s : 0u;
                }
                return to;
            };
#pragma unroll
            for (int s = 0; s < PPT; ++s) idx[s] = i0 + 64 * s;
            const uint32_t on = !zc && n_left <= 64 * (grp - 1) ? close_up(left, n_left) : left;   // probes on codes cost less than this
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                const bool act = (on >> s) & 1u;
                if (__builtin_amdgcn_ballot_w64(act) == 0ull) continue;
                if (PPT > 4) asm volatile("" ::: "memory");   // the probes' fields are read again: kept over the groups they spill 50 registers
                const unsigned long long v = vox[s];
                unsigned long long hs = 0ull;
                bool any = false;
#pragma unroll
                for (int r = 1; r <= NPROBE; ++r) {
                    if (r > a.n_probes) break;
                    const int h = probe(v, r);
                    any |= h != full;
                    hs |= (unsigned long long)(unsigned int)h << (10 * (r - 1));
                }
                vox[s] = hs;
                live |= any && act ? 1u << s : 0u;
                held += __popcll(__builtin_amdgcn_ballot_w64(any && act));
            }
            live = held ? close_up(live, held) : 0u;
        }
        {
            int n = 0;
#pragma unroll
            for (int s = 0; s < PPT; ++s) n += __popcll(__builtin_amdgcn_ballot_w64((live >> s) & 1u));
            if (lane == 0 && n) atomicAdd(&s_live, n);
        }
        __syncthreads();
        // ---- the probe steps, on the survivors
        const int live_total = s_live;
        hopeless = rest - live_total;
        if (live_total > 0) {
            walked = true;
            for (int r = 1; r <= a.n_probes; ++r) {
                const int sh = 10 * (r - 1);
                const int* room = roomb[cur];
#pragma unroll
                for (int s = 0; s < PPT; ++s) {
                    if (64 * s >= held) continue;     // uniform in the wave
                    const int h[1] = {(int)(vox[s] >> sh) & 1023};
                    const bool act[1] = {((live >> s) & 1u) && room[h[0]] > 0};
                    hh[s] = -1;
                    if (__builtin_amdgcn_ballot_w64(act[0]) == 0ull) continue;
                    int rank[1];
                    wave_ranks<1>(h, act, keybits, mine, rank);
                    if (act[0]) hh[s] = h[0] | (rank[0] << 16);
                }
                __syncthreads();
                if (s_live == 0) break;               // uniform: changed again behind the second barrier only
                join_waves<true>(tid, K, cnt, room, roomb[cur ^ 1]);
                __syncthreads();
                int got = 0;
#pragma unroll
                for (int s = 0; s < PPT; ++s) {
                    if (64 * s >= held) continue;
                    const int h = hh[s] >= 0 ? hh[s] & 0xFFFF : 0, f = room[h], rank = (int)mine[h] + (hh[s] >> 16);
                    const bool ok = hh[s] >= 0 && rank < f;
                    if (ok) {
                        const int i = p0 + idx[s], dst = p0 + h * a.S + (h == K - 1 ? cfg.lastcap : a.S) - f + rank;
                        a.inv_perm[(uint32_t)i] = dst;
                        a.perm[(uint32_t)dst] = i;
                        atomicOr(&placed[idx[s] >> 5], 1u << (idx[s] & 31));
                        live &= ~(1u << s);
                    }
                    got += __popcll(__builtin_amdgcn_ballot_w64(ok));
                }
                for (int k = lane; k < K; k += 64) mine[k] = 0u;
                if (lane == 0 && got) {
                    atomicAdd(&s_round[r], got);
                    atomicSub(&s_live, got);
                }
                cur ^= 1;
            }
        }
    }

    // ---- recycle: the j-th point left (by index) takes the j-th free slot (buckets ascending, slots ascending)
    if (walked) __syncthreads();                      // the marks are in place, the counters are free
    if (hopeless > 0 || (walked && s_live > 0)) {
        n_left = 0;
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const int i = i0 + 64 * s;
            if ((left >> s) & 1u) left &= ~(((placed[i >> 5] >> (i & 31)) & 1u) << s);
            n_left += __popcll(__builtin_amdgcn_ballot_w64((left >> s) & 1u));
        }
        if (lane == 0) s_left[wave] = n_left;         // without a walk what it holds already
        // buckets with room, in order: slots before, bucket
        int* slots_before = smem;                     // [K + 1]
        int* bucket_of = smem + (K + 1);              // [K]
        const int* room = roomb[cur];
        const int own = tid < K ? room[tid] : 0;      // K <= 1024
        int tot;                                      // slots (at most 8192) | buckets with room << 16
        int pre = block_excl_scan(own | (own > 0 ? 1 << 16 : 0), &tot, lds17);
        const int opre = pre >> 16, open = tot >> 16;
        pre &= 0xFFFF;
        tot &= 0xFFFF;
        if (own > 0) {
            slots_before[opre] = pre;
            bucket_of[opre] = tid;
        }
        if (tid == 0) slots_before[open] = tot;
        __syncthreads();
        int j0 = 0, all = 0;                          // points left in earlier waves, in all
#pragma unroll
        for (int w = 0; w < SNW; ++w) {
            const int n = s_left[w];
            j0 += w < wave ? n : 0;
            all += n;
        }
        j0 = __builtin_amdgcn_readfirstlane(j0);
        int o = 0;                                    // last bucket whose slots begin at or before j0
        {
            int hi = open;
            while (hi - o > 1) {
                const int mid = (o + hi) >> 1;
                if (__builtin_amdgcn_readfirstlane(slots_before[mid]) <= j0) o = mid; else hi = mid;
            }
        }
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            const bool act = (left >> s) & 1u;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(act);
            if (m == 0ull) continue;
            int q = o;
            if (act) {
                const int j = j0 + bits_below(m);
                int step = 1;
                while (q + step < open && slots_before[q + step] <= j) {
                    q += step;
                    step *= 2;
                }
                for (int hi = min(open, q + step); hi - q > 1;) {
                    const int mid = (q + hi) >> 1;
                    if (slots_before[mid] <= j) q = mid; else hi = mid;
                }
                const int k = bucket_of[q];
                const int dst = k * a.S + (k == K - 1 ? cfg.lastcap : a.S) - room[k] + (j - slots_before[q]);
                if ((uint32_t)dst < (uint32_t)nb) {   // always, while capacities add up to the scan size
                    const int i = p0 + i0 + 64 * s;
                    a.inv_perm[(uint32_t)i] = p0 + dst;
                    a.perm[(uint32_t)(p0 + dst)] = i;
                }
            }
            j0 += __popcll(m);
            o = __builtin_amdgcn_readlane(q, 63 - __builtin_clzll(m));   // of the last of them: the next ones' are not before it
        }
        if (tid == 0) s_round[a.n_probes + 1] = all;
    }
    __syncthreads();
    if (tid < 8) {
        if (single) a.round_count[tid] = s_round[tid];
        else if (s_round[tid]) atomicAdd(&a.round_count[tid], s_round[tid]);
    }
}

constexpr size_t small_lds_bytes(int ppt, int kcap) { return ((size_t)(SNW + 2) * kcap + (size_t)ppt * STH / 32 + (size_t)ppt * STH) * 4; }

template <int PPT>
hipError_t launch_small(const PshArgs& a, hipStream_t stream)
{
    const size_t lds = small_lds_bytes(PPT, a.kcap);
    const hipError_t e = allow_lds((const void*)k_pshs_small<PPT>, small_lds_bytes(PPT, MKMAX));
    if (e != hipSuccess) return e;
    k_pshs_small<PPT><<<a.n_scans, STH, lds, stream>>>(a);
    return hipGetLastError();
}

}  // namespace

// Up to 4096 points always; further for every probe step, each of which is a launch on the launch-per-step path. One scan of a
// cube, room, sensor sweep, us here (there), Z-order-div, scope 1024, six probes: 5000 points 36, 40, 46 (52, 56, 56); 6000 40, 43, 51
// (55, 54, 55); 7000 48, 41, 57 (54, 55, 55); 8192 51, 46, 63 (55, 55, 56); the other hashes at 8192 points 31 to 58 (52 to 55),
// but Z-order-mod on the sweep 73 (55). With two probes 5000 points take 25 and 30 (30 and 31).
// Batches that the one-workgroup-per-scan path takes stay there above 4096 points (100 scans of 8000: 55 against 62, 600 of them
// 140 against 178).
bool psh_small_eligible(long long n, long long max_scan_points, int kcap, int n_probes, bool scans)
{
    return n > 0 && max_scan_points <= 4 * STH + (scans ? 0 : n_probes * STH * 2 / 3) && kcap <= MKMAX;
}

hipError_t psh_small_launch(const PshArgs& args, hipStream_t stream)
{
    PshArgs a = args;
    if (a.n_scans > 1) {
        a.chunk = 8 * STH;
        a.chunk_info = nullptr;
        a.meta_light = 1;   // the scan's own workgroup writes its bucket offsets
        k_psh_meta<<<1, 1024, 0, stream>>>(a);
    }
    if (a.max_scan_points <= 4 * STH) return launch_small<4>(a, stream);
    if (a.max_scan_points <= 6 * STH) return launch_small<6>(a, stream);
    return launch_small<8>(a, stream);
}

}  // namespace f3d
