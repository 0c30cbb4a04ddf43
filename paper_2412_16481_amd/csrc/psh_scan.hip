// PSH bucketing, batch path: ONE workgroup per scan runs all of Algorithms 1 and 2 for its scan in a single launch.
//
// Same schedule and same results as psh.hip and psh_fast.hip (lock step, contenders served by input index). Those
// two spread a scan over many workgroups and need a grid-wide boundary per step; with many scans in a batch the
// scans themselves are the parallel work, and a step boundary is a workgroup barrier.
//
// A step is a count pass (the wave's contenders per bucket, one LDS add each), a prefix over the waves per bucket, and a
// pass that ranks (ballots over the key bits for the 64 points at hand, the wave's running counter for those before) and
// accepts; inside a pass the waves run freely. The direct step takes the scan in blocks of 8192 points, a run of 512 per
// wave, with buckets and voxels in registers between the two passes. (The block is what keeps the writes to `perm` together:
// its points fill about half a line of every bucket. With one run per wave over the whole scan, 16 lines of every bucket were
// being filled at any time, sixteen scans to an XCD evicted them from its L2 half written, and the pass took 190 us
// instead of 70 where the stores were left out.)
//
// Only a point whose probe hits a bucket that still has room can change anything, and room only shrinks. So after the
// direct step all six probes of every point left are hashed at once and looked up in the room the buckets have THEN; a point
// that finds none is done with (it waits for the recycle step), the others go on a list with their six buckets, ten bits each
// (a full bucket standing in for the probes that found none). The probe steps walk that list, 0 to 30 % of the points on
// most inputs and hashes, instead of all points left (45 % after the direct step on uniform cubes, 90 % on sensor sweeps).
//
// The count pass of a probe step reads the list; the contenders it finds, a quarter of the survivors and fewer from step to step, go on
// a queue in LDS, bucket and number, and only those are ranked. What the queue does not hold is read from the list again.
//
// Bound: instruction issue on one compute unit per scan. us per call with every point left walked in every step / with every survivor
// ranked in every step / now: 128 scans of 131 072 points in buckets of 256, 1170 / 501 / 453; 300 of 40 000 in buckets of 128, 629 /
// 360 / 332; 64 sensor sweeps of 30 000 in buckets of 64, 484 / 253 / 236; 100 of 60 000, Z-order-mod, 334 / 167 / 165; 200 of
// 20 000, XOR-div, 138 / 87 / 82; 600 of 20 000 in buckets of 128, - / 296 / 269. (The survivors that have a row as bits in LDS
// instead of marks in the list: 4 to 15 us more with one workgroup per compute unit.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "launch.h"
#include "psh_block.h"

namespace f3d {

namespace {

constexpr int QUEUE_MOST = (1 << 22) - 64;   // survivors of a wave that the queue can name (22 bits beside ten for the bucket)
constexpr int SKMAX = 1024;        // most buckets per scan on this path (ten bits in a list entry; LDS: 72 bytes per bucket)

// dynamic LDS, in 32-bit words: cnt[SNW][K] room[2][K] spare[SNW] queue[SNW][queue_cap]
// The hash function is a template parameter: the kernel holds many scan-wide values in scalar registers, and the
// branches between four hash functions cost enough of them to spill.
// WPE = waves per SIMD the kernel is compiled for: 4 (128 registers, one workgroup per compute unit) or 8 (64
// registers, two workgroups per compute unit: taken when there are more scans than compute units, where the second
// workgroup fills the issue slots the first leaves at its barriers).
template <int HASH, int WPE>
__global__ __launch_bounds__(STH, WPE) void k_pshs_scan(PshArgs a, int32_t* left_idx, int32_t* surv_pos, unsigned long long* voxels,
                                                   unsigned long long* surv_hash, int queue_cap)
{
    // Groups of 64 a wave handles per iteration, all their loads in flight together: stores and loads are waited for in order,
    // so a load an iteration ahead would wait for the stores of this one all the same; more work per wait hides it.
    constexpr int SU = WPE == 4 ? 4 : 2;
    constexpr int DG = WPE == 4 ? 8 : 4;   // groups of 64 in a wave's run of a block of the direct step (twice as many spill: 300 scans 339 -> 360 us)
    extern __shared__ int smem[];
    __shared__ ScanCfg cfg;
    __shared__ ZProbe zps[NPROBE];
    __shared__ uint32_t red[8];
    __shared__ int wleft[SNW];   // points a block of the direct step leaves, by wave
    __shared__ int s_round[8];
    __shared__ int s_full, s_surv;
    __shared__ int lds17[17];
    // Z-order codes of one axis, for coordinates of up to 11 bits (131072 points x 128 scans 491 -> 483 us: three reads for 27 instructions);
    // with two workgroups per compute unit there is no room for it
    constexpr bool TABLE = HASH == 3 && WPE == 4;
    __shared__ uint32_t spread[TABLE ? 2048 : 1];
    if (a.status[0]) return;   // inconsistent batch offsets: flagged by the set-up kernel, nothing to do
    const int b = blockIdx.x;
    const int p0 = a.scan_p0[b], nb = a.scan_p0[b + 1] - p0;
    const int kb0 = a.sbs[b], K = a.sbs[b + 1] - kb0;
    if (nb <= 0 || K <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(smem);
    uint32_t* mine = cnt + wave * K;
    int* roomb[2] = {smem + SNW * K, smem + (SNW + 1) * K};
    int* spare = smem + (SNW + 2) * K;
    uint32_t* queue = reinterpret_cast<uint32_t*>(spare + SNW) + wave * queue_cap;   // this wave's contenders of a probe step
    // The lists: points left by the direct step (number in the scan, voxel), and of those the survivors (position in the first
    // list, number, buckets). Every list of a scan lies in the scan's own stretch of its array.
    int32_t* const surv_idx = reinterpret_cast<int32_t*>(a.key) + p0;
    left_idx += p0;
    surv_pos += p0;
    voxels += p0;
    surv_hash += p0;

    // ---- first row of every bucket of the scan (buckets are full except the last), bounding box
    for (int j = tid; j < K; j += STH) a.offsets[kb0 + j] = p0 + min(j * a.S, nb);
    const Point3* pts = reinterpret_cast<const Point3*>(a.coords) + p0;
    {
        uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
        constexpr int UB = 4;   // points in flight per thread
        for (long long f0 = tid; f0 < nb; f0 += (long long)UB * STH) {
            Point3 v[UB];
#pragma unroll
            for (int j = 0; j < UB; ++j) v[j] = pts[min(f0 + (long long)j * STH, (long long)nb - 1)];   // past the end: the last point again
#pragma unroll
            for (int j = 0; j < UB; ++j) {
                const uint32_t o[3] = {f2ord(v[j].x), f2ord(v[j].y), f2ord(v[j].z)};
#pragma unroll
                for (int t = 0; t < 3; ++t) { mn[t] = min(mn[t], o[t]); mx[t] = max(mx[t], o[t]); }
            }
        }
        if (tid < 3) { red[tid] = 0xFFFFFFFFu; red[4 + tid] = 0u; }
        if (tid < 8) s_round[tid] = 0;
        if (tid == 0) s_surv = 0;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            uint32_t lo = mn[t], hi = mx[t];
            lo = wave_min(lo);
            hi = wave_max(hi);
            if (lane == 0) { atomicMin(&red[t], lo); atomicMax(&red[4 + t], hi); }
        }
        __syncthreads();
        if (tid == 0) compute_cfg(a, b, red, cfg);
    }
    for (int w = tid; w < SNW * K; w += STH) cnt[w] = 0u;
    if (TABLE) {
        spread[tid] = spread11((uint32_t)tid);
        spread[STH + tid] = spread11((uint32_t)(STH + tid));
    }
    __syncthreads();
    for (int k = tid; k < K; k += STH) roomb[0][k] = 0;      // the contenders so far, in the direct step

    const int keybits = max(1, 32 - __clz(max(K - 1, 1)));
    // A point's voxel is kept as its Z-order code where the hash and the probes work on that, else packed.
    const bool zc = HASH == 3 && a.probe_mode == 0;
    if (HASH == 3 && tid < NPROBE) zps[tid] = zprobe_of(cfg, tid + 1);
    const bool narrow = zc && max(max(cfg.vmax[0], cfg.vmax[1]), cfg.vmax[2]) < 1024;   // the code fits 30 bits

    // ---- direct step, block by block
    int total = 0;                          // points left so far
    auto direct_step = [&](auto narrow_tag) __attribute__((always_inline)) {
        constexpr bool NARROW = decltype(narrow_tag)::value;
        for (int b0 = 0; b0 < nb; b0 += 64 * DG * SNW) {
            const int i0 = b0 + wave * (64 * DG) + lane;      // at most 8192 beyond nb, which is 2^20 short of 2^31
            int hh[DG];
            unsigned long long vox[DG];
            uint32_t pass = 0;                                // bit s: the point of group s is passed on
#pragma unroll
            for (int s0 = 0; s0 < DG; s0 += SU) {
                Point3 c[SU];
#pragma unroll
                for (int s = 0; s < SU; ++s) c[s] = pts[(uint32_t)min(i0 + (s0 + s) * 64, nb - 1)];
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int x = voxel_of(c[s].x, cfg.mn[0], a.inv_voxel), y = voxel_of(c[s].y, cfg.mn[1], a.inv_voxel),
                              z = voxel_of(c[s].z, cfg.mn[2], a.inv_voxel);
                    int h;
                    if (NARROW) {
                        const uint32_t code = TABLE ? spread[x & 2047] | (spread[y & 2047] << 1) | (spread[z & 2047] << 2) : (uint32_t)morton3_low(x, y, z);
                        vox[s0 + s] = code;
                        h = zdiv30(code, cfg);
                    } else if (zc) {
                        vox[s0 + s] = cfg.wide ? morton3(x, y, z) : morton3_low(x, y, z);
                        h = hash_code(HASH, vox[s0 + s], cfg);
                    } else {
                        vox[s0 + s] = pack_voxel(x, y, z);
                        h = hash_bucket(HASH, x, y, z, cfg);
                    }
                    hh[s0 + s] = h;
                    if (i0 + (s0 + s) * 64 < nb) atomicAdd(&mine[h], 1u);
                }
            }
            __syncthreads();
            join_waves<false>(tid, K, cnt, roomb[0], roomb[0]);
            __syncthreads();
            int nleft = 0;
#pragma unroll
            for (int s0 = 0; s0 < DG; s0 += SU) {
                int h[SU], rank[SU];
                bool act[SU];
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    h[s] = hh[s0 + s];
                    act[s] = i0 + (s0 + s) * 64 < nb;
                }
                wave_ranks<SU>(h, act, keybits, mine, rank);
#pragma unroll
                for (int s = 0; s < SU; ++s) {
                    const int i = i0 + (s0 + s) * 64;
                    const bool fits = rank[s] < (h[s] == K - 1 ? cfg.lastcap : a.S);
                    if (act[s] && fits) {
                        const uint32_t dst = (uint32_t)(p0 + h[s] * a.S + rank[s]);
                        a.inv_perm[(uint32_t)(p0 + i)] = (int)dst;
                        a.perm[dst] = p0 + i;
                    }
                    const bool on = act[s] && !fits;
                    pass |= on ? 1u << (s0 + s) : 0u;
                    nleft += __popcll(__builtin_amdgcn_ballot_w64(on));
                }
            }
            for (int k = lane; k < K; k += 64) mine[k] = 0u;
            if (lane == 0) wleft[wave] = nleft;
            __syncthreads();
            int at = total;
#pragma unroll
            for (int v = 0; v < SNW; ++v) {
                const int c = wleft[v];
                at += v < wave ? c : 0;
                total += c;
            }
            at = __builtin_amdgcn_readfirstlane(at);
            total = __builtin_amdgcn_readfirstlane(total);
#pragma unroll
            for (int s = 0; s < DG; ++s) {
                const bool on = (pass >> s) & 1u;
                const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
                if (on) {
                    const uint32_t e = (uint32_t)(at + bits_below(m));
                    left_idx[e] = i0 + s * 64;
                    if (NARROW) reinterpret_cast<uint32_t*>(voxels)[e] = (uint32_t)vox[s];   // four of the eight bytes an entry has
                    else voxels[e] = vox[s];
                }
                at += __popcll(m);
            }
        }
    };
    if (HASH == 3 && narrow) direct_step(std::true_type{});
    else direct_step(std::false_type{});
    if (tid == 0) s_round[0] = nb - total;
    for (int k = tid; k < K; k += STH) {    // a thread's own k, as in join_waves
        const int room = max((k == K - 1 ? cfg.lastcap : a.S) - roomb[0][k], 0);
        roomb[1][k] = room;
        if (room == 0) s_full = k;          // some full bucket (there is one if a point was passed on); any will do
    }
    __threadfence_block();                  // the list is read by other threads of the workgroup from here on
    __syncthreads();
    int cur = 1;                            // roomb[cur]: the room the buckets have now
    // wave w takes entries [l0, l1) of the points left, up to SU groups of 64 at a time
    const int per = (total + SNW - 1) / SNW;
    const int l0 = min(wave * per, total), l1 = min(l0 + per, total);

    int nplaced = 0;
    if (total > 0 && a.n_probes > 0) {
        // ---- all probes of the points left, against the room after the direct step
        int nsurv = 0;
        const int full = s_full;
        auto probe_all = [&](auto narrow_tag) __attribute__((always_inline)) {
            constexpr bool NARROW = decltype(narrow_tag)::value;
            const int* room = roomb[cur];
            auto look_up = [&](auto groups, int pos0) __attribute__((always_inline)) {
                constexpr int G = decltype(groups)::value;
                const int entries = min(l1 - pos0, 64 * G);
                // with 64 registers the probes' fields, kept over the loop, spill (118 registers: 300 sweeps of 20000 points 302 -> 329 us;
                // read again each time 232)
                if (HASH == 3 && WPE == 8) asm volatile("" ::: "memory");
                unsigned long long v[G], hs[G];
                int i[G];
                bool any[G];
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    const uint32_t e = (uint32_t)(pos0 + min(s * 64 + lane, entries - 1));
                    i[s] = left_idx[e];
                    v[s] = NARROW ? reinterpret_cast<const uint32_t*>(voxels)[e] : voxels[e];
                    hs[s] = 0ull;
                    any[s] = false;
                }
#pragma unroll
                for (int r = 1; r <= NPROBE; ++r) {
                    if (r > a.n_probes) break;
                    const ZProbe zp = zps[HASH == 3 ? r - 1 : 0];
#pragma unroll
                    for (int s = 0; s < G; ++s) {
                        int h;
                        if (NARROW) {
                            h = zdiv30(zprobe30((uint32_t)v[s], (uint32_t)zp.mask, (uint32_t)zp.step, (uint32_t)zp.lim, (uint32_t)zp.vmax, (r - 1) & 1), cfg);
                        } else if (zc) {
                            h = hash_code(HASH, zprobe(v[s], zp), cfg);
                        } else {
                            int x = (int)(v[s] & 0x1FFFFFull), y = (int)((v[s] >> 21) & 0x1FFFFFull), z = (int)(v[s] >> 42);
                            probe_voxel(a, r, cfg, x, y, z);
                            h = hash_bucket(HASH, x, y, z, cfg);
                        }
                        const bool open = room[h] > 0;
                        any[s] |= open;
                        hs[s] |= (unsigned long long)(unsigned int)(open ? h : full) << (10 * (r - 1));
                    }
                }
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    const bool go = any[s] && s * 64 + lane < entries;
                    const unsigned long long m = __builtin_amdgcn_ballot_w64(go);
                    if (go) {
                        const uint32_t e = (uint32_t)(l0 + nsurv + bits_below(m));
                        surv_pos[e] = pos0 + s * 64 + lane;
                        surv_idx[e] = i[s];
                        surv_hash[e] = hs[s];
                    }
                    nsurv += __popcll(m);
                }
            };
            // Blocks, and the last groups one by one: a wave with a few points left would hash three empty groups beside them (100 scans
            // of 9000 points, Z-order-mod: 77 -> 63 us with that and with the steps ended when the last survivor is placed). Probes
            // that are arithmetic on the code are cheap enough for a block of two or three groups.
            constexpr int ONE_BY_ONE = HASH == 3 ? 1 : SU - 1;
            int pos0 = l0;
            for (; l1 - pos0 > 64 * ONE_BY_ONE; pos0 += 64 * SU) look_up(std::integral_constant<int, SU>{}, pos0);
            for (; pos0 < l1; pos0 += 64) look_up(std::integral_constant<int, 1>{}, pos0);
        };
        if (HASH == 3 && narrow) probe_all(std::true_type{});
        else probe_all(std::false_type{});
        if (lane == 0 && nsurv) atomicAdd(&s_surv, nsurv);
        __threadfence_block();   // a list entry is read by another lane of the wave that wrote it
        __syncthreads();
        // ---- the probe steps, on the survivors
        if (s_surv > 0) {
            const unsigned long long all_full = (unsigned long long)(unsigned int)full;
            for (int r = 1; r <= a.n_probes; ++r) {
                const int sh = 10 * (r - 1);
                const int* room = roomb[cur];
                int nq = 0, stop = nsurv;             // contenders on the queue; survivors from here on are not
                for (int j0 = 0; j0 < nsurv; j0 += 64 * 2 * SU) {
                    unsigned long long e[2 * SU];
#pragma unroll
                    for (int s = 0; s < 2 * SU; ++s) e[s] = surv_hash[(uint32_t)(l0 + min(j0 + s * 64 + lane, nsurv - 1))];
#pragma unroll
                    for (int s = 0; s < 2 * SU; ++s) {
                        const int g0 = j0 + s * 64;
                        if (g0 >= nsurv) break;
                        const int j = g0 + lane, h = (int)(e[s] >> sh) & 1023;
                        const bool on = j < nsurv && room[h] > 0;
                        if (on) atomicAdd(&mine[h], 1u);
                        const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
                        const int more = __popcll(m);
                        if (stop == nsurv && (nq + more > queue_cap || g0 >= QUEUE_MOST)) stop = g0;
                        if (stop == nsurv) {
                            if (on) queue[nq + bits_below(m)] = (uint32_t)h | ((uint32_t)j << 10);
                            nq += more;
                        }
                    }
                }
                __syncthreads();
                if (s_surv == 0) break;               // uniform: changed again behind the second barrier only
                join_waves<true>(tid, K, cnt, room, roomb[cur ^ 1]);
                __syncthreads();
                int got = 0;
                // SU groups of contenders at a time, those on the queue and then the others: where they come from (under way while they
                // are ranked), their ranks, the rows of those that fit
                for (int q0 = 0, j0 = stop; q0 < nq || j0 < nsurv;) {
                    bool on[SU];
                    int hh[SU], jj[SU], dst[SU], pos[SU], idx[SU];
                    if (q0 < nq) {
#pragma unroll
                        for (int s = 0; s < SU; ++s) {
                            const uint32_t e = queue[min(q0 + s * 64 + lane, nq - 1)];
                            on[s] = q0 + s * 64 + lane < nq;
                            hh[s] = (int)(e & 1023u);
                            jj[s] = (int)(e >> 10);
                        }
                        q0 += 64 * SU;
                    } else {
#pragma unroll
                        for (int s = 0; s < SU; ++s) {
                            jj[s] = min(j0 + s * 64 + lane, nsurv - 1);
                            hh[s] = (int)(surv_hash[(uint32_t)(l0 + jj[s])] >> sh) & 1023;
                            on[s] = j0 + s * 64 + lane < nsurv && room[hh[s]] > 0;
                        }
                        j0 += 64 * SU;
                    }
#pragma unroll
                    for (int s = 0; s < SU; ++s) {
                        if (__builtin_amdgcn_ballot_w64(on[s]) == 0ull) continue;
                        pos[s] = surv_pos[(uint32_t)(l0 + jj[s])];
                        idx[s] = surv_idx[(uint32_t)(l0 + jj[s])];
                    }
#pragma unroll
                    for (int s = 0; s < SU; ++s) {
                        const bool act[1] = {on[s]};
                        on[s] = false;
                        if (__builtin_amdgcn_ballot_w64(act[0]) == 0ull) continue;
                        const int h[1] = {hh[s]}, f = room[h[0]];
                        int rank[1];
                        wave_ranks<1>(h, act, keybits, mine, rank);
                        on[s] = act[0] && rank[0] < f;
                        dst[s] = p0 + h[0] * a.S + (h[0] == K - 1 ? cfg.lastcap : a.S) - f + rank[0];
                    }
#pragma unroll
                    for (int s = 0; s < SU; ++s) {
                        const unsigned long long m = __builtin_amdgcn_ballot_w64(on[s]);
                        if (m == 0ull) continue;
                        got += __popcll(m);
                        if (on[s]) {
                            a.inv_perm[(uint32_t)(p0 + idx[s])] = dst[s];
                            a.perm[(uint32_t)dst[s]] = p0 + idx[s];
                            left_idx[(uint32_t)pos[s]] = -1;
                            // from now on it contends for a bucket without room
                            unsigned long long gone = 0ull;
                            for (int t = 0; t < NPROBE; ++t) gone |= all_full << (10 * t);
                            surv_hash[(uint32_t)(l0 + jj[s])] = gone;
                        }
                    }
                }
                if (got) __threadfence_block();       // another lane of the wave may read the buckets of a survivor next
                for (int k = lane; k < K; k += 64) mine[k] = 0u;
                if (lane == 0 && got) {
                    atomicAdd(&s_round[r], got);
                    atomicSub(&s_surv, got);
                }
                nplaced += got;
                cur ^= 1;
            }
        }
    }

    // ---- recycle: the j-th entry left takes the j-th free slot (buckets ascending, slots ascending)
    if (total > 0) {   // uniform
        const int rest = l1 - l0 - nplaced;             // of this wave's entries
        __threadfence_block();                          // entries marked as placed are read by other lanes below
        __syncthreads();                                // everybody is done with the counters
        // buckets with room, in order: slots before, bucket, first free row
        int* slots_before = smem;                       // [K + 1] (the counters' place)
        int* bucket_of = smem + (K + 1);                // [K]
        const int* room = roomb[cur];
        int carry = 0, ocarry = 0;
        for (int k0 = 0; k0 < K; k0 += STH) {
            const int k = k0 + tid;
            const int v = k < K ? room[k] : 0;
            int tot, otot;
            const int pre = block_excl_scan(v, &tot, lds17);
            const int opre = block_excl_scan(v > 0 ? 1 : 0, &otot, lds17);
            if (v > 0) {
                slots_before[ocarry + opre] = carry + pre;
                bucket_of[ocarry + opre] = k;
            }
            carry += tot;
            ocarry += otot;
        }
        if (tid == 0) slots_before[ocarry] = carry;
        if (lane == 0) spare[wave] = rest;
        __syncthreads();
        int j0 = 0, left_total = 0;                     // entries left in earlier waves, in all
        for (int v = 0; v < SNW; ++v) {
            const int c = spare[v];
            j0 += v < wave ? c : 0;
            left_total += c;
        }
        int o = 0;                                      // last bucket whose slots begin at or before j0
        {
            int hi = ocarry;
            while (hi - o > 1) {
                const int mid = (o + hi) >> 1;
                if (slots_before[mid] <= j0) o = mid; else hi = mid;
            }
        }
        for (int pos0 = l0; pos0 < l1; pos0 += 64 * SU) {
            const int entries = min(l1 - pos0, 64 * SU);
            int i[SU];
#pragma unroll
            for (int s = 0; s < SU; ++s) i[s] = left_idx[(uint32_t)(pos0 + min(s * 64 + lane, entries - 1))];
#pragma unroll
            for (int s = 0; s < SU; ++s) {
                const bool act = s * 64 + lane < entries && i[s] >= 0;
                const unsigned long long m = __builtin_amdgcn_ballot_w64(act);
                if (act) {
                    const int j = j0 + bits_below(m);
                    int q = o;
                    while (q + 1 < ocarry && slots_before[q + 1] <= j) ++q;
                    const int k = bucket_of[q];
                    const int dst = p0 + k * a.S + (k == K - 1 ? cfg.lastcap : a.S) - room[k] + (j - slots_before[q]);
                    if ((uint32_t)(dst - p0) < (uint32_t)nb) {   // always, while capacities add up to the scan size
                        a.inv_perm[(uint32_t)(p0 + i[s])] = dst;
                        a.perm[(uint32_t)dst] = p0 + i[s];
                    }
                }
                j0 += __popcll(m);
                while (o + 1 < ocarry && slots_before[o + 1] <= j0) ++o;
            }
        }
        if (tid == 0) s_round[a.n_probes + 1] = left_total;
    }
    __syncthreads();
    if (tid < 8 && s_round[tid]) atomicAdd(&a.round_count[tid], s_round[tid]);
}

}  // namespace

bool psh_scan_eligible(int kcap) { return kcap <= SKMAX; }

hipError_t psh_scan_launch(const PshArgs& args, int32_t* left_idx, int32_t* surv_pos, unsigned long long* voxels, unsigned long long* surv_hash,
                           hipStream_t stream)
{
    PshArgs a = args;
    a.chunk = 2 * STH;
    a.chunk_info = nullptr;
    a.meta_light = 1;   // the scan's own workgroup writes its bucket offsets
    k_psh_meta<<<1, 1024, 0, stream>>>(a);
    if (a.n == 0) return hipGetLastError();
    size_t lds = ((size_t)(SNW + 2) * a.kcap + SNW) * 4;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    const bool two = cus > 0 && a.n_scans > cus && 2 * lds <= 150 * 1024;
    // The queues get what LDS is left beside one or two workgroups, but no more than the points of a wave.
    const size_t most = (two ? 75 : 150) * 1024, room = lds < most ? (most - lds) / (SNW * 4) : 0, all = (size_t)(a.max_scan_points / SNW) + 64;
    const int queue_cap = (int)(room < all ? room : all);
    lds += (size_t)SNW * queue_cap * 4;
    const void* fn[8] = {(const void*)k_pshs_scan<0, 4>, (const void*)k_pshs_scan<1, 4>, (const void*)k_pshs_scan<2, 4>,
                         (const void*)k_pshs_scan<3, 4>, (const void*)k_pshs_scan<0, 8>, (const void*)k_pshs_scan<1, 8>,
                         (const void*)k_pshs_scan<2, 8>, (const void*)k_pshs_scan<3, 8>};
    const int which = (a.hash & 3) + (two ? 4 : 0);
    if (lds > 60000) {
        const hipError_t e = allow_lds(fn[which], most);
        if (e != hipSuccess) return e;
    }
    switch (which) {
        case 0: k_pshs_scan<0, 4><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 1: k_pshs_scan<1, 4><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 2: k_pshs_scan<2, 4><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 3: k_pshs_scan<3, 4><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 4: k_pshs_scan<0, 8><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 5: k_pshs_scan<1, 8><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        case 6: k_pshs_scan<2, 8><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
        default: k_pshs_scan<3, 8><<<a.n_scans, STH, lds, stream>>>(a, left_idx, surv_pos, voxels, surv_hash, queue_cap); break;
    }
    return hipGetLastError();
}

}  // namespace f3d
