// Shared by the two bucketing paths that give a scan to one workgroup (psh_scan.hip, psh_small.hip): ranks inside a wave, the
// prefix over the waves, the probes of a point against the room the buckets have.
#pragma once
#include "psh_common.h"

namespace f3d {

namespace {

constexpr int STH = 1024;          // threads per workgroup
constexpr int SNW = STH / 64;      // waves
constexpr int NPROBE = 6;          // most probe steps (six bucket numbers of ten bits fit 64 bits)

__device__ __forceinline__ unsigned long long pack_voxel(int x, int y, int z)
{
    return (unsigned long long)(uint32_t)x | ((unsigned long long)(uint32_t)y << 21) | ((unsigned long long)(uint32_t)z << 42);
}

struct Point3 {
    float x, y, z;
};

// For U groups of 64, in order: the rank of every active lane among the wave's contenders of its bucket, counted on from
// `mine` (the wave's own row of counters), which is advanced. The first lane of every bucket writes for all. Inactive lanes
// hold a valid bucket too.
template <int U>
__device__ __forceinline__ void wave_ranks(const int (&h)[U], const bool (&act)[U], int keybits, uint32_t* mine, int (&rank)[U])
{
    uint32_t lo[U], hi[U];
#pragma unroll
    for (int s = 0; s < U; ++s) {
        const unsigned long long m = __builtin_amdgcn_ballot_w64(act[s]);
        lo[s] = (uint32_t)m;
        hi[s] = (uint32_t)(m >> 32);
    }
    for (int bit = 0; bit < keybits; ++bit) {             // as match_key, the groups together
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const int t = __builtin_amdgcn_sbfe(h[s], bit, 1);
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(t != 0);
            lo[s] &= ~((uint32_t)bal ^ (uint32_t)t);
            hi[s] &= ~((uint32_t)(bal >> 32) ^ (uint32_t)t);
        }
    }
    // A lane reads what another lane of the wave wrote. Every read and write of `mine` here may be to the same word for all the
    // compiler can tell, so it keeps them in order as they stand, and the barriers keep them from being moved into a branch. (Fences, as
    // in wave_lds_sync, hold back all other accesses too: 128 scans of 131 072 points 498 -> 503 us; volatile accesses 500 -> 508.)
#pragma unroll
    for (int s = 0; s < U; ++s) {
        const unsigned long long m = ((unsigned long long)hi[s] << 32) | lo[s];
        const int below = bits_below(m);
        rank[s] = (int)mine[h[s]] + below;
        __builtin_amdgcn_wave_barrier();
        if (act[s] && below == 0) mine[h[s]] = (uint32_t)(rank[s] + __popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
}

// The waves' counts become the rank of each wave's first contender. TO_ROOM: ranks count from 0, `from` is the room before the
// step and `to` the room after it. Otherwise both are the contenders so far. By all threads, between two barriers.
template <bool TO_ROOM>
__device__ __forceinline__ void join_waves(int tid, int K, uint32_t* cnt, const int* from, int* to)
{
    for (int k = tid; k < K; k += STH) {
        uint32_t run = TO_ROOM ? 0u : (uint32_t)from[k], t[SNW];
#pragma unroll
        for (int v = 0; v < SNW; ++v) t[v] = cnt[v * K + k];
#pragma unroll
        for (int v = 0; v < SNW; ++v) {
            cnt[v * K + k] = run;
            run += t[v];
        }
        to[k] = TO_ROOM ? max(from[k] - (int)run, 0) : (int)run;
    }
}

}  // namespace

}  // namespace f3d
