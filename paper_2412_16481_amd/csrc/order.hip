// Canonical serving order for the rebalancing of Algorithm 2 (Section 4.1 "Bucket rebalancing" leaves the arrival
// order of the contenders of a bucket to the hardware race). Serving them in increasing
// (Z-order code of the voxel, x, y, z, input index) makes the partition of the points independent of the order in
// which they are stored. It is done by sorting the points once by that key and running the index-ordered bucketing on
// the sorted copy; the result is mapped back through the sort order.
//
// The sort is a merge sort on whole keys (112 + 63 bits in three 64-bit words), carrying only the point index: one kernel
// builds the keys and sorts tiles of 2048 positions in LDS, then one kernel per doubling of the sorted length merges
// pairs of runs, a workgroup per 2048 positions of the result. A comparison almost always ends at the first word, which
// holds the scan and the upper 48 bits of the code. The cost does not depend on how the points fall into voxels.
//
// Bound: launches and latency (a merge launch is a chain of a search, two dependent loads and a search in LDS: 10 us at
// 457295 points, the tiles 32 us). A radix sort on 8-bit digits takes 21 passes over these keys, each with its own count,
// scan and scatter, whatever n is. A whole canonical bucketing took 248 us at 1500 points, 521 us at 457295 and 3.44 ms at
// 4 million with such a sort, and took 64 us, 249 us and 1.62 ms with this one (229 us at
// 457295 points since the bucketing that follows takes 89).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "order.h"
#include "psh.h"
#include "psh_common.h"

namespace f3d {
namespace {

constexpr int OT = 256;          // threads per workgroup
constexpr int OE = 2048;         // positions per tile
constexpr int OST = 512;         // threads that sort or merge a tile
constexpr int OPT = OE / OST;    // results per thread

__device__ __forceinline__ int scan_of(const OrderArgs& a, int p)
{
    return a.batch_offsets ? find_scan(a.batch_offsets, a.n_scans, p) : 0;
}

__global__ __launch_bounds__(OT) void k_order_init(OrderArgs a)
{
    const int i = blockIdx.x * OT + threadIdx.x;
    if (i < a.n_scans * 4) a.box[i] = 0xFFFFFFFFu;
}

// per-scan coordinate minimum (Algorithm 1, "compute voxel coordinate"). A workgroup takes OB consecutive positions.
// Almost always they belong to one scan: then the minimum is reduced inside the workgroup and costs three global
// atomics; a workgroup that straddles a scan boundary publishes wave by wave whenever a wave moves on to another scan.
constexpr int OB = OE;
__global__ __launch_bounds__(OT) void k_order_box(OrderArgs a)
{
    __shared__ uint32_t red[3];
    const int tid = threadIdx.x, lane = tid & 63;
    const long long first = (long long)blockIdx.x * OB;
    const long long last = min(first + OB, (long long)a.n) - 1;
    if (first > last) return;
    const int b_first = scan_of(a, (int)first), b_last = scan_of(a, (int)last);
    const bool uniform = b_first == b_last;      // offsets are non-decreasing when they are valid at all
    if (tid < 3) red[tid] = 0xFFFFFFFFu;
    __syncthreads();
    uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    if (uniform) {
        for (long long e = first + tid; e <= last; e += OT) {
#pragma unroll
            for (int t = 0; t < 3; ++t) mn[t] = min(mn[t], f2ord(a.coords[(size_t)e * 3 + t]));
        }
    } else {
        // a lane walks its positions in increasing order, so its scan index only grows: it keeps the minimum of the
        // scan it is in; when any lane of the wave moves on to another scan the whole wave publishes (one atomic per
        // axis if all its lanes were in the same scan, else one per lane and axis)
        int cur = -1;
        const auto flush = [&]() {
            const unsigned long long have = __ballot(cur >= 0);
            if (!have) return;
            const int lead = __shfl(cur, __ffsll((long long)have) - 1, 64);
            if (__ballot(cur >= 0 && cur != lead) == 0) {
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    uint32_t lo = mn[t];
                    for (int d = 32; d >= 1; d >>= 1) lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
                    if (lane == 0) atomicMin(&a.box[lead * 4 + t], lo);
                }
            } else if (cur >= 0) {
#pragma unroll
                for (int t = 0; t < 3; ++t) atomicMin(&a.box[cur * 4 + t], mn[t]);
            }
        };
        for (long long e0 = first; e0 <= last; e0 += OT) {   // the trip count is the same for every lane
            const long long e = e0 + tid;
            const bool ok = e <= last;
            const int b = ok ? scan_of(a, (int)e) : -1;
            if (__ballot(ok && cur >= 0 && b != cur)) {
                flush();
                cur = -1;
                mn[0] = mn[1] = mn[2] = 0xFFFFFFFFu;
            }
            if (ok) {
                cur = b;
#pragma unroll
                for (int t = 0; t < 3; ++t) mn[t] = min(mn[t], f2ord(a.coords[(size_t)e * 3 + t]));
            }
        }
        flush();
    }
    if (!uniform) return;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        uint32_t lo = mn[t];
        for (int d = 32; d >= 1; d >>= 1) lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
        if (lane == 0) atomicMin(&red[t], lo);
    }
    __syncthreads();
    if (tid < 3) atomicMin(&a.box[b_first * 4 + tid], red[tid]);
}

// key of a point: {scan:16 code:63 x:32 y:32 z:32} from the top of the first word down, zero-padded at the end
struct OrderKey {
    unsigned long long a, b, c;
};

// A tile of keys in LDS.
struct KeyTile {
    unsigned long long a[OE], b[OE], c[OE];
};

// key i of the tile comes before key j (equal keys: by position)
__device__ __forceinline__ bool key_less(const KeyTile& k, int i, int j)
{
    const unsigned long long ai = k.a[i], aj = k.a[j];
    if (ai != aj) return ai < aj;
    const unsigned long long bi = k.b[i], bj = k.b[j];
    if (bi != bj) return bi < bj;
    const unsigned long long ci = k.c[i], cj = k.c[j];
    if (ci != cj) return ci < cj;
    return i < j;
}

// Keys of the points (also to `keys`, 24 bytes per point) and the sorted order of every tile of OE positions.
__global__ __launch_bounds__(OST) void k_order_tiles(OrderArgs a)
{
    __shared__ KeyTile k;
    __shared__ uint16_t ord[2][OE];
    const int tid = threadIdx.x;
    const long long first = (long long)blockIdx.x * OE;
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        const int e = u * OST + tid;
        const long long p = first + e;
        OrderKey key = {~0ull, ~0ull, ~0ull};         // past the end: behind every point (a scan index is below 65535)
        if (p < a.n) {
            const int b = scan_of(a, (int)p);
            int v[3];
            uint32_t o[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const float c = a.coords[(size_t)p * 3 + t];
                o[t] = f2ord(c);
                v[t] = voxel_of(c, ord2f(a.box[b * 4 + t]), a.inv_voxel);
            }
            const uint64_t code = morton3(v[0], v[1], v[2]);
            key.a = ((unsigned long long)(uint32_t)b << 48) | (code >> 15);
            key.b = ((code & 0x7FFFull) << 49) | ((unsigned long long)o[0] << 17) | (o[1] >> 15);
            key.c = ((unsigned long long)o[1] << 49) | ((unsigned long long)o[2] << 17);
            a.keys[3 * (size_t)p] = key.a;
            a.keys[3 * (size_t)p + 1] = key.b;
            a.keys[3 * (size_t)p + 2] = key.c;
        }
        k.a[e] = key.a;
        k.b[e] = key.b;
        k.c[e] = key.c;
    }
    __syncthreads();
    {   // four neighbours in order: five exchanges
        static_assert(OPT == 4, "the sorting network below is for four");
        int x[4] = {4 * tid, 4 * tid + 1, 4 * tid + 2, 4 * tid + 3};
        constexpr int net[5][2] = {{0, 1}, {2, 3}, {0, 2}, {1, 3}, {1, 2}};
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int i = x[net[q][0]], j = x[net[q][1]];
            const bool swap = key_less(k, j, i);
            x[net[q][0]] = swap ? j : i;
            x[net[q][1]] = swap ? i : j;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) ord[0][4 * tid + u] = (uint16_t)x[u];
    }
    __syncthreads();
    int cur = 0;
    for (int len = OPT; len < OE; len *= 2) {
        const uint16_t* in = ord[cur];
        const int base = OPT * tid / (2 * len) * (2 * len), d = OPT * tid - base;
        const uint16_t *ra = in + base, *rb = in + base + len;
        int lo = max(0, d - len), hi = min(d, len);   // elements of the first run among the first d of the result
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (key_less(k, ra[mid], rb[d - 1 - mid])) lo = mid + 1; else hi = mid;
        }
        int ia = lo, ib = d - lo;
#pragma unroll
        for (int u = 0; u < OPT; ++u) {
            const bool from_a = ia < len && (ib >= len || key_less(k, ra[min(ia, len - 1)], rb[min(ib, len - 1)]));
            ord[cur ^ 1][OPT * tid + u] = from_a ? ra[ia] : rb[ib];
            ia += from_a ? 1 : 0;
            ib += from_a ? 0 : 1;
        }
        __syncthreads();
        cur ^= 1;
    }
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        const int e = u * OST + tid;
        if (first + e < a.n) a.idx[0][first + e] = (int)first + ord[cur][e];
    }
}

__device__ __forceinline__ OrderKey load_key(const unsigned long long* __restrict__ keys, int i)
{
    return OrderKey{keys[3 * (size_t)i], keys[3 * (size_t)i + 1], keys[3 * (size_t)i + 2]};
}

// x (of the earlier run) comes before y (of the later one) unless y's key is smaller
__device__ __forceinline__ bool before(const OrderKey& x, const OrderKey& y)
{
    if (x.a != y.a) return x.a < y.a;
    if (x.b != y.b) return x.b < y.b;
    return x.c <= y.c;
}

// Merges the sorted runs [base, base + run) and [base + run, base + 2 run) of src into dst, one workgroup per OE results.
__global__ __launch_bounds__(OST) void k_order_merge(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                     const unsigned long long* __restrict__ keys, int n, long long run)
{
    __shared__ KeyTile k;
    __shared__ int32_t idx[OE];
    __shared__ int split[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long out0 = (long long)blockIdx.x * OE;
    const int count = (int)min((long long)OE, (long long)n - out0);
    const long long base = out0 / (2 * run) * (2 * run);
    const int na = (int)min(run, (long long)n - base), nb = (int)max(0ll, min(run, (long long)n - base - run));
    const int32_t *ra = src + base, *rb = src + base + run;      // rb is only read when nb > 0
    if (wave < 2) {
        // how many of the first d results come from the first run: 64 places tried at once, d = where this workgroup's
        // results start (wave 0) and end (wave 1)
        const int d = (int)(out0 - base) + (wave ? count : 0);
        int lo = max(0, d - nb), hi = min(d, na);
        while (lo < hi) {
            const int step = (hi - lo + 63) >> 6;
            const int x = lo + lane * step;
            bool take = false;
            if (x < hi) take = before(load_key(keys, ra[x]), load_key(keys, rb[d - 1 - x]));
            const int yes = __popcll(__builtin_amdgcn_ballot_w64(take));      // a prefix of the lanes
            const int from = lo;
            if (yes > 0) lo = from + (yes - 1) * step + 1;
            if (yes < 64) hi = min(hi, from + yes * step);
        }
        if (lane == 0) split[wave] = lo;
    }
    __syncthreads();
    const int a0 = split[0], la = split[1] - a0, b0 = (int)(out0 - base) - a0, lb = count - la;
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        const int e = u * OST + tid;
        if (e < count) {
            const int i = e < la ? ra[a0 + e] : rb[b0 + e - la];
            const OrderKey key = load_key(keys, i);
            idx[e] = i;
            k.a[e] = key.a;
            k.b[e] = key.b;
            k.c[e] = key.c;
        }
    }
    __syncthreads();
    const int d = min(OPT * tid, count);
    int lo = max(0, d - lb), hi = min(d, la);
    while (lo < hi) {                                 // positions in LDS are in run order: equal keys go to the first run
        const int mid = (lo + hi) >> 1;
        if (key_less(k, mid, la + d - 1 - mid)) lo = mid + 1; else hi = mid;
    }
    int ia = lo, ib = d - lo;
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        if (d + u >= count) break;
        const bool from_a = ia < la && (ib >= lb || key_less(k, ia, la + ib));
        dst[out0 + d + u] = from_a ? idx[ia] : idx[la + ib];
        ia += from_a ? 1 : 0;
        ib += from_a ? 0 : 1;
    }
}

__global__ __launch_bounds__(OT) void k_order_gather(const int32_t* __restrict__ order, const float* __restrict__ coords, int n,
                                                     float* __restrict__ out)
{
    const long long p = (long long)blockIdx.x * OT + threadIdx.x;
    if (p >= n) return;
    const unsigned i = (unsigned)order[p];
    if (i >= (unsigned)n) return;
    out[(size_t)p * 3 + 0] = coords[(size_t)i * 3 + 0];
    out[(size_t)p * 3 + 1] = coords[(size_t)i * 3 + 1];
    out[(size_t)p * 3 + 2] = coords[(size_t)i * 3 + 2];
}

__global__ __launch_bounds__(OT) void k_order_compose(const int32_t* __restrict__ order, const int32_t* __restrict__ perm_sorted,
                                                      const int32_t* __restrict__ inv_sorted, int n, const int32_t* __restrict__ status,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm)
{
    if (status[0]) return;
    const long long p = (long long)blockIdx.x * OT + threadIdx.x;
    if (p >= n) return;
    const unsigned s = (unsigned)perm_sorted[p];
    if (s < (unsigned)n) perm[p] = order[s];
    const unsigned i = (unsigned)order[p];
    if (inv_perm && i < (unsigned)n) inv_perm[i] = inv_sorted[p];
}

}  // namespace

hipError_t order_launch(const OrderArgs& a, const int32_t** order_out, hipStream_t stream)
{
    *order_out = a.idx[0];
    if (a.n <= 0) return hipSuccess;
    const int tiles = (a.n + OE - 1) / OE;
    const int blocks = (a.n + OT - 1) / OT;
    k_order_init<<<(a.n_scans * 4 + OT - 1) / OT, OT, 0, stream>>>(a);
    k_order_box<<<(a.n + OB - 1) / OB, OT, 0, stream>>>(a);
    k_order_tiles<<<tiles, OST, 0, stream>>>(a);
    const int32_t* src = a.idx[0];
    int cur = 1;
    for (long long run = OE; run < a.n; run *= 2) {
        k_order_merge<<<tiles, OST, 0, stream>>>(src, a.idx[cur], a.keys, a.n, run);
        src = a.idx[cur];
        cur ^= 1;
    }
    *order_out = src;
    k_order_gather<<<blocks, OT, 0, stream>>>(src, a.coords, a.n, a.coords_sorted);
    return hipGetLastError();
}

hipError_t order_compose_launch(const int32_t* order, const int32_t* perm_sorted, const int32_t* inv_sorted, int n,
                                const int32_t* status, int32_t* perm, int32_t* inv_perm, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    k_order_compose<<<(n + OT - 1) / OT, OT, 0, stream>>>(order, perm_sorted, inv_sorted, n, status, perm, inv_perm);
    return hipGetLastError();
}

}  // namespace f3d
