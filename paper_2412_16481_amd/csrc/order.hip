// Canonical serving order for the rebalancing of Algorithm 2 (Section 4.1 "Bucket rebalancing" leaves the arrival
// order of the contenders of a bucket to the hardware race). Serving them in increasing
// (Z-order code of the voxel, x, y, z, input index) makes the partition of the points independent of the order in
// which they are stored. It is done by sorting the points once by that key and running the index-ordered bucketing on
// the sorted copy; the result is mapped back through the sort order.
//
// The sort is a merge sort on whole keys (scan, code, x, y, z packed into three 64-bit words), carrying only the point index: one kernel
// cuts the scans into tiles of 2048 positions and takes the tiles' bounding boxes, one builds the keys and sorts the tiles in LDS, then
// one kernel per doubling of the sorted length merges pairs of runs, a workgroup per tile of the result. Runs never reach over the
// end of a scan, so there are as many merges as the longest scan needs. (Batches of more than 512 scans are sorted as one run of
// positions, the scan in front of the key.) The cost does not depend on how the points fall into voxels.
//
// Bound: launches and latency (a merge launch is a chain of a search, two dependent loads and a search in LDS: 10 us at
// 457295 points, the tiles 27 us). A radix sort on 8-bit digits takes 21 passes over these keys, each with its own count,
// scan and scatter, whatever n is. A whole canonical bucketing, us: with such a sort / with runs over scan ends, minima by atomics and the
// code in the upper 63 bits of the key whatever its size / now (the last two in one job; the bucketing behind the sort has become shorter
// between them too): sensor sweeps, 457295 points in four scans 521 / 224 / 178, 914601 in eight - / 299 / 231; cubes, 500000 points in
// 100 scans - / 212 / 128, 60000 in 300 - / 147 / 84, 4 million in eight (buckets of 1024) - / 1626 / 1273; a room of 200000 486 / 209 / 198;
// one scan of 300 points - / 55.8 / 54.1, of 1500 248 / 58.3 / 55.1, of 4 million in buckets of 1024, where the bucketing alone takes
// 1843, - / 3216 / 3152. (A batch of 4 million points took 3440 with the radix sort and 1620 with the first form of this one; how it was cut into
// scans is not on record.) Tiles of 4096 take one merge less and one workgroup per compute unit: 457295 points 1 us less, one
// scan of 1500 12 more, of 200000 16 more.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "order.h"
#include "psh.h"
#include "psh_common.h"

namespace f3d {
namespace {

constexpr int OT = 256;          // threads per workgroup
constexpr int OE = 2048;         // positions per tile
constexpr int OST = 512;        // threads that sort or merge a tile
constexpr int OPT = OE / OST;    // results per thread

constexpr int OSCANS = OST;      // most scans that are sorted each by itself
// Longer scans have their boxes joined once (k_order_join); in others every tile joins them for itself, which is quadratic in the
// tiles. us of a whole canonical bucketing of one scan without / with that launch: 300 000 points 331 / 333, 1 million 661 / 662, 2 million
// 1234 / 1227, 16 million 14 750 / 14 300, 48 million 61 180 / 56 640.
constexpr long long OJOIN = 768 * OE;

// Where tile t of a batch of up to OSCANS scans lies: tiles never straddle scans. Written by k_order_set, with the bounding box of the
// tile's points (ordered ints, minimum xyz at [0..2], maximum at [4..6]) beside it.
struct TileInfo {
    int first, count;   // positions
    int p0, len;        // of the scan
    int t0, tiles;      // first tile of the scan and how many it has
    int scan, ok;
};
static_assert(sizeof(TileInfo) == 32, "the workspace has 32 bytes per tile");

__device__ __forceinline__ TileInfo tile_of(const OrderArgs& a, int t)
{
    if (a.n_scans > 1 && a.n_scans <= OSCANS) return reinterpret_cast<const TileInfo*>(a.tile_info)[t];
    // one scan, or (the keys begin with the scan) one run of positions over all
    const int first = t * OE;
    return TileInfo{first, min(OE, a.n - first), 0, a.n, 0, (a.n + OE - 1) / OE, 0, first < a.n};
}

__device__ __forceinline__ int scan_of(const OrderArgs& a, int p)
{
    return a.batch_offsets ? find_scan(a.batch_offsets, a.n_scans, p) : 0;
}

// Batches of up to OSCANS scans: one workgroup per tile finds its place (a prefix over the scans), writes it down, and the
// bounding box of its points, without atomics. Offsets that are not those of a batch leave no tiles: what follows does nothing, and
// the bucketing flags them.
__global__ __launch_bounds__(OST) void k_order_set(OrderArgs a)
{
    __shared__ TileInfo s_info;
    __shared__ uint32_t red[8];
    __shared__ int lds17[17];
    const int tid = threadIdx.x, lane = tid & 63;
    const int t = blockIdx.x, ns = a.n_scans;
    if (ns == 1) {
        if (tid == 0) s_info = tile_of(a, t);
    } else {
        // thread i looks at scan i; the first wave alone where it holds them all
        int p0 = 0, nb = 0;
        bool good = true;
        if (tid < ns) {
            p0 = a.batch_offsets ? a.batch_offsets[tid] : tid == 0 ? 0 : a.n;
            const int p1 = a.batch_offsets ? a.batch_offsets[tid + 1] : a.n;
            const long long d = (long long)p1 - p0;
            good = d >= 0 && d <= a.max_scan_points && p0 >= 0 && p1 <= a.n && (tid > 0 || p0 == 0) && (tid < ns - 1 || p1 == a.n);
            nb = good ? (int)d : 0;
        }
        const int tiles = (nb + OE - 1) / OE;
        int t0, total, bad;
        if (ns <= 64) {
            const int last = wave_incl_scan(tiles);
            t0 = last - tiles;
            total = __shfl(last, 63, 64);
            bad = __builtin_amdgcn_ballot_w64(!good) != 0ull;
        } else {
            t0 = block_excl_scan(tiles, &total, lds17);
            bad = __syncthreads_or(!good);
        }
        // One thread writes s_info: the one whose scan has the tile, thread 0 where there is none.
        if (t0 <= t && t < t0 + tiles && !bad && tid < ns) {
            TileInfo f;
            f.scan = tid;
            f.t0 = t0;
            f.tiles = tiles;
            f.p0 = p0;
            f.len = nb;
            f.first = p0 + (t - t0) * OE;
            f.count = min(OE, p0 + nb - f.first);
            f.ok = 1;
            s_info = f;
            reinterpret_cast<TileInfo*>(a.tile_info)[t] = f;
        }
        if (tid == 0 && (bad || t >= total)) {
            s_info.ok = 0;
            reinterpret_cast<TileInfo*>(a.tile_info)[t].ok = 0;
        }
    }
    if (tid < 3) {
        red[tid] = 0xFFFFFFFFu;
        red[4 + tid] = 0u;
    }
    __syncthreads();
    if (!s_info.ok) return;
    const float* src = a.coords + (size_t)s_info.first * 3;
    const int nf = s_info.count * 3;
    uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0u, 0u, 0u};
    float v[3 * OPT];
#pragma unroll
    for (int j = 0; j < 3 * OPT; ++j) {          // all loads in flight together; past the end: the axis' first value again
        const int f = tid + j * OST;
        v[j] = src[f < nf ? f : f % 3];
    }
#pragma unroll
    for (int j = 0; j < 3 * OPT; ++j) {
        const uint32_t o = f2ord(v[j]);
        const int ax = (tid + j * OST) % 3;
#pragma unroll
        for (int x = 0; x < 3; ++x)
            if (ax == x) { mn[x] = min(mn[x], o); mx[x] = max(mx[x], o); }
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        uint32_t lo = mn[x], hi = mx[x];
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0) { atomicMin(&red[x], lo); atomicMax(&red[4 + x], hi); }
    }
    __syncthreads();
    if (tid < 8) a.tile_box[t * 8 + tid] = red[(tid & 3) < 3 ? tid : 0];
}

// Scans of many tiles: the workgroup of the first joins the boxes of all of them in place of its own.
__global__ __launch_bounds__(OST) void k_order_join(OrderArgs a)
{
    __shared__ uint32_t red[8];
    const int tid = threadIdx.x;
    const TileInfo ti = tile_of(a, blockIdx.x);
    if (!ti.ok || (int)blockIdx.x != ti.t0) return;
    if (tid < 8) red[tid] = tid < 4 ? 0xFFFFFFFFu : 0u;
    __syncthreads();
    uint32_t* const boxes = a.tile_box + (size_t)ti.t0 * 8;
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
    for (int t = tid; t < ti.tiles; t += OST) {
#pragma unroll
        for (int x = 0; x < 3; ++x) { lo[x] = min(lo[x], boxes[(size_t)t * 8 + x]); hi[x] = max(hi[x], boxes[(size_t)t * 8 + 4 + x]); }
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        lo[x] = wave_min(lo[x]);
        hi[x] = wave_max(hi[x]);
        if ((tid & 63) == 0) { atomicMin(&red[x], lo[x]); atomicMax(&red[4 + x], hi[x]); }
    }
    __syncthreads();                                  // every box has been read
    if (tid < 8) boxes[tid] = red[tid];
}

// Batches of more scans: their minima by atomics.
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

// Key of a point: scan (16 bits), code, x, y, z (32 bits each), from the top of the first word down, zero-padded at the end. The code
// takes as many bits as the scan's largest (63 in batches of many scans): what stands in front of x is then nearly always
// in the first word, and some of x too, and a comparison seldom looks at the second.
struct OrderKey {
    unsigned long long a, b, c;
};

__device__ __forceinline__ OrderKey make_key(int scan, uint64_t code, int bits, uint32_t x, uint32_t y, uint32_t z)
{
    const uint64_t u = ((uint64_t)x << 32) | y, w = (uint64_t)z << 32;
    const uint64_t h0 = (code << (64 - bits)) | (u >> bits), h1 = (u << (64 - bits)) | (w >> bits), h2 = w << (64 - bits);   // 0 < bits < 64
    return OrderKey{((uint64_t)(uint32_t)scan << 48) | (h0 >> 16), (h0 << 48) | (h1 >> 16), (h1 << 48) | (h2 >> 16)};
}

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
template <bool FEW>   // a batch of up to OSCANS scans
__global__ __launch_bounds__(OST) void k_order_tiles(OrderArgs a)
{
    __shared__ KeyTile k;
    __shared__ uint16_t ord[2][OE];
    __shared__ uint32_t box[8];
    const int tid = threadIdx.x;
    const TileInfo ti = tile_of(a, blockIdx.x);
    if (!ti.ok) return;
    if (FEW && tid < 64) {                            // the boxes of the scan's tiles
        uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
        for (int t = tid; t < (a.joined ? 1 : ti.tiles); t += 64) {
            const uint32_t* b = a.tile_box + (size_t)(ti.t0 + t) * 8;
#pragma unroll
            for (int x = 0; x < 3; ++x) { lo[x] = min(lo[x], b[x]); hi[x] = max(hi[x], b[4 + x]); }
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            lo[x] = wave_min(lo[x]);
            hi[x] = wave_max(hi[x]);
            if (tid == 0) { box[x] = lo[x]; box[4 + x] = hi[x]; }
        }
    }
    float c[OPT][3];
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        const int e = min(u * OST + tid, ti.count - 1);
#pragma unroll
        for (int x = 0; x < 3; ++x) c[u][x] = a.coords[(size_t)(ti.first + e) * 3 + x];
    }
    int bits = 63;
    if (FEW) {                                        // of the largest code: that of the far corner of the box
        __syncthreads();
        bits = 1;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const float far = ord2f(box[4 + x]);
            const int v = far == far ? voxel_of(far, ord2f(box[x]), a.inv_voxel) : F3D_VOXEL_MAX;   // a NaN says nothing of the others
            if (v > 0) bits = max(bits, 3 * (31 - __clz(v)) + x + 1);
        }
    }
#pragma unroll
    for (int u = 0; u < OPT; ++u) {
        const int e = u * OST + tid;
        OrderKey key = {~0ull, ~0ull, ~0ull};         // past the end: behind every point (a scan index is below 65535)
        if (e < ti.count) {
            const size_t p = (size_t)(ti.first + e);
            const int b = FEW ? ti.scan : scan_of(a, (int)p);
            int v[3];
#pragma unroll
            for (int x = 0; x < 3; ++x) v[x] = voxel_of(c[u][x], ord2f(FEW ? box[x] : a.box[b * 4 + x]), a.inv_voxel);
            key = make_key(b, morton3(v[0], v[1], v[2]), bits, f2ord(c[u][0]), f2ord(c[u][1]), f2ord(c[u][2]));
            a.keys[3 * p] = key.a;
            a.keys[3 * p + 1] = key.b;
            a.keys[3 * p + 2] = key.c;
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
        if (e < ti.count) a.idx[0][ti.first + e] = ti.first + ord[cur][e];
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

// Merges the sorted runs [base, base + run) and [base + run, base + 2 run) of a scan's (of all) positions of src into dst, one
// workgroup per tile of results.
__global__ __launch_bounds__(OST) void k_order_merge(OrderArgs a, const int32_t* __restrict__ src_all, int32_t* __restrict__ dst_all, int run)
{
    __shared__ KeyTile k;
    __shared__ int32_t idx[OE];
    __shared__ int split[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TileInfo ti = tile_of(a, blockIdx.x);
    if (!ti.ok) return;
    const unsigned long long* __restrict__ keys = a.keys;
    const int32_t* __restrict__ src = src_all + ti.p0;
    int32_t* __restrict__ dst = dst_all + ti.p0;
    const int out0 = ti.first - ti.p0, count = ti.count;
    const int base = (int)((long long)out0 / (2ll * run) * (2ll * run));
    const int na = min(run, ti.len - base), nb = max(0, min(run, ti.len - base - run));
    const int32_t *ra = src + base, *rb = src + base + run;      // rb is only read when nb > 0
    if (nb == 0) {                                    // the last run has no partner yet
#pragma unroll
        for (int u = 0; u < OPT; ++u) {
            const int e = u * OST + tid;
            if (e < count) dst[out0 + e] = src[out0 + e];
        }
        return;
    }
    if (wave < 2) {
        // how many of the first d results come from the first run: 64 places tried at once, d = where this workgroup's
        // results start (wave 0) and end (wave 1)
        const int d = out0 - base + (wave ? count : 0);
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
    const int a0 = split[0], la = split[1] - a0, b0 = out0 - base - a0, lb = count - la;
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

hipError_t order_launch(const OrderArgs& args, const int32_t** order_out, hipStream_t stream)
{
    OrderArgs a = args;
    *order_out = a.idx[0];
    if (a.n <= 0) return hipSuccess;
    const bool few = a.n_scans <= OSCANS;
    const int tiles = few ? a.n / OE + a.n_scans : (a.n + OE - 1) / OE;
    const int blocks = (a.n + OT - 1) / OT;
    const long long longest = few && a.max_scan_points < a.n ? a.max_scan_points : a.n;
    if (few) {
        k_order_set<<<tiles, OST, 0, stream>>>(a);
        a.joined = longest > OJOIN;
        if (a.joined) k_order_join<<<a.n_scans == 1 ? 1 : tiles, OST, 0, stream>>>(a);
        k_order_tiles<true><<<tiles, OST, 0, stream>>>(a);
    } else {
        k_order_init<<<(a.n_scans * 4 + OT - 1) / OT, OT, 0, stream>>>(a);
        k_order_box<<<(a.n + OB - 1) / OB, OT, 0, stream>>>(a);
        k_order_tiles<false><<<tiles, OST, 0, stream>>>(a);
    }
    const int32_t* src = a.idx[0];
    int cur = 1;
    for (long long run = OE; run < longest; run *= 2) {
        k_order_merge<<<tiles, OST, 0, stream>>>(a, src, a.idx[cur], (int)run);
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
