// Internal interface between the C ABI (flash3d_api.hip) and the attention kernel (attn.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace f3d {

// How to divide a non-negative int by a value the launch knows: a shift (powers of two), else the upper half of a product
// where that is exact for every dividend in question, else (magic 0) an ordinary division.
struct Divide {
    uint32_t magic;
    int shift;      // -1: not a power of two
};
inline Divide make_divide(int d, long long most)   // dividends 0 .. most
{
    Divide r{0, -1};
    if (d > 0 && (d & (d - 1)) == 0) {
        r.shift = 0;
        while ((1 << r.shift) < d) ++r.shift;
    } else if (most * d < (1ll << 32)) {
        r.magic = (uint32_t)((1ull << 32) / (unsigned)d + 1);   // more than 2^32/d by less than one: off by less than most/2^32 < 1/d
    }
    return r;
}

struct AttnArgs {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    uint16_t* out;
    float* lse;                // null, or [n, H]: natural-log sum of exponentials of every row's scaled scores (bucket-major)
    const int32_t* out_perm;   // null: out is bucket-major; else the result of bucket-major row p goes to row out_perm[p]
    const int32_t* perm;     // may be null
    const int32_t* offsets;
    const int32_t* sbs;      // scan_bucket_start
    int n;
    int n_scans;
    int m;        // buckets per scope
    int mode;     // 0 plain, 1 shift, 2 stride
    int shift;
    int stride;
    int H;
    int C;        // row pitch in elements = heads * head_dim
    float c_log2; // softmax scale * log2(e)
    float q_pow2; // head_dim 32, bfloat16: a power of two, at most 1, that goes into the query (exactly), and
    float s_mul;  // head_dim 32: what is left of c_log2, multiplied onto the score
    int n_slots;  // scope slots over all scans (upper bound, surplus workgroups exit)
    int qblocks;  // query blocks per scope = ceil(bucket_cap / attn_block_rows(...))
    int extra;    // spare slots per scan: 2 (plain, shift) or stride + 1
    Divide by_m, by_t, by_mt, by_h, by_blocks;   // buckets per scope, stride, their product, heads, row blocks of a scope
    int f16;      // 0: q, k, v, out are bfloat16; 1: binary16 (forward only)
};

// Backward pass: the forward arguments (f.out = the forward output O, f.lse = its log-sum-exp, f.out_perm = where a
// gradient row goes, null = bucket-major) plus the incoming gradient and the three outgoing ones.
struct AttnBwdArgs {
    AttnArgs f;
    const uint16_t* dout;   // bf16 [n, C], gradient of the bucket-major output rows
    float* dsum;            // workspace [n, H]: sum over the head's channels of dO * O
    uint16_t* dq;           // bf16 [n, C]
    uint16_t* dk;
    uint16_t* dv;
    float scale;            // softmax scale (the forward's c_log2 divided by log2 e)
    int d_first;            // dq overwrites the forward output at other rows: D is summed by a kernel of its own, first
    int ahead;              // the score products run a tile ahead (always with two tiles); 0: the form for short scopes
    int tiles;              // tiles of 32 rows a wave owns (1 or 2): queries in the dQ kernel, keys in the dK/dV kernel
    int kblocks;            // ceil(bucket_cap / (128 * tiles)): row blocks of a scope (f.qblocks is the same)
    // one kernel for all three gradients
    int tasks;              // scope slots x heads, rounded up to a multiple of 8
    int done;               // tasks it takes of each eighth of them (those of an XCD); the two kernels take the others
    int cap;                // most rows of a scope
    float* scratch;         // workspace of scopes of several passes: [workgroups][cap][head_dim]
};
constexpr int ATTN_BWD_ONE_WAVES = 8;     // of a workgroup, 64 keys each
constexpr int ATTN_BWD_ONE_ROWS = 2048;   // the longest scope it takes: 16 bytes of LDS per row

hipError_t attn_bwd_one_launch(const AttnBwdArgs& a, int head_dim, int grid, hipStream_t stream);
hipError_t attn_bwd_launch(const AttnBwdArgs& a, int head_dim, hipStream_t stream);

int attn_block_rows(int head_dim, long long slots, int heads, int bucket_cap);   // query rows one workgroup covers
hipError_t attn_launch(const AttnArgs& a, int head_dim, int block_rows, hipStream_t stream);

}  // namespace f3d
