// Index build at prefill: promotion of the initial centroids, nearest-centroid assignment on the
// matrix cores, deterministic per-cluster means, and the node -> page layout (Sec. 4.1-4.2,
// Alg. 2 of the paper restricted to two levels and iterated as Lloyd rounds).
#include <algorithm>
#include <type_traits>

#include "ice_internal.h"

namespace ice {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// a.lo*b.lo + a.hi*b.hi + c on packed bf16 pairs, fp32 accumulate (v_dot2_f32_bf16)
__device__ inline float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

__device__ inline uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// ------------------------------------------------------------------------------------------------
// Transformed keys (Sec. 4.2, Eq. 2): T_K(k) = [k / c, sqrt(1 - ||k||^2 / c^2)] with c >= the largest
// key norm.  Distances are only compared, so everything is kept times c: the key itself plus ONE
// more coordinate a(k) = sqrt(c^2 - ||k||^2), stored as bf16 beside the keys; c^2 is the largest
// squared norm of the unit's prefill keys (a later key with a larger norm gets a(k) = 0).
// Pass 1: squared norms (16 lanes per key, fixed summation order) and their maximum per workgroup;
// pass 2: the maximum per unit and the extra coordinate.  (A maximum passes over NaN: whether a norm is one, or 2^118 and
// more, goes beside it, for `large_keys`.)
// Bound by one read of the keys.  The workgroups leave their maxima side by side and pass 2 reduces
// them: one atomic maximum per wave on the unit's word puts thousands of updates on one or two cache
// lines (16 units x 23457 keys, 96 MB: 76 us for the atomic form; the whole six-round build went from
// 753 to 692 us without them).
__global__ __launch_bounds__(256) void key_norms_kernel(Dev d, const bf16_t *__restrict__ K, int n, float *n2_out, float *max_out) {
    // 256 keys per workgroup (16 at a time, 16 lanes each)
    __shared__ float wmax[4], wlarge[4];
    const int u = blockIdx.y, row = threadIdx.x >> 4, ch = threadIdx.x & 15;
    float mx = 0.f;
    u64 large = 0ull;
    uint4 w[16];  // the workgroup's 64 KB of key rows are requested at once (read once: streaming loads)
#pragma unroll
    for (int it = 0; it < 16; ++it) {
        const int i = blockIdx.x * 256 + it * 16 + row;
        w[it] = i < n ? load16_stream((const uint4 *)(K + ((size_t)u * n + i) * kD) + ch) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int it = 0; it < 16; ++it) {
        const int i = blockIdx.x * 256 + it * 16 + row;
        const float n2 = key_sqnorm16(w[it]);  // (uniform over the 16 lanes of a key: no divergent reduction)
        if (i < n) {
            if (ch == 0) n2_out[(size_t)u * d.max_tokens + i] = n2;
            mx = fmaxf(mx, n2);
        }
        large |= __ballot(!(n2 < 0x1p118f));  // (rows past the end are zeros)
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if ((threadIdx.x & 63) == 0) {
        wmax[threadIdx.x >> 6] = mx;
        wlarge[threadIdx.x >> 6] = large != 0ull ? 1.f : 0.f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const size_t at = (size_t)u * d.max_tokens + blockIdx.x;
        max_out[at] = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
        max_out[(size_t)d.U * d.max_tokens + at] = fmaxf(fmaxf(wlarge[0], wlarge[1]), fmaxf(wlarge[2], wlarge[3]));
    }
}
__global__ __launch_bounds__(256) void key_aug_kernel(Dev d, int n, const float *n2_in, const float *max_in) {
    __shared__ float wmax[4], wlarge[4];
    const int u = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    const float n2 = i < n ? n2_in[(size_t)u * d.max_tokens + i] : 0.f;
    float c2 = 0.f, large = 0.f;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += 256) {
        c2 = fmaxf(c2, max_in[(size_t)u * d.max_tokens + b]);
        large = fmaxf(large, max_in[((size_t)d.U + u) * d.max_tokens + b]);
    }
    for (int off = 1; off < 64; off <<= 1) c2 = fmaxf(c2, __shfl_xor(c2, off));
    const u64 any_large = __ballot(large > 0.f);
    if ((threadIdx.x & 63) == 0) {
        wmax[threadIdx.x >> 6] = c2;
        wlarge[threadIdx.x >> 6] = any_large != 0ull ? 1.f : 0.f;
    }
    __syncthreads();
    c2 = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        d.c2[u] = c2;
        d.large_keys[u] = wlarge[0] + wlarge[1] + wlarge[2] + wlarge[3] > 0.f;
    }
    if (i < n) d.kaug[(size_t)u * d.max_tokens + i] = key_extra_coordinate(c2, n2);
}

void launch_key_aug(const Dev &d, const bf16_t *K, int n, hipStream_t st) {
    // (order and packed are free until the first assignment)
    float *n2 = (float *)d.order, *part = (float *)d.packed;
    hipLaunchKernelGGL(key_norms_kernel, dim3((n + 255) / 256, d.U), dim3(256), 0, st, d, K, n, n2, part);
    hipLaunchKernelGGL(key_aug_kernel, dim3((n + 255) / 256, d.U), dim3(256), 0, st, d, n, n2, part);
}

// A build's scratch at the start of a unit's key tiles, which the page layout overwrites in any case (see Near)
constexpr int kNearHead = 6, kNearHeadBytes = 256;
__device__ inline char *near_scratch(const Dev &d, int u) { return (char *)(d.Kp + (size_t)u * d.max_pages * d.s * kD); }

// ------------------------------------------------------------------------------------------------
// Initial centroids = the promoted keys (Alg. 2, "random promotion" with an exact count): cluster c
// of unit u starts at key init_idx[u][c], or, without a list, at a hashed position inside the c-th
// of C equal strata of the sequence (distinct by construction).  One wave per centroid row; rows
// >= C are padding (zero vector, infinite norm) in both centroid buffers.
__global__ __launch_bounds__(64) void init_centroids_kernel(Dev d, const bf16_t *K, int n,
                                                            const int *init_idx, uint64_t seed, int cur) {
    const int c = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
    uint32_t *cb0 = (uint32_t *)(d.cent_bf16[cur] + ((size_t)u * d.Cpad + c) * kD);
    uint32_t *cb1 = (uint32_t *)(d.cent_bf16[cur ^ 1] + ((size_t)u * d.Cpad + c) * kD);
    if (lane == 0) d.moved[(size_t)u * d.Cpad + c] = d.touched[(size_t)u * d.Cpad + c] = 0;
    if (c == 0 && lane == 0 && !d.tk) d.large_keys[u] = 0;  // (transformed keys: set already)
    if (c == 0 && lane < kNearHead) ((int *)near_scratch(d, u))[lane] = 0;
    if (c >= d.C) {
        cb0[lane] = 0u;
        cb1[lane] = 0u;
        if (lane == 0) {
            d.cnorm[cur][(size_t)u * d.Cpad + c] = INFINITY;
            d.cnorm[cur ^ 1][(size_t)u * d.Cpad + c] = INFINITY;
            if (d.tk) d.caug[cur][(size_t)u * d.Cpad + c] = d.caug[cur ^ 1][(size_t)u * d.Cpad + c] = 0;
        }
        return;
    }
    int idx;
    if (init_idx) {
        idx = init_idx[(size_t)u * d.C + c];
        idx = idx < 0 ? 0 : (idx >= n ? n - 1 : idx);
    } else {
        long long lo = (long long)c * n / d.C, hi = (long long)(c + 1) * n / d.C;
        idx = (int)(lo + (long long)(splitmix64(seed ^ ((uint64_t)u << 32) ^ (uint64_t)c) % (uint64_t)(hi - lo)));
    }
    const uint32_t w = ((const uint32_t *)(K + ((size_t)u * n + idx) * kD))[lane];
    const float lo = bf16_lo(w), hi = bf16_hi(w);
    cb0[lane] = w;
    ((float2 *)(d.centroid + ((size_t)u * d.C + c) * kD))[lane] = make_float2(lo, hi);
    float nn = wave_sum(lo * lo + hi * hi);
    if (lane == 0) {
        if (d.tk) {  // the promoted key's extra coordinate
            const bf16_t a = d.kaug[(size_t)u * d.max_tokens + idx];
            const float af = bf16_to_f32(a);
            d.caug[cur][(size_t)u * d.Cpad + c] = a;
            d.cent_aug[(size_t)u * d.C + c] = af;
            nn += af * af;
        }
        d.cnorm[cur][(size_t)u * d.Cpad + c] = nn;
        d.init_idx[(size_t)u * d.C + c] = idx;
    }
}

void launch_init_centroids(const Dev &d, const bf16_t *K, int n, const int *init_idx, uint64_t seed, int cur,
                           hipStream_t st) {
    hipLaunchKernelGGL(init_centroids_kernel, dim3(d.Cpad, d.U), dim3(64), 0, st, d, K, n, init_idx, seed, cur);
}

// Caller-supplied bf16 centroids [U][C][128] -> live centroid buffer (padding + squared norms).
__global__ __launch_bounds__(64) void load_centroids_kernel(Dev d, const bf16_t *cent, int cur) {
    const int c = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
    uint32_t *cb = (uint32_t *)(d.cent_bf16[cur] + ((size_t)u * d.Cpad + c) * kD);
    if (c >= d.C) {
        cb[lane] = 0u;
        if (lane == 0) d.cnorm[cur][(size_t)u * d.Cpad + c] = INFINITY;
        return;
    }
    const uint32_t w = ((const uint32_t *)(cent + ((size_t)u * d.C + c) * kD))[lane];
    cb[lane] = w;
    const float lo = bf16_lo(w), hi = bf16_hi(w);
    const float nn = wave_sum(lo * lo + hi * hi);
    if (lane == 0) d.cnorm[cur][(size_t)u * d.Cpad + c] = nn;
}

void launch_load_centroids(const Dev &d, const bf16_t *cent, int cur, hipStream_t st) {
    hipLaunchKernelGGL(load_centroids_kernel, dim3(d.Cpad, d.U), dim3(64), 0, st, d, cent, cur);
}

// Recompute the bf16 rounding and squared norm of every centroid from the fp32 centroids.
__global__ __launch_bounds__(64) void refresh_centroids_kernel(Dev d, int cur) {
    const int c = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
    uint32_t *cb = (uint32_t *)(d.cent_bf16[cur] + ((size_t)u * d.Cpad + c) * kD);
    if (c >= d.C) {
        cb[lane] = 0u;
        if (lane == 0) d.cnorm[cur][(size_t)u * d.Cpad + c] = INFINITY;
        return;
    }
    const float2 m = ((const float2 *)(d.centroid + ((size_t)u * d.C + c) * kD))[lane];
    const bf16_t b0 = f32_to_bf16(m.x), b1 = f32_to_bf16(m.y);
    cb[lane] = (uint32_t)b0 | ((uint32_t)b1 << 16);
    const float lo = bf16_to_f32(b0), hi = bf16_to_f32(b1);
    const float nn = wave_sum(lo * lo + hi * hi);
    if (lane == 0) d.cnorm[cur][(size_t)u * d.Cpad + c] = nn;
}

void launch_refresh_centroids(const Dev &d, int cur, hipStream_t st) {
    hipLaunchKernelGGL(refresh_centroids_kernel, dim3(d.Cpad, d.U), dim3(64), 0, st, d, cur);
}

// The copy of every cluster's tail-page state that the insertions work on (fill and key sum).
__global__ __launch_bounds__(256) void refresh_tails_kernel(Dev d) {
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6), u = blockIdx.y, lane = threadIdx.x & 63;
    if (c >= d.C) return;
    const size_t cl = (size_t)u * d.C + c;
    const int tail = d.cluster_tail[cl];
    float2 ps = make_float2(0.f, 0.f);
    int fill = d.s;
    if (tail >= 0) {
        const size_t pg = (size_t)u * d.max_pages + tail;
        fill = d.page_fill[pg];
        ps = ((const float2 *)(d.page_sum + pg * kD))[lane];
    }
    ((float2 *)(d.tail_sum + cl * kD))[lane] = ps;
    if (lane == 0) d.tail_fill[cl] = fill;
}
void launch_refresh_tails(const Dev &d, hipStream_t st) {
    hipLaunchKernelGGL(refresh_tails_kernel, dim3((d.C + 3) / 4, d.U), dim3(256), 0, st, d);
}

// An import in one launch: the caller's arrays are copied, what is derived from them is formed from the
// caller's copies beside that (the centroids' bf16 rounding and squared norms for both buffers, the tail
// pages' state), and the decode state is set.  Bound by the copy; apart, twelve copies and seven small
// launches cost their start-up and drain each (32 units x 8392 tokens, 385 MB read and written: 71 us in one launch;
// a turn of 200 tokens took 252 us with them apart and 211 with this).
// Blocks [0, copy_blocks) copy 32 KB each, the next cluster_blocks take four clusters each (one wave per
// cluster), the rest the score slots and the units' counters.
constexpr int kImportArrays = 12, kImportChunk = 32768;
struct ImportArgs {
    const char *src[kImportArrays];
    char *dst[kImportArrays];
    size_t bytes[kImportArrays];
    unsigned first[kImportArrays];  // first copy block of the array
    const float *centroid, *page_sum;
    const int *cluster_tail, *page_fill;
    unsigned copy_blocks, cluster_blocks;
    int n_tokens;
};
__global__ __launch_bounds__(256) void import_kernel(Dev d, ImportArgs a) {
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned blk = blockIdx.x;
    if (blk < a.copy_blocks) {
        int x = 0;
#pragma unroll
        for (int i = 1; i < kImportArrays; ++i) x = blk >= a.first[i] ? i : x;
        const size_t at = (size_t)(blk - a.first[x]) * kImportChunk, left = a.bytes[x] - at;
        const u32x4 *src = (const u32x4 *)(a.src[x] + at);
        u32x4 *dst = (u32x4 *)(a.dst[x] + at);
        if (left >= (size_t)kImportChunk) {
            u32x4 w[8];  // (of uint4 structures the compiler keeps a copy in scratch memory)
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = src[i * 256 + tid];
#pragma unroll
            for (int i = 0; i < 8; ++i) dst[i * 256 + tid] = w[i];
        } else {
            const int n16 = (int)(left / 16), n4 = (int)(left / 4);
            for (int i = tid; i < n16; i += 256) dst[i] = src[i];
            for (int i = n16 * 4 + tid; i < n4; i += 256) ((uint32_t *)dst)[i] = ((const uint32_t *)src)[i];
        }
        return;
    }
    blk -= a.copy_blocks;
    if (blk < a.cluster_blocks) {
        const unsigned row = blk * 4 + (tid >> 6);
        if (row >= (unsigned)d.U * d.Cpad) return;
        const int u = (int)(row / d.Cpad), c = (int)(row % d.Cpad);
        if (c >= d.C) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                ((uint32_t *)(d.cent_bf16[b] + (size_t)row * kD))[lane] = 0u;
                if (lane == 0) d.cnorm[b][row] = INFINITY;
            }
            return;
        }
        const size_t cl = (size_t)u * d.C + c;
        const float2 m = ((const float2 *)(a.centroid + cl * kD))[lane];
        const int tail = a.cluster_tail[cl];
        const bf16_t b0 = f32_to_bf16(m.x), b1 = f32_to_bf16(m.y);
        const float lo = bf16_to_f32(b0), hi = bf16_to_f32(b1);
        const float nn = wave_sum(lo * lo + hi * hi);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            ((uint32_t *)(d.cent_bf16[b] + (size_t)row * kD))[lane] = (uint32_t)b0 | ((uint32_t)b1 << 16);
            if (lane == 0) d.cnorm[b][row] = nn;
        }
        float2 ps = make_float2(0.f, 0.f);
        int fill = d.s;
        if (tail >= 0 && tail < d.max_pages) {
            const size_t pg = (size_t)u * d.max_pages + tail;
            fill = a.page_fill[pg];
            ps = ((const float2 *)(a.page_sum + pg * kD))[lane];
        }
        ((float2 *)(d.tail_sum + cl * kD))[lane] = ps;
        if (lane == 0) d.tail_fill[cl] = fill;
        return;
    }
    const size_t i = ((size_t)(blk - a.cluster_blocks) * 256 + tid) * 4, ns = (size_t)d.U * d.max_pages;
    if (i + 4 <= ns) {
        ((uint4 *)d.scores)[i / 4] = make_uint4(~0u, ~0u, ~0u, ~0u);
    } else {
        for (size_t x = i; x < ns; ++x) d.scores[x] = ~0u;
    }
    const size_t u = i / 4;
    if (u < (size_t)d.U) { d.n_tokens[u] = a.n_tokens; d.counter[u] = 0; d.attn_arrive[u] = 0; }
}

void launch_import(const Dev &d, const void *const *src, void *const *dst, const size_t *bytes, const ice_index_view_t &v, hipStream_t st) {
    ImportArgs a;
    unsigned blocks = 0;
    for (int i = 0; i < kImportArrays; ++i) {
        a.src[i] = (const char *)src[i];
        a.dst[i] = (char *)dst[i];
        a.bytes[i] = bytes[i];
        a.first[i] = blocks;
        blocks += (unsigned)((bytes[i] + kImportChunk - 1) / kImportChunk);
    }
    a.centroid = v.centroid; a.page_sum = v.page_sum; a.cluster_tail = v.cluster_tail; a.page_fill = v.page_fill;
    a.copy_blocks = blocks;
    a.cluster_blocks = (unsigned)(((size_t)d.U * d.Cpad + 3) / 4);
    a.n_tokens = v.n_tokens;
    const size_t state = std::max<size_t>(((size_t)d.U * d.max_pages + 3) / 4, (size_t)d.U);  // one thread per four score slots and per unit
    hipLaunchKernelGGL(import_kernel, dim3(a.copy_blocks + a.cluster_blocks + (unsigned)((state + 255) / 256)), dim3(256), 0, st, d, a);
}

// ------------------------------------------------------------------------------------------------
// Sorting the tokens by cluster (ascending position inside a cluster), range by range: a unit's tokens
// are cut into R ranges of L, one workgroup each, and every range is sorted by itself (`order`, stable
// counting sort) with every cluster's piece (first slot, members) beside it (`range_off`).  The members of
// a cluster in ascending position are its pieces of range 0, 1, ...: what reads members (the means, the
// page layout) finds member j through the pieces' lengths (Pieces), so no pass over the
// whole unit ties the ranges together: one launch per round, bound by its latencies.  (With a second
// launch that turned the ranges' totals into unit-wide positions the two took 17.2 us per round at
// 8 units x 32768 tokens x 512 clusters and 32 us at 131072 x 2048, most of it reading R totals per
// cluster in every workgroup; this one takes 6.1 and 16 us, and the means
// read their lists at 3 to 6 us more.  A fifth wave in the means that prepared the next cluster's list while
// four summed was slower, 24 against 17.3 us: its chain of list reads is the longer one.)
// A range is cut into W segments, one per wave.  A wave walks its segment 64 tokens at a time: lanes
// with the same cluster find each other bit by bit of the id (ballots), the first of them moves the
// segment's counter of that cluster past all of them, and a token's rank among its cluster's
// members of the segment stays in its register.  The counters are then scanned over segments and
// clusters and every token's slot is counter + rank.  W x Cpad counters of 4 bytes fit 144 KB.
constexpr int kSortCounters = 36864, kSortMaxSeg = 2048;  // LDS counters; tokens per segment at most

static int sort_segments(int Cpad) {
    int W = 16;
    while (W * Cpad > kSortCounters) W /= 2;  // (Cpad <= 8192: W >= 4)
    return W;
}
static int sort_max_len(int Cpad) { return sort_segments(Cpad) * kSortMaxSeg; }
static int sort_range_len(int U, int n, int Cpad) {
    // short ranges keep the chip busy, few ranges keep the reading of their pieces short: at most 64 per
    // unit and one workgroup per CU unless even the longest ranges are more (256 units x 32768 tokens: two
    // ranges 80 us and the means 426, one range 94 and 411; 64 units: eight ranges 24 and 115, four 20 and 109)
    int L = 1024;
    while (L < sort_max_len(Cpad) && L < n && ((n + L - 1) / L > 64 || (long long)U * ((n + L - 1) / L) > 256)) L *= 2;
    return L;
}
// Whether a build's assignment sorts its runs itself (a run is then a range of the sort): one slice of centroids, at most
// kFusedRun tiles per workgroup (their winners sit in LDS), one workgroup per CU and at most 128 ranges per unit.  A launch and
// the reading of the winners less per round; assignment and sort by themselves and in one, us: 8 units x 4000 x 62 5.2 + 5.8 and
// 7.6, 8 x 16384 x 256 13.0 + 6.3 and 15.8, 8 x 32768 x 512 34.7 + 7.2 and 38.1, 16 x 23457 x 366 (transformed) 40.9 + 9.0 and 46.0.
// What reads the members pays for shorter ranges: a wave holds 64 pieces of a cluster, and beyond 64 ranges a cluster that is
// not listed in LDS (kMemberSlots) is searched piece by piece.  So more than 64 ranges are for clusters of about 330 members and
// fewer.  Whole builds of ten rounds, by themselves and in one: 32 ranges 8 x 32768 x 512 517 and 486, clusters of 2048 8 x 32768 x 16
// 706 and 673; 79 ranges 1 x 20000 x 60 213 and 189, x 40 243 and 241; 128 ranges 1 x 32768 x 512 246 and 219, x 100 (328 members) 226
// and 202, transformed 286 and 282; but x 80 (410) 246 and 248, transformed 285 and 302, x 16 376 and 423; 2 x 65536 x 200 (328) 344 and
// 345, x 128 345 and 355, x 32 transformed 650 and 792.
constexpr int kFusedRun = 16, kFusedMembers = 336;
static int assign_run(int U, int n, int slices);
bool sort_is_fused(const Dev &d, int n) {
    if (d.Cpad > 512) return false;
    const int run = assign_run(d.U, n, 1), R = (n + run * kAssignTile - 1) / (run * kAssignTile);
    return run <= kFusedRun && R <= (n <= (long long)kFusedMembers * d.C ? 128 : 64) && (long long)d.U * R <= 256;
}
// tokens per range of the sort
static int sort_len(const Dev &d, int n) { return sort_is_fused(d, n) ? assign_run(d.U, n, 1) * kAssignTile : sort_range_len(d.U, n, d.Cpad); }
size_t sort_ranges_max(int U, int max_tokens, int Cpad) {
    const int L = sort_max_len(Cpad);
    return std::max<size_t>(std::max(256, U), (size_t)U * (((size_t)max_tokens + L - 1) / L));
}

// The thread's number out of its wave's, worked out where it is asked for.
__device__ inline int thread_of(int wave) {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return wave * 64 + lane;
}

// NG: groups of 64 tokens per wave at most.  MASK: the lanes of a group with the same cluster meet in a 64-bit lane mask per
// cluster in LDS (OR, read back, clear) instead of by ballots: cheaper per group, but the masks have to be cleared and
// take 8 more bytes per counter, so it is for long ranges (256 units x 32768 tokens: 78 us with ballots, 69 so).
// The sort of tokens [rb, re) of unit u, its range r of R, by a workgroup of NWV waves; W segments of `seg` tokens.
// winner(i): what is known of token i's cluster, cluster(.): which it is (apart, so that nothing is waited for where it is
// loaded), best_of(i): what goes to best_out.  Every thread comes here.
template <int NWV, int NG, bool MASK, typename Winner, typename Cluster, typename BestOf>
__device__ inline void sort_range(const Dev &d, int tid, int u, int n, int r, int R, int rb, int re, int seg, int W, int nbits, int round, int goes,
                                  int *pos_all, float *best_out, int *assign_out, Winner winner, Cluster cluster, BestOf best_of) {
    constexpr int NT = NWV * 64;
    __shared__ int wsum[NWV];
    __shared__ int carry;
    const int lane = tid & 63, wave = tid >> 6;
    const int Cpad = d.Cpad;
    const int beg = min(re, rb + wave * seg), end = wave < W ? min(re, beg + seg) : beg;  // this wave's tokens
    uint32_t v[NG];
    // The last round's clusters.  The registers of the longest form hold a few of them at a time, requested kAhead groups ahead.
    constexpr int kAhead = NG <= 16 ? NG : 8;
    int was[kAhead];
    const int *assign = d.assign + (size_t)u * d.max_tokens;
    auto token = [&](int j) { return min(beg + j * 64 + lane, re - 1); };  // (past the end: read and dropped, no branch around the loads)
#pragma unroll
    for (int j = 0; j < NG; ++j) v[j] = winner(token(j));
    if (round > 0) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) was[j] = assign[token(j)];
    }
    if (goes == 0) return;  // (no centroid moved: nor did a token)
    for (int x = tid; x < W * Cpad / 4 * (MASK ? 3 : 1); x += NT) ((int4 *)pos_all)[x] = make_int4(0, 0, 0, 0);  // (Cpad is a multiple of 32)
    if (tid == 0) carry = 0;
    __syncthreads();
    // ---- rank inside the segment (row `wave` of the counters is this wave's alone)
    int *pos = pos_all + (wave < W ? wave : 0) * Cpad;
    u64 *mask = (u64 *)(pos_all + W * Cpad) + (size_t)(wave < W ? wave : 0) * Cpad;  // (MASK)
    const u64 lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < NG; ++j) {  // v[j]: from here on cluster << 16 | rank
        const int i = beg + j * 64 + lane;
        const bool valid = i < end;
        // (always < C for finite keys; a key with no finite score may come out with a padding row: it goes to the last
        // cluster, so that every token has a page whatever its key holds)
        const int a = (int)min(cluster(v[j]), (uint32_t)d.C - 1u);
        v[j] = (uint32_t)a << 16;
        if (beg + j * 64 >= end) continue;  // (wave-uniform)
        u64 peers;
        if constexpr (MASK) {
            if (valid) atomicOr(&mask[a], 1ull << lane);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            peers = valid ? mask[a] : 0ull;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (valid) mask[a] = 0ull;
        } else {
            peers = __ballot(valid);
            for (int b = 0; b < nbits; ++b) {
                const bool bit = (a >> b) & 1;
                const u64 m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
        }
        if (valid) {
            const int base = pos[a];
            v[j] |= (uint32_t)(base + (int)__popcll(peers & lt));
            if ((peers & lt) == 0ull) pos[a] = base + (int)__popcll(peers);
            d.assign[(size_t)u * d.max_tokens + i] = a;
            if (assign_out) assign_out[(size_t)u * n + i] = a;
            if (best_out) best_out[(size_t)u * n + i] = best_of(i);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (the LDS unit executes a wave's accesses in order)
        if constexpr (kAhead < NG) {
            if (round > 0) {
                const int b = was[j % kAhead];
                if (valid && a != b) d.touched[(size_t)u * Cpad + a] = d.touched[(size_t)u * Cpad + b] = 1;
                if (j + kAhead < NG) was[j % kAhead] = assign[token(j + kAhead)];
            }
        }
    }
    if (kAhead == NG && round > 0) {  // a later round of a build: the clusters that lost or gained a token are marked
        // (a range without such a token could be left as it is, but finding that out for the whole workgroup takes as long
        // as sorting 1024 tokens: 6.3 us with the exit taken or not)
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const int i = beg + j * 64 + lane;
            if (i < end) {
                const int a = (int)(v[j] >> 16), b = was[j % kAhead];
                if (a != b) d.touched[(size_t)u * Cpad + a] = d.touched[(size_t)u * Cpad + b] = 1;
            }
        }
    }
    __syncthreads();
    // ---- scan over segments and clusters
    uint32_t *off = d.range_off + ((size_t)u * R + r) * Cpad;
    for (int c0 = 0; c0 < Cpad; c0 += NT) {
        const int c = c0 + tid;
        int t[NWV], tot = 0;
#pragma unroll
        for (int w = 0; w < NWV; ++w) {
            t[w] = c < Cpad && w < W ? pos_all[w * Cpad + c] : 0;
            tot += t[w];
        }
        const int incl = wave_scan_add(tot);
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int ex = carry + incl - tot;
#pragma unroll
        for (int w = 0; w < NWV; ++w) ex += w < wave ? wsum[w] : 0;
        if (c < Cpad) {
            off[c] = (uint32_t)ex << 16 | (uint32_t)tot;  // (both at most 32768)
            int run = ex;
#pragma unroll
            for (int w = 0; w < NWV; ++w) {
                if (w < W) pos_all[w * Cpad + c] = run;
                run += t[w];
            }
        }
        __syncthreads();
        if (c0 + NT >= Cpad) break;
        if (tid == NT - 1) carry = ex + tot;  // (threads past Cpad add nothing)
        __syncthreads();
    }
    // ---- place
    int *order = d.order + (size_t)u * d.max_tokens + rb;
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        const int i = beg + j * 64 + lane;
        if (i < end) order[pos[v[j] >> 16] + (int)(v[j] & 0xFFFFu)] = i;
    }
}

// ------------------------------------------------------------------------------------------------
// A key's winner in memory: round's number (its low 19 bits) << 45 | ordered score << 13 | ~cluster (its low 13 bits).  Slices
// of the centroids meet by atomic maxima of such words, and a later round's are above those of the rounds before: nothing is
// cleared between rounds.  (A launch that did took 6 us of 440 at 8 units x 131072 x 2048, 5 of 33 at 2 x 32768 x 2048.)  In
// LDS, inside one round: ordered score << 32 | ~cluster.
constexpr int kMaxClusters = 8192;
__device__ inline u64 winner_word(u64 best, uint32_t round) {
    return (u64)round << 45 | (best >> 32) << 13 | (best & (kMaxClusters - 1));
}
__device__ inline u64 winner_of_word(u64 w) { return (w >> 13) << 32 | (0xFFFFFFFFu & ~(uint32_t)(kMaxClusters - 1)) | ((uint32_t)w & (kMaxClusters - 1)); }
__device__ inline uint32_t cluster_of_word(uint32_t low) { return ~low & (kMaxClusters - 1); }
// zero winners, where no round's are there
__global__ __launch_bounds__(256) void clear_winners_kernel(Dev d, int n) {
    const int u = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) d.packed[(size_t)u * d.max_tokens + i] = 0ull;
}

// ------------------------------------------------------------------------------------------------
// Nearest centroid on the matrix cores.
//   score(i, c) = k_i . mu~_c - ||mu~_c||^2 / 2      (argmax score == argmin ||k_i - mu~_c||^2)
// A dense (keys x 128) by (128 x centroids) contraction: v_mfma_f32_32x32x16_bf16 with the
// centroids as the A operand (rows) and the keys as the B operand (columns), so one lane ends up
// with 16 centroid scores of ONE key per 32x32 tile and the argmax over centroids stays in-lane.
// The accumulator is seeded with -||mu~||^2/2, so the epilogue is compare/select only.
//
// A workgroup of 8 waves covers CW * CT * 32 centroids (wave w keeps CT tiles of 32 centroids in
// registers for its whole life) and streams its share of the unit's keys through LDS in tiles of
// 256 keys (direct global -> LDS loads into unpadded rows whose 16-byte chunks are swizzled by row,
// so the 32-row operand reads are bank-conflict free).  When CW < 8 the remaining waves split the
// key tile instead.  Per key
// the waves' candidates meet in an LDS 64-bit max of (ordered score, ~centroid id): the exact fp32
// maximum with the lowest centroid id on ties.  More than CW*CT*32 centroids are covered by
// blockIdx.y slices that meet the same way in global memory.
//
// In-lane argmax over the 16 scores of one accumulator tile: a tournament with three entries per
// node.  The value of a node is one v_max3; its index follows by equality with that value, the
// first of the three entries winning ties (lowest element index), i.e. two v_cmp and two v_cndmask:
// 5 vector operations for every two entries removed, 38 per tile (a binary tournament of (value,
// index) pairs needs 45, and measured 2 % slower; carrying the index bits as lane masks on the
// scalar unit needs 30 vector + ~40 scalar operations and measured 5 % slower: what limits the
// kernel is the number of instructions a wave has to issue per MFMA).  The index comes out as the
// local centroid id 8 (v / 4) + v % 4 of element v.  Written level by level (all maxima, then all
// comparisons, then all selects) so that a comparison and the select that consumes its lane mask
// need not be adjacent.
__device__ inline float max3f(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }
__device__ inline void argmax16(const f32x16 &x, float &m, uint32_t &idx) {
    auto id = [](int v) { return (uint32_t)(8 * (v >> 2) + (v & 3)); };
    float t1[6], t2[2];
    uint32_t i1[6], i2[2];
    bool ea[5], eb[5];
#pragma unroll
    for (int p = 0; p < 5; ++p) t1[p] = max3f(x[3 * p], x[3 * p + 1], x[3 * p + 2]);
    t1[5] = x[15];
    t2[0] = max3f(t1[0], t1[1], t1[2]);
    t2[1] = max3f(t1[3], t1[4], t1[5]);
#pragma unroll
    for (int p = 0; p < 5; ++p) {
        ea[p] = x[3 * p] == t1[p];
        eb[p] = x[3 * p + 1] == t1[p];
    }
    const bool fa0 = t1[0] == t2[0], fb0 = t1[1] == t2[0], fa1 = t1[3] == t2[1], fb1 = t1[4] == t2[1];
    const bool g = t2[1] > t2[0];
#pragma unroll
    for (int p = 0; p < 5; ++p) {
        const uint32_t t = eb[p] ? id(3 * p + 1) : id(3 * p + 2);
        i1[p] = ea[p] ? id(3 * p) : t;
    }
    i1[5] = id(15);
    const uint32_t u0 = fb0 ? i1[1] : i1[2], u1 = fb1 ? i1[4] : i1[5];
    i2[0] = fa0 ? i1[0] : u0;
    i2[1] = fa1 ? i1[3] : u1;
    m = g ? t2[1] : t2[0];
    idx = g ? i2[1] : i2[0];
}
// LDS layout of a 256-row tile (keys, or the centroid block while it is staged): rows of 256 bytes
// without padding, the 16-byte chunk c of row r stored in slot c ^ (r & 15).  A fragment read (lane
// = row r, chunk 2 ks + half) then hits 16 different 16-byte bank groups per 16 lanes (measured: the
// full 160 B/clk/CU), and a wave can write four whole rows with ONE direct global -> LDS load (lane
// l lands at 16 l; it fetches chunk (l & 15) ^ (row & 15) of its row), so a key tile never passes
// through registers.  With the extra coordinate (transformed keys) each row has a 32-byte
// companion (the coordinate, then zeros: the two chunks of a ninth contraction step) in a
// separate array.
__host__ __device__ constexpr int assign_lds_bytes(bool aug) {
    return 2 * 256 * 256 + (aug ? 2 * 256 * 32 : 0) + 2 * 256 * 8;
}

// While every coordinate is below 2^59 (here its bf16 bits; transformed keys: every squared norm below 2^118) so are the
// means', and all scores of a build are finite.
constexpr uint32_t kLargeKey = (127 + 59) << 7;

// One workgroup's run of keys [k0, kend) of unit u against slice `slice` of the centroids.  go: see round_goes (nullptr: the
// caller knows that the unit goes); returns whether it goes.  won != nullptr: [kend - k0] (LDS) the run's winners as well.
// look: also looks for large keys.
template <int CT, int CW, bool AUG, bool FULL>
__device__ __forceinline__ bool assign_slice(const Dev &d, const bf16_t *__restrict__ K, const bf16_t *__restrict__ cent,
                                             const float *__restrict__ cnorm, int n, int u, int slice, int k0, int kend, int zsplit,
                                             int Cpad, int cur, const int *__restrict__ go, uint32_t round, uint16_t *won, bool look, char *smem) {
    constexpr int KW = 8 / CW;
    constexpr int KS = AUG ? 9 : 8;  // 16-wide steps of the contraction
    char *keys = smem;                                                // [2][256][256 B], chunks swizzled
    uint4 *kext = (uint4 *)(smem + 2 * kAssignTile * 256);            // (AUG) [2][256][2] companion chunks
    u64 *best = (u64 *)(smem + 2 * kAssignTile * 256 + (AUG ? 2 * kAssignTile * 32 : 0));  // [2][256]
    // byte offset of chunk c of row r inside a buffer
    auto slot = [](int r, int c) { return r * 256 + ((c ^ (r & 15)) << 4); };

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, col = lane & 31, half = lane >> 5;
    // Wave (cw, kw) holds CT centroid tiles of the slice: neighbours when every slice is full (FULL), else cw
    // and cw + CW.  Waves w and w + 4 share a SIMD: tiles missing at the slice's end are spread over the
    // SIMDs that way (with all eight waves on the centroids tile t belongs to SIMD t mod 4; with fewer
    // the upper four waves take the columns in a shifted order), and a wave skips what it does not have
    // (ctv), so a slice costs what its fullest SIMD holds: 12 tiles run in 3/4 of the time of 16.
    constexpr int CS = FULL ? 1 : CW;  // distance between a wave's tiles
    const int kw = wave / CW, cw = FULL || CW == 8 ? wave % CW : (wave + (wave >> 2) * (CW / 2)) % CW;
    const int wt0 = FULL ? cw * CT : cw, tile0 = slice * CW * CT + wt0;
    const int ctv = __builtin_amdgcn_readfirstlane(tile0 * 32 >= Cpad ? 0 : CT == 2 && (tile0 + CS) * 32 < Cpad ? 2 : 1);
    const int ntiles = (kend - k0 + kAssignTile - 1) / kAssignTile;
    const bf16_t *Ku = K + (size_t)u * n * kD;

    ICE_BSTAMP(0);
    // Prologue.  The workgroup's block of centroid rows goes to LDS with fully coalesced 16-byte
    // loads (the staging area is the key buffers, not yet in use) and every wave then picks its
    // MFMA fragments from there: reading the fragments straight from global memory touches 32
    // separate rows per load instruction.  The first key tile is in flight meanwhile.
    constexpr int R = CW * CT * 32;  // centroid rows of this workgroup
    const int crow0 = slice * R;
    uint4 cst[R / 32];
    {
        const bf16_t *csrc = cent + ((size_t)u * Cpad + crow0) * kD;
#pragma unroll
        for (int i = 0; i < R / 32; ++i) {
            const int id = tid + 512 * i, row = id >> 4, ch = id & 15;
            cst[i] = crow0 + row < Cpad ? ((const uint4 *)(csrc + (size_t)row * kD))[ch] : make_uint4(0, 0, 0, 0);
        }
    }
    // accumulator seeds -||mu~||^2 / 2 (rows past Cpad: -inf), resident for the whole kernel: element v
    // of a lane of half h belongs to local centroid 8 (v / 4) + 4 h + v % 4 of its tile
    f32x16 seed[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int row0 = (tile0 + ct * CS) * 32;
        if (row0 < Cpad) {
            const float *wn = cnorm + (size_t)u * Cpad + row0;
#pragma unroll
            for (int v = 0; v < 16; ++v) seed[ct][v] = -0.5f * wn[8 * (v >> 2) + 4 * half + (v & 3)];
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) seed[ct][v] = -INFINITY;
        }
    }

    const int goes = go ? go[2 * u] : 1;
    // The first key tile travels through registers (it is requested before the centroid block is
    // staged in the very buffers it goes to); every later tile goes straight to LDS.
    uint32_t stage_aug = 0;  // (AUG) extra coordinate of key `tid` of the next tile, threads 0..255
    auto load_aug = [&](int t) {
        if constexpr (AUG) {
            const int key = k0 + t * kAssignTile + tid;
            stage_aug = tid < kAssignTile && key < kend ? d.kaug[(size_t)u * d.max_tokens + key] : 0u;
        }
    };
    auto store_aug = [&](int buf) {
        if constexpr (AUG) {
            // (the thread worked out again: kept in scratch memory, where registers end, it is waited for in front of the barrier)
            const int t = thread_of(__builtin_amdgcn_readfirstlane(wave));
            if (t < kAssignTile) *(uint32_t *)&kext[(buf * kAssignTile + t) * 2] = stage_aug;  // (the other 28 bytes stay zero)
        }
    };
    // rows past the end of the range are never written back: they may hold any valid key
    auto request_tile = [&](int t, int buf) {
        const int base = k0 + t * kAssignTile;
        const int ch = tid & 15, r16 = (tid >> 4) & 15;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = (tid >> 4) + 32 * i;
            const int key = min(base + row, kend - 1);
            const uint4 *src = (const uint4 *)(Ku + (size_t)key * kD) + (ch ^ r16);
            char *dst = keys + buf * (kAssignTile * 256) + (4 * wave + 32 * i) * 256;  // this wave's four rows
            lds_dma16(src, dst);
        }
    };
    u32x4 first[8];  // (the grid leaves no workgroup without keys: ntiles >= 1)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int id = tid + 512 * i, row = id >> 4, ch = id & 15;
        const int key = min(k0 + row, kend - 1);
        first[i] = ((const u32x4 *)(Ku + (size_t)key * kD))[ch];
    }
    load_aug(0);
    if (goes == 0) return false;  // (a later round of a unit whose centroids stayed: every winner stands)
#pragma unroll
    for (int i = 0; i < R / 32; ++i) {
        const int id = tid + 512 * i, row = id >> 4, ch = id & 15;
        *(uint4 *)(keys + slot(row, ch)) = cst[i];
    }
    if constexpr (AUG) {
        // the centroids' extra coordinate, then 15 zeros (both buffers' 512 rows: the zeros serve the keys as well)
        static_assert(2 * kAssignTile == 512, "one thread per row");
        const uint32_t a = tid < R && crow0 + tid < Cpad ? d.caug[cur][(size_t)u * Cpad + crow0 + tid] : 0u;
        kext[tid * 2] = make_uint4(a, 0, 0, 0);
        kext[tid * 2 + 1] = make_uint4(0, 0, 0, 0);
    }
    if (tid < 2 * kAssignTile) best[tid] = 0ull;
    __syncthreads();
    // centroid operand, resident for the whole kernel
    bf16x8 A[CT][KS];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int r = (wt0 + ct * CS) * 32 + col;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) A[ct][ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(keys + slot(r, 2 * ks + half)));
        if constexpr (AUG) A[ct][8] = __builtin_bit_cast(bf16x8, kext[r * 2 + half]);
    }
    __syncthreads();  // every wave holds its fragments before the first key tile overwrites them
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int id = tid + 512 * i, row = id >> 4, ch = id & 15;
        *(u32x4 *)(keys + slot(row, ch)) = first[i];
    }
    if constexpr (AUG) asm volatile("" : "+v"(stage_aug));  // (as in the loop below)
    store_aug(0);
    __syncthreads();
    // byte address of this lane's fragment chunk ks in row `col` of buffer 0; sub-tiles and the
    // other buffer are constant offsets from it
    uint32_t frag[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) frag[ks] = (uint32_t)slot(col, 2 * ks + half);
    ICE_BSTAMP(1);

    constexpr int NSUB = 8 / KW;  // 32-key sub-tiles of this wave per tile
    const uint32_t inv_cid0 = 0xFFFFFFFFu - (uint32_t)(tile0 * 32 + 4 * half);  // low word for local centroid id 0
    for (int t = 0; t < ntiles; ++t) {
        const int buf = t & 1;
        u64 *bestt = best + buf * kAssignTile;
        ICE_WSTAMP(t, 0);
        if (t + 1 < ntiles) {
            request_tile(t + 1, buf ^ 1);
            load_aug(t + 1);
        }
        if constexpr (!AUG) {
            if (look) {  // largest magnitude of the tile's keys (this thread's share), as 16-bit patterns: NaN is above all
                typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
                u16x2 top = {0, 0};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint4 w = *(const uint4 *)(keys + buf * (kAssignTile * 256) + (tid + 512 * i) * 16);
                    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, x[j] & 0x7FFF7FFFu));
                }
                if (max(top.x, top.y) >= kLargeKey) d.large_keys[u] = 1;
            }
        }
        // Software pipeline over "slots" j = (sub-tile i, centroid tile ct): while the matrix cores
        // run the 8-MFMA chain of slot j+1 into one accumulator set, the vector unit
        // reduces slot j's 16 scores per lane from the other set (argmax16).  The key operand of a
        // sub-tile is read from LDS one sub-tile ahead.
        bf16x8 B[2][KS];
        auto load_b = [&](int i, bf16x8 (&dst)[KS]) {
            const char *sub = keys + buf * (kAssignTile * 256) + (kw + i * KW) * 32 * 256;  // (32 rows: r & 15 is col & 15)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) dst[ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(sub + frag[ks]));
            if constexpr (AUG) dst[8] = __builtin_bit_cast(bf16x8, kext[(buf * kAssignTile + (kw + i * KW) * 32 + col) * 2 + half]);
        };
        auto compute = [&](auto tiles_held) {
            constexpr int CTV = decltype(tiles_held)::value, NSLOT = NSUB * CTV;
            f32x16 acc[2];
            auto chain = [&](int j, f32x16 &dst) {
                const int i = j / CTV, ct = j % CTV;
                dst = seed[ct];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ct][ks], B[i & 1][ks], dst, 0, 0, 0);
            };
            load_b(0, B[0]);
            if (CTV == 1 && NSUB > 1) load_b(1, B[1]);
            chain(0, acc[0]);
            float sv = 0.f;
            uint32_t sidx = 0;
#pragma unroll
            for (int j = 0; j < NSLOT; ++j) {
                const int i = j / CTV, ct = j % CTV;
                // LDS reads for the sub-tile whose first chain is issued in the NEXT iteration
                if ((j + 2) % CTV == 0 && (j + 2) / CTV < NSUB && (j + 2) / CTV >= 1 && !(CTV == 1 && j + 2 == 1))
                    load_b((j + 2) / CTV, B[((j + 2) / CTV) & 1]);
                if (j + 1 < NSLOT) chain(j + 1, acc[(j + 1) & 1]);
                // element v of this lane has local centroid id ct*32*CS + 8*(v/4) + v%4 (+ 4*half), ascending in v
                float m;
                uint32_t li;
                argmax16(acc[j & 1], m, li);
                if (ct == 0) {
                    sv = m;
                    sidx = li;
                } else {
                    const bool gt = m > sv;
                    sv = gt ? m : sv;
                    sidx = gt ? li + 32u * CS * ct : sidx;
                }
                if (ct == CTV - 1) {
                    const u64 pk = ((u64)f32_ordered(sv + 0.0f) << 32) | (u64)(inv_cid0 - sidx);
                    atomicMax(&bestt[(kw + i * KW) * 32 + col], pk);
                }
            }
        };
        if (FULL || ctv == CT) compute(std::integral_constant<int, CT>{});  // (wave-uniform)
        else if (CT == 2 && ctv == 1) compute(std::integral_constant<int, 1>{});
        ICE_BSTAMP(2 + 2 * (t & 3));
        ICE_WSTAMP(t, 1);
        if (t + 1 < ntiles) {
            wait_lds_dma();  // this wave's share of the next tile is in LDS
            store_aug(buf ^ 1);
        }
        // (the coordinates count as arrived here in every wave and on every path: a wait left for the next such load would
        // cover the direct loads issued before it, i.e. come before the contraction: 54 against 46 us, 16 units x 23457 x 366)
        if constexpr (AUG) asm volatile("" : "+v"(stage_aug));
        ICE_WSTAMP(t, 2);
        __syncthreads();
        ICE_WSTAMP(t, 3);
        ICE_BSTAMP(3 + 2 * (t & 3));
        // the per-key winners of this tile leave through the first 256 threads; the other buffer
        // collects the next tile meanwhile, and this one is not touched again before the barrier
        // of the next tile
        if (tid < kAssignTile) {
            const int key = k0 + t * kAssignTile + tid;
            if (key < kend) {
                u64 *dst = d.packed + (size_t)u * d.max_tokens + key;
                const u64 b = bestt[tid], w = winner_word(b, round);
                if (zsplit == 1) *dst = w;
                else atomicMax(dst, w);
                if (won) won[t * kAssignTile + tid] = (uint16_t)(0xFFFFFFFFu - (uint32_t)b);
            }
            bestt[tid] = 0ull;
        }
    }
    return true;
}

template <int CT, int CW, bool AUG, bool FULL>
__global__ __launch_bounds__(512) void assign_kernel(const bf16_t *__restrict__ K, const bf16_t *__restrict__ cent,
                                                      const float *__restrict__ cnorm, int n, int keys_per_wg, int zsplit,
                                                      int Cpad, int cur, const int *__restrict__ go, int round, int fused, int look, Dev d) {  // (scalars first: preloaded at wave start)
    extern __shared__ __align__(16) char smem[];
    const int u = blockIdx.z, k0 = blockIdx.x * keys_per_wg, kend = min(n, k0 + keys_per_wg);
    uint16_t *won = (uint16_t *)(smem + assign_lds_bytes(AUG));  // [keys_per_wg] (fused)
    if (fused && blockIdx.x == 0 && threadIdx.x == 0) d.any_moved[2 * u + (round & 1)] = 0;  // (for this round's means)
    if (!assign_slice<CT, CW, AUG, FULL>(d, K, cent, cnorm, n, u, blockIdx.y, k0, kend, zsplit, Cpad, cur, go, round % kRoundNumbers, fused ? won : nullptr,
                                           look != 0 && blockIdx.y == 0, smem)) return;
    if (fused) {  // the run is a range of the sort as well
        __syncthreads();    // (the winners are there; the key tiles are not needed any more)
        sort_range<8, kFusedRun / 2, false>(d, threadIdx.x, u, n, blockIdx.x, gridDim.x, k0, kend, keys_per_wg / 8, 8, 32 - __builtin_clz((unsigned)Cpad - 1u),
                                            round, 1, (int *)smem, nullptr, nullptr, [=](int i) { return (uint32_t)won[i - k0]; }, [](uint32_t w) { return w; },
                                            [](int) { return 0.f; });
    }
}

// How a later round is cut (reassign_kernel), in one way and in the other.
struct RoundPlan {
    int run, wgs;                // moved centroids: 256-key tiles per workgroup, workgroups per unit
    int all_run, all_wgs, slices;  // all centroids: the same, workgroups per unit and slice
    int fixed, per_key;          // for takes_all: the prologues of the slices of all centroids, a run's keys against them
    long long limit;             // ... and what all centroids cost (2 n times, by rounds of 256 workgroups)
    long long all_turns;         // rounds of 256 workgroups of all centroids
    int tiles;                   // 32-centroid tiles of a slice, as they are dealt to four SIMDs
};

// Whether the full contraction of a unit costs no more than `moved` of its centroids, which hold `keys` of its n keys,
// and then the keys of which the winner is not known.  In contractions of 256 keys x 32 centroids: the centroids of a
// slice are dealt to four SIMDs, a slice's prologue costs about 16 of them, and of the keys whose centroid moved about half
// are listed (of 32768 keys and 512 clusters 0.34 to 0.5 of them in the benchmark's mixture, 0.4 to 0.55 without structure).
__device__ inline bool takes_all(const RoundPlan &p, int moved, int keys, int n) {
    const int S = (moved + 511) / 512, own = 16 * (S - 1) + 4 * ((moved - 512 * (S - 1) + 127) / 128);
    // (whole numbers, 2 n times: every workgroup of the unit comes to the same)
    return (long long)(p.run * own + 16 * S + p.fixed) * 2 * n + (long long)keys * p.per_key >= p.limit;
}

// What `moved` says of a unit: of the 16 centroids from 16 x on a mask and the keys they hold.
__device__ inline uint32_t moved_of_16(const uint32_t *moved, int x, int &keys) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 w = ((const uint4 *)moved)[4 * x + i];
        m |= ((w.x & 1u) | (w.y & 1u) << 1 | (w.z & 1u) << 2 | (w.w & 1u) << 3) << (4 * i);
        keys += (int)((w.x & 1u) * (w.x >> 1) + (w.y & 1u) * (w.y >> 1) + (w.z & 1u) * (w.z >> 1) + (w.w & 1u) * (w.w >> 1));
    }
    return m;
}

// Slices of at most 512 centroids that meet through an atomic maximum in `packed`.
int assign_slices(const Dev &d) { return (d.Cpad + 511) / 512; }

// Key tiles per workgroup: the run for which the chip's rounds of 256 workgroups, each its tiles plus a prologue worth
// about one, come out shortest (as for assign_kernel, whose grid also counts the slices).
static int assign_run(int U, int n, int slices) {
    const int ktiles = (n + kAssignTile - 1) / kAssignTile;
    int run = 1;
    long long best_cost = -1;
    for (int g = 1; g <= ktiles && g <= 4096;) {  // g workgroups per unit and slice: the fewest for each length of run
        const int r = (ktiles + g - 1) / g;
        const long long wgs = (long long)((ktiles + r - 1) / r) * slices * U;
        const long long cost = (wgs + 255) / 256 * (r + 1);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; run = r; }
        if (wgs > 256 * 64 || r == 1) break;  // (more, shorter runs only repeat the prologue)
        g = (ktiles + r - 2) / (r - 1);
    }
    return run;
}

// whether a centroid of the unit moved in the round before round t: element 2 u of the result (all units go in the first round)
static const int *round_goes(const Dev &d, int t) { return t > 0 ? d.any_moved + ((t - 1) & 1) : nullptr; }

void launch_assign(const Dev &d, const bf16_t *K, int n, int cur, int t, bool fused, bool look, hipStream_t st) {
    const int tiles = d.Cpad / 32;
    int CT = tiles == 1 ? 1 : 2, CW = 1;
    while (CW < 8 && CW * CT < tiles) CW *= 2;
    const int zsplit = assign_slices(d);
    // A workgroup fills a CU (132-148 KB of LDS, 8 waves of 226-256 registers) and takes a run of key tiles
    // of one unit, any number of them: the run for which the chip's rounds of 256 workgroups, each its
    // tiles plus a prologue worth about one tile, come out shortest.  (Runs of a power of two tiles only:
    // 16 units x 92 tiles, 12 of 16 centroid tiles, transformed, are 192 workgroups of 8 tiles and took
    // 56 us, 256 of 6 with the tiles dealt over the SIMDs 43; a ten-round build of 8 units x 40001 keys
    // with 625 clusters, 160 workgroups of 8 tiles against 256 of 10, 1314 us against 1031.)
    const int keys_per_wg = assign_run(d.U, n, zsplit) * kAssignTile;
    dim3 grid((n + keys_per_wg - 1) / keys_per_wg, zsplit, d.U);
    const size_t lds = assign_lds_bytes(d.tk != 0) + (fused ? (size_t)keys_per_wg * 2 : 0);
    if (zsplit > 1 && t % kRoundNumbers == 0) hipLaunchKernelGGL(clear_winners_kernel, dim3((n + 255) / 256, d.U), dim3(256), 0, st, d, n);
    const bool full = tiles % (CT * CW) == 0;
#define ICE_ASSIGN_F(ct, cw, aug, full)                                                             \
    do {                                                                                            \
        allow_dynamic_lds((const void *)assign_kernel<ct, cw, aug, full>, lds);                     \
        hipLaunchKernelGGL((assign_kernel<ct, cw, aug, full>), grid, dim3(512), lds, st, K, d.cent_bf16[cur], d.cnorm[cur], n, \
                           keys_per_wg, zsplit, d.Cpad, cur, round_goes(d, t), t, fused ? 1 : 0, look ? 1 : 0, d);  \
    } while (0)
#define ICE_ASSIGN_A(ct, cw, aug)                                                                   \
    do {                                                                                            \
        if (full) ICE_ASSIGN_F(ct, cw, aug, true);                                                  \
        else ICE_ASSIGN_F(ct, cw, aug, (ct * cw <= 2));  /* (one or two tiles are always full: no such variant) */ \
    } while (0)
#define ICE_ASSIGN(ct, cw)                                                                          \
    do {                                                                                            \
        if (d.tk) ICE_ASSIGN_A(ct, cw, true);                                                       \
        else ICE_ASSIGN_A(ct, cw, false);                                                           \
    } while (0)
    if (CT == 1) ICE_ASSIGN(1, 1);
    else if (CW == 1) ICE_ASSIGN(2, 1);
    else if (CW == 2) ICE_ASSIGN(2, 2);
    else if (CW == 4) ICE_ASSIGN(2, 4);
    else ICE_ASSIGN(2, 8);
#undef ICE_ASSIGN
#undef ICE_ASSIGN_A
#undef ICE_ASSIGN_F
}

// ------------------------------------------------------------------------------------------------
// The assignment of a later round.  Between two rounds many centroids stay where they are, bit for bit (clusters of
// about 64 keys in 128 dimensions settle fast: of 512 clusters over 32768 keys of the benchmark's mixture 79 % moved
// after the second round, 50 % after the third, then 29, 18, 5, 2 and below 1 %; of as many clusters of keys without any
// structure 75, 71, 70, 68, 68, 67, 64 %), and a score is the
// same bits whichever slot of the matrix instruction it comes out of.  So the winner among the centroids that did not
// move is known from the last round for every key whose own centroid did not, and what the full contraction
// would leave in `packed` follows from less of it:
//   moved  every key against the moved centroids only (`d.moved`, listed in ascending id in LDS), winner m.  With `old` the
//          last round's winner (score, ~id), which no centroid that stayed can beat:
//            m >  old: m;   m <= old and old's centroid stayed: old;   m == old (its score came out the same): old;
//            m <  old and old's centroid moved: a centroid that stayed may lie between, the key is listed;
//   again  the listed keys, gathered, against all centroids.
// A unit for which that is no less work (takes_all) goes through the full contraction, by the same code as a round of
// assign_kernel.  So does one with keys that are not finite, or so large that a score may not be (`large_keys`): what the
// contraction leaves of a key among whose scores are NaN depends on where in a tile they are (argmax16: nine of them side by
// side hide their lane's others).
// One workgroup takes a run of 256-key tiles through moved and again; more than 512 centroids are slices that it takes one
// after the other, its keys' winners so far in `tmp`.  A slice of few tiles splits the keys among the waves instead of
// the centroids (slice<CW>: CW waves share the centroids of a key).  In a unit that takes all, workgroups are cut over
// slices as well.  Bound as assign_kernel is while many centroids move, by the read of the keys once few do.
// `tmp` and the key lists are scratch at the start of the unit's key tiles (behind Near's head), 12 of the 256 bytes per token
// that the page layout overwrites in any case.
enum { kMovedCentroids = 1, kListedKeys = 2 };  // what a pass over the keys is about
__host__ __device__ inline int reassign_lds_bytes(bool aug, int Cpad) {
    return 2 * 256 * 256 + 2 * 256 * 8 + 512 * 4 + (aug ? 1024 * 4 : 0) + Cpad * 2 + Cpad / 8;
}
__device__ inline bool ordered_is_nan(uint32_t k) { return k > 0xFF800000u || k < 0x007FFFFFu; }

// One slice of at most 512 of a job's centroids (places c0 .. of its list) against its keys, by a workgroup of 8 waves: CW waves share
// the centroids of a key, the others split a key tile.  The job says which keys (nk of them: key_of(place), rows_of(tile, rows): a
// thread's eight rows of a tile, 32 apart) and which centroids (ncent, centroid(place)), what is loaded ahead of a tile's
// contraction (ahead) and counts as arrived behind it (arrived), and takes the winners: take(place, best, c0, lane), where
// best = ordered score << 32 | ~place of the centroid.
template <bool AUG, int CW, bool FULL, typename Job>
__device__ __forceinline__ void later_slice(const Dev &d, const bf16_t *Ku, const bf16_t *__restrict__ cent, const float *__restrict__ cnorm, int u, int Cpad,
                                            int cur, int wave, int c0, int &tid, char *keys, u64 *best, float *seeds, uint32_t *kext, uint32_t *cext, Job &job) {
    constexpr int KS = AUG ? 9 : 8;
    constexpr int KW = 8 / CW, NSUB = 8 / KW, R = CW * 64;
    auto slot = [](int r, int c) { return r * 256 + ((c ^ (r & 15)) << 4); };
    // (worked out in every slice and tile: hoisted out of the forms and the loops, the lanes' addresses would not fit the
    // registers, and kept in memory instead they would be waited for)
    tid = thread_of(wave);
    const int lane = tid & 63, col = lane & 31, half = lane >> 5;
    constexpr int CS = FULL ? 1 : CW;  // distance between a wave's two tiles (dealt over the SIMDs as in assign_kernel)
    const int kw = wave / CW, cw = FULL || CW == 8 ? wave % CW : (wave + (wave >> 2) * (CW / 2)) % CW;
    const int wt0 = FULL ? cw * 2 : cw, nt = (min(512, job.ncent - c0) + 31) / 32;
    const int ctv = wt0 >= nt ? 0 : wt0 + CS < nt ? 2 : 1;
    const int ntiles = (job.nk + kAssignTile - 1) / kAssignTile;
    // ---- prologue: the slice's centroid rows through LDS into the waves' operand registers (the first key tile goes
    // through registers: the rows are staged where it belongs)
    u32x4 first[8];
    {
        int key[8];
        job.rows_of(0, tid, key);
#pragma unroll
        for (int i = 0; i < 8; ++i) first[i] = ((const u32x4 *)(Ku + (size_t)key[i] * kD))[tid & 15];
    }
    uint4 cst[R / 32];
#pragma unroll
    for (int i = 0; i < R / 32; ++i) {
        const int id = tid + 512 * i, pos = c0 + (id >> 4);
        const uint4 w = ((const uint4 *)(cent + ((size_t)u * Cpad + job.centroid(min(pos, job.ncent - 1))) * kD))[id & 15];
        cst[i] = pos < job.ncent ? w : make_uint4(0, 0, 0, 0);
    }
    float seed_in = -INFINITY;
    uint32_t cext_in = 0u, kext_in = 0u;
    if (tid < R && c0 + tid < job.ncent) {
        const int c = job.centroid(c0 + tid);
        seed_in = -0.5f * cnorm[(size_t)u * Cpad + c];
        if constexpr (AUG) cext_in = d.caug[cur][(size_t)u * Cpad + c];
    }
    auto load_aug = [&](int t) {
        if constexpr (AUG) {
            const int pos = t * kAssignTile + tid;
            kext_in = tid < kAssignTile && pos < job.nk ? d.kaug[(size_t)u * d.max_tokens + job.key_of(pos)] : 0u;
        }
    };
    auto store_aug = [&](int buf) {
        if constexpr (AUG) {
            if (tid < kAssignTile) kext[buf * kAssignTile + tid] = kext_in;
        }
    };
    load_aug(0);
#pragma unroll
    for (int i = 0; i < R / 32; ++i) {
        const int id = tid + 512 * i;
        *(uint4 *)(keys + slot(id >> 4, id & 15)) = cst[i];
    }
    if (tid < R) {
        seeds[tid] = seed_in;
        if constexpr (AUG) cext[tid] = cext_in;
    }
    __syncthreads();
    bf16x8 A[2][KS];
    f32x16 seed[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int t0 = (wt0 + ct * CS) * 32, r = t0 + col;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) A[ct][ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(keys + slot(r, 2 * ks + half)));
        if constexpr (AUG) A[ct][8] = __builtin_bit_cast(bf16x8, make_uint4(half ? 0u : cext[r], 0, 0, 0));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float4 w = *(const float4 *)(seeds + t0 + 8 * v + 4 * half);
            seed[ct][4 * v] = w.x; seed[ct][4 * v + 1] = w.y; seed[ct][4 * v + 2] = w.z; seed[ct][4 * v + 3] = w.w;
        }
    }
    __syncthreads();  // every wave holds its fragments before the first key tile overwrites them
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int id = tid + 512 * i;
        *(u32x4 *)(keys + slot(id >> 4, id & 15)) = first[i];
    }
    store_aug(0);
    __syncthreads();
    uint32_t frag[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) frag[ks] = (uint32_t)slot(col, 2 * ks + half);
    const uint32_t inv0 = 0xFFFFFFFFu - (uint32_t)(c0 + wt0 * 32 + 4 * half);  // low word of a winner: ~(place in the list)

    for (int t = 0; t < ntiles; ++t) {
        const int buf = t & 1;
        u64 *bestt = best + buf * kAssignTile;
        tid = thread_of(wave);
        if (t + 1 < ntiles) {
            const int ch = tid & 15, r16 = (tid >> 4) & 15;
            int key[8];
            job.rows_of(t + 1, tid, key);
            load_aug(t + 1);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                lds_dma16((const uint4 *)(Ku + (size_t)key[i] * kD) + (ch ^ r16), keys + (buf ^ 1) * (kAssignTile * 256) + (4 * wave + 32 * i) * 256);
        }
        job.ahead(t, tid, c0);
        auto load_b = [&](int i, bf16x8 (&dst)[KS]) {
            const char *sub = keys + buf * (kAssignTile * 256) + (kw + i * KW) * 32 * 256;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) dst[ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(sub + frag[ks]));
            if constexpr (AUG) {
                const uint32_t e = kext[buf * kAssignTile + (kw + i * KW) * 32 + col];
                dst[8] = __builtin_bit_cast(bf16x8, make_uint4(half ? 0u : e, 0, 0, 0));
            }
        };
        auto chain = [&](int ct, const bf16x8 (&b)[KS], f32x16 &dst) {
            dst = seed[ct];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ct][ks], b[ks], dst, 0, 0, 0);
        };
        float sv = 0.f;
        uint32_t sidx = 0;
        auto reduce = [&](const f32x16 &acc, int i, int ct, int ctv_of) {  // as in assign_kernel
            float m;
            uint32_t li;
            argmax16(acc, m, li);
            asm("" : "+v"(li));  // (worked out in any case: as a branch around its selects it ends the pipeline of chains)
            if (ct == 0) {
                sv = m;
                sidx = li;
            } else {
                const bool gt = m > sv;
                sv = gt ? m : sv;
                sidx = gt ? li + 32u * CS * ct : sidx;
            }
            if (ct == ctv_of - 1)
                atomicMax(&bestt[(kw + i * KW) * 32 + col], ((u64)f32_ordered(sv + 0.0f) << 32) | (u64)(inv0 - sidx));
        };
        const int subs = min(8, (job.nk - t * kAssignTile + 31) / 32);  // 32-key sub-tiles with keys
        auto compute = [&](auto tiles_held) __attribute__((always_inline)) {
            constexpr int CTV = decltype(tiles_held)::value, NSLOT = NSUB * CTV;
            if (subs > 4) {  // (the software pipeline of assign_kernel)
                bf16x8 B[2][KS];
                f32x16 acc[2];
                load_b(0, B[0]);
                if (CTV == 1 && NSUB > 1) load_b(1, B[1]);
                chain(0, B[0], acc[0]);
#pragma unroll
                for (int j = 0; j < NSLOT; ++j) {
                    const int i = j / CTV, ct = j % CTV, i1 = (j + 1) / CTV;
                    if ((j + 2) % CTV == 0 && (j + 2) / CTV < NSUB && (j + 2) / CTV >= 1 && !(CTV == 1 && j + 2 == 1))
                        load_b((j + 2) / CTV, B[((j + 2) / CTV) & 1]);
                    if (j + 1 < NSLOT) chain((j + 1) % CTV, B[i1 & 1], acc[(j + 1) & 1]);
                    reduce(acc[j & 1], i, ct, CTV);
                }
            } else {  // a tile of few keys: no work for the empty sub-tiles
                for (int i = 0; kw + i * KW < subs; ++i) {
                    bf16x8 B[KS];
                    f32x16 acc[CTV];
                    load_b(i, B);
#pragma unroll
                    for (int ct = 0; ct < CTV; ++ct) chain(ct, B, acc[ct]);
#pragma unroll
                    for (int ct = 0; ct < CTV; ++ct) reduce(acc[ct], i, ct, CTV);
                }
            }
        };
        if (FULL || ctv == 2) compute(std::integral_constant<int, 2>{});  // (wave-uniform)
        else if (ctv == 1) compute(std::integral_constant<int, 1>{});
        if (t + 1 < ntiles) {
            wait_lds_dma();
            asm volatile("" : "+v"(kext_in));
            store_aug(buf ^ 1);
        }
        // (what was requested ahead counts as arrived here for every lane: a wait left for a later place would also
        // cover the next tile's direct loads)
        job.arrived();
        __syncthreads();
        // the tile's winners, first 256 threads (a key's are the same thread's in every slice)
        if (tid < kAssignTile) {
            const u64 b = bestt[tid];
            bestt[tid] = 0ull;
            job.take(t * kAssignTile + tid, b, c0, lane);
        }
    }
}

// every slice of the job's centroids from place c_first on
template <bool AUG, typename Job>
__device__ __forceinline__ void later_slices(const Dev &d, const bf16_t *Ku, const bf16_t *__restrict__ cent, const float *__restrict__ cnorm, int u, int Cpad,
                                             int cur, int wave, int c_first, int &tid, char *keys, u64 *best, float *seeds, uint32_t *kext, uint32_t *cext, Job &job) {
    for (int c0 = c_first; c0 < job.ncent; c0 += 512) {
        const int nt = (min(512, job.ncent - c0) + 31) / 32;
#define ICE_SLICE(cw, full) later_slice<AUG, cw, full>(d, Ku, cent, cnorm, u, Cpad, cur, wave, c0, tid, keys, best, seeds, kext, cext, job)
        if (nt <= 2) ICE_SLICE(1, false);
        else if (nt <= 4) ICE_SLICE(2, false);
        else if (nt <= 8) ICE_SLICE(4, false);
        else if (nt < 16) ICE_SLICE(8, false);
        else ICE_SLICE(8, true);
#undef ICE_SLICE
    }
}

// The keys and centroids of reassign_kernel's two passes
struct ReassignJob {
    int job, nk, ncent, k0, Cpad;
    uint32_t round;
    u64 *packed, *tmp;
    uint32_t *fails;
    const uint16_t *list, *bits;
    int *sh_fails;
    u64 last_word, sofar;
    __device__ __forceinline__ int key_of(int pos) const {
        int key = k0 + min(pos, nk - 1);
        if (job == kListedKeys) {
            key = (int)fails[min(pos, nk - 1)];
            asm volatile("" : "+v"(key));  // (see rows_of)
        }
        return key;
    }
    // (The listed keys are waited for where they are loaded: left to the compiler the wait is at every use, in the other pass
    // too, and each key row waits for the one before.)
    __device__ __forceinline__ void rows_of(int t, int tid, int (&key)[8]) const {
        const int base = t * kAssignTile + (tid >> 4);
        if (job == kListedKeys) {
#pragma unroll
            for (int i = 0; i < 8; ++i) key[i] = (int)fails[min(base + 32 * i, nk - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(key[i]));
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) key[i] = k0 + min(base + 32 * i, nk - 1);
        }
    }
    __device__ __forceinline__ int centroid(int pos) const { return job == kMovedCentroids ? (int)list[pos] : pos; }
    // (the last slice of the moved centroids: what the tile's keys are compared with, in flight during the contraction)
    __device__ __forceinline__ void ahead(int t, int tid, int c0) {
        last_word = sofar = 0ull;  // (the last round's winner as it is in memory: taken apart here it would be waited for)
        if (job == kMovedCentroids && c0 + 512 >= ncent && tid < kAssignTile) {
            const int key = key_of(t * kAssignTile + tid);
            last_word = packed[key];
            if (c0 > 0) sofar = tmp[key];
        }
    }
    __device__ __forceinline__ void arrived() { asm volatile("" : "+v"(last_word), "+v"(sofar)); }
    __device__ __forceinline__ void take(int pos, u64 b, int c0, int lane) {
        const bool valid = pos < nk, last = c0 + 512 >= ncent;
        bool fail = false;
        const int key = key_of(pos);
        if (valid && !(job == kMovedCentroids && last)) {
            u64 *dst = (job == kMovedCentroids ? tmp : packed) + key;
            if (job != kMovedCentroids) b = winner_word(b, round);
            if (c0 > 0) atomicMax(dst, b);  // (nothing waits for it)
            else *dst = b;
        } else if (valid) {
            const u64 old = winner_of_word(last_word);
            b = max(b, sofar);
            const uint32_t at = ~(uint32_t)b, own = min(~(uint32_t)old, (uint32_t)Cpad - 1u);
            const uint32_t id = at < (uint32_t)ncent ? list[at] : 0x7FFFFFFFu;  // (a place past the list: no centroid)
            const u64 m = (b & 0xFFFFFFFF00000000ull) | (u64)(0xFFFFFFFFu - id);
            const bool own_moved = (bits[own >> 4] >> (own & 15u)) & 1u;
            fail = ordered_is_nan((uint32_t)(b >> 32)) || ordered_is_nan((uint32_t)(old >> 32)) || (own_moved && m < old);
            if (!fail && m > old) packed[key] = winner_word(m, round);
        }
        if (job == kMovedCentroids && last) {
            const u64 f = __ballot(fail);
            int at = 0;
            if (lane == 0 && f) at = atomicAdd(sh_fails, (int)__popcll(f));
            at = __builtin_amdgcn_readfirstlane(at);
            if (fail) fails[at + (int)__popcll(f & ((1ull << lane) - 1ull))] = (uint32_t)key;
        }
    }
};

// A workgroup's part of the round of unit blockIdx.y.  in_full: the unit goes through the full contraction in any case.
template <bool AUG, bool ALL_FULL>  // ALL_FULL: every slice of the centroids is full (FULL of assign_slice)
__device__ __forceinline__ void reassign_unit(const bf16_t *K, const bf16_t *cent, const float *cnorm, int n, int Cpad,
                                              int cur, const int *go, int round, int fused, bool in_full, RoundPlan &plan, Dev &d, char *smem) {
    char *keys = smem;                                             // [2][256][256 B], chunks swizzled as in assign_slice
    u64 *best = (u64 *)(smem + 2 * kAssignTile * 256);             // [2][256]
    float *seeds = (float *)(best + 2 * kAssignTile);              // [512] of the slice at hand
    uint32_t *kext = (uint32_t *)(seeds + 512);                    // (AUG) [2][256] the keys' extra coordinates
    uint32_t *cext = kext + 2 * kAssignTile;                       // (AUG) [512] the centroids' of the slice at hand
    uint16_t *list = (uint16_t *)(kext + (AUG ? 1024 : 0));        // [Cpad] moved centroids, ascending
    uint16_t *bits = list + Cpad;                                  // [Cpad / 16] the same as a mask
    uint16_t *won = (uint16_t *)(smem + assign_lds_bytes(AUG));    // (all centroids, fused) the run's winners
    __shared__ int sh_wave[8], sh_keys[8], sh_fails;

    const int u = blockIdx.y;
    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u64 *packed = d.packed + (size_t)u * d.max_tokens;

    if (fused && blockIdx.x == 0 && tid == 0) d.any_moved[2 * u + (round & 1)] = 0;  // (for this round's means)
    // ---- which centroids moved
    ICE_PIN(plan.limit); ICE_PIN(plan.per_key); ICE_PIN(plan.fixed); ICE_PIN(plan.run);  // (not fetched behind the barrier)
    int ncent = 0;
    bool all;
    {
        const int lane = tid & 63, goes = go[2 * u], large = __builtin_amdgcn_readfirstlane(d.large_keys[u]);
        uint32_t m = 0;
        int held = 0;
        if (tid * 16 < Cpad) m = moved_of_16(d.moved + (size_t)u * Cpad, tid, held);
        if (goes == 0) return;  // (none: every winner stands)
        const int cnt = __popc(m), incl = wave_scan_add(cnt);
        held = wave_scan_add(held);
        if (lane == 63) { sh_wave[wave] = incl; sh_keys[wave] = held; }
        if (tid == 0) sh_fails = 0;
        __syncthreads();
        int pos = incl - cnt, total_held = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const int x = sh_wave[w];
            pos += w < wave ? x : 0;
            ncent += x;
            total_held += sh_keys[w];
        }
        ncent = __builtin_amdgcn_readfirstlane(ncent);
        all = in_full || large != 0 || takes_all(plan, ncent, __builtin_amdgcn_readfirstlane(total_held), n);
        if (!all) {
            if (tid * 16 < Cpad) bits[tid] = (uint16_t)m;
            for (; m; m &= m - 1) list[pos++] = (uint16_t)(tid * 16 + __ffs(m) - 1);
            if (tid < 2 * kAssignTile) best[tid] = 0ull;
            __syncthreads();
        }
    }
    const int nbits = 32 - __builtin_clz((unsigned)Cpad - 1u);
    if (all) {
        const int keys_per_wg = plan.all_run * kAssignTile, which = blockIdx.x / plan.all_wgs, k0 = (blockIdx.x - which * plan.all_wgs) * keys_per_wg;
        const int kend = min(n, k0 + keys_per_wg);
        if (which >= plan.slices) return;
        assign_slice<2, 8, AUG, ALL_FULL>(d, K, cent, cnorm, n, u, which, k0, kend, plan.slices, Cpad, cur, nullptr,
                                          round % kRoundNumbers, fused ? won : nullptr, false, smem);
        if (fused) {  // (one slice: a range of the sort, as in assign_kernel)
            __syncthreads();
            sort_range<8, kFusedRun / 2, false>(d, thread_of(wave), u, n, blockIdx.x, plan.all_wgs, k0, kend, keys_per_wg / 8, 8, nbits, round, 1, (int *)smem,
                                                nullptr, nullptr, [=](int i) { return (uint32_t)won[i - k0]; }, [](uint32_t w) { return w; }, [](int) { return 0.f; });
        }
        return;
    }
    if ((int)blockIdx.x >= plan.wgs) return;
    const int keys_per_wg = plan.run * kAssignTile, k0 = blockIdx.x * keys_per_wg;
    const bf16_t *Ku = K + (size_t)u * n * kD;
    u64 *tmp = (u64 *)(near_scratch(d, u) + kNearHeadBytes);
    uint32_t *fails = (uint32_t *)(tmp + n) + k0;

    ReassignJob job{kMovedCentroids, min(n, k0 + keys_per_wg) - k0, ncent, k0, Cpad, (uint32_t)(round % kRoundNumbers), packed, tmp, fails, list, bits, &sh_fails, 0ull, 0ull};
    for (;;) {
        later_slices<AUG>(d, Ku, cent, cnorm, u, Cpad, cur, wave, 0, tid, keys, best, seeds, kext, cext, job);
        if (job.job != kMovedCentroids) break;
        wait_vmem();  // (the key lists of all waves are read by all)
        __threadfence_block();
        __syncthreads();
        job.nk = __builtin_amdgcn_readfirstlane(sh_fails);
        if (job.nk == 0) break;
        job.job = kListedKeys;
        job.ncent = Cpad;
    }
    if (fused) {  // the run is a range of the sort as well
        wait_vmem();
        __threadfence_block();
        __syncthreads();
        const uint32_t *pk = (const uint32_t *)packed;
        sort_range<8, kFusedRun / 2, false>(d, thread_of(wave), u, n, blockIdx.x, plan.wgs, k0, min(n, k0 + keys_per_wg), keys_per_wg / 8, 8, nbits, round, 1,
                                            (int *)smem, nullptr, nullptr, [=](int i) { return pk[2 * i]; }, cluster_of_word, [](int) { return 0.f; });
    }
}

template <bool AUG, bool ALL_FULL>
__global__ __launch_bounds__(512) void reassign_kernel(const bf16_t *__restrict__ K, const bf16_t *__restrict__ cent,
                                                       const float *__restrict__ cnorm, int n, int Cpad, int cur,
                                                       const int *__restrict__ go, int round, int fused, RoundPlan plan, Dev d) {  // (scalars first: preloaded at wave start)
    extern __shared__ __align__(16) char smem[];
    reassign_unit<AUG, ALL_FULL>(K, cent, cnorm, n, Cpad, cur, go, round, fused, false, plan, d, smem);
}

static RoundPlan round_plan(const Dev &d, int n) {
    const int ktiles = (n + kAssignTile - 1) / kAssignTile;
    RoundPlan p;
    p.slices = assign_slices(d);
    p.run = assign_run(d.U, n, 1);
    p.wgs = (ktiles + p.run - 1) / p.run;
    p.all_run = assign_run(d.U, n, p.slices);
    p.all_wgs = (ktiles + p.all_run - 1) / p.all_run;
    auto turns = [](long long wgs) { return (wgs + 255) / 256; };
    p.tiles = p.slices > 1 ? 16 : 4 * ((d.Cpad + 127) / 128);
    p.fixed = 16 * p.slices;
    p.per_key = p.run * p.tiles * p.slices;
    // (the moved centroids' launch in as many rounds of the chip as it takes)
    p.all_turns = turns((long long)d.U * p.all_wgs * p.slices);
    p.limit = p.all_turns * (p.all_run * p.tiles + 16) * 2 * n / turns((long long)d.U * p.wgs);
    return p;
}

// Rounds by reassign_kernel instead of assign_kernel: from the third on (the first means move nearly all centroids), above
// 256 clusters and where the whole contraction is at least four tiles of 256 keys x 512 centroids per workgroup.  A unit that
// takes all of it pays about 0.6 us for finding that out, from four tiles on 1 %; keys that settle gain many times that.  Builds of ten
// rounds, us, without and with it, for keys that settle (the benchmark's mixture) and keys without structure: 8 units x 32768 x 512
// (four tiles) 528 and 485, 604 and 609, transformed 601 and 553, 679 and 684; 2 x 32768 x 2048 (four) 313 and 308, 511 and 519;
// 4 x 65536 x 1024 (eight) 819 and 674, 897 and 904; 8 x 131072 x 2048 (64) 4930 and 2969, 5257 and 5268.  Below the line 8 x 24576 x
// 512 (three) 380 and 354, 475 and 485; 4 x 32768 x 512 (two) 317 and 312, 384 and 391; 1 x 16384 x 1024 (one) 163 and 165, 242 and 248.
// (Eight tiles of centroids or fewer are contracted in about the time that their keys take to come in: with 256 clusters
// 64 x 32768 2417 and 2440, 8 x 131072 1356 and 1415, 1564 and 1603, though 128 x 16384 2346 and 2270.)
// Larger builds go by the centroids near a key's own (near_pays); the figures above are without that.
bool reassign_pays(const Dev &d, int n) {
    if (d.Cpad <= 256) return false;
    const RoundPlan p = round_plan(d, n);
    return p.all_turns * p.all_run * p.tiles >= 64;
}

void launch_reassign(const Dev &d, const bf16_t *K, int n, int cur, int t, bool fused, hipStream_t st) {
    const RoundPlan p = round_plan(d, n);
    const size_t lds = std::max<size_t>(reassign_lds_bytes(d.tk != 0, d.Cpad), assign_lds_bytes(d.tk != 0) + (fused ? (size_t)p.all_run * kAssignTile * 2 : 0));
    const dim3 grid(std::max(p.wgs, p.all_wgs * p.slices), d.U);
#define ICE_REASSIGN(aug, full)                                                                                            \
    do {                                                                                                                   \
        allow_dynamic_lds((const void *)reassign_kernel<aug, full>, lds);                                                  \
        hipLaunchKernelGGL((reassign_kernel<aug, full>), grid, dim3(512), lds, st, K, d.cent_bf16[cur], d.cnorm[cur], n, d.Cpad, \
                           cur, round_goes(d, t), t, fused ? 1 : 0, p, d);                                                   \
    } while (0)
    const bool full = d.Cpad / 32 % 16 == 0;
    if (d.tk) { if (full) ICE_REASSIGN(true, true); else ICE_REASSIGN(true, false); }
    else { if (full) ICE_REASSIGN(false, true); else ICE_REASSIGN(false, false); }
#undef ICE_REASSIGN
}

// The members of cluster c in ascending position, out of the ranges' sorted pieces: member j sits in the last piece that
// starts at or before it.  A wave holds 64 pieces at a time, one per lane: `first` = members in the pieces before the lane's
// own, `from` = index into the unit's `order` of its first one.  Nothing is kept per range, so any number of ranges will do.
struct Pieces {
    const uint32_t *off;  // the unit's range_off, at cluster c
    int Cpad, R, L;
    __device__ uint32_t word(int r) const { return r < R ? off[(size_t)r * Cpad] : 0u; }
    // pieces r0 .. r0 + 63, `before` members in front of them; returns the members up to their end (the same on every lane)
    __device__ int load(int r0, int lane, int before, int &first, int &from, int &cnt) const {
        return take(word(r0 + lane), r0, lane, before, first, from, cnt);
    }
    // ... of which the lane's word is at hand
    __device__ int take(uint32_t o, int r0, int lane, int before, int &first, int &from, int &cnt) const {
        const int r = r0 + lane;
        cnt = (int)(o & 0xFFFFu);
        const int incl = wave_scan_add(cnt);
        first = before + incl - cnt;
        from = r * L + (int)(o >> 16);
        return before + __builtin_amdgcn_readlane(incl, 63);
    }
    // index into `order` of member j, which is in the 64 pieces at hand (all lanes take part, j differs by lane)
    __device__ static int find(int first, int from, int j) {
        int x = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) x += __shfl(first, x + step) <= j ? step : 0;
        return __shfl(from, x) + j - __shfl(first, x);
    }
    // the same over all pieces, 64 at a time, for lanes' j in [j0, j0 + 64) (all lanes take part; -1 past the last member)
    __device__ int search(int j0, int j, int lane) const {
        int index = -1;
        for (int r0 = 0, before = 0; r0 < R && before < j0 + 64; r0 += 64) {
            int first, from, cnt;
            const int end = load(r0, lane, before, first, from, cnt);
            if (end > j0) {  // (wave-uniform)
                const int at = find(first, from, j);
                index = j >= before && j < end ? at : index;
            }
            before = end;
        }
        return index;
    }
};
constexpr int kFewPieces = 8;

// ------------------------------------------------------------------------------------------------
// The assignment of a later round: keys that can only have gone to a centroid near their own, and the others.
//
// Between two rounds a key of a settled cluster has few centroids to choose from.  Let a be the (moved) centroid that won it
// last, b the best of a list of centroids near a, da and db their distances from the key, and T a distance from a that no
// centroid outside the list falls below.  A centroid c outside is at least |a - c| - da away, so it loses to b where
//   |a - c| >= T > da + db.
// In the benchmark's mixture (131072 keys, 2048 centroids, 5 % outliers) that leaves 23 % of the keys after the first
// round and 10 to 12 % after the later ones, with 1 to 4 centroids near enough to matter.  The winning cluster that all
// keys against all centroids would leave in `packed` follows from three launches (the score and the round beside it may be an earlier
// round's, where a key was settled and stayed, or not looked at):
//   near_lists  per centroid a: up to 32 centroids next to it in ascending id, T, and whether its keys have to be looked at: a centroid
//               that is near enough to matter for one of them moved, its members changed, or T fell below what they need.
//               Clusters to be looked at are listed in chunks of 64 members.
//   near        per chunk: the keys against the list (one 32 x 32 tile per 32 keys).  The winner is written where it is another
//               one; a key that the test leaves open is marked, with the score of its own centroid.
//   marked      the marked keys, gathered: those whose own centroid stayed, against the centroids that moved (no other one can
//               have overtaken), the others against all.
// A score is the same bits whichever slot of the matrix instruction it comes out of, and a margin for the scores' rounding
// (near_need) stands in the test, so the winner is the one that all of them would leave.
// A unit takes reassign_kernel's way instead, by the same code, for the rest of the build: where it has keys that are not finite or
// so large that a score may not be (`large_keys`: what the contraction leaves of a key among whose scores are NaN depends on
// where in a tile they are; argmax16: nine of them side by side hide their lane's others), and once too many of its keys were marked
// in a round, or would be in the first one as far as one key of every second cluster tells (keys of little structure: near_in_vain).
// The round in which it turns goes through the full contraction: the scores in `packed` are the last round's only behind one.
//
// `Near`: what the three leave for each other, scratch at the start of the unit's key tiles: 256 bytes and at most 114 of the 256 bytes per
// token there (n tokens, C <= n).
constexpr int kNearList = 32, kNearChunk = 64;
constexpr int kNearGroups = 12;   // a list's threshold: this many groups of 16 centroids have a member at or above it
constexpr int kMaxNearTokens = 1 << 24;  // (an item holds a cluster in 13 bits and a chunk in 19)
constexpr int kNearMaxClusters = 4096;   // (what near_lists holds of a unit in LDS)
struct Near {
    int *head;           // items; marked keys in even rounds, in odd ones; near_turned; (8 bytes) workgroups that looked at keys ahead in
                         // round 1 << 40 | these keys << 20 | those of them that will be marked
    uint32_t *list;      // [kNearMaxClusters / 512][n] marked's keys, per slice of the centroids
    unsigned char *open; // [n] 0: settled; else marked: near_mark of the round if the key's own centroid moved, 1 if it stayed
    uint16_t *near;      // [C][kNearList] ascending, the centroid itself among them, 0xFFFF behind the last
    float *reach;        // [C] T
    float *need;         // [C] what T has to exceed for every settled key
    float *few;          // [C] squared distance within which few centroids were when it was last worked out (0: a dozen and more are the same as this one; its keys
                         // stay open)
    uint32_t *items;     // [C + n / kNearChunk]
};
__device__ inline Near near_of(const Dev &d, int u, int n) {
    Near x;
    char *p = near_scratch(d, u);
    x.head = (int *)p;
    p += kNearHeadBytes;
    x.list = (uint32_t *)p;
    p += (size_t)(kNearMaxClusters / 512) * n * 4;
    x.open = (unsigned char *)p;
    p += (n + 63) / 64 * 64;
    x.near = (uint16_t *)p;
    p += (size_t)d.C * kNearList * 2;
    x.reach = (float *)p;
    x.need = x.reach + d.C;
    x.few = x.need + d.C;
    x.items = (uint32_t *)(x.few + d.C);
    return x;
}
// Whether a unit's keys are settled too seldom: so many of them were marked in a round, or (sample) so many of those that round 1 looked
// at ahead will be.  Ten rounds, us, this way throughout and turned in round 1, by the spread of the components (the benchmark's: 0.3), behind
// it the share of the keys that were looked at ahead and left open and the share that was marked in round 1:
//                          0.5                         0.52                        0.55                        0.6
//   8 x 131072 x 2048      2613  3354  0.34 0.49       2811  3359  0.45 0.62       3184  3373  0.66 0.80       3698  3402  0.89 0.96
//   2 x 131072 x 2048      1024  1139                  1093  1153                  1192  1148                  1289  1151
//   8 x 65536 x 1024       1104  1203  0.26 0.39       1178  1201  0.35 0.51       1266  1199  0.55 0.72       1412  1199  0.88 0.93
//   64 x 32768 x 512       2667  2872  0.25 0.28       2798  2867  0.28 0.36       3129  2893  0.43 0.52       3609  2891  0.68 0.83
// Two of the three launches cost the same for any number of clusters, a full round does not: with more of them fewer settled keys pay.
__device__ inline bool near_in_vain(int open, int of, int Cpad, bool sample) {
    const int limit = Cpad <= 768 ? (sample ? 8 : 9) : Cpad <= 1024 ? (sample ? 9 : 12) : (sample ? 12 : 15);  // twentieths
    return (long long)open * 20 > (long long)of * limit;
}
// The round in which unit u turned, 0: it did not.  joint: a build's units turn together.  (While the chip holds a round's workgroups
// at once, or nearly, a unit that takes the other way is what the others wait for: 64 x 32768 x 512 of spread 0.5, of which some turned,
// 3187, and 2667 and 2872 with none and all.  In more turns than two a unit's work adds to the others'.)
__device__ inline int *near_turned(const Dev &d, int u, int joint) { return (int *)near_scratch(d, joint ? 0 : u) + 3; }
__device__ inline unsigned near_mark(int round) { return 128u | ((unsigned)round & 127u); }

// The margin for rounding.  A score s(c) = k . c - |c|^2 / 2 is a chain of 129 (transformed keys: 130) fp32 additions of exact
// products: off by at most E(c) = g (|k| |c| + |c|^2), g = 2^-15 (four times (d + 2) 2^-24).  With D = |a - c| >= T > da + db:
//   s(b) - s(c) = (dc^2 - db^2) / 2 >= (D - da - db)^2 / 2,
//   E(b) + E(c) <= g (4 |k|^2 + 3 |a|^2 + 6 D^2)        (|c|^2 <= 2 |a|^2 + 2 D^2, |b|^2 <= 2 |k|^2 + 2 D^2),
// so c loses in fp32 as well where D - (da + db) > sqrt(8 g (|k|^2 + |a|^2)) + sqrt(12 g) D; sqrt(12 g) < 0.0195, hence the factor
// 1.025, which covers the rounding of these lines too.  da^2 and db^2 come out of scores, |k|^2 - 2 s, at most
// 2 g (5 |k|^2 + 4 db^2) too low: 32 g (|k|^2 + |a|^2) is added to them.  Whatever is not a number leaves the key open.
// Below 2^-126 an operation is off by up to 2^-126 more, whatever its result (2^-149 where subnormal numbers are kept): a score, a
// norm or a distance by at most 2^-118.  Counting |k|^2 + |a|^2 as 2^-90 more covers that many times over: the slack that this
// adds to the test is above 2^-51, its square above 2^-103.
constexpr float kNearFloor = 0x1p-90f;
__host__ __device__ inline float near_need(float k2, float a2, float sa, float sb) {
    const float w = k2 + a2 + kNearFloor, up = 0x1p-10f * w;
    const float da = sqrtf(fmaxf(k2 - 2.f * sa, 0.f) + up), db = sqrtf(fmaxf(k2 - 2.f * sb, 0.f) + up);
    return (da + db + sqrtf(0x1p-12f * w)) * 1.025f;
}
// a lower bound of the squared distance of a and a centroid of score at most s against it (the same bound on the score; what
// is lost below 2^-126 stands in near_need)
__host__ __device__ inline float near_dist2(float a2, float s) { return fmaxf((a2 * (1.f - 0x1p-11f) - 2.f * s) * (1.f - 0x1p-11f), 0.f); }

// Up to 32 rows of 256 bytes into a wave's own LDS tile (chunk c of row r in slot c ^ (r & 15)), lane first + r saying where row r is
__device__ inline void stage_rows(const bf16_t *base, int row_of_lane, int first, int rows, char *tile, int lane) {
    const int g = lane >> 4, i = lane & 15;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        if (4 * x >= rows) break;  // (wave-uniform)
        const int rr = 4 * x + g;
        const int row = __shfl(row_of_lane, first + rr);
        lds_dma16((const uint4 *)(base + (size_t)row * kD) + (i ^ (rr & 15)), tile + x * 1024);
    }
}
__device__ inline void read_rows(const char *tile, int lane, bf16x8 *out) {
    const int col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(tile + col * 256 + (((2 * ks + half) ^ (col & 15)) << 4)));
}

// Per centroid the ones near it.  A workgroup of 8 waves takes 64 centroids (the B operand, in registers) against all of the
// unit's, 32 at a time per wave, for the mask of those whose score reaches a limit.  The limit stands for a distance: within which
// few centroids are, and no further than the centroid's keys need (with something to spare, more where the centroid or its members
// are other ones than in the last round).  For the first list a pass over all of them finds the maximum of every group of 16, of which
// the kNearGroups-th largest (its upper 16 bits) is taken.  Bound by the round trips to the centroid rows, one tile's behind the other's.
constexpr int kNearA = 64;
// a wave's tiles of rows (two where they fit), the centroids' squared norms, the groups' maxima (the workgroup's own rows first)
__host__ __device__ inline int near_tiles(int Cpad) { return Cpad <= 2048 ? 2 : 1; }
__host__ __device__ inline int near_lists_lds_bytes(int Cpad) {
    const int maxima = kNearA * (Cpad / 16 + 2) * 2;
    return 8 * 8192 * near_tiles(Cpad) + Cpad * 4 + (maxima > 16384 ? maxima : 16384);  // (at most 153 KB)
}
template <bool AUG>
__global__ __launch_bounds__(512) void near_lists_kernel(const bf16_t *__restrict__ cent, const float *__restrict__ cnorm, int n, int Cpad, int cur,
                                                         const bf16_t *__restrict__ K, const int *__restrict__ go, int round, int R, int L, int joint, Dev d) {
    constexpr int KS = AUG ? 9 : 8;
    extern __shared__ __align__(16) char smem[];
    __shared__ float limit[kNearA];
    __shared__ int sampled, will_be_open;
    __shared__ __align__(4) uint16_t moved[kNearMaxClusters / 16];
    __shared__ int chunks[kNearA], found[kNearA];
    const int nbuf = near_tiles(Cpad);
    float *norms = (float *)(smem + 8 * 8192 * nbuf);  // [Cpad]
    char *own_rows = (char *)(norms + Cpad);
    uint16_t *gmax = (uint16_t *)own_rows;            // [kNearA][Cpad / 16 + 2] upper halves of the groups' ordered maxima
    uint32_t *hits = (uint32_t *)gmax;                // [kNearA][Cpad / 32 + 1] afterwards: the list as a mask
    const int groups = Cpad / 16, gstride = groups + 2, tiles = Cpad / 32, hstride = tiles + 1;
    // (a unit's workgroups on few dies: its rows stay in their L2)
    const int u = blockIdx.x % d.U, block = blockIdx.x / d.U, a0 = block * kNearA, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63;
    char *tile_lds = smem + wave * nbuf * 8192;
    const bf16_t *cu = cent + (size_t)u * Cpad * kD;
    const float *wn = cnorm + (size_t)u * Cpad;
    const Near x = near_of(d, u, n);
    auto request = [&](int t, int buf) {  // rows of a tile, direct to LDS
        const int g = lane >> 4, i = lane & 15;
        const uint4 *src = (const uint4 *)(cu + (size_t)t * 32 * kD);
#pragma unroll
        for (int y = 0; y < 8; ++y) lds_dma16(src + (4 * y + g) * 16 + (i ^ (4 * (y & 3) + g)), tile_lds + buf * 8192 + y * 1024);
    };
    int *turned = near_turned(d, u, joint);
    // whether the unit does not go this way in this round
    auto ends = [&] {
        const int goes = go[2 * u], off = *turned, large = d.large_keys[u], open = x.head[1 + ((round - 1) & 1)];
        // (a unit that turns in this very launch is not looked at: the waves of a workgroup might see it turn between them)
        const bool over = goes == 0 || (off != 0 && off != round), turns = large != 0 || near_in_vain(open, n, Cpad, false);
        if (tid == 0 && turns && !over) *turned = round;
        return over || turns;
    };
    // (Where a CU takes several workgroups one after the other, each would wait for its rows in vain: 256 units x 512 clusters that
    // turned 42 us a launch, 6 so.  Where it takes one, the rows are on their way while the flags are: 20.0 us at 8 units x 2048, 21.2 else.)
    if (gridDim.x > 256 && ends()) return;
    if (wave < 2) stage_rows(cu, min(a0 + 32 * wave + (lane & 31), Cpad - 1), 0, 32, own_rows + wave * 8192, lane);
    // a scan's first tiles
    auto request_first = [&] {
        if (wave < tiles) request(wave, 0);
        if (nbuf > 1 && wave + 8 < tiles) request(wave + 8, 1);
    };
    request_first();
    for (int i = tid; i < Cpad / 4; i += 512) ((float4 *)norms)[i] = ((const float4 *)wn)[i];
    const bool out = gridDim.x <= 256 && ends();
    uint32_t mv = 0;
    int held = 0;
    if (tid < groups) mv = moved_of_16(d.moved + (size_t)u * Cpad, tid, held);
    float a2 = 0.f, need = 0.f, few = 0.f;
    int members = 0;
    uint32_t own_word = 0, own_extra[2] = {0, 0};
    if constexpr (AUG) {
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) own_extra[ct] = d.caug[cur][(size_t)u * Cpad + min(a0 + 32 * ct + (lane & 31), Cpad - 1)];
    }
    const bool real = tid < kNearA && a0 + tid < d.C;
    if (real) {
        a2 = wn[a0 + tid];
        members = d.cluster_cnt[(size_t)u * d.C + a0 + tid];
        own_word = d.moved[(size_t)u * Cpad + a0 + tid];
        if (round > 1) {
            need = x.need[a0 + tid];
            few = x.few[a0 + tid];
        }
    }
    wait_lds_dma();  // (also for a workgroup that leaves here: nothing lands in its LDS any more)
    if (out) return;
    if (block == 0 && tid == 0) x.head[1 + (round & 1)] = 0;
    if (tid < groups) moved[tid] = (uint16_t)mv;
    if (wave == 0) {  // (kNearA == 64)
        // (near_dist2 of score_at(x) is x)
        auto score_at = [&](float dist2) { return 0.5f * (a2 * (1.f - 0x1p-11f) - dist2 * (1.f + 0x1p-11f)); };
        const float w = (own_word != 0u ? 1.3f : 1.02f) * need;
        limit[tid] = fmaxf(need > 0.f ? score_at(w * w) : -INFINITY, score_at(few));
        chunks[tid] = (members + kNearChunk - 1) / kNearChunk;
        if (tid == 0) sampled = will_be_open = 0;
    }
    lds_barrier();
    bf16x8 B[2][KS];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        read_rows(own_rows + ct * 8192, lane, B[ct]);
        if constexpr (AUG) B[ct][8] = __builtin_bit_cast(bf16x8, make_uint4(lane >= 32 ? 0u : own_extra[ct], 0, 0, 0));
    }
    lds_barrier();  // (read before the maxima go there)
    // every tile of this wave: use(tile, ct, scores)
    auto scan = [&](auto use) {
        const int col = lane & 31, half = lane >> 5;
        for (int t = wave, y = 0; t < tiles; t += 8, ++y) {
            const int buf = y & (nbuf - 1);
            uint32_t extra = 0;
            if constexpr (AUG) extra = d.caug[cur][(size_t)u * Cpad + t * 32 + col];
            // (behind the first tile nothing but tiles is on its way: the next one's eight loads may be)
            if (!AUG && nbuf > 1 && y > 0 && t + 8 < tiles) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else wait_lds_dma();
            bf16x8 A[KS];
            f32x16 seed;
            read_rows(tile_lds + buf * 8192, lane, A);
            if constexpr (AUG) A[8] = __builtin_bit_cast(bf16x8, make_uint4(half ? 0u : extra, 0, 0, 0));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float4 w = *(const float4 *)(norms + t * 32 + 8 * v + 4 * half);
                seed[4 * v] = -0.5f * w.x; seed[4 * v + 1] = -0.5f * w.y; seed[4 * v + 2] = -0.5f * w.z; seed[4 * v + 3] = -0.5f * w.w;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (read before the next tile may land there)
            if (t + 8 * nbuf < tiles) request(t + 8 * nbuf, buf);
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                f32x16 acc = seed;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ks], B[ct][ks], acc, 0, 0, 0);
                use(t, ct, acc);
            }
        }
    };
    // the kNearGroups-th largest group maximum of four centroids side by side (the chain of one is ballot, count, compare)
    const int k = min(kNearGroups, groups / 2);
    auto kth = [&](auto words) {
        constexpr int NJ = decltype(words)::value, NA = NJ > 2 ? 1 : 4;
        for (int i = 0; i < kNearA / 8; i += NA) {
            const int a = wave * (kNearA / 8) + i;
            uint32_t v[NA][NJ], at[NA];
#pragma unroll
            for (int y = 0; y < NA; ++y) {
                at[y] = 0;
#pragma unroll
                for (int j = 0; j < NJ; ++j) v[y][j] = 64 * j + lane < groups ? gmax[(a + y) * gstride + 64 * j + lane] : 0u;
            }
#pragma unroll
            for (int b = 15; b >= 0; --b) {
#pragma unroll
                for (int y = 0; y < NA; ++y) {
                    const uint32_t trial = at[y] | 1u << b;
                    int cnt = 0;
#pragma unroll
                    for (int j = 0; j < NJ; ++j) cnt += (int)__popcll(__ballot(v[y][j] >= trial));
                    at[y] = cnt >= k ? trial : at[y];
                }
            }
#pragma unroll
            for (int y = 0; y < NA; ++y)
                if (lane == 0) limit[a + y] = ordered_f32(max(at[y] << 16, 0x00800000u));  // (above -inf, the padding rows' score)
        }
    };
    // masks to lists, eight centroids per wave, NA side by side
    auto lists = [&](auto words) {
        constexpr int NJ = decltype(words)::value, NA = NJ > 1 ? 1 : 4;
        for (int i = 0; i < kNearA / 8; i += NA) {
            uint32_t w[NA][NJ];
            int at[NA][NJ], m[NA];
            bool ok[NA];
#pragma unroll
            for (int y = 0; y < NA; ++y) {
                const int al = wave * (kNearA / 8) + i + y, a = a0 + al;
                bool own = false, any = false;
                m[y] = 0;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int t = 64 * j + lane;
                    w[y][j] = t < tiles ? hits[al * hstride + t] : 0u;
                    const int cnt = __popc(w[y][j]), incl = wave_scan_add(cnt);
                    at[y][j] = m[y] + incl - cnt;
                    m[y] += __builtin_amdgcn_readlane(incl, 63);
                    own |= t == a >> 5 && (w[y][j] >> (a & 31) & 1u) != 0u;
                    any |= (w[y][j] & (t < tiles ? *(const uint32_t *)(moved + 2 * t) : 0u)) != 0u;
                }
                ok[y] = m[y] <= kNearList && __ballot(own) != 0ull;  // (else too many, as of centroids that are alike: no list)
                const u64 some = __ballot(any);
                if (lane == 0) found[al] = (ok[y] ? m[y] : 0) | (some != 0ull ? 64 : 0);
            }
#pragma unroll
            for (int y = 0; y < NA; ++y) {
                const int a = a0 + wave * (kNearA / 8) + i + y;
                if (a >= d.C) continue;  // (wave-uniform)
                uint16_t *out = x.near + (size_t)a * kNearList;
                if (ok[y]) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        for (uint32_t z = w[y][j]; z; z &= z - 1) out[at[y][j]++] = (uint16_t)(32 * (64 * j + lane) + __ffs(z) - 1);
                }
                if (lane < kNearList && lane >= (ok[y] ? m[y] : 0)) out[lane] = (uint16_t)(!ok[y] && lane == 0 ? a : 0xFFFF);
            }
        }
    };
    const int col = lane & 31, half = lane >> 5;
    bool no_lists = false;
    if (round == 1) {
        scan([&](int t, int ct, const f32x16 &acc) {
            float m = max3f(acc[0], acc[1], acc[2]);
#pragma unroll
            for (int v = 3; v < 15; v += 2) m = max3f(m, acc[v], acc[v + 1]);
            m = fmaxf(m, acc[15]);
            gmax[(32 * ct + col) * gstride + 2 * t + half] = (uint16_t)(f32_ordered(m) >> 16);
        });
        request_first();
        lds_barrier();
        if (groups <= 64) kth(std::integral_constant<int, 1>{});
        else if (groups <= 128) kth(std::integral_constant<int, 2>{});
        else kth(std::integral_constant<int, 4>{});
        lds_barrier();
        if (wave == 0) few = near_dist2(a2, limit[tid]);
        // one key of every second cluster: does its list settle it, as far as the distance from its own centroid says
        const int g = lane >> 4, ch = lane & 15, al = wave * (kNearA / 8) + 2 * g, c = min(a0 + al, d.C - 1);
        const uint32_t word = ch < R ? d.range_off[((size_t)u * R + ch) * Cpad + c] : 0u;  // (a member in the first 16 ranges, mostly)
        const uint32_t has = (uint32_t)(__ballot((word & 0xFFFFu) != 0u) >> (16 * g)) & 0xFFFFu;
        const int r = has ? __ffs(has) - 1 : 0;
        const int at = r * L + (int)((uint32_t)__shfl((int)word, 16 * g + r) >> 16);
        const int tok = has ? d.order[(size_t)u * d.max_tokens + at] : 0;
        const uint4 x4 = ((const uint4 *)(K + ((size_t)u * n + tok) * kD))[ch], c4 = ((const uint4 *)(cu + (size_t)c * kD))[ch];
        const uint32_t xs[4] = {x4.x, x4.y, x4.z, x4.w}, cs[4] = {c4.x, c4.y, c4.z, c4.w};
        float d2 = 0.f;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const float lo = bf16_lo(xs[y]) - bf16_lo(cs[y]), hi = bf16_hi(xs[y]) - bf16_hi(cs[y]);
            d2 += lo * lo + hi * hi;
        }
        if constexpr (AUG) {
            const float e = bf16_to_f32(d.kaug[(size_t)u * d.max_tokens + tok]) - bf16_to_f32(d.caug[cur][(size_t)u * Cpad + c]);
            d2 += ch == 0 ? e * e : 0.f;
        }
        d2 = row16_sum(d2);
        const bool sample = has != 0u && a0 + al < d.C && ch == 0;
        const u64 all = __ballot(sample), open_too = __ballot(sample && !(4.25f * d2 < near_dist2(wn[c], limit[al])));
        if (lane == 0 && all) {
            atomicAdd(&sampled, (int)__popcll(all));
            if (open_too) atomicAdd(&will_be_open, (int)__popcll(open_too));
        }
        lds_barrier();
        const int of = sampled, will = will_be_open;
        // (the unit's last workgroup says whether it turns; one that sees little but open keys needs no lists)
        if (tid == 0) {
            u64 sum = 1ull << 40 | (u64)of << 20 | (u64)will;
            sum += atomicAdd((u64 *)(x.head + 4), sum);
            if ((int)(sum >> 40) == (d.C + kNearA - 1) / kNearA && near_in_vain((int)(sum & 0xFFFFFu), (int)(sum >> 20 & 0xFFFFFu), Cpad, true)) *turned = 1;
        }
        no_lists = will * 4 > of * 3;
    }
    if (no_lists) {  // (workgroup-uniform)
        wait_lds_dma();
        for (int i = tid; i < kNearA * kNearList; i += 512) {
            const int a = a0 + i / kNearList;
            if (a < d.C) x.near[(size_t)a * kNearList + i % kNearList] = (uint16_t)(i % kNearList == 0 ? a : 0xFFFF);
        }
        if (tid < kNearA) found[tid] = 0;
    } else {
        const float lim0 = limit[col], lim1 = limit[32 + col];
        scan([&](int t, int ct, const f32x16 &acc) {
            const float lim = ct ? lim1 : lim0;
            uint32_t m = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) m |= acc[v] >= lim ? 1u << (8 * (v >> 2) + (v & 3)) : 0u;
            m <<= 4 * half;
            m |= (uint32_t)__shfl_xor((int)m, 32);
            if (half == 0) hits[(32 * ct + col) * hstride + t] = m;
        });
        lds_barrier();
        if (tiles <= 64) lists(std::integral_constant<int, 1>{});
        else lists(std::integral_constant<int, 2>{});
        lds_barrier();
    }
    if (tid >= kNearA) return;
    // one thread per centroid
    int mine = 0;
    if (real) {
        const int f = found[tid];
        const int m = f & 63;
        const float dist2 = near_dist2(a2, limit[tid]), reach = m > 0 ? sqrtf(dist2) * (1.f - 0x1p-20f) : 0.f;
        x.reach[a0 + tid] = reach;
        // (how many there are follows the centroids' moves: a list that came out too long is left out for once, a short one may grow)
        x.few[a0 + tid] = m == 0 ? 0.5f * dist2 : m < kNearGroups / 2 && dist2 > 0.95f * few ? 1.2f * few : few;
        if ((f & 64) != 0 || own_word != 0u || !(reach > need) || round == 1) {
            mine = chunks[tid];
            x.need[a0 + tid] = 0.f;
        }
    }
    const int incl = wave_scan_add(mine), total = __builtin_amdgcn_readlane(incl, 63);
    int base = 0;
    if (lane == 0 && total > 0) base = atomicAdd(&x.head[0], total);
    base = __builtin_amdgcn_readfirstlane(base);
    const int to = base + incl - mine;
    constexpr int kAlone = 8;
    for (int c = 0; c < min(mine, kAlone); ++c) x.items[to + c] = (uint32_t)(a0 + tid) | (uint32_t)c << 13;
    for (u64 left = __ballot(mine > kAlone); left; left &= left - 1ull) {  // (a large cluster's chunks by the whole wave)
        const int l = (int)__builtin_ctzll(left), cnt = __builtin_amdgcn_readlane(mine, l), first = __builtin_amdgcn_readlane(to, l);
        for (int c = kAlone + lane; c < cnt; c += 64) x.items[first + c] = (uint32_t)(a0 + l) | (uint32_t)c << 13;
    }
}

// The keys of the listed chunks against their centroids' lists, one wave per chunk of 64 members: the list's rows (A operand) and
// the keys' (B, 32 at a time) through the wave's own LDS, so no wave waits for another; the next chunk is looked up and its
// rows are requested while this one's are worked on.  Bound by the read of the keys and, where
// chunks are few, by the chain chunk -> piece -> entry -> row.
// NP: as in means_kernel (1 piece per cluster, at most kFewPieces, more).
template <bool AUG, int NP>
__global__ __launch_bounds__(64) void near_kernel(const bf16_t *__restrict__ K, const bf16_t *__restrict__ cent, const float *__restrict__ cnorm,
                                                  int n, int Cpad, int cur, const int *__restrict__ go, int round, int R, int L, int joint, Dev d) {
    constexpr int KS = AUG ? 9 : 8;
    __shared__ __align__(16) char rows[2][8192];
    __shared__ __align__(16) float seeds[32];
    const int u = blockIdx.x % d.U, lane = threadIdx.x, col = lane & 31, half = lane >> 5;  // (a unit's workgroups on few dies: its rows stay in their L2)
    const Near x = near_of(d, u, n);
    const int goes = go[2 * u], off = *near_turned(d, u, joint), items = __builtin_amdgcn_readfirstlane(x.head[0]), step = gridDim.x / d.U;
    int it = blockIdx.x / d.U;
    if (it >= items || goes == 0 || off != 0) return;
    // (rows of the list's tile that no centroid is staged into keep finite numbers: they count with a seed of -inf)
#pragma unroll
    for (int i = 0; i < 16; ++i) *(uint4 *)(&rows[0][0] + (i * 64 + lane) * 16) = make_uint4(0, 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const bf16_t *Ku = K + (size_t)u * n * kD, *cu = cent + (size_t)u * Cpad * kD;
    const int *order = d.order + (size_t)u * d.max_tokens;
    u64 *packed = d.packed + (size_t)u * d.max_tokens;
    const uint32_t tag = (uint32_t)(round % kRoundNumbers);
    struct Chunk {
        int c, j0, id, cnt;
        float reach, a2;
        uint32_t moved, word;
    };
    auto look_up = [&](uint32_t item) {
        Chunk k;
        k.c = (int)(item & 8191u);
        k.j0 = (int)(item >> 13) * kNearChunk;
        const size_t row = (size_t)u * Cpad + k.c;
        k.word = Pieces{d.range_off + (size_t)u * R * Cpad + k.c, Cpad, R, L}.word(NP == 1 ? 0 : lane);
        k.id = x.near[(size_t)k.c * kNearList + col];
        k.reach = x.reach[k.c];
        k.a2 = cnorm[row];
        k.cnt = d.cluster_cnt[(size_t)u * d.C + k.c];
        k.moved = d.moved[row];
        return k;
    };
    auto token = [&](const Chunk &k) -> int {  // member j0 + lane, -1 past the last
        const int j = k.j0 + lane;
        const Pieces pieces = {d.range_off + (size_t)u * R * Cpad + k.c, Cpad, R, L};
        int at;
        if constexpr (NP == 1) {
            at = (int)(k.word >> 16) + j;
        } else if constexpr (NP == kFewPieces) {
            at = 0;
            int before = 0;
#pragma unroll
            for (int r = 0; r < NP; ++r) {
                const uint32_t w = __builtin_amdgcn_readlane(k.word, r);
                if (j >= before) at = r * L + (int)(w >> 16) + j - before;
                before += (int)(w & 0xFFFFu);
            }
        } else if (R <= 64) {
            int first, from, own;
            pieces.take(k.word, 0, lane, 0, first, from, own);
            at = Pieces::find(first, from, j);
        } else {
            at = pieces.search(k.j0, j, lane);
        }
        int tok = -1;
        if (j < k.cnt) tok = order[at];
        return tok;
    };
    // The rows of a chunk go to two tiles: its list's and its first 32 keys'; then the other keys' to where the list's were and the
    // next chunk's list to where the first keys' were; then the next chunk's first keys to where the other keys' were.
    auto list_rows = [&](const Chunk &k, char *to) {
        stage_rows(cu, k.id == 0xFFFF ? k.c : k.id, 0, (int)__popcll(__ballot(lane < 32 && k.id != 0xFFFF)), to, lane);
    };
    auto key_rows = [&](const Chunk &k, int tok, int first, char *to) {
        const int any = __builtin_amdgcn_readfirstlane(tok);  // (a chunk has a member)
        stage_rows(Ku, tok >= 0 ? tok : any, first, min(k.cnt - k.j0 - first, 32), to, lane);
    };
    Chunk k = look_up(__builtin_amdgcn_readfirstlane(x.items[it]));
    uint32_t item1 = it + step < items ? x.items[it + step] : 0u;
    int tok = token(k);
    list_rows(k, rows[0]);
    key_rows(k, tok, 0, rows[1]);
    for (int p = 0;; p ^= 1) {
        char *list_at = rows[p], *keys_at = rows[1 - p];
        const int c = k.c, listed = k.id == 0xFFFF ? c : k.id;
        float seed_in = -INFINITY;
        uint32_t cext = 0, kext = 0;
        if (k.id != 0xFFFF) seed_in = -0.5f * cnorm[(size_t)u * Cpad + k.id];
        if constexpr (AUG) {
            cext = d.caug[cur][(size_t)u * Cpad + listed];
            kext = d.kaug[(size_t)u * d.max_tokens + max(tok, 0)];
        }
        const u64 is_own = __ballot(lane < 32 && k.id == c);
        const int own_at = (int)__builtin_ctzll(is_own | 1ull << 32) & 31;  // (c is in its list)
        const int own_v = (own_at >> 3) * 4 + (own_at & 3), own_half = own_at >> 2 & 1;
        const float reach = k.reach, a2 = k.a2;
        k.cnt = __builtin_amdgcn_readfirstlane(k.cnt);
        const bool own_moved = (__builtin_amdgcn_readfirstlane((int)k.moved) & 1) != 0, more = k.cnt - k.j0 > 32;
        // the next chunk
        it += step;
        const bool goes_on = it < items;
        Chunk k1 = k;
        if (goes_on) k1 = look_up(__builtin_amdgcn_readfirstlane(item1));
        if (it + step < items) item1 = x.items[it + step];
        wait_lds_dma();
        if (lane < 32) seeds[lane] = seed_in;
        bf16x8 A[KS], B[KS];
        f32x16 seed;
        read_rows(list_at, lane, A);
        if constexpr (AUG) A[8] = __builtin_bit_cast(bf16x8, make_uint4(half ? 0u : cext, 0, 0, 0));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float4 w = *(const float4 *)(seeds + 8 * v + 4 * half);
            seed[4 * v] = w.x; seed[4 * v + 1] = w.y; seed[4 * v + 2] = w.z; seed[4 * v + 3] = w.w;
        }
        read_rows(keys_at, lane, B);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (read before the next rows may land there)
        if (more) key_rows(k, tok, 32, list_at);
        int tok1 = -1;
        if (goes_on) {
            tok1 = token(k1);
            list_rows(k1, keys_at);
        }
        float need_max = 0.f;
        // the keys in B: members 32 h .. of the chunk
        auto settle = [&](int h) __attribute__((always_inline)) {
            const int key = __shfl(tok, 32 * h + col);
            float k2 = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const uint4 w = __builtin_bit_cast(uint4, B[ks]);
                k2 = dot2(w.w, w.w, dot2(w.z, w.z, dot2(w.y, w.y, dot2(w.x, w.x, k2))));
            }
            k2 += __shfl_xor(k2, 32);
            if constexpr (AUG) {
                const uint32_t e = __shfl(kext, 32 * h + col);
                B[8] = __builtin_bit_cast(bf16x8, make_uint4(half ? 0u : e, 0, 0, 0));
                const float f = __uint_as_float(e << 16);
                k2 += f * f;
            }
            f32x16 acc = seed;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ks], B[ks], acc, 0, 0, 0);
            float sa = acc[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) sa = v == own_v ? acc[v] : sa;
            sa = __shfl(sa, col + 32 * own_half);
            float m;
            uint32_t li;
            argmax16(acc, m, li);
            const u64 mine = ((u64)f32_ordered(m + 0.0f) << 32) | (u64)(31u - (li + 4u * half));
            const u64 other = ((u64)(uint32_t)__shfl_xor((int)(uint32_t)(mine >> 32), 32) << 32) | (u64)(uint32_t)__shfl_xor((int)(uint32_t)mine, 32);
            const u64 best = mine > other ? mine : other;
            const int won = __shfl(listed, (int)(31u - (uint32_t)best));
            const float need = near_need(k2, a2, sa, ordered_f32((uint32_t)(best >> 32)));
            const bool settled = reach > need;
            if (half == 0 && key >= 0) {
                x.open[key] = (unsigned char)(settled ? 0u : own_moved ? near_mark(round) : 1u);
                // (an open key: its own centroid's score as it is now, which the marked keys' pass compares with)
                const u64 word_of = settled ? (best & 0xFFFFFFFF00000000ull) | (u64)(0xFFFFFFFFu - (uint32_t)won)
                                            : ((u64)f32_ordered(sa + 0.0f) << 32) | (u64)(0xFFFFFFFFu - (uint32_t)c);
                if (!settled || won != c) packed[key] = winner_word(word_of, tag);
                if (settled) need_max = fmaxf(need_max, need);
            }
        };
        settle(0);
        if (more) {  // (wave-uniform)
            wait_lds_dma();
            read_rows(list_at, lane, B);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        if (goes_on) key_rows(k1, tok1, 0, list_at);
        if (more) settle(1);
        uint32_t top = row16_max_u32(__float_as_uint(need_max));  // (no need is negative)
        top = max(top, (uint32_t)__shfl_xor((int)top, 16));
        if (lane == 0 && top != 0u) atomicMax((int *)&x.need[c], (int)top);
        if (!goes_on) break;
        k = k1;
        tok = tok1;
    }
}

// The marked keys of a run (see above; a unit that turned: reassign_unit).  The workgroup that has slice x of
// the centroids takes the keys whose own centroid moved against that slice (they meet in `packed`, as in assign_kernel), and
// its share of the others against the centroids that moved (listed in ascending id in LDS, 512 at a time): with `old`
// the word of the key's own centroid, the winner m stands where m > old.
// Bound by its prologues where few keys are marked, as assign_kernel is else.
struct MarkedJob {
    bool moved;             // against the centroids that moved (`list`), else against all
    int nk, ncent, dir, slices;
    uint32_t round;
    u64 *packed;
    const uint32_t *keys;   // key x is keys[dir * x]
    const uint16_t *list;
    u64 last_word;
    __device__ __forceinline__ int key_of(int pos) const {
        int key = (int)keys[dir * min(pos, nk - 1)];
        asm volatile("" : "+v"(key));  // (waited for where it is loaded, see ReassignJob)
        return key;
    }
    __device__ __forceinline__ void rows_of(int t, int tid, int (&key)[8]) const {
        const int base = t * kAssignTile + (tid >> 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) key[i] = (int)keys[dir * min(base + 32 * i, nk - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(key[i]));
    }
    __device__ __forceinline__ int centroid(int pos) const { return moved ? (int)list[pos] : pos; }
    // (the moved centroids: what the tile's keys are compared with, in flight during the contraction)
    __device__ __forceinline__ void ahead(int t, int tid, int) {
        last_word = 0ull;  // (as it is in memory: taken apart here it would be waited for)
        if (moved && tid < kAssignTile) last_word = packed[key_of(t * kAssignTile + tid)];
    }
    __device__ __forceinline__ void arrived() { asm volatile("" : "+v"(last_word)); }
    __device__ __forceinline__ void take(int pos, u64 b, int, int) {
        if (pos >= nk) return;
        const int key = key_of(pos);
        if (!moved) {
            const u64 w = winner_word(b, round);
            if (slices > 1) atomicMax(packed + key, w);  // (nothing waits for it)
            else packed[key] = w;
        } else {
            const uint32_t at = ~(uint32_t)b;  // (a place in the list)
            const u64 m = (b & 0xFFFFFFFF00000000ull) | (u64)(0xFFFFFFFFu - list[min(at, (uint32_t)ncent - 1u)]);
            if (m > winner_of_word(last_word)) packed[key] = winner_word(m, round);
        }
    }
};

template <bool AUG, bool ALL_FULL>  // ALL_FULL: every slice of the centroids is full (FULL of assign_slice)
__global__ __launch_bounds__(512) void marked_kernel(const bf16_t *__restrict__ K, const bf16_t *__restrict__ cent,
                                                     const float *__restrict__ cnorm, int n, int Cpad, int cur, const int *__restrict__ go,
                                                     int round, int fused, int joint, RoundPlan plan, Dev d) {  // (scalars first: preloaded at wave start)
    extern __shared__ __align__(16) char smem[];
    char *keys = smem;                                             // [2][256][256 B], chunks swizzled as in assign_slice
    u64 *best = (u64 *)(smem + 2 * kAssignTile * 256);             // [2][256]
    float *seeds = (float *)(best + 2 * kAssignTile);              // [512] of the slice at hand
    uint32_t *kext = (uint32_t *)(seeds + 512);                    // (AUG) [2][256] the keys' extra coordinates
    uint32_t *cext = kext + 2 * kAssignTile;                       // (AUG) [512] the centroids' of the slice at hand
    uint16_t *list = (uint16_t *)(kext + (AUG ? 1024 : 0));        // [Cpad] moved centroids, ascending
    __shared__ int sh_wave[8], sh_marked[2];

    const int u = blockIdx.y;
    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u64 *packed = d.packed + (size_t)u * d.max_tokens;
    const int slices = plan.slices, wgs = plan.all_wgs, keys_per_wg = plan.all_run * kAssignTile, which = blockIdx.x / wgs, range = blockIdx.x - which * wgs;
    const int k0 = range * keys_per_wg, kend = min(n, k0 + keys_per_wg);
    const int nbits = 32 - __builtin_clz((unsigned)Cpad - 1u);
    int *head = (int *)near_scratch(d, u);

    int goes_in = go[2 * u], turned_in = *near_turned(d, u, joint);  // (nothing in this launch changes it)
    asm volatile("" : "+v"(goes_in), "+v"(turned_in));               // (one trip for both)
    const int goes = __builtin_amdgcn_readfirstlane(goes_in), turned = __builtin_amdgcn_readfirstlane(turned_in);
    if (turned != 0 || which >= slices) {  // (one branch: as two the transformed forms kept addresses in scratch memory)
        if (turned == 0) return;
        reassign_unit<AUG, ALL_FULL>(K, cent, cnorm, n, Cpad, cur, go, round, fused, turned == round, plan, d, smem);
        return;
    }
    if (fused && blockIdx.x == 0 && tid == 0) d.any_moved[2 * u + (round & 1)] = 0;  // (for this round's means)
    if (goes == 0) return;  // (no centroid moved: every winner stands)
    if (blockIdx.x == 0 && tid == 0) head[0] = 0;  // (for the next round's near_lists)
    // ---- which centroids moved, and the run's marked keys: whose own centroid moved from the front of the key list on,
    // the others from its end
    int ncent = 0, n_all, n_moved;
    uint32_t *marked;
    {
        const Near x = near_of(d, u, n);
        marked = x.list + (size_t)which * n + k0;
        const int lane = tid & 63;
        uint32_t m = 0;
        int held = 0;
        if (tid * 16 < Cpad) m = moved_of_16(d.moved + (size_t)u * Cpad, tid, held);
        const int cnt = __popc(m), incl = wave_scan_add(cnt);
        if (lane == 63) sh_wave[wave] = incl;
        if (tid < 2) sh_marked[tid] = 0;
        if (tid < 2 * kAssignTile) best[tid] = 0ull;
        __syncthreads();
        int pos = incl - cnt;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const int y = sh_wave[w];
            pos += w < wave ? y : 0;
            ncent += y;
        }
        ncent = __builtin_amdgcn_readfirstlane(ncent);
        for (; m; m &= m - 1) list[pos++] = (uint16_t)(tid * 16 + __ffs(m) - 1);
        __syncthreads();  // (sh_wave is used again)
        const uint32_t mark = near_mark(round);
        const unsigned char *open = x.open + k0;
        const int len = kend - k0;
        // 16 keys from i0 on: those whose own centroid moved, and the others (masks)
        auto split = [&](int i0, uint32_t &front, uint32_t &back) {
            uint4 w = make_uint4(0, 0, 0, 0);
            if (i0 < len) w = *(const uint4 *)(open + i0);  // (k0 is a multiple of 256)
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
            front = back = 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t v = ws[e >> 2] >> (8 * (e & 3)) & 255u;
                front |= v == mark ? 1u << e : 0u;
                back |= v != 0u && v != mark ? 1u << e : 0u;
            }
            const uint32_t valid = i0 + 16 <= len ? 0xFFFFu : (1u << max(len - i0, 0)) - 1u;
            front &= valid;
            back &= valid;
        };
        int others = 0;
        for (int b = 16 * tid; b < len; b += 16 * 512) {
            uint32_t front, back;
            split(b, front, back);
            others += __popc(back);
        }
        others = __builtin_amdgcn_readlane(wave_scan_add(others), 63);
        if (lane == 0) sh_wave[wave] = others;
        __syncthreads();
        others = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) others += sh_wave[w];
        others = __builtin_amdgcn_readfirstlane(others);
        // One pass of all marked keys against all centroids, in the first round (no winner of a round before stands behind the marks) and
        // where the others cost no more there than by themselves against the moved ones: in tiles of 256 keys x 512 centroids, of
        // which a pass's prologue takes about 3/4, x = others / 256 and 3/4 of a tile per 512 moved centroids + x * moved / all.
        // (Else the workgroup has every slices-th 16 of them.)
        const bool one_pass = round == 1 || (long long)others * (Cpad - ncent) <= 192ll * ((ncent + 511) / 512) * Cpad;
        for (int b = 0; b < len; b += 16 * 512) {
            const int i0 = b + 16 * tid;
            uint32_t front, back;
            split(i0, front, back);
            if (one_pass) front |= back;
            if (one_pass || (i0 >> 4) % slices != which) back = 0;
            const int nf = __popc(front), nb = __popc(back), scan = wave_scan_add(nf | nb << 16);
            int base_f = 0, base_b = 0;
            if (lane == 63) {
                base_f = atomicAdd(&sh_marked[0], scan & 0xFFFF);
                base_b = atomicAdd(&sh_marked[1], scan >> 16);
            }
            int pf = __builtin_amdgcn_readlane(base_f, 63) + (scan & 0xFFFF) - nf, pb = __builtin_amdgcn_readlane(base_b, 63) + (scan >> 16) - nb;
            for (; front; front &= front - 1) marked[pf++] = (uint32_t)(k0 + i0 + __ffs(front) - 1);
            for (; back; back &= back - 1) marked[len - 1 - pb++] = (uint32_t)(k0 + i0 + __ffs(back) - 1);
        }
        wait_vmem();  // (the key lists of all waves are read by all)
        __threadfence_block();
        __syncthreads();
        n_all = __builtin_amdgcn_readfirstlane(sh_marked[0]);
        n_moved = __builtin_amdgcn_readfirstlane(sh_marked[1]);
        const int count = (which == 0 ? n_all : 0) + n_moved;
        if (tid == 0 && count > 0) atomicAdd(&head[1 + (round & 1)], count);
    }
    const bf16_t *Ku = K + (size_t)u * n * kD;

    MarkedJob job{false, n_all, min(Cpad, (which + 1) * 512), 1, slices, (uint32_t)(round % kRoundNumbers), packed, marked, list, 0ull};
    int c_first = which * 512;
    for (;;) {
        if (job.nk > 0) later_slices<AUG>(d, Ku, cent, cnorm, u, Cpad, cur, wave, c_first, tid, keys, best, seeds, kext, cext, job);
        if (job.moved) break;
        job.moved = true;
        job.nk = n_moved;
        job.keys = marked + (kend - k0 - 1);
        job.dir = -1;
        job.ncent = ncent;
        c_first = 0;
        __syncthreads();
    }
    if (fused) {  // the run is a range of the sort as well
        wait_vmem();
        __threadfence_block();
        __syncthreads();
        const uint32_t *pk = (const uint32_t *)packed;
        sort_range<8, kFusedRun / 2, false>(d, thread_of(wave), u, n, range, wgs, k0, kend, keys_per_wg / 8, 8, nbits, round, 1,
                                            (int *)smem, nullptr, nullptr, [=](int i) { return pk[2 * i]; }, cluster_of_word, [](int) { return 0.f; });
    }
}

// Rounds this way, from the second on, where a full one is at least 16 tiles of 256 keys x 512 centroids per workgroup (about 110 us).
// Builds of ten rounds, us, by the centroids that moved from the third round on (reassign_kernel) and so: 8 units x 131072 x 2048 with
// 5 % outliers (64 tiles) 3690 and 2300; the benchmark's mixture 8 x 131072 x 1024 (32) 2554 and 1588, x 1310 transformed 3189 and 2030,
// 64 x 32768 x 512 (32) 2720 and 2204, 8 x 65536 x 1024 (16) 1080 and 924, 2 x 131072 x 2048 (16) 1040 and 852, 16 x 32768 x 768 (16)
// 904 and 864, 256 x 32768 x 512 10920 and 8690; below the line 8 x 49152 x 768 (12) 819 and 775, 1 x 131072 x 2048 (8) 687 and 662, 4 x
// 65536 x 1024 (8) 677 and 685, 2 x 32768 x 2048 (4) 302 and 377, 8 x 32768 x 512 (4) 492 and 567.  Keys that the near centroids do not
// settle pay for finding that out and for two empty launches (3.5 us each) in each later round.  Without any structure: 8 x 131072 x 2048 5090 and
// 5220, 64 x 32768 x 512 3820 and 3920, 8 x 65536 x 1024 1557 and 1644; components of spread 0.6: 3048 and 3154, 2730 and 2825, 1053 and 1145,
// 2 x 131072 x 2048 996 and 1086, 16 x 32768 x 768 897 and 983.  (The line leaves out the gains of 3 to 6 % right below it: such keys
// lose more there, 8 x 49152 x 768 without structure 1176 and 1248.)
// And from 16384 keys and 32 keys per cluster on (20 from 32768 keys on): the lists of near centroids are worked out per cluster, by all
// centroids.  From there on 256 units x 16384 x 512 (32 keys) 4600 and 4200, 64 x 32768 x 1024 (32) 3070 and 2630, 48 x 32768 x 1536 (21) 3320 and
// 2980; below 64 x 20480 x 1024 (20) 1880 and 1910, 256 x 12288 x 512 (24) 3410 and 3440, 64 x 16384 x 1024 (16) 1535 and 1690, 256 x 8192 x 512 (16)
// 2380 and 2700, 300 x 6100 x 300 (20) 1920 and 2340, 32 x 16384 x 2048 (8) 1325 and 1605, 600 x 4000 x 450 (9) 3630 and 4970.  (The line leaves
// out gains that components of spread 0.45 and 0.6 turn into losses, 64 x 32768 x 2048 (16) 4960 and 4830, 4400 and 4560, 4820 and 5140, 256 x 9600 x 300
// (32) 2440 and 2400, 2610 and 2675, 2640 and 2800; and 16 x 65536 x 4096 (16) 3330 and 3000.)
// Of the 2300 us of 8 x 131072 x 2048: first round 440, then near_lists 32 and eight times 19, near 80 to 18, marked 130 to 32,
// sort 16, means 55 to 14 each, page copy 190.
// With up to 512 clusters the first of these rounds (the first lists, nearly all keys looked at) takes longer than a full one, and the later ones
// have to make up for it: from four rounds on, up to 384 clusters six.  Two, three, four and six rounds: 256 x 32768 x 512 4240 and 4420, 5530 and 5515, 6710
// and 6315, 8320 and 7370; 256 x 24576 x 384 2815 and 3060, 3610 and 3820, 4320 and 4370, 5490 and 5130; 512 x 16384 x 260 3620 and 3980, 4625 and 4980, 5525
// and 5715, 6980 and 6740.  Above 512 two rounds do: 128 x 20480 x 640 1870 and 1815, 48 x 32768 x 1536 1712 and 1718, 8 x 131072 x 2048 1269 and 1044.
constexpr int kNearMinSteps = 16;
bool near_pays(const Dev &d, int n, int rounds) {
    if (rounds < (d.Cpad <= 384 ? 6 : d.Cpad <= 512 ? 4 : 2)) return false;
    if (d.Cpad > kNearMaxClusters || n > kMaxNearTokens || !reassign_pays(d, n)) return false;
    if (n < 16384 || n < (n < 32768 ? 32ll : 20ll) * d.C) return false;
    const RoundPlan p = round_plan(d, n);
    return p.all_turns * p.all_run * p.tiles >= 16 * kNearMinSteps;
}

void launch_near(const Dev &d, const bf16_t *K, int n, int cur, int t, bool fused, hipStream_t st) {
    const RoundPlan p = round_plan(d, n);
    const int joint = p.all_turns <= 2 ? 1 : 0;
    const int L = sort_len(d, n), R = (n + L - 1) / L;
    const int *go = round_goes(d, t);
    const size_t near_lds = near_lists_lds_bytes(d.Cpad);
#define ICE_NEAR_LISTS(aug)                                                                                                \
    do {                                                                                                                   \
        allow_dynamic_lds((const void *)near_lists_kernel<aug>, near_lds);                                                 \
        hipLaunchKernelGGL(near_lists_kernel<aug>, dim3((d.C + kNearA - 1) / kNearA * d.U), dim3(512), near_lds, st, d.cent_bf16[cur], d.cnorm[cur], n, \
                           d.Cpad, cur, K, go, t, R, L, joint, d);                                                                  \
    } while (0)
    if (d.tk) ICE_NEAR_LISTS(true);
    else ICE_NEAR_LISTS(false);
#undef ICE_NEAR_LISTS
    // as many waves as the chip holds at once, at most one per chunk
    const int waves = (int)std::min<long long>((2048 + d.U - 1) / d.U, (long long)d.C + n / kNearChunk);
#define ICE_NEAR(aug, np)                                                                                                  \
    hipLaunchKernelGGL((near_kernel<aug, np>), dim3(waves * d.U), dim3(64), 0, st, K, d.cent_bf16[cur], d.cnorm[cur], n, d.Cpad, cur, go, t, R, L, joint, d)
#define ICE_NEAR_P(aug)                                                                                                    \
    do {                                                                                                                   \
        if (R == 1) ICE_NEAR(aug, 1);                                                                                      \
        else if (R <= kFewPieces) ICE_NEAR(aug, kFewPieces);                                                               \
        else ICE_NEAR(aug, 0);                                                                                             \
    } while (0)
    if (d.tk) ICE_NEAR_P(true);
    else ICE_NEAR_P(false);
#undef ICE_NEAR_P
#undef ICE_NEAR
    const size_t lds = std::max<size_t>(reassign_lds_bytes(d.tk != 0, d.Cpad), assign_lds_bytes(d.tk != 0) + (fused ? (size_t)p.all_run * kAssignTile * 2 : 0));
#define ICE_MARKED(aug, full)                                                                                              \
    do {                                                                                                                   \
        allow_dynamic_lds((const void *)marked_kernel<aug, full>, lds);                                                    \
        hipLaunchKernelGGL((marked_kernel<aug, full>), dim3(std::max(p.wgs, p.all_wgs * p.slices), d.U), dim3(512), lds, st, K, d.cent_bf16[cur], \
                           d.cnorm[cur], n, d.Cpad, cur, go, t, fused ? 1 : 0, joint, p, d);                               \
    } while (0)
    const bool full = d.Cpad / 32 % 16 == 0;
    if (d.tk) { if (full) ICE_MARKED(true, true); else ICE_MARKED(true, false); }
    else { if (full) ICE_MARKED(false, true); else ICE_MARKED(false, false); }
#undef ICE_MARKED
}

void near_bounds(int n, const float *k2, const float *a2, const float *sa, const float *sb, float *need, float *dist2) {
    for (int i = 0; i < n; ++i) {
        need[i] = near_need(k2[i], a2[i], sa[i], sb[i]);
        dist2[i] = near_dist2(a2[i], sb[i]);
    }
}

void build_plan(const Dev &d, int n, int rounds, int *plan) {
    plan[0] = sort_is_fused(d, n) ? 1 : 0;
    plan[1] = sort_len(d, n);
    plan[2] = (n + plan[1] - 1) / plan[1];
    plan[3] = near_pays(d, n, rounds) ? 1 : rounds > 2 && reassign_pays(d, n) ? 2 : 0;
    plan[4] = assign_run(d.U, n, 1);
    plan[5] = assign_slices(d);
}

// ------------------------------------------------------------------------------------------------
// The sort by itself
template <int NG, bool MASK>
__global__ __launch_bounds__(1024) void range_sort_kernel(Dev d, int n, int L, int W, int nbits, int round, float *best_out,
                                                          int *assign_out) {
    extern __shared__ __align__(16) int pos_all[];  // [W][Cpad]
    const int r = blockIdx.x, u = blockIdx.y;
    const int goes = round > 0 ? d.any_moved[2 * u + ((round - 1) & 1)] : 1;
    if (r == 0 && threadIdx.x == 0) d.any_moved[2 * u + (round & 1)] = 0;  // (for this round's means)
    // (a winner's low word holds its cluster; the whole of it is read only for best_out)
    const u64 *packed = d.packed + (size_t)u * d.max_tokens;
    const uint32_t *pk = (const uint32_t *)packed;
    sort_range<16, NG, MASK>(d, threadIdx.x, u, n, r, gridDim.x, r * L, min(n, r * L + L), L / W, W, nbits, round, goes, pos_all, best_out, assign_out,
                             [=](int i) { return pk[2 * i]; }, cluster_of_word, [=](int i) { return -2.0f * ordered_f32((uint32_t)(packed[i] >> 13)); });
}

void launch_sort(const Dev &d, int n, int t, float *best_out, int *assign_out, hipStream_t st) {
    const int L = sort_len(d, n), R = (n + L - 1) / L, W = sort_segments(d.Cpad);
    int nbits = 0;
    while ((1 << nbits) < d.Cpad) ++nbits;
    const bool masks = L / W > 4 * 64 && W * d.Cpad * 3 <= kSortCounters;
    const size_t lds = (size_t)W * d.Cpad * (masks ? 12 : 4);
#define ICE_SORT(ng, mk)                                                                                                   \
    do {                                                                                                                   \
        allow_dynamic_lds((const void *)range_sort_kernel<ng, mk>, lds);                                                   \
        hipLaunchKernelGGL((range_sort_kernel<ng, mk>), dim3(R, d.U), dim3(1024), lds, st, d, n, L, W, nbits, t, best_out, assign_out); \
    } while (0)
    if (L / W <= 4 * 64) ICE_SORT(4, false);
    else if (L / W <= 16 * 64) { if (masks) ICE_SORT(16, true); else ICE_SORT(16, false); }
    else { if (masks) ICE_SORT(32, true); else ICE_SORT(32, false); }
#undef ICE_SORT
}

// One wave counts the members of a cluster and lists their indexes into `order` in slots[0..kMemberSlots), piece by piece,
// as long as they fit and no piece has more than kMemberPiece of them (*listed): one read per member instead of a search.
constexpr int kMemberSlots = 512, kMemberPiece = 32;
constexpr int kAugAlone = 256, kAugChunk = 1024;
__device__ inline int list_members(const Pieces &pieces, uint32_t word0, int lane, int *slots, bool *listed) {
    int total = 0;
    bool ok = true;
    for (int r0 = 0; r0 < pieces.R; r0 += 64) {
        int first, from, cnt;
        total = pieces.take(r0 == 0 ? word0 : pieces.word(r0 + lane), r0, lane, total, first, from, cnt);
        ok = ok && total <= kMemberSlots && __ballot(cnt > kMemberPiece) == 0ull;
        for (int e = 0; ok && __ballot(e < cnt) != 0ull; ++e)
            if (e < cnt) slots[first + e] = from + e;
    }
    *listed = ok;
    return total;
}

// The key rows of one clustering pass are read by assign, then by means (and once more by paginate).
// While they fit the chip's last-level cache (256 MB) the second reader finds them there; beyond
// that every pass streams from HBM, and the non-temporal hint is what gets the most out of it.
static bool keys_exceed_cache(const Dev &d, int n) { return (size_t)d.U * (size_t)n * kD * sizeof(bf16_t) >= ((size_t)256 << 20); }

// ------------------------------------------------------------------------------------------------
// Centroid update: one workgroup of four waves per cluster.  Wave w gathers the w-th quarter of the
// cluster's members in sorted order (key rows of 256 contiguous bytes, 16 lanes x 16 bytes, four
// rows per load) and sums them in fp32 in a fixed order; the four partial sums meet in LDS and are
// added in wave order, so the result is the same on every run (no floating-point atomics) and a
// large cluster costs a quarter of the dependent round trips.  Writes sum, count, mean, and the
// bf16 rounding + squared norm of the mean into the OTHER centroid buffer; an empty cluster keeps
// its centroid.
// NP: 1, a cluster is one piece; kFewPieces, at most that many, which every wave fetches with one load and picks from per
// member; 0, more, which the first wave lists in LDS for all (or every wave searches, see list_members).  Bound by the key
// rows where units are many and by the chain piece -> entry -> row where they are few.  Measured (us; pieces looked up one
// after the other and no entry ahead, as it is, and over one contiguous list per cluster, which takes a unit-wide sort):
// 256 units x 32768 tokens x 512 clusters, one piece, 429, 411, 410; 40 units, four pieces, 77.5, 68.5, 66; 32 units, eight,
// 59 through LDS, 56.4, 53.5; 8 units x 131072 x 2048, 32 pieces, 61.7, 60.7, 55; 2 x 131072 x 64, clusters of thousands, 131, 108, 103.
// (Eight waves per SIMD: 256 units 418 us with seven; the last form keeps two registers in scratch for it, 62 -> 60.6 at 8 units.)
template <bool STREAM, int NP>
__global__ __launch_bounds__(256, 8) void means_kernel(Dev d, const bf16_t *__restrict__ K, int n, int cur, int R, int L, int round, int last) {
    __shared__ float4 part_sum[3][16][2];
    __shared__ int slots[kMemberSlots], sh_cnt, sh_listed;
    __shared__ float aug_lds[kAugChunk];
    const int u = blockIdx.y, c = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = lane >> 4, ch = lane & 15;
    const size_t row = (size_t)u * d.Cpad + c;
    const int *order = d.order + (size_t)u * d.max_tokens;
    const Pieces pieces = {d.range_off + (size_t)u * R * d.Cpad + c, d.Cpad, R, L};
    // (requested ahead of the flags, which mostly say that it was in vain, late in a build)
    uint32_t word0 = pieces.word(NP == 1 ? 0 : lane);
    if (round > 0) {
        const int goes = d.any_moved[2 * u + ((round - 1) & 1)], touched = d.touched[row], had_moved = d.moved[row];
        asm volatile("" : "+v"(word0));
        if (goes == 0) return;  // (no centroid of the unit moved in the last round: both buffers hold the same, no token moved)
        if (touched == 0) {     // the members of the last round: the same mean
            if (wave == 0 && had_moved != 0) {
                if (g == 0) ((uint4 *)(d.cent_bf16[cur ^ 1] + row * kD))[ch] = ((const uint4 *)(d.cent_bf16[cur] + row * kD))[ch];
                if (lane == 0) {
                    d.cnorm[cur ^ 1][row] = d.cnorm[cur][row];
                    if (d.tk) d.caug[cur ^ 1][row] = d.caug[cur][row];
                    d.moved[row] = 0;
                }
            }
            return;
        }
    }
    int before[kFewPieces], from[kFewPieces], cnt = 0, first = 0, first_at = 0;
    bool listed = false;
    if constexpr (NP == 1) {
        const uint32_t o = word0;
        from[0] = (int)(o >> 16);
        cnt = (int)(o & 0xFFFFu);
    } else if constexpr (NP == kFewPieces) {
        const uint32_t o = word0;
#pragma unroll
        for (int r = 0; r < kFewPieces; ++r) {
            const uint32_t x = __builtin_amdgcn_readlane(o, r);  // (no members past the last piece)
            before[r] = cnt;
            from[r] = r * L + (int)(x >> 16);
            cnt += (int)(x & 0xFFFFu);
        }
    } else {
        if (wave == 0) {
            bool ok;
            const int m = list_members(pieces, word0, lane, slots, &ok);
            if (lane == 0) {
                sh_cnt = m;
                sh_listed = ok;
            }
        }
        lds_barrier();
        cnt = sh_cnt;
        listed = sh_listed != 0;
        int own;
        if (!listed && R <= 64) pieces.take(word0, 0, lane, 0, first, first_at, own);
    }
    // lane l: the token of member j0 + l, -1 from `end` on (all lanes take part)
    auto member = [&](int j0, int end) -> int {
        const int j = j0 + lane;
        int at;
        if constexpr (NP == 1) {
            at = from[0] + j;
        } else if constexpr (NP == kFewPieces) {
            at = from[0] + j;
#pragma unroll
            for (int r = 1; r < kFewPieces; ++r)
                if (j >= before[r]) at = from[r] + j - before[r];
        } else {
            if (listed) at = slots[min(j, kMemberSlots - 1)];
            else if (R <= 64) at = Pieces::find(first, first_at, j);
            else at = pieces.search(j0, j, lane);
        }
        int tok = -1;
        if (j < end) tok = order[at];
        return tok;
    };
    const bf16_t *Ku = K + (size_t)u * n * kD;
    const int quarter = (cnt + 3) / 4;
    const int lo = min(cnt, wave * quarter), hi = min(cnt, lo + quarter);
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    // Group g of a wave sums rows g, g+4, g+8, ... of the wave's range in that order.  The member
    // list is read 64 entries at a time (one per lane) and the rows are fetched eight per group at
    // once, so a wave keeps 8 KB of key rows in flight instead of one dependent load pair per step.
    // The next 64 entries are looked up while the rows of these are on their way.
    int mine = member(lo, hi);
    for (int base = lo; base < hi; base += 64) {
        int next = -1;
        const int rows = min(64, hi - base);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h * 32 >= rows) break;
            uint4 w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int tok = __shfl(mine, 4 * (h * 8 + k) + g);
                w[k] = tok >= 0 ? load16<STREAM>((const uint4 *)(Ku + (size_t)tok * kD) + ch) : make_uint4(0, 0, 0, 0);
            }
            if (h == 0 && base + 64 < hi) next = member(base + 64, hi);
#pragma unroll
            for (int k = 0; k < 8; ++k) {  // rows past the end add +0
                acc[0] += bf16_lo(w[k].x); acc[1] += bf16_hi(w[k].x);
                acc[2] += bf16_lo(w[k].y); acc[3] += bf16_hi(w[k].y);
                acc[4] += bf16_lo(w[k].z); acc[5] += bf16_hi(w[k].z);
                acc[6] += bf16_lo(w[k].w); acc[7] += bf16_hi(w[k].w);
            }
        }
        mine = next;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        acc[j] += __shfl_xor(acc[j], 16);
        acc[j] += __shfl_xor(acc[j], 32);
    }
    // (transformed keys) sum of the members' extra coordinates: lane-strided partial sums in member order by the first
    // wave, requested before the waves meet.  Beyond kAugAlone members all four waves look them up and leave the
    // coordinates in LDS, kAugChunk at a time, for the first one to add (by itself it took 116 us at clusters of thousands,
    // 2 units x 131072 x 64, against 58 over one contiguous list).
    float aug_part = 0.f;
    if (d.tk) {
        const bf16_t *extra = d.kaug + (size_t)u * d.max_tokens;
        const bool alone = cnt <= kAugAlone;
        for (int j0 = 0; j0 < cnt; j0 += kAugChunk) {
            constexpr int NB = 4;  // 64 members each
            static_assert(kAugAlone == 64 * NB && kAugChunk == 4 * kAugAlone, "four look-ups per wave at a time");
            int tok[NB];
            float a[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = alone ? i : 4 * i + wave;
                tok[i] = -1;
                if (j0 + 64 * b < cnt && (wave == 0 || !alone)) tok[i] = member(j0 + 64 * b, cnt);  // (wave-uniform)
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                a[i] = 0.f;
                if (tok[i] >= 0) a[i] = bf16_to_f32(extra[tok[i]]);
            }
            if (alone) {
#pragma unroll
                for (int i = 0; i < NB; ++i) aug_part += a[i];  // (no coordinate is negative: +0 past the end changes nothing)
                break;
            }
            if (j0 > 0) __syncthreads();  // (the first wave has added the last chunk)
#pragma unroll
            for (int i = 0; i < NB; ++i) aug_lds[(4 * i + wave) * 64 + lane] = a[i];
            __syncthreads();
            if (wave == 0)
                for (int b = 0; b < 4 * NB && j0 + 64 * b < cnt; ++b) aug_part += aug_lds[64 * b + lane];
        }
    }
    // what the last assignment saw of the centroid (in flight while the waves meet)
    uint4 was = make_uint4(0, 0, 0, 0);
    float was_norm = 0.f;
    if (wave == 0 && !last) {  // (behind the last round nobody asks)
        was = ((const uint4 *)(d.cent_bf16[cur] + row * kD))[ch];
        was_norm = d.cnorm[cur][row];
    }
    if (wave > 0 && g == 0) {
        part_sum[wave - 1][ch][0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        part_sum[wave - 1][ch][1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w) {
        const float4 p0 = part_sum[w][ch][0], p1 = part_sum[w][ch][1];
        acc[0] += p0.x; acc[1] += p0.y; acc[2] += p0.z; acc[3] += p0.w;
        acc[4] += p1.x; acc[5] += p1.y; acc[6] += p1.z; acc[7] += p1.w;
    }
    float mu[8];
    float *cen = d.centroid + ((size_t)u * d.C + c) * kD + ch * 8;
    if (cnt > 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) mu[j] = acc[j] / (float)cnt;
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) mu[j] = cen[j];
    }
    uint32_t pk[4];
    float nn = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bf16_t b0 = f32_to_bf16(mu[2 * j]), b1 = f32_to_bf16(mu[2 * j + 1]);
        pk[j] = (uint32_t)b0 | ((uint32_t)b1 << 16);
        const float f0 = bf16_to_f32(b0), f1 = bf16_to_f32(b1);
        nn += f0 * f0 + f1 * f1;
    }
    nn = row16_sum(nn);
    bool moved = __ballot(was.x != pk[0] || was.y != pk[1] || was.z != pk[2] || was.w != pk[3]) != 0ull;  // (last: no matter)
    if (d.tk) {
        // the centroid's extra coordinate: mean of the members' extra coordinates (the fixed wave
        // reduction of the partial sums above)
        const float asum = wave_sum(aug_part);
        const float e = cnt > 0 ? asum / (float)cnt : d.cent_aug[(size_t)u * d.C + c];
        const bf16_t eb = f32_to_bf16(e);
        const float ef = bf16_to_f32(eb);
        if (lane == 0) {
            d.csum_aug[(size_t)u * d.C + c] = asum;
            d.cent_aug[(size_t)u * d.C + c] = e;
            d.caug[cur ^ 1][row] = eb;
        }
        moved |= d.caug[cur][row] != eb;
        nn += ef * ef;
    }
    moved |= __float_as_uint(was_norm) != __float_as_uint(nn);  // (a promoted key's is summed in another order)
    // (stored here and not where it is known: the first loads' wait would cover an earlier store)
    if (lane == 0) {
        d.cluster_cnt[(size_t)u * d.C + c] = cnt;
        d.moved[row] = (uint32_t)cnt << 1 | (moved ? 1u : 0u);
        if (moved) d.any_moved[2 * u + (round & 1)] = 1;
        d.touched[row] = 0;
    }
    if (g == 0) {
        float *sum = d.cluster_sum + ((size_t)u * d.C + c) * kD + ch * 8;
        ((float4 *)sum)[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        ((float4 *)sum)[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
        ((float4 *)cen)[0] = make_float4(mu[0], mu[1], mu[2], mu[3]);
        ((float4 *)cen)[1] = make_float4(mu[4], mu[5], mu[6], mu[7]);
        ((uint4 *)(d.cent_bf16[cur ^ 1] + ((size_t)u * d.Cpad + c) * kD))[ch] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        if (ch == 0) d.cnorm[cur ^ 1][(size_t)u * d.Cpad + c] = nn;
    }
}

void launch_means(const Dev &d, const bf16_t *K, int n, int cur, int t, bool last, hipStream_t st) {
    const int L = sort_len(d, n), R = (n + L - 1) / L;
#define ICE_MEANS(np)                                                                                                     \
    do {                                                                                                                  \
        if (keys_exceed_cache(d, n)) hipLaunchKernelGGL((means_kernel<true, np>), dim3(d.C, d.U), dim3(256), 0, st, d, K, n, cur, R, L, t, last ? 1 : 0); \
        else hipLaunchKernelGGL((means_kernel<false, np>), dim3(d.C, d.U), dim3(256), 0, st, d, K, n, cur, R, L, t, last ? 1 : 0); \
    } while (0)
    if (R == 1) ICE_MEANS(1);
    else if (R <= kFewPieces) ICE_MEANS(kFewPieces);
    else ICE_MEANS(0);
#undef ICE_MEANS
}

// ------------------------------------------------------------------------------------------------
// Node -> pages (Sec. 4.1): clusters in id order, members in ascending position, cut every s
// tokens; consecutive page ids.  One wave per page copies the s key rows and s value rows into
// the page's contiguous tiles, records their positions, and forms the representative: the fp32
// sum of the page's keys in slot order (one add per slot), divided by the fill, rounded to bf16.
//
// layout_kernel, one workgroup per unit, goes first: the exclusive scan of the clusters' page counts
// (`page_base`, n_pages, tails) and every page's cluster, found by a search over the scan in LDS.  With
// `arm` it also sets the unit's counters for the decode calls (a build; not a re-run of the stage).
__global__ __launch_bounds__(1024) void layout_kernel(Dev d, int n, int arm) {
    extern __shared__ int pb[];  // [C + 1]
    __shared__ int wsum[16];
    __shared__ int carry;
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, C = d.C;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int c0 = 0; c0 < C; c0 += 1024) {
        const int c = c0 + tid;
        const size_t cl = (size_t)u * C + c;
        const int cnt = c < C ? d.cluster_cnt[cl] : 0, pages = (cnt + d.s - 1) / d.s;
        int incl = wave_scan_add(pages);
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int ex = carry + incl - pages;
        for (int w = 0; w < wave; ++w) ex += wsum[w];
        if (c < C) {
            pb[c] = ex;
            d.page_base[cl] = ex;
            d.cluster_tail[cl] = cnt > 0 ? ex + pages - 1 : -1;
            if (cnt == 0) {  // (the state of the other clusters' tail pages follows with those pages)
                d.tail_fill[cl] = d.s;
                for (int x = 0; x < kD / 4; ++x) ((float4 *)(d.tail_sum + cl * kD))[x] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        __syncthreads();
        if (tid == 1023) carry = ex + pages;
        __syncthreads();
    }
    const int np = carry;
    if (tid == 0) {
        d.n_pages[u] = np;
        if (arm) { d.n_tokens[u] = n; d.counter[u] = 0; d.attn_arrive[u] = 0; }
    }
    for (int p = tid; p < d.max_pages; p += 1024) {
        int c = -1;
        if (p < np) {  // largest c with pb[c] <= p (clusters without pages are skipped)
            int lo = 0, hi = C;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (pb[mid] <= p) lo = mid; else hi = mid;
            }
            c = lo;
        }
        d.page_cluster[(size_t)u * d.max_pages + p] = c;
    }
}

template <bool STREAM>
__global__ __launch_bounds__(256) void paginate_kernel(Dev d, const bf16_t *__restrict__ K,
                                                        const bf16_t *__restrict__ V, int n, int R, int L, int arm) {
    extern __shared__ __align__(16) char smem[];  // [4][s][128] bf16
    const int u = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int p = blockIdx.x * 4 + wave;
    if (p >= d.max_pages) return;
    const int s = d.s;
    const size_t pg = (size_t)u * d.max_pages + p;
    const int c = d.page_cluster[pg];
    if (arm && lane == 0) d.scores[pg] = 0xFFFFFFFFu;  // (empty)
    if (c < 0) {  // unused page: clear its table entries
        if (lane == 0) d.page_fill[pg] = 0;
        for (int t = lane; t < s; t += 64) d.page_pos[pg * s + t] = -1;
        return;
    }
    const size_t cl = (size_t)u * d.C + c;
    const int r0 = (p - d.page_base[cl]) * s, cnt = d.cluster_cnt[cl], fill = min(s, cnt - r0);
    const Pieces pieces = {d.range_off + (size_t)u * R * d.Cpad + c, d.Cpad, R, L};
    const int at = pieces.search(r0, r0 + lane, lane);
    int mine = -1;  // slot `lane`'s token (s <= 64)
    if (lane < fill) mine = d.order[(size_t)u * d.max_tokens + at];
    const int g = lane >> 4, ch = lane & 15;
    bf16_t *tile = (bf16_t *)smem + (size_t)wave * s * kD;
    for (int t4 = 0; t4 < s; t4 += 4) {
        const int slot = t4 + g;
        const bool valid = slot < fill;
        const int tok = __shfl(mine, slot);
        uint4 kw = make_uint4(0, 0, 0, 0), vw = kw;
        if (valid) {
            kw = load16<STREAM>((const uint4 *)(K + ((size_t)u * n + tok) * kD) + ch);
            vw = load16<STREAM>((const uint4 *)(V + ((size_t)u * n + tok) * kD) + ch);
        }
        store16<STREAM>((uint4 *)(d.Kp + (pg * s + slot) * kD) + ch, kw);
        store16<STREAM>((uint4 *)(d.Vp + (pg * s + slot) * kD) + ch, vw);
        ((uint4 *)(tile + (size_t)slot * kD))[ch] = kw;
    }
    if (lane < s) d.page_pos[pg * s + lane] = mine;
    if (lane == 0) d.page_fill[pg] = fill;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the tile writes above are visible to the wave
    float a0 = 0.f, a1 = 0.f;
    for (int t = 0; t < fill; ++t) {
        const uint32_t w = ((const uint32_t *)(tile + (size_t)t * kD))[lane];
        a0 = a0 + bf16_lo(w);
        a1 = a1 + bf16_hi(w);
    }
    ((float2 *)(d.page_sum + pg * kD))[lane] = make_float2(a0, a1);
    const float f = (float)fill;
    ((uint32_t *)(d.rep + pg * kD))[lane] = (uint32_t)f32_to_bf16(a0 / f) | ((uint32_t)f32_to_bf16(a1 / f) << 16);
    if (r0 + fill == cnt) {  // the cluster's last page: what an insertion needs of it, beside the cluster
        ((float2 *)(d.tail_sum + cl * kD))[lane] = make_float2(a0, a1);
        if (lane == 0) d.tail_fill[cl] = fill;
    }
}

void launch_paginate(const Dev &d, const bf16_t *K, const bf16_t *V, int n, bool arm, hipStream_t st) {
    const int L = sort_len(d, n), R = (n + L - 1) / L;
    const size_t lds = (size_t)4 * d.s * kD * 2;
    hipLaunchKernelGGL(layout_kernel, dim3(d.U), dim3(1024), (size_t)(d.C + 1) * 4, st, d, n, arm ? 1 : 0);
#define ICE_PAGINATE(stream)                                                                                               \
    do {                                                                                                                   \
        hipLaunchKernelGGL(paginate_kernel<stream>, dim3((d.max_pages + 3) / 4, d.U), dim3(256), lds, st, d, K, V, n, R, L, arm ? 1 : 0); \
    } while (0)
    if (keys_exceed_cache(d, n)) ICE_PAGINATE(true);
    else ICE_PAGINATE(false);
#undef ICE_PAGINATE
}

// ------------------------------------------------------------------------------------------------
// The level above the clusters (Sec. 3.3: every point's parent is a point one level up).  A small
// Lloyd iteration over the unit's C bf16 centroids as points, one workgroup per unit:
//   promote  top node t starts at the centroid in the middle of the t-th of n_top equal strata of the
//            cluster ids;
//   assign   every cluster to the nearest top node: ||t~||^2 - 2 c . t~, fp32 accumulate on the matrix cores
//            (16 clusters x 16 nodes per v_mfma_f32_16x16x32_bf16 chain) against the nodes' bf16 rounding held
//            in LDS, lowest id on ties;
//   means    the clusters of a node are listed in ascending id (one wave per node walks the
//            assignment with lane masks) and summed in that order in fp32, four dimensions per thread;
//            an empty node keeps its position.
// The state left is the last assignment and the means of that assignment, as for the clusters.
// LDS: [n_top][128] bf16 rows, [n_top] norms, [n_top + 1] list starts, [C] assignment, [C] member list.
__global__ __launch_bounds__(1024) void top_level_kernel(Dev d, const bf16_t *__restrict__ cent, int n_top, int iters) {
    extern __shared__ __align__(16) char smem[];
    const int u = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int C = d.C;
    uint4 *rows = (uint4 *)smem;                                   // [n_top][16]
    float *norm = (float *)(smem + (size_t)n_top * 256);           // [n_top]
    int *start = (int *)(norm + n_top);                            // [n_top + 1]
    int *asg = start + n_top + 1;                                  // [C]
    int *members = asg + C;                                        // [C]
    const bf16_t *pts = cent + (size_t)u * d.Cpad * kD;            // the clusters' bf16 centroids: the points
    float *tc = d.top_cent + (size_t)u * kTopMax * kD;
    // promote
    for (int x = tid; x < n_top * 16; x += 1024) {
        const int t = x >> 4, ch = x & 15;
        const int c = (int)(((long long)(2 * t + 1) * C) / (2 * n_top));
        const uint4 w = ((const uint4 *)(pts + (size_t)c * kD))[ch];
        rows[x] = w;
        float *dst = tc + (size_t)t * kD + ch * 8;
        dst[0] = bf16_lo(w.x); dst[1] = bf16_hi(w.x); dst[2] = bf16_lo(w.y); dst[3] = bf16_hi(w.y);
        dst[4] = bf16_lo(w.z); dst[5] = bf16_hi(w.z); dst[6] = bf16_lo(w.w); dst[7] = bf16_hi(w.w);
        if (ch == 0) d.top_init[(size_t)u * kTopMax + t] = c;
    }
    __syncthreads();
    for (int it = 0; it < iters; ++it) {
        for (int t = tid; t < n_top; t += 1024) {
            float nn = 0.f;
            for (int ch = 0; ch < 16; ++ch) {
                const uint4 w = rows[t * 16 + ch];
                nn += bf16_lo(w.x) * bf16_lo(w.x) + bf16_hi(w.x) * bf16_hi(w.x) + bf16_lo(w.y) * bf16_lo(w.y) + bf16_hi(w.y) * bf16_hi(w.y) +
                      bf16_lo(w.z) * bf16_lo(w.z) + bf16_hi(w.z) * bf16_hi(w.z) + bf16_lo(w.w) * bf16_lo(w.w) + bf16_hi(w.w) * bf16_hi(w.w);
            }
            norm[t] = nn;
        }
        __syncthreads();
        // assign on the matrix cores: a wave takes 16 clusters at a time as the columns of the B operand (lane
        // (g, n): dims [32 ks + 8 g, +8) of cluster n) and walks the nodes 16 at a time as the rows of A, read from
        // LDS; lane (g, n) ends with nodes 4g .. 4g+3 of the tile against cluster n and keeps the best, lowest node
        // id on ties; the four row groups meet by lane exchange
        {
            const int g = lane >> 4, i16 = lane & 15;
            const int ptiles = (C + 15) >> 4, ntiles = (n_top + 15) >> 4;
            auto cluster_rows = [&](int pt, uint4 (&b)[4]) {
                const int c = pt * 16 + i16;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    b[ks] = make_uint4(0, 0, 0, 0);
                    if (c < C) b[ks] = ((const uint4 *)(pts + (size_t)c * kD))[ks * 4 + g];
                }
            };
            uint4 b[4], bn[4];
            if (wave < ptiles) cluster_rows(wave, b);
            for (int pt = wave; pt < ptiles; pt += 16) {
                const int c = pt * 16 + i16;
                if (pt + 16 < ptiles) cluster_rows(pt + 16, bn);  // (the next tile's rows are on their way during this one)
                u64 best = ~0ull;
                for (int nt = 0; nt < ntiles; ++nt) {
                    const int node_a = nt * 16 + i16;
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        uint4 a = make_uint4(0, 0, 0, 0);
                        if (node_a < n_top) a = rows[node_a * 16 + ks * 4 + g];
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b[ks]), acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int node = nt * 16 + 4 * g + j;
                        const float val = __builtin_fmaf(-2.0f, acc[j], node < n_top ? norm[node] : INFINITY);
                        if (node < n_top && !(val != val)) {
                            const u64 key = ((u64)f32_ordered(val) << 32) | (u64)(uint32_t)node;
                            best = key < best ? key : best;
                        }
                    }
                }
                u64 o = __shfl_xor(best, 16);
                best = o < best ? o : best;
                o = __shfl_xor(best, 32);
                best = o < best ? o : best;
                if (g == 0 && c < C) {
                    const int bi = best == ~0ull ? 0 : (int)(uint32_t)best;
                    asg[c] = bi;
                    d.top_of[(size_t)u * C + c] = bi;
                }
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) b[ks] = bn[ks];
            }
        }
        __syncthreads();
        // list the clusters of every node in ascending id: counts, starts, then placement
        for (int t = wave; t < n_top; t += 16) {
            int cnt = 0;
            for (int c0 = 0; c0 < C; c0 += 64) cnt += (int)__popcll(__ballot(c0 + lane < C && asg[c0 + lane] == t));
            if (lane == 0) start[t + 1] = cnt;
        }
        __syncthreads();
        if (tid == 0) {
            start[0] = 0;
            for (int t = 0; t < n_top; ++t) start[t + 1] += start[t];
        }
        __syncthreads();
        for (int t = wave; t < n_top; t += 16) {
            int base = start[t];
            for (int c0 = 0; c0 < C; c0 += 64) {
                const bool is = c0 + lane < C && asg[c0 + lane] == t;
                const u64 bal = __ballot(is);
                if (is) members[base + (int)__popcll(bal & ((1ull << lane) - 1ull))] = c0 + lane;
                base += (int)__popcll(bal);
            }
        }
        __syncthreads();
        // means: (node, four dimensions) per thread, members in list order
        for (int x = tid; x < n_top * 32; x += 1024) {
            const int t = x >> 5, qd = x & 31;
            const int lo = start[t], cnt = start[t + 1] - lo;
            float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
            constexpr int MB = 32;  // rows requested at once (the sum itself stays in list order)
            for (int i0 = 0; i0 < cnt; i0 += MB) {
                uint2 w[MB];
#pragma unroll
                for (int x = 0; x < MB; ++x) {
                    w[x] = make_uint2(0u, 0u);
                    if (i0 + x < cnt) w[x] = ((const uint2 *)(pts + (size_t)members[lo + i0 + x] * kD))[qd];
                }
#pragma unroll
                for (int x = 0; x < MB; ++x)
                    if (i0 + x < cnt) { a0 += bf16_lo(w[x].x); a1 += bf16_hi(w[x].x); a2 += bf16_lo(w[x].y); a3 += bf16_hi(w[x].y); }
            }
            float *dst = tc + (size_t)t * kD + qd * 4;
            if (cnt > 0) {
                const float f = (float)cnt;
                a0 /= f; a1 /= f; a2 /= f; a3 /= f;
                dst[0] = a0; dst[1] = a1; dst[2] = a2; dst[3] = a3;
            } else {
                a0 = dst[0]; a1 = dst[1]; a2 = dst[2]; a3 = dst[3];
            }
            ((uint2 *)rows)[t * 32 + qd] = make_uint2((uint32_t)f32_to_bf16(a0) | ((uint32_t)f32_to_bf16(a1) << 16),
                                                      (uint32_t)f32_to_bf16(a2) | ((uint32_t)f32_to_bf16(a3) << 16));
            if (qd == 0) d.top_cnt[(size_t)u * kTopMax + t] = cnt;
        }
        __syncthreads();
    }
    // the nodes' bf16 rows for the search (rows from n_top on: zero)
    uint4 *dst = (uint4 *)(d.top_bf16 + (size_t)u * kTopMax * kD);
    for (int x = tid; x < kTopMax * 16; x += 1024) dst[x] = x < n_top * 16 ? rows[x] : make_uint4(0, 0, 0, 0);
}

void launch_top_level(const Dev &d, int cur, int n_top, int iters, hipStream_t st) {
    const size_t lds = (size_t)n_top * 256 + (size_t)(2 * n_top + 1) * 4 + (size_t)d.C * 8;
    allow_dynamic_lds((const void *)top_level_kernel, lds);
    hipLaunchKernelGGL(top_level_kernel, dim3(d.U), dim3(1024), lds, st, d, d.cent_bf16[cur], n_top, iters);
}

}  // namespace ice

ICE_PROF_EXPORT(ice_debug_prof_build)
