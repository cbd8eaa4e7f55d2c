// Device code shared by the decode-step kernels (flat and hierarchical page selection): vector
// types, packed-bf16 dot products, the query operand of the scoring / logit MFMAs, and sparse
// paged attention over a list of pages.
#pragma once
#include "ice_internal.h"

namespace ice {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short bf16x4s __attribute__((ext_vector_type(4)));  // operand type of the 16x16x16 bf16 MFMA builtin
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned long long u64;

// a.lo*b.lo + a.hi*b.hi + c on packed bf16 pairs, fp32 accumulate (v_dot2_f32_bf16)
__device__ inline float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
__device__ inline float dot8(const uint4 &a, const uint4 &b) {
    return dot2(a.w, b.w, dot2(a.z, b.z, dot2(a.y, b.y, dot2(a.x, b.x, 0.f))));
}

// The places of the n winners (composites with ~id in the low word, LDS) in ascending id order: put(place, winner) on one lane
// each, by waves `part` of `parts`.  A wave keeps up to kPlaceBlocks * 64 winners' ids on its lanes and takes winners part,
// part + parts, ...: one comparison and one count of its lane mask per 64 ids.  Longer lists by one thread per winner that
// reads them all from LDS.  8 units x 32768 tokens, a whole step, us, so, by one thread per winner, and with the blocks read from LDS
// for every winner: 128 pages 23.2, 29.3, 24.8; 256 23.7, 26.3, 30.2; 300 26.7, 27.8, 34.1; 1000 50.4, 51.5, 143 (in the second
// column other parts of the step were slower too).
constexpr int kPlaceBlocks = 4;
template <int NB, typename Put>
__device__ inline void place_by_id_blocks(const u64 *win, int n, int part, int parts, int lane, Put put) {
    uint32_t lo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) lo[b] = 64 * b + lane < n ? (uint32_t)win[64 * b + lane] : 0u;  // (no id is as high as ~0)
    for (int t0 = part; t0 < n; t0 += 64 * parts) {  // (64 of the wave's winners at a time, one per lane)
        const u64 w = win[min(t0 + lane * parts, n - 1)];
        int place = 0;
        const int cnt = min(64, (n - t0 + parts - 1) / parts);
        for (int x = 0; x < cnt; ++x) {
            const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, x);
            int pos = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) pos += (int)__popcll(__ballot(lo[b] > mine));
            place = lane == x ? pos : place;
        }
        if (lane < cnt) put(place, w);
    }
}
template <typename Put>
__device__ inline void place_by_id(const u64 *win, int n, int part, int parts, int lane, Put put) {
    if (__builtin_expect(n <= 64, 1)) {  // (all of them side by side on the lanes: one trip to LDS)
        const u64 w = win[min(lane, max(n - 1, 0))];
        const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
        for (int t = part; t < n; t += parts) {  // (t is the same for the whole wave)
            const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)lo, t), score = (uint32_t)__builtin_amdgcn_readlane((int)hi, t);
            const int pos = (int)__popcll(__ballot(lane < n && lo > mine));
            if (lane == 0) put(pos, ((u64)score << 32) | mine);
        }
    } else if (__builtin_expect(n <= 64 * kPlaceBlocks, 1)) {
        place_by_id_blocks<kPlaceBlocks>(win, n, part, parts, lane, put);
    } else {
        for (int t = part * 64 + lane; t < n; t += parts * 64) {
            const u64 mine = win[t];
            int pos = 0;
            for (int j = 0; j < n; ++j) pos += (uint32_t)win[j] > (uint32_t)mine ? 1 : 0;
            put(pos, mine);
        }
    }
}

// The `need` best of n <= kRankMax distinct 64-bit composites (LDS), best first, into sel[0 .. need), by the NW waves of a
// workgroup (a barrier in front and behind is the caller's).  Bound by vector instructions (four waves to a SIMD) and the trips to
// LDS.  rank_blocks: every wave holds all of them on its lanes and counts, for each of its share, those above it with a lane
// mask.  rank_lanes: up to 64 lanes to a composite walk a part of the list each; it is the flat step's with eight waves, two such
// workgroups to a CU.  (16 waves: 84 of 512 0.8 and 2.3 us, the step of 8 units x 2300 pages, about 25 listed, 11.89 and 12.07.  Eight
// waves, of which a wave's share is twice as long: 312 units x 460 pages 35.3 and 34.9, 368 pages of 32 tokens 28.9 and 28.6; where there is one
// such workgroup to a CU no difference but with long lists: 8 units x 2300 pages, 16 kept, 12.6 and 12.6, 64 kept 19.3 and 19.0, 32 x 2300,
// 32 kept, 19.2 and 19.1, 128 x 1150 23.6 and 23.6, 256 x 2300 33.5 and 33.4, 2 x 300 10.6 and 10.6.)
constexpr int kRankMax = 512;
template <int NW>
__device__ inline void rank_lanes(const u64 *cand, int n, int need, int tid, u64 *sel) {
    constexpr int NT = NW * 64;
    static_assert(kRankMax <= NT, "a lane to a composite at least");
    int lp = 0;
    while (lp < 6 && (n << (lp + 1)) <= NT) ++lp;
    const int parts = 1 << lp, i = tid >> lp, part = tid & (parts - 1), len = (n + parts - 1) >> lp;
    const u64 mine = i < n ? cand[i] : ~0ull;
    int rank = 0;
#pragma unroll 4
    for (int j = part * len; j < min(n, (part + 1) * len); ++j) rank += cand[j] > mine;
    // sum over the `parts` lanes of a candidate: DPP inside a 16-lane row, shuffles beyond
    if (parts >= 2) rank += (int)dpp_u32<0xB1>((uint32_t)rank);
    if (parts >= 4) rank += (int)dpp_u32<0x4E>((uint32_t)rank);
    if (parts >= 8) rank += (int)dpp_u32<0x141>((uint32_t)rank);
    if (parts >= 16) rank += (int)dpp_u32<0x140>((uint32_t)rank);
    if (parts >= 32) rank += __shfl_xor(rank, 16);
    if (parts >= 64) rank += __shfl_xor(rank, 32);
    if (part == 0 && i < n && rank < need) sel[rank] = mine;
}
template <int NB, int NW>
__device__ inline void rank_blocks(const u64 *cand, int n, int need, int wave, int lane, u64 *sel) {
    u64 c[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) c[b] = 64 * b + lane < n ? cand[64 * b + lane] : 0ull;
    const u64 own = cand[min(wave + lane * NW, n - 1)];  // this wave's: wave, wave + NW, ... (at most 64: n <= 64 NW)
    const int cnt = (n - wave + NW - 1) / NW;
    int rank = 0;
    for (int x = 0; x < cnt; ++x) {
        const u64 mine = (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(own >> 32), x) << 32 |
                         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)own, x);
        int r = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) r += (int)__popcll(__ballot(c[b] > mine));
        rank = lane == x ? r : rank;
    }
    if (lane < cnt && rank < need) sel[rank] = own;
}
template <int NW>
__device__ inline void rank_composites(const u64 *cand, int n, int need, int wave, int lane, u64 *sel) {
    static_assert(kRankMax <= 64 * NW, "a wave's share on its lanes");
    if (n <= 64) rank_blocks<1, NW>(cand, n, need, wave, lane, sel);
    else if (n <= 128) rank_blocks<2, NW>(cand, n, need, wave, lane, sel);
    else if (n <= 256) rank_blocks<4, NW>(cand, n, need, wave, lane, sel);
    else rank_blocks<kRankMax / 64, NW>(cand, n, need, wave, lane, sel);
}

// The set bits of a mask of `words` 32-bit words (LDS) in ascending order, by one wave: out[0], out[1], ...
__device__ inline void list_bits(const uint32_t *mask, int words, int lane, int *out) {
    int before = 0;
    for (int w0 = 0; w0 < words; w0 += 64) {
        uint32_t w = w0 + lane < words ? mask[w0 + lane] : 0u;
        const int cnt = __popc(w), incl = wave_scan_add(cnt);
        int pos = before + incl - cnt;
        for (; w; w &= w - 1) out[pos++] = 32 * (w0 + lane) + __ffs(w) - 1;
        before += __builtin_amdgcn_readlane(incl, 63);
    }
}

// Sparse paged attention over a list of pages (Eq. 1 with the mask set on the tokens of the listed
// pages), for one unit, by the NW waves of the calling workgroup.  Wave w streams pages w, w+NW, ...;
// a page's key tile and value tile are each s x 256 contiguous bytes.  Per 16-token block:
//   logits   one v_mfma_f32_16x16x32_bf16 chain, A = the G query rows, B = the 16 key rows (lane
//            (g, r) reads bytes [64*ks + 16*g, +16) of key row r).  Head h sits in row 4 (h % 4) + h / 4 of A, so lane (g, r)
//            gets the logits of token r for heads g and g + 4: with the heads in rows 0, 1, ... one row group of lanes
//            held up to four heads and the others none, i.e. four times the vector instructions of the softmax, and
//            16 waves of a CU share four vector units (8 units x 16 pages, from the tiles' request to the last wave's sums:
//            2.95 us then, 2.5 now; 32 x 512 rows by position 8.9 and 8.4);
//   softmax  running maximum and denominator per head, shared by the whole wave (DPP row maxima),
//            fp32; the 16 x G weights cross to the matrix-operand layout via LDS;
//   values   also on the matrix cores: out[head][dim] += sum_token p[head][token] v[token][dim] as
//            v_mfma_f32_16x16x16_bf16 with A = the weights, split into two bf16 terms (p = hi + lo,
//            relative error 2^-16, so the fp32 softmax survives), and B = the value rows.  Lane
//            (g, c) loads value rows 4t+g, 16 bytes each (1 KiB per load instruction): it holds
//            tokens {g, 4+g, 8+g, 12+g} x dims 8c..8c+7, which is exactly the B operand of eight
//            column tiles if tile j is made of dims {8c + j} and contraction slot 4g+i stands for
//            token 4i+g (a permutation of the sum); two byte-permutes per tile pack it.
// The NW waves are merged by the (max, sum, output) rule.  page_of(x) names the x-th listed page
// (x differs by lane); `red` is LDS scratch of attend_scratch_floats() floats; aside(part, parts) is work of the
// caller that needs no barrier: the waves that the output leaves idle do it beside the others, each its part.  (In front of the last
// barrier, or while the first tiles are on their way, it was 0.3 us longer for 16 winners.)
__host__ __device__ constexpr int attend_scratch_floats(int G, int NW) { return NW * (G * (kD + 2) + 16 * 8); }

// the head in row r of the attention's query operand, -1: a zero row
template <int G>
__device__ inline int operand_head(int r) {
    const int hg = r >> 2, v = r & 3;
    return v < (G + 3) / 4 && hg < (G < 4 ? G : 4) ? hg + 4 * v : -1;
}
template <int G>
__device__ inline void load_query_operand(const bf16_t *q, int u, int lane, bf16x8 (&qa)[4], float *sumsq) {
    const int g = lane >> 4, h = operand_head<G>(lane & 15);
    float nn = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const uint4 w = h >= 0 ? ((const uint4 *)(q + ((size_t)u * G + h) * kD))[ks * 4 + g] : make_uint4(0, 0, 0, 0);
        qa[ks] = __builtin_bit_cast(bf16x8, w);
        nn += dot8(w, w);
    }
    if (sumsq) *sumsq = nn;
}

// Split-row form of the scoring contraction.  In the plain form lane (g, c) of a B operand reads
// 16 bytes of row c at 64*ks + 16*g, so one load instruction touches half a 128-byte line of each of
// 16 rows.  Here a load instruction covers whole lines: lanes c and c+8 read the two 64-byte halves
// of a line of row c%8, i.e. column c < 8 of the B operand carries dims [64t, 64t+32) of the row and
// column c+8 dims [64t+32, 64t+64) (t = 0, 1: two MFMAs per 8 rows, as many as before per byte).
// The A operand holds every query row twice: row h with the dims of the lower halves, row G+h with
// those of the upper halves (load_query).  Output (row h, column c < 8) and (row G+h, column c+8) are then the
// two halves of q_h . row_c; the other outputs are discarded.  A pair of 8-row blocks shares one
// exchange: lanes c < 8 keep the first block, lanes c >= 8 the second, each sends the partner
// (lane xor kXor) the half it does not keep, and lane (.., c) ends with the scores of row c of the
// 16 for its heads.
template <int G>
struct SplitRow {
    static_assert(G == 1 || G == 2 || G == 4 || G == 8, "2G query rows must fit the 16 operand rows");
    static constexpr int kDG = G >= 4 ? G / 4 : 0;  // 16-lane row groups between row h and row G+h
    static constexpr int kDV = G >= 4 ? 0 : G;      // accumulator slots between them
    static constexpr int kXor = 8 + 16 * kDG;
    static constexpr int kHV = G < 4 ? G : 4;       // heads per lane

    // The A operand straight from memory: lane (g, c) holds q_c dims [64t + 8g, +8) for c < G and
    // q_{c-G} dims [64t + 32 + 8g, +8) for G <= c < 2G (t = 0, 1), zeros from row 2G on.  *inv_norm =
    // 1 / max(||q_h||, 1e-20) on the lanes with c = h and c = G + h.
    __device__ static void request_query(const bf16_t *q, int u, int lane, uint4 (&w)[2]) {
        const int g = lane >> 4, c = lane & 15;
        const int upper = c >= G ? 1 : 0, h = c - G * upper;
        const uint4 *row = (const uint4 *)(q + ((size_t)u * G + h) * kD);
#pragma unroll
        for (int t = 0; t < 2; ++t) w[t] = c < 2 * G ? row[8 * t + 4 * upper + g] : make_uint4(0, 0, 0, 0);
    }
    __device__ static void take_query(const uint4 (&w)[2], bf16x8 (&qs)[2], float *inv_norm) {
        float nn = 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            qs[t] = __builtin_bit_cast(bf16x8, w[t]);
            nn += dot8(w[t], w[t]);
        }
        nn += __shfl_xor(nn, 16);
        nn += __shfl_xor(nn, 32);
        nn += __shfl_xor(nn, G);  // the other half of the row
        *inv_norm = 1.0f / fmaxf(sqrtf(nn), 1e-20f);
    }
    __device__ static void load_query(const bf16_t *q, int u, int lane, bf16x8 (&qs)[2], float *inv_norm) {
        uint4 w[2];
        request_query(q, u, lane, w);
        take_query(w, qs, inv_norm);
    }
    // The operand of the logit MFMAs (lane (g, r): dims [32ks + 8g, +8) of the head in row r, zeros where there is none) out of
    // the split one, by lane exchange: no second trip to memory for the query rows.
    __device__ static void to_plain(const bf16x8 (&qs)[2], int lane, bf16x8 (&qa)[4]) {
        const int h = operand_head<G>(lane & 15);
        const uint4 zero = make_uint4(0, 0, 0, 0);
        const int src = (lane & 48) + max(h, 0);  // row h holds the lower halves of q_h, row G + h the upper ones
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint4 w = __builtin_bit_cast(uint4, qs[t]);
            uint4 lo, up;
            lo.x = __shfl(w.x, src);
            lo.y = __shfl(w.y, src);
            lo.z = __shfl(w.z, src);
            lo.w = __shfl(w.w, src);
            up.x = __shfl(w.x, src + G);
            up.y = __shfl(w.y, src + G);
            up.z = __shfl(w.z, src + G);
            up.w = __shfl(w.w, src + G);
            qa[2 * t] = __builtin_bit_cast(bf16x8, h >= 0 ? lo : zero);
            qa[2 * t + 1] = __builtin_bit_cast(bf16x8, h >= 0 ? up : zero);
        }
    }
    // uint4 index inside a 16-row block (rows of 16 uint4) of the load that feeds MFMA t of 8-row
    // block blk
    __device__ static int word(int lane, int blk, int t) {
        const int g = lane >> 4, c = lane & 15;
        return (8 * blk + (c & 7)) * 16 + 8 * t + 4 * (c >> 3) + g;
    }
    // lanes whose result is a row's score: row c of the 16, heads 4 * head_group(lane) + v
    __device__ static bool owner(int lane) { return (lane >> 4) == ((lane & 8) ? kDG : 0); }
    __device__ static int head_group(int lane) { return (lane >> 4) - ((lane & 8) ? kDG : 0); }
    // max over the group's heads of (q_h . row) * inv[v]; acc0 / acc1 = accumulators of the two blocks
    __device__ static float score(const f32x4 &acc0, const f32x4 &acc1, const float (&inv)[4], int lane) {
        const bool hi = (lane & 8) != 0;
        float sc = -INFINITY;
#pragma unroll
        for (int v = 0; v < kHV; ++v) {
            const float a0 = (kDV && hi) ? acc0[(v + kDV) & 3] : acc0[v];
            const float a1 = (kDV && hi) ? acc1[(v + kDV) & 3] : acc1[v];
            const float tot = (hi ? a1 : a0) + __shfl_xor(hi ? a0 : a1, kXor);
            sc = fmaxf(sc, tot * inv[v]);
        }
        if (G > 4) sc = fmaxf(sc, __shfl_xor(sc, 16));
        return sc;
    }
};

// With PARTIAL the workgroup attends to a share of a unit's pages and leaves, instead of the output,
// what a later merge needs: per head h the unnormalised sum at out[h * (kD + 2) + j], the running
// maximum at [.. + kD] and the denominator at [.. + kD + 1] (`out` then points at the workgroup's own
// block and `u` only addresses the pages).
// RES: what is attended besides the pages (kNoRows, kDenseRows, kGatheredRows: see Resident).
// FILLS: the pages' fills are fetched ahead of all but the wave's first page (one lane per page), so that rows past
// a page's fill are not read: worth it where the bytes count (many units with several pages per wave, a window
// beside the pages), not where a few units wait for one or two round trips (attend_by_fills).
template <int G, int NW, int RES, bool PARTIAL, bool FILLS, typename PageOf, typename Aside>
__device__ inline void attend_pages(const Dev &d, int u, const bf16x8 (&qa)[4], PageOf page_of, int ns, Resident res,
                                    float *__restrict__ out, float *red, Aside aside) {
    constexpr int HV = (G + 3) / 4;  // heads per lane: g + 4 v, v < HV, on lanes (g, .) with g < G
    float(*wacc)[G][kD] = (float(*)[G][kD])red;                   // [NW][G][128]
    float(*wm)[G] = (float(*)[G])(red + NW * G * kD);             // [NW][G]
    float(*wl)[G] = (float(*)[G])(red + NW * G * (kD + 1));       // [NW][G]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane >> 4, ch = lane & 15;
    float *px = red + NW * G * (kD + 2) + wave * (16 * 8);        // [16 tokens][8 heads] weights of this wave
    const float scale = 0.08838834764831845f;  // 1/sqrt(128)
    const int s = d.s;
    // lane (g, r): m, l of heads g + 4 v (wave-wide maxima, own-token denominators);
    // acc[j][v] = output of head g + 4 v, dim 8r+j
    float m[HV], l[HV];
    f32x4 acc[8];
#pragma unroll
    for (int v = 0; v < HV; ++v) { m[v] = -INFINITY; l[v] = 0.f; }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bool first = true;
    // one 16-token block whose key pieces (kb) and value rows (vt) are in registers, its first nv tokens
    // (nv >= 1) taking part; next_keys() / next_values() request the next block into kb / vt
    uint4 kb[4], vt[4];
    auto block = [&](int nv, auto next_keys, auto next_values) __attribute__((always_inline)) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ks], __builtin_bit_cast(bf16x8, kb[ks]), z, 0, 0, 0);
        next_keys();
        const bool tok_ok = ch < nv;  // this lane's logits belong to token ch of the block
        float pw[HV], alpha[HV];
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            const float zz = tok_ok ? z[v] * scale : -INFINITY;
            float mx = zz;
            mx = fmaxf(mx, dpp_f32<0xB1>(mx));
            mx = fmaxf(mx, dpp_f32<0x4E>(mx));
            mx = fmaxf(mx, dpp_f32<0x141>(mx));
            mx = fmaxf(mx, dpp_f32<0x140>(mx));   // block maximum of head g + 4 v on all 16 lanes of the row
            const float mn = fmaxf(m[v], mx);     // finite: every block has at least one token
            alpha[v] = __expf(m[v] - mn);
            pw[v] = __expf(zz - mn);
            l[v] = l[v] * alpha[v] + pw[v];
            m[v] = mn;
        }
        if (g < G) {  // (head g + 4 v in slot HV g + v)
            if constexpr (HV == 2) *(float2 *)(px + ch * 8 + 2 * g) = make_float2(pw[0], pw[1]);
            else px[ch * 8 + g] = pw[0];
        }
        __builtin_amdgcn_wave_barrier();
        // A operand: lane (g, r) holds p[head in row r][token 4i+g], i = 0..3, as hi + lo bf16 terms
        float pa[4];
        const bool row_used = operand_head<G>(ch) >= 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float t = px[(4 * i + g) * 8 + HV * (ch >> 2) + (ch & (HV - 1))];  // (unconditional read, then select: no branch)
            pa[i] = row_used ? t : 0.f;
        }
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[i] = __float_as_uint(pa[i]) & 0xFFFF0000u;
            lo[i] = __float_as_uint(pa[i] - __uint_as_float(hi[i]));
        }
        const v2u ahi = {__builtin_amdgcn_perm(hi[1], hi[0], 0x07060302u), __builtin_amdgcn_perm(hi[3], hi[2], 0x07060302u)};
        const v2u alo = {__builtin_amdgcn_perm(lo[1], lo[0], 0x07060302u), __builtin_amdgcn_perm(lo[3], lo[2], 0x07060302u)};
        if (!first) {  // rescale what earlier blocks left (same lanes hold the factors)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int v = 0; v < HV; ++v) acc[j][v] *= alpha[v];
        }
        first = false;
        if (nv < 16) {  // a partly filled block: rows past the end must not reach the matrix core
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * t + g >= nv) vt[t] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // column tile j: dims {8c + j}; contraction slot 4g+i = token 4i+g
            const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
            const uint32_t w0 = j < 2 ? vt[0].x : j < 4 ? vt[0].y : j < 6 ? vt[0].z : vt[0].w;
            const uint32_t w1 = j < 2 ? vt[1].x : j < 4 ? vt[1].y : j < 6 ? vt[1].z : vt[1].w;
            const uint32_t w2 = j < 2 ? vt[2].x : j < 4 ? vt[2].y : j < 6 ? vt[2].z : vt[2].w;
            const uint32_t w3 = j < 2 ? vt[3].x : j < 4 ? vt[3].y : j < 6 ? vt[3].z : vt[3].w;
            const v2u bv = {__builtin_amdgcn_perm(w1, w0, sel), __builtin_amdgcn_perm(w3, w2, sel)};
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4s, ahi), __builtin_bit_cast(bf16x4s, bv), acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4s, alo), __builtin_bit_cast(bf16x4s, bv), acc[j], 0, 0, 0);
        }
        next_values();
        __builtin_amdgcn_wave_barrier();  // the next block overwrites px
    };
    // a block of contiguous rows: rows from nv on are not read (row nv - 1 stands in for them)
    auto load_keys = [&](const uint4 *rows, int nv) {
        const uint4 *src = rows + min(ch, nv - 1) * 16 + g;
#pragma unroll
        for (int t = 0; t < 4; ++t) kb[t] = src[4 * t];
    };
    auto load_values = [&](const uint4 *rows, int nv) {
#pragma unroll
        for (int t = 0; t < 4; ++t) vt[t] = (rows + min(4 * t + g, nv - 1) * 16)[ch];
    };
    // this wave's resident blocks: rj, rj + NW, ... below rend, dealt where the pages leave off
    int rj = 0, rend = 0, nres = 0;
    if constexpr (RES != kNoRows) {
        nres = RES == kGatheredRows ? max(0, min(res.cnt[u], res.n)) : res.n;
        rj = res.b0 + ((wave - ns) % NW + NW) % NW;
        rend = min(res.b1, (nres + 15) >> 4);
    }
    if constexpr (RES == kNoRows && !FILLS) {
        // the first 16-token block of a page is fetched before its fill count is known (one fewer
        // dependent round trip); slots >= fill may hold stale bytes and are masked after the load
        for (int x = tid >> 6; x < ns; x += NW) {
            const int p = page_of(x);
            if ((unsigned)p >= (unsigned)d.max_pages) continue;  // not a page id: ignored
            const size_t pg = (size_t)u * d.max_pages + p;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                kb[t] = ((const uint4 *)(d.Kp + (pg * s + ch) * kD))[t * 4 + g];
                vt[t] = ((const uint4 *)(d.Vp + (pg * s + 4 * t + g) * kD))[ch];
            }
            const int fill = d.page_fill[pg];
            ICE_STAMP(8);
            for (int b0 = 0; b0 < fill; b0 += 16) {
                if (b0 > 0) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        kb[t] = ((const uint4 *)(d.Kp + (pg * s + b0 + ch) * kD))[t * 4 + g];
                        vt[t] = ((const uint4 *)(d.Vp + (pg * s + b0 + 4 * t + g) * kD))[ch];
                    }
                }
                block(fill - b0, [] {}, [] {});
            }
        }
    } else if constexpr (RES != kGatheredRows) {
        // Contiguous blocks: the pages' (16 tokens at a time), then the dense run's.  Everything that says
        // which block comes next is the same for the whole wave.  The wave's pages are taken 64 at a time,
        // one per lane (id, fill); `live` = those still to come that hold tokens.
        int x0 = wave, id = -1, fl = 0, i = 0, b0 = 0, fill = 0;
        u64 live = 0ull;
        const uint4 *nk = nullptr, *nval = nullptr;  // the block requested next: key rows, value rows, tokens from there on
        int nnv = 0;
        auto tile = [&](int page, int from, int nv) {
            const size_t row = ((size_t)u * d.max_pages + page) * s + from;
            nk = (const uint4 *)(d.Kp + row * kD);
            nval = (const uint4 *)(d.Vp + row * kD);
            nnv = nv;
        };
        auto refill = [&] {
            const int xl = x0 + lane * NW;
            id = -1;
            fl = 0;
            if (xl < ns) id = page_of(xl);
            if ((unsigned)id < (unsigned)d.max_pages) fl = d.page_fill[(size_t)u * d.max_pages + id];  // (not a page id: ignored)
            live = __ballot(fl > 0);
        };
        auto next = [&]() -> bool {
            if (b0 + 16 < fill) {  // this page goes on
                b0 += 16;
                tile(__builtin_amdgcn_readlane(id, i), b0, fill - b0);
                return true;
            }
            b0 = fill = 0;
            while (live == 0ull && x0 + 64 * NW < ns) {
                x0 += 64 * NW;
                refill();
            }
            if (live != 0ull) {
                i = (int)__builtin_ctzll(live);
                live &= live - 1ull;
                fill = __builtin_amdgcn_readlane(fl, i);
                tile(__builtin_amdgcn_readlane(id, i), 0, fill);
                return true;
            }
            if constexpr (RES == kDenseRows) {
                if (rj < rend) {
                    const size_t row = (size_t)u * res.n + 16 * rj;
                    nk = (const uint4 *)(res.k + row * kD);
                    nval = (const uint4 *)(res.v + row * kD);
                    nnv = nres - 16 * rj;
                    rj += NW;
                    return true;
                }
            }
            return false;
        };
        // The first page's first block is requested before anything else, its fill included (all 16 slots are
        // there to be read, slots past the fill are masked); the ids and fills of the others follow.
        if (x0 < ns) {
            id = __builtin_amdgcn_readfirstlane(page_of(x0));
            if ((unsigned)id < (unsigned)d.max_pages) {
                tile(id, 0, 16);
                load_keys(nk, 16);
                load_values(nval, 16);
                fl = d.page_fill[(size_t)u * d.max_pages + id];
            }
            ICE_STAMP(8);
            if (x0 + NW < ns) refill();
            fill = __builtin_amdgcn_readfirstlane(fl);
            live &= ~1ull;
        }
        int nv = fill;
        bool have = fill > 0;
        if (!have && next()) {  // (no page, or an empty one, at the head of the list)
            have = true;
            nv = nnv;
            load_keys(nk, nv);
            load_values(nval, nv);
        }
        while (have) {
            if constexpr (RES == kDenseRows) {
                // the next block's keys are requested as soon as the logits have consumed this one's, its values behind
                // this block's value contraction
                have = next();
                block(nv, [&] { if (have) load_keys(nk, nnv); }, [&] { if (have) load_values(nval, nnv); });
            } else {
                block(nv, [] {}, [] {});
                have = next();
                if (have) {
                    load_keys(nk, nnv);
                    load_values(nval, nnv);
                }
            }
            nv = nnv;
        }
    }
    if constexpr (RES == kGatheredRows) {
        // Gathered rows: a block's 16 positions sit on lanes ch, the next block's are fetched while this one is
        // worked on.  List entries past the unit's count are read (the list has res.n of them) and not used.
        const int *pl = res.pos + (size_t)u * res.n;
        const uint4 *kbase = (const uint4 *)(res.k + (size_t)u * res.rows * kD), *vbase = (const uint4 *)(res.v + (size_t)u * res.rows * kD);
        auto position = [&](int j) { return min(max(pl[min(16 * j + ch, res.n - 1)], 0), res.rows - 1); };
        auto gather_keys = [&](int row) {
            const uint4 *src = kbase + (size_t)row * 16 + g;
#pragma unroll
            for (int t = 0; t < 4; ++t) kb[t] = src[4 * t];
        };
        auto gather_values = [&](int row) {
#pragma unroll
            for (int t = 0; t < 4; ++t) vt[t] = (vbase + (size_t)__shfl(row, 4 * t + g) * 16)[ch];
        };
        if (rj < rend) {
            int row = position(rj);
            gather_keys(row);
            gather_values(row);
            int row1 = position(rj + NW);
            for (; rj + NW < rend; rj += NW) {
                row = row1;
                row1 = position(rj + 2 * NW);
                block(nres - 16 * rj, [&] { gather_keys(row); }, [&] { gather_values(row); });
            }
            block(nres - 16 * rj, [] {}, [] {});
        }
    }
    ICE_STAMP(10);
#pragma unroll
    for (int v = 0; v < HV; ++v) {
        l[v] = row16_sum(l[v]);
        if (g < G) {  // (with more than four heads every g + 4 v is one)
            float *dst = &wacc[wave][g + 4 * v][ch * 8];
            *(float4 *)dst = make_float4(acc[0][v], acc[1][v], acc[2][v], acc[3][v]);
            *(float4 *)(dst + 4) = make_float4(acc[4][v], acc[5][v], acc[6][v], acc[7][v]);
            if (ch == 0) { wm[wave][g + 4 * v] = m[v]; wl[wave][g + 4 * v] = l[v]; }
        }
    }
    __syncthreads();
    ICE_STAMP(11);
    // per head: the waves' merge weights exp(m_w - M) / L, one 16-lane row per head, one lane per wave
    static_assert(NW <= 16, "one DPP row holds the waves of a head");
    if (tid < 16 * G) {
        const int h = tid >> 4, w = tid & 15;
        const float mw = w < NW ? wm[w][h] : -INFINITY, lw = w < NW ? wl[w][h] : 0.f;
        float M = mw;
        M = fmaxf(M, dpp_f32<0xB1>(M));
        M = fmaxf(M, dpp_f32<0x4E>(M));
        M = fmaxf(M, dpp_f32<0x141>(M));
        M = fmaxf(M, dpp_f32<0x140>(M));
        const float e = M == -INFINITY ? 0.f : __expf(mw - M);
        const float L = row16_sum(lw * e);
        if constexpr (PARTIAL) {  // (device-scope words: another workgroup merges them)
            if (w < NW) wm[w][h] = e;
            if (w == 0) {
                __hip_atomic_store(out + h * (kD + 2) + kD, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(out + h * (kD + 2) + kD + 1, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            if (w < NW) wm[w][h] = L > 0.f ? e / L : 0.f;
        }
    }
    __syncthreads();
    constexpr int OW = G * kD / 64;  // waves' worth of outputs
    if constexpr (OW < NW) {
        if (wave >= OW) {
            aside(wave - OW, NW - OW);
            return;
        }
    }
    for (int o = tid; o < G * kD; o += NW * 64) {
        const int h = o / kD, j = o % kD;
        float O = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) O += wacc[w][h][j] * wm[w][h];
        if constexpr (PARTIAL) __hip_atomic_store(out + h * (kD + 2) + j, O, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else out[((size_t)u * G + h) * kD + j] = O;
    }
    if constexpr (OW >= NW) aside(wave, NW);
}

}  // namespace ice
