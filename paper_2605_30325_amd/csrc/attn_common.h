// Declarations shared by the attention kernels: launch arguments, vector types and the die-aware work split.  Not part of the public ABI.
#pragma once

#include "direct_load.h"
#include "veda_internal.h"

namespace veda {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct AttnArgs {
    const HeadGeom* heads;
    const uint8_t* tile_head;
    const int32_t* xcd_cum;    // pair items, walk mode
    const AttnItem* items;     // items of the table mode, by workgroup
    const uint64_t* tile_real; // real slots of every tile (plan table)
    const char* q;             // tiled Q, or null when q_tok is given
    const char* q_tok;         // Q in token order (bf16 kernel only): gathered by the kernel itself
    int64_t sq_b, sq_h, sq_n;  // its strides in bytes
    const char* k;             // tiled K, or null when k_tok is given
    const char* k_tok;         // K in token order (bf16 kernel only): key tiles gathered row by row
    int64_t sk_b, sk_h, sk_n;  // its strides in bytes
    const int32_t* tile_n0;    // token index of slot 0 of every tile (plan table)
    const char* v;
    const uint64_t* valid_mask;
    const int32_t* row_ptr;
    const int32_t* col_idx;
    char* out;
    float* lse;
    int64_t total_tiles, rows;
    int64_t so_b, so_h, so_n;  // output strides in bytes
    int64_t tokens;
    int n_heads, T, H, W;
    float scale_log2;          // softmax_scale * log2(e)
    // scale_log2 = scale_pow2 * scale_resid, scale_pow2 a power of two and 1 <= scale_resid < 2: with the
    // plan's exact-logit-scale option the bf16 kernel multiplies Q by scale_pow2 (exact in bf16) and the
    // logits by scale_resid on their way into the exponential, so no rounding of Q comes between the
    // inputs and the products; without it Q is multiplied by scale_log2 and rounded to bf16 once
    float scale_pow2, scale_resid;
    int split_tiles;           // fp32 kernel: split products up to this many kept key tiles of a query tile
};

// Workgroups are dealt round-robin to the 8 dies (XCDs), each with its own L2, all sharing
// the 256 MB memory-side cache.  Die x = blockIdx.x % 8 takes the x-th eighth of every head's
// query tiles and walks the heads in order: all dies then work on the same head at the same
// time (its K/V, ~120 MB at 220k tokens, stay in the memory-side cache), and the workgroups
// sharing an L2 hold neighbouring query tiles, whose kept key tiles overlap.
// The work item is a pair of adjacent query tiles; xcd_cum is the plan's table of them, `at` the workgroup's number.  Returns false
// for the padding workgroups of dies with fewer items.
// The head is found with one load per lane and a ballot: a binary search is log2(heads) loads one after the
// other, at the head of every workgroup's life (see union_build for what the whole of it costs).
__device__ inline bool xcd_work(const int32_t* __restrict__ xcd_cum, const HeadGeom* __restrict__ heads,
                                int n_heads, int at, int& head, int& item) {
    const int x = at % kXcd, local = at / kXcd, lane = threadIdx.x & 63;
    const int32_t* cum = xcd_cum + x * (n_heads + 1);
    // cum[0] = 0, ascending: the last head whose first item is <= local
    static_assert(kMaxHeads <= 128, "two entries per lane");
    const int c0 = lane < n_heads ? cum[lane] : 0x7fffffff, c1 = 64 + lane < n_heads ? cum[64 + lane] : 0x7fffffff;
    if (local >= cum[n_heads]) return false;
    head = __popcll(__ballot(local >= c0)) + __popcll(__ballot(local >= c1)) - 1;
    const int first = __builtin_amdgcn_readlane(head < 64 ? c0 : c1, head & 63);
    const int n = heads[head].n_pairs;
    item = x * (n / kXcd) + (x < n % kXcd ? x : n % kXcd) + (local - first);
    return true;
}

// Work item p of a head -> its query tiles: A always, B = A's neighbour along g.pair_ax if it
// exists (the last layer of an odd-sized axis has none).
__device__ inline void pair_tiles(const HeadGeom& g, int p, int& qiA, int& qiB, bool& hasB) {
    if (g.pair_ax == 3) {            // halves of a 128-token tile
        qiA = 2 * p; qiB = qiA + 1; hasB = true;
    } else if (g.pair_ax == 2) {
        const int half = (g.nw + 1) / 2, tw2 = p % half, rest = p / half;
        qiA = rest * g.nw + 2 * tw2; qiB = qiA + 1; hasB = 2 * tw2 + 1 < g.nw;
    } else if (g.pair_ax == 1) {
        const int half = (g.nh + 1) / 2, tw = p % g.nw, th2 = (p / g.nw) % half, tt = p / (g.nw * half);
        qiA = (tt * g.nh + 2 * th2) * g.nw + tw; qiB = qiA + g.nw; hasB = 2 * th2 + 1 < g.nh;
    } else {
        const int plane = g.nh * g.nw, rest = p % plane, tt2 = p / plane;
        qiA = 2 * tt2 * plane + rest; qiB = qiA + plane; hasB = 2 * tt2 + 1 < g.nt;
    }
    if (!hasB) qiB = qiA;
}

// What this workgroup computes, or false for nothing: its entry of the plan's table, or (walk mode: two lists at most) the
// pair that xcd_work gives it.
template <bool kTable> __device__ __forceinline__ bool attn_work(const AttnArgs& a, AttnItem& it) {
    if constexpr (kTable) {
        typedef const __attribute__((address_space(4))) int32_t* const_i32_t;
        const const_i32_t src = (const_i32_t)(uintptr_t)(a.items + blockIdx.x);   // scalar loads
        it.head = src[0];
        it.n_tiles = src[1];
#pragma unroll
        for (int t = 0; t < 4; ++t) it.tile[t] = src[2 + t];
        it.waves = (uint32_t)src[6];
        it.partners = src[7];
        return it.head >= 0;
    } else {
        int pair;
        bool hasB;
        if (!xcd_work(a.xcd_cum, a.heads, a.n_heads, blockIdx.x, it.head, pair)) return false;
        pair_tiles(a.heads[it.head], pair, it.tile[0], it.tile[1], hasB);
        it.n_tiles = hasB ? 2 : 1;
        it.tile[2] = it.tile[3] = it.tile[0];
        it.partners = hasB && a.heads[it.head].n_tiles > kF32SplitTiles ? 1 : 0;
        const uint32_t b = hasB ? 1u : kItemIdle;
        it.waves = kItemSecond << 8 | b << 16 | (b | kItemSecond) << 24;
        return true;
    }
}

// Sum over the lanes up to and with this one, by DPP.
__device__ __forceinline__ int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Position of the n-th set bit (from 0) of m; n < popcount(m).
__device__ inline int nth_bit(uint64_t m, int n) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const int c = __popcll((m >> pos) & ((1ull << w) - 1ull));
        if (n >= c) { n -= c; pos += w; }
    }
    return pos;
}

__device__ inline int rho(int m) {  // swap bits 2 and 3
    return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// x of this lane and x of lane ^ 32, without a trip through LDS: the swap exchanges lanes 32-63
// of its first operand with lanes 0-31 of its second, leaving (low half, low half) in one
// register and (high half, high half) in the other.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi) {
    lo = x;
    hi = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
}
__device__ __forceinline__ float max_with_other_half(float x) {
    float lo, hi;
    both_halves(x, lo, hi);
    asm("v_max_f32 %0, %0, %1" : "+v"(lo) : "v"(hi));   // fmaxf would quiet both first
    return lo;
}
__device__ __forceinline__ float sum_with_other_half(float x) {
    float lo, hi;
    both_halves(x, lo, hi);
    return lo + hi;
}

// Launches the query-tile-pair bf16 kernel (attn_pair.hip) on plan pl's geometry; a.xcd_cum must be
// its pair table.  grouped: pl is the inner plan of 128-token tiles and the CSR counts whole tiles.
// exact: the power-of-two / residual split of the logit scale (AttnArgs::scale_pow2, scale_resid).
// walk: merge the kept lists inside the loop instead of building the step table first.
veda_status launch_sparse_attn_bf16_pair(const veda_plan* pl, const AttnArgs& a, bool grouped, bool exact, bool walk,
                                         hipStream_t s);

// The fp32 kernel (attn_f32.hip): same work items (a.xcd_cum must be the plan's pair table), tiled Q, K, V only.
veda_status launch_sparse_attn_f32(const veda_plan* pl, const AttnArgs& a, bool walk, hipStream_t s);

}  // namespace veda
