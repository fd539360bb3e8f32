// The union of the kept lists of a workgroup's query tiles as a step table in LDS (Sec. 4.3: a
// workgroup visits only kept key tiles; here several query tiles share one visit).
//
// A workgroup that owns N query tiles visits every key tile kept by at least one of them once.
// Walking the N lists with scalar loads inside the main loop costs a wave a scalar-memory
// round trip per step, and while one is in flight the compiler can only wait for LDS operand
// reads by waiting for everything.  So the walk is done up front, by all threads at once:
//   1. every list is turned into a bitmap over the head's key tiles (LDS atomics);
//   2. a block-wide prefix sum over the population counts of the OR of the bitmaps numbers the
//      kept key tiles in ascending order: these are the steps;
//   3. the table of steps is filled kUnionChunk entries at a time, one entry per thread: the
//      thread finds the bitmap word of its step by binary search in the prefix sums, the bit by
//      counting, and stores (key tile, who keeps it, the tile's anchor token, its validity mask).
// The main loop reads one 16-byte entry per step from LDS, steps ahead.  The table is a ring of
// two chunks; a chunk is refilled when the loop has left it.
// Padding.  A key tile at a ragged edge of the grid may hold real tokens in few of its eight 8-slot chunks.
// With four or fewer the step is a half step: the chunks that hold real tokens are gathered to the front on
// their way into LDS (a chunk is 16 bytes of a V^T row and eight K rows, so both move freely) and one 32-key
// block of products serves the tile.  A tile with no real token at all (the second half of a 128-token tile)
// is neither loaded nor computed.  A tile with five or more such chunks is a full step: it needs both blocks.
// Lists may come in any order (the union is visited in ascending order regardless) and must not
// name a tile twice in a row of the CSR (the attention entry points' contract).
#pragma once

#include "attn_common.h"

namespace veda {

constexpr int kUnionMaxWords = 512;                 // bitmap words: list entries name at most 16384 different tiles
constexpr int kUnionMaxTiles = kUnionMaxWords * 32;

// What a step does with its key tile, beside the keeper bits 0..3 of its flags.
constexpr int kStepHalf = 16;    // one 32-key block after gathering chunks
constexpr int kStepEmpty = 32;   // nothing to attend to
constexpr int kStepWhole = 64;   // no padding: the common case, told apart by one test
constexpr int kStepPart = 256;   // both blocks, some padding

// Validity mask of a key tile -> kind of step.  Half: lo = mask of the 32 gathered slots, hi = the
// four chunks they come from, one byte each (places without a chunk name one that is all padding: V is zero
// there).  Otherwise lo, hi = the mask itself.
__device__ __forceinline__ int step_kind(uint64_t vm, uint32_t& lo, uint32_t& hi) {
    lo = (uint32_t)vm;
    hi = (uint32_t)(vm >> 32);
    if (vm == ~0ull) return kStepWhole;
    // Tiles with five or more chunks in use are told by counting: in walk mode this runs on the scalar unit inside the
    // main loop, and gathering what is then not used cost more than half steps gave on large grids (24 heads of
    // 219,600 tokens, walk mode 35.4 -> 34.8 ms, without any kinds 34.6; from the table 33.2 -> 32.9, of which the rest
    // is fewer tests per load in the main loop).
    uint64_t used = vm | (vm >> 4);   // bit 0 of every byte that is not zero
    used |= used >> 2;
    used |= used >> 1;
    const int chunks = __popcll(used & 0x0101010101010101ull);
    if (chunks > 4) return kStepPart;
    if (chunks == 0) return kStepEmpty;
    uint32_t mask = 0u, from = 0u, none = 0u;
    int n = 0;
    for (int c = 0; c < 8; ++c) {
        const uint32_t byte = (uint32_t)(vm >> (8 * c)) & 255u;
        if (byte == 0u) none = (uint32_t)c;
        else {
            mask |= byte << (8 * n);
            from |= (uint32_t)c << (8 * n);
            ++n;
        }
    }
    for (int i = n; i < 4; ++i) from |= none << (8 * i);
    lo = mask;
    hi = from;
    return kStepHalf;
}

// x: key tile | flags << 16 (keepers, kind; 0 = past the last step); y: anchor token; z, w: step_kind's lo, hi.
struct __align__(16) UnionEntry { int32_t x, y; uint32_t z, w; };

// kChunk: table entries filled at a time (a power of two); the ring holds two chunks.
template <int N, int kChunk> struct UnionLds {
    static constexpr int kRingEntries = 2 * kChunk;
    UnionEntry tab[kRingEntries];
    uint32_t bm[N][kUnionMaxWords];
    int32_t prefix[kUnionMaxWords];
    int32_t wave_sum[16];
};

// What comes before the first product of a workgroup is a chain of loads and barriers: 15 % of a call at 32 kept
// tiles, 10 % at 63 (the second resident workgroup computes meanwhile).  Finding the head by ballot (xcd_work), asking
// for the lists before the bitmaps are cleared and filling the whole ring in one go took 40 heads of 21x30x52 at
// one kept tile from 371 to 364 us; union_table after that: 4 heads of 9x18x18, 2 samples, 25 % kept (d = 64, whole call)
// 73.9 -> 72.4 us, 40 heads of 21x30x52 at 5 % 1906 -> 1895.

// The lists' entries into their bitmaps, which are clear.  early: the first kThreads of each.
template <int N, int kThreads>
__device__ __forceinline__ void union_mark(uint32_t (&bm)[N][kUnionMaxWords], const int32_t* const (&cols)[N], const int (&n)[N],
                                           const int (&early)[N], int lists, int n_tiles, int tid) {
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if (t >= lists) break;
        auto mark = [&](int j) {
            if ((unsigned)j < (unsigned)n_tiles) atomicOr(&bm[t][j >> 5], 1u << (j & 31));
        };
        mark(early[t]);
        for (int i = tid + kThreads; i < n[t]; i += kThreads) mark(cols[t][i]);
    }
}

// Steps 1 and 2 over many key tiles (kUnionDirectTiles).  All threads of the workgroup call it; it ends with a barrier.  Returns the number of kept key tiles.
template <int N, int kThreads, int kChunk>
__device__ inline int union_build(UnionLds<N, kChunk>& u, const int32_t* const (&cols)[N], const int (&n)[N], const int (&early)[N],
                                  int lists, int n_tiles, int tid) {
    static_assert(kUnionMaxWords % kThreads == 0, "whole words per thread");
    constexpr int kPer = kUnionMaxWords / kThreads;
    const int words = (n_tiles + 31) >> 5;
    for (int w = tid; w < words; w += kThreads)
#pragma unroll
        for (int t = 0; t < N; ++t) u.bm[t][w] = 0u;
    __syncthreads();
    union_mark<N, kThreads>(u.bm, cols, n, early, lists, n_tiles, tid);
    __syncthreads();
    // exclusive prefix sum of the words' population counts: kPer consecutive words per thread
    int cnt[kPer], mine = 0;
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const int w = tid * kPer + p;
        uint32_t all = 0u;
        if (w < words) {
#pragma unroll
            for (int t = 0; t < N; ++t) all |= u.bm[t][w];
        }
        cnt[p] = __popc(all);
        mine += cnt[p];
    }
    int incl = mine;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
    }
    if (lane == 63) u.wave_sum[wave] = incl;
    __syncthreads();
    int off = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        const int s = u.wave_sum[w];
        off += w < wave ? s : 0;
        total += s;
    }
    int run = off + incl - mine;
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        u.prefix[tid * kPer + p] = run;
        run += cnt[p];
    }
    __syncthreads();
    return total;
}

// Step 3: entries [first, first + kCount) of the step sequence into their places in the ring
// (entry s lives at s % (2 kChunk)).  No barrier inside: the caller separates it from the readers
// of these places.  total: number of steps.  kGrouped: the lists name whole 128-token tiles and
// every kept one makes two steps, its 64-slot halves 2o and 2o+1 (vmask, n0s are indexed by half),
// kept by all N query tiles alike.
template <int N, int kThreads, int kChunk, bool kGrouped, int kCount = kChunk>
__device__ inline void union_fill(UnionLds<N, kChunk>& u, int first, int total, int n_tiles, const uint64_t* __restrict__ vmask,
                                  const int32_t* __restrict__ n0s, int tid) {
    const int words = (n_tiles + 31) >> 5;
    for (int i = tid; i < kCount; i += kThreads) {
        const int step = first + i;
        const int s = kGrouped ? step >> 1 : step;   // position in the ascending union
        UnionEntry e = {0, 0, 0u, 0u};
        if (step < total) {
            int lo = 0, hi = words - 1;   // the last word whose prefix is <= s holds step s
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (u.prefix[mid] <= s) lo = mid; else hi = mid - 1;
            }
            uint32_t b[N], all = 0u;
#pragma unroll
            for (int t = 0; t < N; ++t) {
                b[t] = u.bm[t][lo];
                all |= b[t];
            }
            for (int k = s - u.prefix[lo]; k > 0; --k) all &= all - 1u;
            if (all == 0u) all = 1u;   // cannot happen for s < total; keeps the index below in range regardless
            const int bit = __ffs((int)all) - 1;
            const int j = kGrouped ? 2 * (lo * 32 + bit) + (step & 1) : lo * 32 + bit;
            int fl = 0;
#pragma unroll
            for (int t = 0; t < N; ++t) fl |= (int)((b[t] >> bit) & 1u) << t;
            if (kGrouped) fl = (1 << N) - 1;
            const int kind = step_kind(vmask[j], e.z, e.w);
            e.x = j | ((kind == kStepEmpty ? kind : fl | kind) << 16);
            e.y = n0s[j];
        }
        u.tab[step & (2 * kChunk - 1)] = e;
    }
}

// Lists over few key tiles: the whole table at once.  A thread stands for a key tile (of every kThreads-th) instead of a step, so
// the tiles' masks and anchors are asked for before the lists have come and neither a search nor a second trip to memory
// follows them; a bitmap word to a lane of a wavefront, so that every wavefront numbers the steps for itself.
constexpr int kUnionDirectTiles = 2048;

template <int N, int kThreads, bool kGrouped> struct UnionEarly {
    static constexpr int kTurns = kUnionDirectTiles / kThreads, kHalves = kGrouped ? 2 : 1;
    int col[N];                     // the thread's first entry of every list, or -1
    uint64_t vm[kTurns][kHalves];   // its key tiles'
    int32_t n0[kTurns][kHalves];

    __device__ __forceinline__ void ask(const int32_t* const (&cols)[N], const int (&n)[N], int lists, int n_tiles,
                                        const uint64_t* __restrict__ vmask, const int32_t* __restrict__ n0s, int tid) {
#pragma unroll
        for (int t = 0; t < N; ++t) col[t] = t < lists && tid < n[t] ? cols[t][tid] : -1;
#pragma unroll
        for (int i = 0; i < kTurns; ++i) {
            if (i * kThreads >= n_tiles || n_tiles > kUnionDirectTiles) break;
            const int j = i * kThreads + tid < n_tiles ? i * kThreads + tid : n_tiles - 1;
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                vm[i][h] = vmask[kHalves * j + h];
                n0[i][h] = n0s[kHalves * j + h];
            }
        }
    }
};

// Steps 1 and 2, and step 3 for the whole ring.  cols[t], n[t]: list t (global memory).  n_tiles: the range of the list entries; lists: how
// many of the N there are.  All threads of the workgroup call it; it ends with a barrier.  Returns the number of
// kept key tiles; with kGrouped each makes two steps.
template <int N, int kThreads, int kChunk, bool kGrouped>
__device__ inline int union_table(UnionLds<N, kChunk>& u, const UnionEarly<N, kThreads, kGrouped>& early, const int32_t* const (&cols)[N],
                                  const int (&n)[N], int lists, int n_tiles, const uint64_t* __restrict__ vmask,
                                  const int32_t* __restrict__ n0s, int tid) {
    if (n_tiles > kUnionDirectTiles) {
        const int total = union_build<N, kThreads, kChunk>(u, cols, n, early.col, lists, n_tiles, tid);
        union_fill<N, kThreads, kChunk, kGrouped, 2 * kChunk>(u, 0, kGrouped ? 2 * total : total, n_tiles, vmask, n0s, tid);
        __syncthreads();
        return total;
    }
    constexpr int kWords = kUnionDirectTiles / 32, kRing = 2 * kChunk, kHalves = kGrouped ? 2 : 1;
    static_assert(kWords == 64 && kThreads % 64 == 0, "a word to a lane");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < N * kWords; i += kThreads) u.bm[i / kWords][i % kWords] = 0u;
    for (int i = tid; i < kRing; i += kThreads) u.tab[i] = UnionEntry{0, 0, 0u, 0u};
    __syncthreads();
    union_mark<N, kThreads>(u.bm, cols, n, early.col, lists, n_tiles, tid);
    __syncthreads();
    uint32_t word = 0u;
#pragma unroll
    for (int t = 0; t < N; ++t) word |= u.bm[t][lane];
    const int upto = wave_scan(__popc(word)), before = upto - __popc(word), total = __builtin_amdgcn_readlane(upto, 63);
    if (wave == 0) u.prefix[lane] = before;   // for union_fill
#pragma unroll
    for (int i = 0; i < UnionEarly<N, kThreads, kGrouped>::kTurns; ++i) {
        if (i * kThreads >= n_tiles) break;
        const int at = i * (kThreads / 32) + 2 * wave;   // word of lanes 0-31
        const bool up = lane >= 32;
        const uint32_t w0 = (uint32_t)__builtin_amdgcn_readlane((int)word, at), w1 = (uint32_t)__builtin_amdgcn_readlane((int)word, at + 1);
        const int s0 = __builtin_amdgcn_readlane(before, at), s1 = __builtin_amdgcn_readlane(before, at + 1);
        const uint32_t w = up ? w1 : w0;
        const int bit = lane & 31, s = (up ? s1 : s0) + __popc(w & ((1u << bit) - 1u));
        if (((w >> bit) & 1u) && kHalves * s < kRing) {
            int fl = 0;
            if (kGrouped) {
                fl = (1 << N) - 1;
            } else {
#pragma unroll
                for (int t = 0; t < N; ++t) fl |= (int)((u.bm[t][at + (up ? 1 : 0)] >> bit) & 1u) << t;
            }
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                const int j = kHalves * (i * kThreads + tid) + h;
                u.tab[kHalves * s + h] = UnionEntry{j | fl << 16, early.n0[i][h], (uint32_t)early.vm[i][h], (uint32_t)(early.vm[i][h] >> 32)};
            }
        }
    }
    __syncthreads();
    // the kinds, a step to a thread: above, few threads of a turn have one
    for (int i = tid; i < kRing; i += kThreads) {
        if (i >= kHalves * total) break;
        UnionEntry e = u.tab[i];
        const uint64_t vm = (uint64_t)e.w << 32 | e.z;
        const int kind = step_kind(vm, e.z, e.w);
        e.x = kind == kStepEmpty ? (e.x & 0xffff) | kind << 16 : e.x | kind << 16;
        u.tab[i] = e;
    }
    __syncthreads();
    return total;
}

// One step as the main loop holds it (all fields wave-uniform, in scalar registers).
struct UnionStep {
    int j;         // key tile (head-local)
    int fl;        // bit t: query tile t of the workgroup keeps it; its kind; 0 = past the end
    uint64_t vm;   // validity mask of key tile j; half steps: step_kind's lo | hi << 32
    int n0;        // token index of its slot 0
};

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef const __attribute__((address_space(3))) i32x4* lds_i32x4_ptr;

// The raw entry of step s (the same address in every lane), and its fields once it has arrived.
template <int kChunk> __device__ __forceinline__ i32x4 union_read(uint32_t tab_lds, int s) {
    return *(lds_i32x4_ptr)(uintptr_t)(tab_lds + (uint32_t)(s & (2 * kChunk - 1)) * 16u);
}
__device__ __forceinline__ UnionStep union_step(const i32x4& raw) {
    UnionStep e;
    const int x = __builtin_amdgcn_readfirstlane(raw[0]);
    e.j = x & 0xffff;
    e.fl = x >> 16;
    e.n0 = __builtin_amdgcn_readfirstlane(raw[1]);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(raw[2]), hi = (uint32_t)__builtin_amdgcn_readfirstlane(raw[3]);
    e.vm = (uint64_t)hi << 32 | lo;
    return e;
}

}  // namespace veda
