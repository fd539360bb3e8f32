// Target tile scores of full attention and tile recall -- the supervision side of the method
// (Sec. 4.1 "Target: Full-Attention Score Construction", Eq. 3: S_tgt[i][j] = max over the
// token pairs of (query tile i, key tile j) of Softmax(Q K^T / sqrt(d)); Sec. 4.3 "Efficient
// Ground-Truth Heatmap Generation": exact pooled scores in two passes without storing the
// attention map, optionally for a subset of query tiles; Sec. 3.2: Recall@k).
//
// The softmax couples all keys of a query row, so every query tile walks all key tiles of
// its head twice: pass 1 forms the row maximum m_u and the denominator l_u with an online
// softmax, pass 2 forms the logits again and reduces exp(s_uv - m_u) / l_u over each 64 x 64
// block.  exp is monotone, so the block maximum needs one exponential per query row and
// block: exp(max_v s_uv - m_u) / l_u, then the maximum over the rows u.  Both passes stay in
// one kernel: m_u and l_u never leave the registers.  With scratch (veda_tile_heatmap_ws) the block's
// max_v s_uv of pass 1 are kept, 4 bytes per row and key tile where the products of that block read 16 KB, and pass 2
// only reads those: the same bits without forming the logits again.
//
// The same kernel serves bf16 and fp32 (v_mfma_f32_32x32x16_bf16 or v_mfma_f32_32x32x2_f32, fp32
// accumulation): S^T = K Q^T, so a lane owns a query row and its registers run over keys.  A workgroup holds the
// real rows of as many consecutive query tiles as fit its four waves of 32 (geometry.h, heat_items; with a list, up to four
// tiles), packed: rows do not know each other before their maxima meet, in LDS, per tile.  Two tiles to a workgroup, whatever
// they hold, before: 12 heads of 21x30x52 (27 % of the tiles hold 32 rows or fewer) whole call 4.91 -> 4.49 ms, one tile
// in 16 of 40 heads of 21x45x80 8.41 -> 8.14, fp32 search of 9x24x32, whose 16x2x2 tiles hold 36 rows, 9.5 -> 7.5.  Pass 1 is bound by its exponentials (one per pair of tokens, with the
// fused multiply-add before and the addition after it: 48 vector operations per 8 products), pass 2 by the
// products; the exponentials of one 32-key block are therefore formed behind the products of the next, and the
// reference of the softmax stays where it is until a sum outgrows it.
// Measured, the heat map alone, before and after: 12 heads of 624 tiles, bf16, d = 128, 10.0 -> 7.9 ms; one in 16
// of the query tiles of 40 heads of 21x45x80, mixed shapes, 23.1 -> 11.6 ms (listed tiles used to run one to a
// workgroup); 8 heads of 144 tiles, fp32, d = 128, 19.1 -> 3.0 ms (on the vector units before).  Tried and left out: 64 rows
// per wave, four tiles per workgroup (half the operand reads and loads: 8.3 and 11.7 ms, fp32 3.9), a ring of
// three or four K tiles (0.5 ms slower: it costs a resident workgroup and the loads are not what is waited for).
// With scratch, whole calls of the supervision side (gathers, heat map, both top-k, recall), two walks and one: 12 heads
// of 624 tiles 8.0 -> 5.0 ms, one in 16 tiles of 40 heads of 21x45x80 13.4 -> 8.8 ms; of the gain, masks
// on the scalar unit and no register copies at the ends of branches gave a fifth,
// handing work items out as asked for 12 % of the second case.  Operand addresses that never change (two steps to a turn of the
// loop, the slot a constant) and maxima that quiet no NaN first (61 vector instructions per 8 products, 48 of them the exponentials'
// three): 4.49 -> 4.15 ms and 8.14 -> 7.72.  While a compute unit is busy its vector units then issue 80 % of the cycles and its matrix
// pipes 50 %.  The bf16 forms spill 6 to 19 registers (d = 64 with a list none): what a work item keeps from its start for its end,
// stored and read once per item, not in the walk.  Tried: the additions on the matrix pipe (v_mfma_f32_4x4x1, one a lane), 5.25 ms: they queue behind the products.
// Padding: a wave runs only the blocks that hold real rows, and key tiles with few real keys are half steps (attn_union.h).
#include <type_traits>

#include "attn_common.h"
#include "attn_union.h"

namespace veda {

struct HeatArgs {
    const HeadGeom* heads;
    const uint8_t* tile_head;
    const HeatItem* table;        // the plan's work items; unused with a query list
    const int32_t* query_tiles;   // optional: global tile ids to process
    int64_t n_query_tiles;
    const char* q;
    const char* k;
    const uint64_t* valid_mask;
    float* heat;
    int64_t total_tiles, score_elems;
    int n_heads;
    float scale_log2;             // softmax_scale * log2(e)
    float2* rows;                 // optional: (ref, 1/l) of every row, token order
    int have_rows;                // read them instead of running pass 1
    int64_t tokens;
    int T, H, W;
    uint32_t* taken;              // one-walk mode: work items handed out, per die, kHeatTakenStride apart; null = one each
    float* maxima;                // one-walk mode: kept block maxima, max_tiles * 128 floats per workgroup
    int64_t max_tiles;            // tiles of the largest head
    uint32_t items, batch;        // work items of a sample; samples
};

// Maximum over the 32 rows of a wave (x alike in both lane halves), wave-uniform: within 16 lanes by DPP, the
// two groups through scalar registers.
__device__ __forceinline__ float rows_max(float x) {
    const auto step = [](float v, auto ctrl) __attribute__((always_inline)) {
        return fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true)));
    };
    x = step(x, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
    x = step(x, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
    x = step(x, std::integral_constant<int, 0x141>{});   // row_half_mirror
    x = step(x, std::integral_constant<int, 0x140>{});   // row_mirror
    return fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0)),
                 __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16)));
}

// One operand fragment: 16 bytes per lane, chunk 2f + hh of a K or Q row, and the products it takes part in.
template <typename E> struct HeatFrag;
template <> struct HeatFrag<uint16_t> {
    typedef bf16x8 type;
    static __device__ __forceinline__ f32x16 mul(type k, type q, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q, c, 0, 0, 0);
    }
};
template <> struct HeatFrag<uint32_t> {
    typedef __attribute__((ext_vector_type(4))) float type;
    static __device__ __forceinline__ f32x16 mul(type k, type q, f32x16 c) {
#pragma unroll
        for (int t = 0; t < 4; ++t) c = __builtin_amdgcn_mfma_f32_32x32x2f32(k[t], q[t], c, 0, 0, 0);
        return c;
    }
};

constexpr int kHeatTakenStride = 16;   // counters of the dies, 64 bytes apart
constexpr int kHeatFold = 32;          // steps after which the running part of a denominator is put away
constexpr float kHeatNoRef = -3e38f;   // reference before the first key: everything finite outgrows it
// A lane's sum over its 16 keys of a block above this moves the reference.  At most 16 where the reference is
// the row's maximum, so rows of even logits stay below it.
constexpr float kHeatSlack = 32.0f;

// exp2(t) / l of a block's largest logit.  The instruction returns 0 below 2^-126; fp32 target scores keep the order of
// tiles that far below their row's maximum, so there the exponential is formed 2^64 higher and the score rounded once.
// (One score per query row and block.  8 heads of 144 tiles, d = 128: the second pass alone 1.46 -> 1.47 ms, d = 64
// 0.73 -> 0.74, both passes 3.0 ms either way.)
template <typename E> __device__ __forceinline__ float heat_score(float t, float inv_l) {
    if (sizeof(E) == 2) return __builtin_amdgcn_exp2f(t) * inv_l;
    const bool low = t < -126.0f;
    const float p = __builtin_amdgcn_exp2f(low ? t + 64.0f : t) * inv_l;
    return low ? p * 0x1p-64f : p;
}

// Scores as unsigned numbers of the same order, so that wavefronts meet in LDS with an integer maximum: 0 where there is none, 1
// for NaN (the largest only where there is nothing else, as with fmaxf).
__device__ __forceinline__ uint32_t heat_key(float x) {
    const uint32_t u = __float_as_uint(x);
    return x != x ? 1u : u ^ (uint32_t)((int)u >> 31 | (int)0x80000000);
}
__device__ __forceinline__ float heat_of_key(uint32_t key) {
    if (key <= 1u) return key ? __builtin_nanf("") : 0.0f;
    return __uint_as_float(key & 0x80000000u ? key ^ 0x80000000u : ~key);
}

// The listed query tiles of this workgroup (up to four), their head and their number, or false: the split is in
// geometry.h.  The heads' full and thin entries in the window are counted in LDS and their kinds kept there as bytes; every
// wave then finds the same head and the same entries.  LDS: kListWindow bytes and a word per head, free again on return.
// Finding the p-th item here leaves no workgroup that only exits: with one workgroup per entry, those that had a pair
// alternated with those that did not in an ordinary list, and the hardware deals workgroups out in turn, over the dies
// and inside them, so half the chip had nothing.  Measured, one workgroup per entry and now: one tile in 16 of 40 heads of
// 21x45x80, one shape, bf16 13.7 -> 10.0 ms (mixed shapes 11.7-12.6 -> 11.5, in no order 14.3 -> 11.7); all tiles of
// 12 heads of 624 in order, bf16 11.4 -> 7.9 and fp32 128 -> 64.6 ms (without a list 7.75 and 64.2), in no order
// 8.8 -> 7.8 and 77 -> 64.2; all 57,600 of 40 heads at d = 64 142 -> 87 ms; 8 tiles of 2 heads 15.3 -> 15.9 us.  A
// contiguous piece of the list for each die, followers still exiting, is not enough (13.1, 13.3 and 121 ms).
__device__ inline bool listed_tiles(const HeatArgs& a, int item, char* smem, int tid, int& head, int& n_own, int (&own)[4]) {
    static_assert(kMaxHeads == 128, "two heads per lane, a head and a kind in a byte");
    const int lane = tid & 63;
    const int per = (int)list_window_blocks(kListWindow, a.n_heads), p = item % per;
    const int64_t begin = (int64_t)(item / per) * kListWindow;
    const int m = (int)(a.n_query_tiles - begin < kListWindow ? a.n_query_tiles - begin : kListWindow);
    const int32_t* list = a.query_tiles + begin;
    uint8_t* kinds = reinterpret_cast<uint8_t*>(smem);          // 2 head + (1 if thin)
    int* count = reinterpret_cast<int*>(smem + kListWindow);    // full | thin << 16
    if (tid < kMaxHeads) count[tid] = 0;
    __syncthreads();
    for (int i = tid; i < m; i += 256) {
        const int g = list[i], h = a.tile_head[g];
        const bool thin = __popcll(a.valid_mask[g]) <= 32;
        kinds[i] = (uint8_t)(2 * h + (thin ? 1 : 0));
        atomicAdd(&count[h], thin ? 1 << 16 : 1);
    }
    __syncthreads();
    // items of heads `lane` and 64 + lane, and of all heads up to them
    auto items = [&](int h) { return list_items(count[h] & 0xffff, (int)((uint32_t)count[h] >> 16)); };
    const int n0 = items(lane), n1 = items(64 + lane);
    const int upto0 = wave_scan(n0);
    int upto1 = __builtin_amdgcn_readlane(upto0, 63);
    if (a.n_heads > 64) upto1 += wave_scan(n1);
    head = __popcll(__ballot(upto0 <= p)) + __popcll(__ballot(upto1 <= p));
    const bool any = head < kMaxHeads;
    n_own = 0;
    if (any) {
        const int q = p - __builtin_amdgcn_readlane(head < 64 ? upto0 - n0 : upto1 - n1, head & 63);
        const int both = __builtin_amdgcn_readfirstlane(count[head]), full = both & 0xffff, thin = (int)((uint32_t)both >> 16);
        // entries of rank first .. first + want - 1 of a kind
        auto find = [&](int kind, int first, int want) {
            int before = 0;
            for (int i0 = 0; i0 < m && want > 0; i0 += 64) {
                const uint64_t same = __ballot(i0 + lane < m && kinds[i0 + lane < m ? i0 + lane : 0] == 2 * head + kind);
                const int upto = before + __popcll(same);
                for (; want > 0 && first < upto; ++first, --want) {
                    const int at = list[i0 + nth_bit(same, first - before)];
                    if (n_own == 0) own[0] = at; else if (n_own == 1) own[1] = at; else if (n_own == 2) own[2] = at; else own[3] = at;
                    ++n_own;
                }
                before = upto;
            }
        };
        const int along = full & 1 ? (thin < 2 ? thin : 2) : 0;   // thin entries that go with the last full one
        if (q < (full + 1) / 2) {
            const bool last = 2 * q + 1 == full;
            find(0, 2 * q, last ? 1 : 2);
            if (last && along) find(1, 0, along);
        } else {
            const int first = along + 4 * (q - (full + 1) / 2);
            find(1, first, thin - first < 4 ? thin - first : 4);
        }
    }
    __syncthreads();
    return any;
}

// Workgroups on a compute unit: two K tiles of fp32 at d = 128 are 65 KB of LDS, elsewhere the registers decide.  One walk
// keeps a place for each (three where two fit: 8.12 instead of 8.10 ms for 12 heads of 288 tiles, a third of them listed 3.68 instead
// of 3.56; bf16 at d = 64, five where four fit: 12 heads of 624, a third listed, 1.23 instead of 1.18 ms).
// fp32 at d = 64: a fourth fits where all tiles are asked for, and is slower (12 heads of 624 tiles 17.6 -> 18.2 ms).
constexpr int heat_resident(bool bf16, int d, bool grouped, bool listed) {
    if (!bf16) return d == 128 ? 2 : 3;
    return d == 128 || (listed && !grouped) ? 4 : 5;
}

// kGrouped: 128-token tiles.  The geometry in `a` is that of the 64-slot halves; a whole tile is a
// workgroup and two consecutive key steps, and its block maximum the maximum over them.
// kOneWalk: the logits are formed once.  Pass 1 keeps the largest raw logit of every row and key tile in scratch, one
// place per workgroup and written over for its next work item; pass 2 reads those instead of forming the products again.
template <typename E, int D, bool kGrouped, bool kListed, bool kOneWalk>
__global__ __launch_bounds__(256, heat_resident(sizeof(E) == 2, D, kGrouped, kListed)) void tile_heatmap_kernel(HeatArgs a) {
    typedef HeatFrag<E> F;
    typedef typename F::type frag;
    typedef const __attribute__((address_space(3))) frag* lds_frag_ptr;
    constexpr int kRowB = D * (int)sizeof(E), kKBytes = kTile * kRowB, kKChunks = kRowB / 16;
    constexpr int kF = kRowB / 32;               // fragments of a row
    constexpr int kLoads = kKBytes / 1024 / 4;   // direct-load instructions per wave per K tile
    constexpr int kGroup = kLoads < 4 ? kLoads : 4;
    constexpr int kAhead = 4;
    constexpr int kExps = 16 / kF;               // exponentials behind one fragment's products
    // dynamic LDS only, so the base is the workgroup's LDS origin (the XOR swizzle needs address bits 4-9 of
    // the base clear): two K slots, then the results of 64 steps for each of the workgroup's query tiles
    extern __shared__ __align__(1024) char smem[];
    uint32_t (*part)[64] = reinterpret_cast<uint32_t (*)[64]>(smem + 2 * kKBytes);   // heat_key
    int* out_tile = reinterpret_cast<int*>(part + kHeatTiles);                       // the tiles

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int idx = lane & 31, hh = lane >> 5;
    for (int i = tid; i < kHeatTiles * 64; i += 256) (&part[0][0])[i] = 0u;   // read after the barriers of the walk

    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x;
    // A work item is a few query tiles of one head, with 128 rows between them or a little less.
    auto run = [&](uint32_t work) __attribute__((always_inline)) {
    const int64_t b = work / a.items;
    const int at = (int)(work - (uint32_t)b * a.items);
    constexpr bool kOwn = kListed && !kGrouped;
    int head, first = 0, n_own = 0, own[4] = {0, 0, 0, 0};
    if constexpr (kOwn) {
        if (!listed_tiles(a, at, smem, tid, head, n_own, own)) return;
    } else if constexpr (kListed) {   // a listed 128-token tile fills a workgroup
        first = 2 * a.query_tiles[at];
        head = a.tile_head[first];
        first -= a.heads[head].tile_off;
        n_own = 2;
    } else {
        typedef const __attribute__((address_space(4))) int32_t* const_i32_t;
        const const_i32_t src = (const_i32_t)(uintptr_t)(a.table + at);
        head = src[0];
        first = src[1];
        n_own = src[2];
    }
    const HeadGeom hg = a.heads[head];
    const int n = hg.n_tiles;
    const int64_t head_tile0 = b * a.total_tiles + hg.tile_off;
    const char* kt = a.k + head_tile0 * kKBytes;
    typedef const __attribute__((address_space(4))) uint64_t* const_u64_t;
    const const_u64_t vmask = (const_u64_t)(uintptr_t)(a.valid_mask + hg.tile_off);
    // The item's tiles as far as their rows fit; a mask with more real slots than the grid gives leaves some for another turn.
    for (int t0 = 0; t0 < n_own;) {
    // This lane's row: the real slots of the query tiles in order, 32 per wave.
    const int row = 32 * wave + idx;
    int qi = 0, slot = 0, out = 0, rows = 0, t1 = t0;
    bool q_real = false;
    for (; t1 < n_own; ++t1) {
        const int i = !kOwn ? first + t1 : (t1 == 0 ? own[0] : t1 == 1 ? own[1] : t1 == 2 ? own[2] : own[3]) - hg.tile_off;
        const uint64_t mask = vmask[i];
        const int more = __popcll(mask);
        if (rows + more > 128) break;
        if (row >= rows && row < rows + more) {
            qi = i;
            slot = nth_bit(mask, row - rows);
            out = kGrouped ? 0 : t1 - t0;
            q_real = true;
        }
        if (tid == 0) out_tile[t1 - t0] = i;
        rows += more;
    }
    const int outs = kGrouped ? 1 : t1 - t0;
    t0 = t1;
    const bool active = __builtin_amdgcn_readfirstlane(32 * wave < rows ? 1 : 0);
    frag qf[kF];
    float2* row_sums = nullptr;   // where this lane's are kept
    {
        const char* qrow = a.q + (head_tile0 + qi) * kKBytes + slot * kRowB + 16 * hh;
#pragma unroll
        for (int f = 0; f < kF; ++f) qf[f] = *reinterpret_cast<const frag*>(qrow + 32 * f);
        if (a.rows && q_real) {
            // a slot without a token has no place there, whatever the mask says of it
            const int token = slot_token(hg, qi, slot, a.T, a.H, a.W);
            q_real = token >= 0;
            if (q_real) row_sums = a.rows + (b * a.n_heads + head) * a.tokens + token;
        }
    }
    uint32_t rows_real = (uint32_t)__ballot(q_real);
    const int out0 = __builtin_amdgcn_readfirstlane(out);
    // 32 rows of one tile: results need no telling apart
    const bool plain = rows_real == ~0u && __ballot(out != out0) == 0ull;

    // global -> LDS copy plan: see the attention kernels.
    uint32_t k_src[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int krow = (wave * kLoads + j) * (1024 / kRowB) + lane / kKChunks, kpos = lane % kKChunks;
        k_src[j] = krow * kRowB + ((kpos ^ (krow & (kKChunks - 1))) << 4) - 1024u * (j % kGroup);
    }
    const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t wave_lds = smem_base + (uint32_t)wave * (kLoads * 1024);
    const uint32_t k0 = smem_base + idx * kRowB + ((hh ^ (idx & (kKChunks - 1))) << 4);
    // step_kind of 64 key tiles at a time, one per lane; the next 64 masks are fetched a step before their turn
    // (the wait for the tile loads that ends every step covers them).
    struct Key { int kind; uint32_t lo, hi; };
    const uint64_t* vmask_g = a.valid_mask + hg.tile_off;
    uint64_t vm_next = 0ull;
    Key k64;
    auto fetch_masks = [&](int j) __attribute__((always_inline)) { vm_next = j + lane < n ? vmask_g[j + lane] : 0ull; };
    auto key_of = [&](int j) __attribute__((always_inline)) {   // call for j = 0, 1, 2, ... in order
        if ((j & 63) == 0) k64.kind = step_kind(vm_next, k64.lo, k64.hi);
        Key e;
        e.kind = __builtin_amdgcn_readlane(k64.kind, j & 63);
        e.lo = (uint32_t)__builtin_amdgcn_readlane((int)k64.lo, j & 63);
        e.hi = (uint32_t)__builtin_amdgcn_readlane((int)k64.hi, j & 63);
        if ((j & 63) == 62) fetch_masks(j + 2);
        return e;
    };
    auto load_k = [&](int j_tile, const Key& e, int sl) __attribute__((always_inline)) {
        if (e.kind == kStepEmpty || (e.kind == kStepHalf && wave >= 2)) return;   // half: only the first 32 rows are read
        const char* src = kt + (int64_t)j_tile * kKBytes;
        uint32_t moved[2] = {0u, 0u};   // the eight-slot chunks of this wave's first and last eight rows, moved: by how much
        if (e.kind == kStepHalf) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c = 2 * wave + u;
                moved[u] = (((e.hi >> (8 * c)) & 255u) - (uint32_t)c) * (8 * kRowB);
            }
        }
#pragma unroll
        for (int g = 0; g < kLoads / kGroup; ++g) {
            uint32_t off[kGroup];
#pragma unroll
            for (int u = 0; u < kGroup; ++u) off[u] = k_src[g * kGroup + u] + moved[(g * kGroup + u) * 2 / kLoads];
            dma16_group_to_lds<kGroup>(wave_lds + (uint32_t)sl * kKBytes + g * (kGroup * 1024), src, off);
        }
    };
    // The walk over the key tiles: two K tiles in LDS, loads one step ahead.
    Key e0, e1;
    auto walk_begin = [&]() __attribute__((always_inline)) {
        fetch_masks(0);
        e0 = e1 = key_of(0);
        load_k(0, e0, 0);
        wait_vmcnt<0>();
        __syncthreads();
    };
    auto step_begin = [&](int j) __attribute__((always_inline)) {
        if (j + 1 < n) {
            e1 = key_of(j + 1);
            load_k(j + 1, e1, (j + 1) & 1);
        }
    };
    auto step_end = [&]() __attribute__((always_inline)) {
        e0 = e1;
        wait_vmcnt<0>();
        __syncthreads();
    };
#define VEDA_KF(block, f) (*(lds_frag_ptr)(uintptr_t)(kx[f] + (block) * (uint32_t)(32 * kRowB)))   // block 2P, 2P + 1: of slot P

    // Raw dot products of this wave's rows with the 32 keys of an LDS block; `behind(f)` is vector work placed
    // behind the products of fragment f.
    uint32_t kx[kF];   // operand addresses of slot 0's first block; the others are constant distances away
#pragma unroll
    for (int f = 0; f < kF; ++f) kx[f] = k0 ^ (uint32_t)(f << 5);
    // body(j, P) for every key tile j, its slot P = j % 2 a constant
    auto walk = [&](auto body) __attribute__((always_inline)) {
        for (int j = 0;;) {
            body(j, std::integral_constant<uint32_t, 0u>{});
            if (++j == n) break;
            body(j, std::integral_constant<uint32_t, 1u>{});
            if (++j == n) break;
        }
    };
    auto products = [&](f32x16& s, uint32_t block, auto behind) __attribute__((always_inline)) {
        const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        frag kf[kF];
#pragma unroll
        for (int f = 0; f < kAhead; ++f) kf[f] = VEDA_KF(block, f);
#pragma unroll
        for (int f = 0; f < kF; ++f) {
            if (f + kAhead < kF) kf[f + kAhead] = VEDA_KF(block, f + kAhead);
            s = F::mul(kf[f], qf[f], f == 0 ? zero : s);
            behind(f);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // padded keys of a block: register i is key 8*(i/4) + 4*hh + i%4
    auto mask_keys = [&](f32x16& s, uint32_t mask) __attribute__((always_inline)) {
        if (mask == ~0u) return;
        asm volatile("" ::: "memory");   // keeps this a branch, taken at edge tiles only
        // a register's two keys as a lane mask, on the scalar unit: the vector unit is what pass 1 waits for
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int bit = 8 * (i >> 2) + (i & 3);
            const uint32_t lo = (uint32_t)((int)(mask << (31 - bit)) >> 31), up = (uint32_t)((int)(mask << (27 - bit)) >> 31);
            s[i] = __builtin_amdgcn_inverse_ballot_w64((uint64_t)up << 32 | lo) ? s[i] : -INFINITY;
        }
    };
    // relative to ref, log2 units
    auto logit = [&](float x, float ref) __attribute__((always_inline)) { return fmaf(x, a.scale_log2, -ref); };

    // ---- pass 1: reference (log2 units) and denominator of this lane's row over the keys of its lane half ----
    // The denominator is kept as a finished part and that of the last kHeatFold steps, so that its rounding
    // errors grow with the root of those, not of the key tiles.
    float ref = kHeatNoRef, l = 0.0f, l_part = 0.0f;
    // Adds a block's exponentials to the denominator: sum holds them at the present reference.  A row whose sum
    // is out of range (in either lane half) first moves its reference to the block's maximum; the rule looks at
    // the row alone, so results do not depend on which rows share a wave.
    auto settle = [&](const f32x16& s, float sum) __attribute__((always_inline)) {
        if (__builtin_expect(__any(!(sum <= kHeatSlack)), 0)) {
            asm volatile("" ::: "memory");
            const float over = max_with_other_half(sum <= kHeatSlack ? 0.0f : 1.0f);
            float mx = s[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
            mx = max_with_other_half(mx) * a.scale_log2;
            if (over > 0.0f && mx > ref) {
                const float shrink = __builtin_amdgcn_exp2f(ref - mx);
                l *= shrink;
                l_part *= shrink;
                ref = mx;
                sum = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(logit(s[i], mx));
            }
        }
        l_part += sum;
    };
    // One walk: the largest raw logits of this wave's rows, [key tile][32 rows], nothing for tiles without a real key.
    float* const kept = kOneWalk ? a.maxima + ((int64_t)block * 4 + wave) * a.max_tiles * 32 : nullptr;
    if (!kOneWalk && a.have_rows) {
        // nothing to do
    } else if (walk_begin(); active) {
        // s1 holds the block whose exponentials are still to come: they are formed behind the next products, and with
        // them the maximum of its tile, `last`
        f32x16 s0, s1;
        float sum, mx = -INFINITY;
        int last = -1;
        auto maxima = [&](const f32x16& s, int f, bool first) __attribute__((always_inline)) {
            if (!kOneWalk) return;
#pragma unroll
            for (int i = f * kExps; i < (f + 1) * kExps; ++i) mx = fmaxf(first && i == 0 ? -INFINITY : mx, s[i]);
        };
        auto keep = [&]() __attribute__((always_inline)) {
            if (!kOneWalk || last < 0) return;
            float* const rows = kept + (int64_t)last * 32;
            rows[idx] = max_with_other_half(mx);   // alike in both halves
        };
        auto exps = [&](const f32x16& s, int f) __attribute__((always_inline)) {
#pragma unroll
            for (int i = f * kExps; i < (f + 1) * kExps; ++i) {
                const float p = __builtin_amdgcn_exp2f(logit(s[i], ref));
                sum = i == 0 ? p : sum + p;
            }
        };
#pragma unroll
        for (int i = 0; i < 16; ++i) s1[i] = -INFINITY;
        walk([&](int j, auto P) __attribute__((always_inline)) {
            step_begin(j);
            if (e0.kind != kStepEmpty) {
                products(s0, 2u * P, [&](int f) __attribute__((always_inline)) { exps(s1, f); maxima(s1, f, false); });
                asm volatile("" : "+v"(sum), "+v"(mx));   // they stay behind the products: the branches below would take them along
                keep();
                last = j;
                settle(s1, sum);
                mask_keys(s0, e0.lo);
                if (e0.kind == kStepHalf) {
                    // moves of this branch alone: as a plain copy the other branch would carry sixteen as well
#pragma unroll
                    for (int i = 0; i < 16; ++i) s1[i] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s0[i]), 0xE4, 0xf, 0xf, true));   // quad_perm [0,1,2,3]
                    mx = -INFINITY;
                } else {
                    products(s1, 2u * P + 1u, [&](int f) __attribute__((always_inline)) { exps(s0, f); maxima(s0, f, true); });
                    asm volatile("" : "+v"(sum), "+v"(mx));
                    settle(s0, sum);   // before the mask's branch: the exponentials would move behind it
                    mask_keys(s1, e0.hi);
                }
            }
            if ((j & (kHeatFold - 1)) == kHeatFold - 1) {
                l += l_part;
                l_part = 0.0f;
            }
            step_end();
        });
#pragma unroll
        for (int f = 0; f < kF; ++f) { exps(s1, f); maxima(s1, f, false); }
        keep();
        settle(s1, sum);
    } else {   // a wave without rows loads and meets the others
        for (int j = 0; j < n; ++j) {
            step_begin(j);
            step_end();
        }
    }
    float inv_l;
    if (!kOneWalk && a.have_rows) {
        const float2 known = row_sums ? *row_sums : make_float2(0.0f, 0.0f);
        ref = known.x;
        inv_l = known.y;
    } else {
        inv_l = 1.0f / sum_with_other_half(l + l_part);   // the lane halves hold different keys
        if (row_sums && hh == 0) *row_sums = make_float2(ref, inv_l);
    }

    // ---- pass 2: block maxima of exp2(s - ref) / l ----
    // whole-tile score blocks hold a quarter of the half-tile ones
    const int n_cols = kGrouped ? n >> 1 : n;
    float* const heat = a.heat + b * a.score_elems + (kGrouped ? hg.score_off / 4 : hg.score_off);
    float mine = 0.0f;   // plain: block maximum of step 64*m + lane
    // After the barrier that ends step j: every 64 steps, and at the end, the maxima go out, a tile's in one store.
    auto publish = [&](int j) __attribute__((always_inline)) {
        if ((j & 63) != 63 && j != n - 1) return;
        if (active && plain) atomicMax(&part[out0][lane], heat_key(mine));
        __syncthreads();
        for (int o = wave; o < outs; o += 4) {
            float v = heat_of_key(part[o][lane]);
            part[o][lane] = 0u;
            const int from = j & ~63;
            float* const hrow = heat + (int64_t)(kGrouped ? out_tile[0] >> 1 : out_tile[o]) * n_cols;
            if (kGrouped) {
                v = fmaxf(v, __shfl_xor(v, 1));
                if (!(lane & 1) && from + lane <= j) hrow[(from + lane) >> 1] = v;
            } else if (from + lane <= j) {
                hrow[from + lane] = v;
            }
        }
        __syncthreads();
        mine = 0.0f;
    };
    if constexpr (kOneWalk) {
        // A lane takes a key tile and goes through the wave's rows, whose reference and denominator are then scalars.
        __syncthreads();   // what other lanes of this wave kept is read below; the last key tile has been read
        // rows after which another tile's come, or none
        const int next_out = __shfl_down(q_real ? out : -1, 1);   // by all lanes
        uint32_t ends = (uint32_t)__ballot(q_real && (idx == 31 || next_out != out));
        for (int from = 0; from < n; from += 64) {
            if (active) {
                const int tile = from + lane < n ? from + lane : n - 1;
                const float4* src = reinterpret_cast<const float4*>(kept + tile * 32);
                float4 x[8];
#pragma unroll
                for (int g = 0; g < 8; ++g) x[g] = src[g];
                const bool empty = vmask_g[tile] == 0ull;
                asm volatile("" : "+v"(ref), "+v"(inv_l), "+v"(out));   // 96 scalars, formed where they are used: kept, they would spill
                auto take = [&](int i) __attribute__((always_inline)) {
                    const float4& v = x[i >> 2];
                    const float m = (i & 3) == 0 ? v.x : (i & 3) == 1 ? v.y : (i & 3) == 2 ? v.z : v.w;
                    const float row_ref = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ref), i));
                    const float row_inv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv_l), i));
                    return heat_score<E>(logit(m, row_ref), row_inv);
                };
                if (plain) {
                    float best = take(0);
#pragma unroll
                    for (int i = 1; i < 32; ++i) best = fmaxf(best, take(i));
                    mine = empty ? 0.0f : best;
                } else {
                    float best = __builtin_nanf("");   // fmaxf takes the other
                    asm volatile("" : "+s"(rows_real), "+s"(ends));   // so are the tests of their bits
#pragma unroll
                    for (int i = 0; i < 32; ++i) {
                        if ((rows_real >> i) & 1u) best = fmaxf(best, take(i));
                        if ((ends >> i) & 1u) {
                            atomicMax(&part[__builtin_amdgcn_readlane(out, i)][lane], heat_key(empty ? 0.0f : best));
                            best = __builtin_nanf("");
                        }
                    }
                }
            }
            publish(from + 63 < n ? from + 63 : n - 1);
        }
        continue;
    }
    walk_begin();
    if (active) {
        walk([&](int j, auto P) __attribute__((always_inline)) {
            step_begin(j);
            float best = 0.0f;
            if (e0.kind != kStepEmpty) {
                f32x16 s0, s1;
                products(s0, 2u * P, [](int) {});
                mask_keys(s0, e0.lo);
                float mx = s0[0];
                auto maxima = [&](const f32x16& s, int f) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = f * kExps; i < (f + 1) * kExps; ++i) mx = fmaxf(mx, s[i]);
                };
                if (e0.kind == kStepHalf) {
                    s1 = s0;
                } else {
                    products(s1, 2u * P + 1u, [&](int f) __attribute__((always_inline)) { maxima(s0, f); });
                    asm volatile("" : "+v"(mx));   // the maxima stay behind the products
                    mask_keys(s1, e0.hi);
                }
#pragma unroll
                for (int f = 0; f < kF; ++f) maxima(s1, f);
                const float score = heat_score<E>(logit(max_with_other_half(mx), ref), inv_l);
                if (plain) best = rows_max(score);
                else if (q_real && hh == 0) atomicMax(&part[out][j & 63], heat_key(score));
            } else if (!plain && q_real && hh == 0) {
                atomicMax(&part[out][j & 63], heat_key(0.0f));
            }
            mine = lane == (j & 63) ? best : mine;
            step_end();
            publish(j);
        });
    } else {
        for (int j = 0; j < n; ++j) {
            step_begin(j);
            step_end();
            publish(j);
        }
    }
    }   // tiles of the item
    };   // run
#undef VEDA_KF

    // With more items than places in the scratch a workgroup goes on with the next one of its die.  Handed out as they
    // are asked for: a fixed share each left a quarter of the chip idle at the end where tiles differ (one in 16 of 40
    // heads of 21x45x80, mixed shapes).
    const uint32_t die = block % kXcd;
    uint32_t* const next = reinterpret_cast<uint32_t*>(out_tile + kHeatTiles);
    for (uint32_t work = block;;) {
        run(work);
        if (!kOneWalk || a.taken == nullptr) return;
        if (tid == 0) *next = (gridDim.x / kXcd + atomicAdd(a.taken + die * kHeatTakenStride, 1u)) * kXcd + die;
        __syncthreads();
        work = (uint32_t)__builtin_amdgcn_readfirstlane((int)*next);
        __syncthreads();
        if (work >= a.items * a.batch) return;
    }
}

__global__ void heat_taken_clear_kernel(uint32_t* taken) { taken[threadIdx.x * kHeatTakenStride] = 0u; }

// Recall@k: a wavefront counts, row by row, the key tiles the two kept lists share (lists of
// distinct tiles in any order); integer atomics keep the per-head totals order-independent.
// The tiles of list b become a bitmap in LDS that those of list a are looked up in (12 heads
// of 624 rows at k = 63: 85 us comparing all pairs, 22 us so; 40 heads of 21x45x80, 5 % kept: 516 and 89 us).  Rows longer than the
// bitmap, or with an entry that is no tile of theirs, compare all pairs.
struct RecallArgs {
    int32_t k[kMaxHeads];
    int64_t col_off[kMaxHeads];
    int64_t nnz_per_batch;
};

constexpr int kRecallWords = 512;   // bitmap words of a row: 16384 key tiles
// Consecutive rows of a wavefront, to save atomics on the totals.  One, two, four and eight: 12 heads of 624 rows 76, 40,
// 24.5 and 20 us for the whole call; 40 heads of 1440 385, 218, 114 and 62; 4 heads of 75 9.4, 8.4, 9.1 and 12.5 (too few
// wavefronts).
constexpr int kRecallRows = 4;

__global__ __launch_bounds__(256) void recall_count_kernel(const HeadGeom* __restrict__ heads,
                                                           const uint8_t* __restrict__ tile_head, RecallArgs args,
                                                           const int32_t* __restrict__ col_a,
                                                           const int32_t* __restrict__ col_b,
                                                           unsigned long long* __restrict__ counts,
                                                           int64_t total_tiles, int64_t rows, int n_heads) {
    __shared__ uint32_t bitmap[4][kRecallWords];
    const int lane = threadIdx.x & 63;
    uint32_t* bits = bitmap[threadIdx.x >> 6];
    const int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kRecallRows;
    int64_t total_of = -1;   // (batch, head) that `common` counts for
    int common = 0;
    auto sync = []() {   // LDS of one wavefront: its own operations in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int64_t row = first; row < first + kRecallRows && row < rows; ++row) {
        const int64_t b = row / total_tiles, g = row - b * total_tiles;
        const int head = tile_head[g], n = heads[head].n_tiles;
        const int k = args.k[head];
        if (b * n_heads + head != total_of) {
            if (lane == 0 && common) atomicAdd(&counts[total_of], (unsigned long long)common);
            total_of = b * n_heads + head;
            common = 0;
        }
        const int64_t off = b * args.nnz_per_batch + args.col_off[head] + (g - heads[head].tile_off) * k;
        const int32_t* la = col_a + off;
        const int32_t* lb = col_b + off;
        bool strange = n > 32 * kRecallWords;
        if (!strange) {
            for (int w = lane; w < (n + 31) / 32; w += 64) bits[w] = 0u;
            sync();
            for (int y = lane; y < k; y += 64) {
                const int v = lb[y];
                if ((unsigned)v < (unsigned)n) atomicOr(&bits[v >> 5], 1u << (v & 31));
                else strange = true;
            }
            sync();
            int hits = 0;
            for (int x = lane; x - lane < k; x += 64) {
                const int v = x < k ? la[x] : 0;
                if ((unsigned)v >= (unsigned)n) strange = true;
                hits += __popcll(__ballot(x < k && (unsigned)v < (unsigned)n && ((bits[v >> 5] >> (v & 31)) & 1u)));
            }
            sync();   // before the next row's bitmap
            strange = __any(strange);
            if (!strange) common += hits;
        }
        if (strange) {
            for (int x = 0; x < k; ++x) {
                const int want = la[x];
                bool hit = false;
                for (int y = lane; y < k; y += 64) hit |= lb[y] == want;
                common += __any(hit) ? 1 : 0;
            }
        }
    }
    if (lane == 0 && common) atomicAdd(&counts[total_of], (unsigned long long)common);
}

__global__ void recall_clear_kernel(unsigned long long* counts, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) counts[i] = 0ull;
}

__global__ void recall_finish_kernel(const HeadGeom* __restrict__ heads, RecallArgs args,
                                     const unsigned long long* __restrict__ counts, float* __restrict__ recall,
                                     int n_heads, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int head = i % n_heads;
    recall[i] = (float)((double)counts[i] / ((double)heads[head].n_tiles * (double)args.k[head]));
}

}  // namespace veda

namespace veda {

constexpr size_t kHeatTakenBytes = kXcd * kHeatTakenStride * sizeof(uint32_t);   // at the start of the scratch

static int64_t heat_item_count(const veda_plan* pl, int64_t n_listed) {
    const veda_plan* ip = pl->inner ? pl->inner : pl;
    return n_listed == 0 ? (int64_t)ip->heat_blocks : pl->inner ? n_listed : list_blocks(n_listed, pl->prob.heads);
}

static int64_t heat_max_tiles(const veda_plan* pl) {
    const veda_plan* ip = pl->inner ? pl->inner : pl;
    int64_t n = 0;
    for (const HeadGeom& g : ip->heads) n = g.n_tiles > n ? g.n_tiles : n;
    return n;
}

// One walk: the workgroups of a launch, each with a place in the scratch.  As many as are resident at once, fewer where their
// scratch would pass 2 GiB, down to half (a head of 8192 tiles in bf16: 76.8 ms on 1024 places, 4.3 GB; 90.6 on 512; 132 in two walks
// without scratch).
static int64_t heat_places(const veda_plan* pl, bool listed) {
    const int64_t all = 256 * heat_resident(pl->prob.dtype == VEDA_BF16, pl->prob.head_dim, pl->inner != nullptr, listed);
    const int64_t fit = (((int64_t)2 << 30) - (int64_t)kHeatTakenBytes) / (heat_max_tiles(pl) * 128 * (int64_t)sizeof(float)) / kXcd * kXcd;
    return fit >= all ? all : fit > all / 2 ? fit : all / 2;
}

}  // namespace veda

// All entry points; rows: optional row sums, read if have_rows; workspace: optional.
static veda_status target_heatmap(const veda_plan* pl, const void* q_tiled, const void* k_tiled, const uint64_t* valid_mask,
                                  float softmax_scale, const int32_t* query_tiles, int64_t n_query_tiles, float2* rows,
                                  int have_rows, float* heat, void* workspace, size_t workspace_bytes, void* stream) {
    using namespace veda;
    if (!pl || !q_tiled || !k_tiled || !valid_mask || !heat) return VEDA_ERR_INVALID_ARG;
    if (!(softmax_scale > 0.0f) || !(softmax_scale < INFINITY)) return VEDA_ERR_INVALID_ARG;
    if (query_tiles ? (n_query_tiles < 1 || n_query_tiles > pl->total_tiles) : n_query_tiles != 0)
        return VEDA_ERR_INVALID_ARG;
    if (!aligned16(q_tiled) || !aligned16(k_tiled)) return VEDA_ERR_UNSUPPORTED;
    const int d = pl->prob.head_dim;
    const bool bf16 = pl->prob.dtype == VEDA_BF16;
    // 128-token tiles (bf16 only): the kernel walks their 64-slot halves, heat counts whole tiles
    const veda_plan* ip = pl->inner ? pl->inner : pl;
    HeatArgs a;
    a.heads = ip->d_heads;
    a.tile_head = ip->d_tile_head;
    a.query_tiles = query_tiles;
    a.n_query_tiles = query_tiles ? n_query_tiles : 0;
    a.q = (const char*)q_tiled; a.k = (const char*)k_tiled;
    a.valid_mask = valid_mask;
    a.heat = heat;
    a.total_tiles = ip->total_tiles;
    a.score_elems = pl->score_elems;
    a.n_heads = pl->prob.heads;
    a.scale_log2 = softmax_scale * kLog2e;
    a.rows = rows;
    a.have_rows = have_rows;
    a.tokens = pl->tokens();
    a.T = pl->prob.T; a.H = pl->prob.H; a.W = pl->prob.W;
    hipStream_t s = (hipStream_t)stream;
    a.table = ip->d_heat_items;
    const int64_t items = heat_item_count(pl, a.n_query_tiles);
    a.items = (uint32_t)items;
    a.batch = (uint32_t)pl->prob.batch;
    a.maxima = nullptr;
    a.taken = nullptr;
    a.max_tiles = heat_max_tiles(pl);
    int64_t blocks = items * pl->prob.batch;
    if (blocks > 0x7fffffff) return VEDA_ERR_UNSUPPORTED;
    if (workspace) {
        if (reinterpret_cast<uintptr_t>(workspace) & 15u) return VEDA_ERR_UNSUPPORTED;
        const int64_t places = heat_places(pl, query_tiles != nullptr);
        const bool share = blocks > places;
        blocks = share ? places : blocks;
        if (workspace_bytes < kHeatTakenBytes + (size_t)(blocks * a.max_tiles) * 128 * sizeof(float)) return VEDA_ERR_WORKSPACE;
        a.maxima = reinterpret_cast<float*>((char*)workspace + kHeatTakenBytes);
        if (share) {
            a.taken = reinterpret_cast<uint32_t*>(workspace);
            hipLaunchKernelGGL(heat_taken_clear_kernel, dim3(1), dim3(kXcd), 0, s, a.taken);
        }
    }
    // a dimension holds fewer than 2^32 threads: samples of many padding workgroups go along the second
    dim3 grid((unsigned)blocks), block(256);
    if (blocks >= (int64_t)1 << 24) grid = dim3((unsigned)items, (unsigned)pl->prob.batch);
    const size_t smem = (size_t)2 * kTile * d * pl->elem_size() + kHeatTiles * (64 + 1) * sizeof(uint32_t) + 16;
    auto launch = [&](auto kern) {
        if (smem > 64 * 1024)
            VEDA_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        hipLaunchKernelGGL(kern, grid, block, smem, s, a);
        return launch_status("veda_tile_heatmap");
    };
#define VEDA_LAUNCH_HEAT(E, DD, GG)                                                                      \
    (workspace ? query_tiles ? launch(tile_heatmap_kernel<E, DD, GG, true, true>)                        \
                             : launch(tile_heatmap_kernel<E, DD, GG, false, true>)                       \
               : query_tiles ? launch(tile_heatmap_kernel<E, DD, GG, true, false>)                       \
                             : launch(tile_heatmap_kernel<E, DD, GG, false, false>))
    if (bf16 && pl->inner) return d == 128 ? VEDA_LAUNCH_HEAT(uint16_t, 128, true) : VEDA_LAUNCH_HEAT(uint16_t, 64, true);
    if (bf16) return d == 128 ? VEDA_LAUNCH_HEAT(uint16_t, 128, false) : VEDA_LAUNCH_HEAT(uint16_t, 64, false);
    return d == 128 ? VEDA_LAUNCH_HEAT(uint32_t, 128, false) : VEDA_LAUNCH_HEAT(uint32_t, 64, false);
#undef VEDA_LAUNCH_HEAT
}

extern "C" size_t veda_plan_heatmap_workspace_bytes(const veda_plan* pl, int64_t n_query_tiles) {
    using namespace veda;
    if (!pl || n_query_tiles < 0 || n_query_tiles > pl->total_tiles) return 0;
    const int64_t blocks = heat_item_count(pl, n_query_tiles) * pl->prob.batch, places = heat_places(pl, n_query_tiles > 0);
    return kHeatTakenBytes + (size_t)((blocks < places ? blocks : places) * heat_max_tiles(pl)) * 128 * sizeof(float);
}

extern "C" veda_status veda_tile_heatmap(const veda_plan* pl, const void* q_tiled, const void* k_tiled,
                                         const uint64_t* valid_mask, float softmax_scale,
                                         const int32_t* query_tiles, int64_t n_query_tiles, float* heat,
                                         void* stream) {
    return target_heatmap(pl, q_tiled, k_tiled, valid_mask, softmax_scale, query_tiles, n_query_tiles, nullptr, 0, heat, nullptr, 0,
                          stream);
}

extern "C" veda_status veda_tile_heatmap_ws(const veda_plan* pl, const void* q_tiled, const void* k_tiled,
                                            const uint64_t* valid_mask, float softmax_scale, const int32_t* query_tiles,
                                            int64_t n_query_tiles, float* row_sums, float* heat, void* workspace,
                                            size_t workspace_bytes, void* stream) {
    // a list that has no size of scratch is a bad list, not too little scratch
    if (!pl || (query_tiles ? n_query_tiles < 1 || n_query_tiles > pl->total_tiles : n_query_tiles != 0)) return VEDA_ERR_INVALID_ARG;
    if (!workspace) return VEDA_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(row_sums) & 7u) return VEDA_ERR_UNSUPPORTED;
    return target_heatmap(pl, q_tiled, k_tiled, valid_mask, softmax_scale, query_tiles, n_query_tiles,
                          reinterpret_cast<float2*>(row_sums), 0, heat, workspace, workspace_bytes, stream);
}

extern "C" veda_status veda_tile_heatmap_rows(const veda_plan* pl, const void* q_tiled, const void* k_tiled,
                                              const uint64_t* valid_mask, float softmax_scale, float* row_sums,
                                              int32_t have_row_sums, float* heat, void* stream) {
    if (!row_sums || have_row_sums < 0 || have_row_sums > 1) return VEDA_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(row_sums) & 7u) return VEDA_ERR_UNSUPPORTED;
    return target_heatmap(pl, q_tiled, k_tiled, valid_mask, softmax_scale, nullptr, 0, reinterpret_cast<float2*>(row_sums),
                          have_row_sums, heat, nullptr, 0, stream);
}

extern "C" veda_status veda_tile_recall(const veda_plan* pl, const int32_t* k_per_head, const int32_t* col_idx_a,
                                        const int32_t* col_idx_b, float* recall, void* workspace,
                                        size_t workspace_bytes, void* stream) {
    using namespace veda;
    if (!pl || !k_per_head || !col_idx_a || !col_idx_b || !recall) return VEDA_ERR_INVALID_ARG;
    const int n = pl->prob.batch * pl->prob.heads;
    if (!workspace || workspace_bytes < sizeof(unsigned long long) * (size_t)n) return VEDA_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 7u) return VEDA_ERR_UNSUPPORTED;
    RecallArgs args;
    int64_t off = 0;
    for (int h = 0; h < pl->prob.heads; ++h) {
        const int nt = pl->heads[h].n_tiles;
        if (k_per_head[h] < 1 || k_per_head[h] > nt) return VEDA_ERR_INVALID_ARG;
        args.k[h] = k_per_head[h];
        args.col_off[h] = off;
        off += (int64_t)nt * k_per_head[h];
    }
    args.nnz_per_batch = off;
    hipStream_t s = (hipStream_t)stream;
    unsigned long long* counts = (unsigned long long*)workspace;
    const int64_t rows = pl->total_tiles * pl->prob.batch;
    hipLaunchKernelGGL(recall_clear_kernel, dim3((n + 255) / 256), dim3(256), 0, s, counts, n);
    hipLaunchKernelGGL(recall_count_kernel, dim3((unsigned)((rows + 4 * kRecallRows - 1) / (4 * kRecallRows))), dim3(256), 0, s,
                       pl->d_heads, pl->d_tile_head, args, col_idx_a, col_idx_b, counts, pl->total_tiles, rows, pl->prob.heads);
    hipLaunchKernelGGL(recall_finish_kernel, dim3((n + 255) / 256), dim3(256), 0, s, pl->d_heads, args, counts,
                       recall, pl->prob.heads, n);
    return launch_status("veda_tile_recall");
}

// ---- squared Frobenius distance between two token-order tensors, per (batch, head) ----------
// (Eq. 8 / Alg. 1: the error a candidate tiling is scored by).  Two deterministic stages: 64
// workgroups per (batch, head) each reduce a contiguous share of the tokens in double precision
// (fixed tree inside the workgroup), then one thread adds the 64 partial sums in order.
namespace veda {

constexpr int kErrParts = 64;

template <typename E> __device__ __forceinline__ float err_elem(const char* p, int c);
template <> __device__ __forceinline__ float err_elem<uint16_t>(const char* p, int c) {
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(p)[c] << 16);
}
template <> __device__ __forceinline__ float err_elem<uint32_t>(const char* p, int c) {
    return reinterpret_cast<const float*>(p)[c];
}

template <typename E>
__global__ __launch_bounds__(256) void sqerr_partial_kernel(const char* __restrict__ a, int64_t ab, int64_t ah, int64_t an,
                                                            const char* __restrict__ b, int64_t bb, int64_t bh, int64_t bn,
                                                            double* __restrict__ partial, int64_t tokens, int d,
                                                            int n_heads) {
    __shared__ double red[256];
    const int part = blockIdx.x, head = blockIdx.y, bt = blockIdx.z;
    const int64_t per = (tokens + kErrParts - 1) / kErrParts;
    const int64_t lo = part * per, hi = lo + per < tokens ? lo + per : tokens;
    const char* pa = a + bt * ab + head * ah;
    const char* pb = b + bt * bb + head * bh;
    double acc = 0.0;
    for (int64_t e = lo * d + threadIdx.x; e < hi * d; e += 256) {
        const int64_t n = e / d;
        const int c = (int)(e - n * d);
        const float diff = err_elem<E>(pa + n * an, c) - err_elem<E>(pb + n * bn, c);
        acc += (double)diff * (double)diff;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[((int64_t)bt * n_heads + head) * kErrParts + part] = red[0];
}

__global__ void sqerr_finish_kernel(const double* __restrict__ partial, double* __restrict__ err, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = 0.0;
    for (int p = 0; p < kErrParts; ++p) acc += partial[(int64_t)i * kErrParts + p];
    err[i] = acc;
}

}  // namespace veda

extern "C" veda_status veda_output_sqerr(const veda_plan* pl, const void* a, veda_strides sa, const void* b,
                                         veda_strides sb, double* err, void* workspace, size_t workspace_bytes,
                                         void* stream) {
    using namespace veda;
    if (!pl || !a || !b || !err) return VEDA_ERR_INVALID_ARG;
    const int d = pl->prob.head_dim, es = pl->elem_size();
    if (sa.n < d || sb.n < d || sa.b < 0 || sa.h < 0 || sb.b < 0 || sb.h < 0) return VEDA_ERR_INVALID_ARG;
    const int n = pl->prob.batch * pl->prob.heads;
    if (!workspace || workspace_bytes < sizeof(double) * (size_t)n * kErrParts) return VEDA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 7u) || (reinterpret_cast<uintptr_t>(err) & 7u)) return VEDA_ERR_UNSUPPORTED;
    hipStream_t s = (hipStream_t)stream;
    double* partial = (double*)workspace;
    dim3 grid(kErrParts, (unsigned)pl->prob.heads, (unsigned)pl->prob.batch);
    if (es == 2)
        hipLaunchKernelGGL(sqerr_partial_kernel<uint16_t>, grid, dim3(256), 0, s, (const char*)a, sa.b * es, sa.h * es,
                           sa.n * es, (const char*)b, sb.b * es, sb.h * es, sb.n * es, partial, pl->tokens(), d,
                           pl->prob.heads);
    else
        hipLaunchKernelGGL(sqerr_partial_kernel<uint32_t>, grid, dim3(256), 0, s, (const char*)a, sa.b * es, sa.h * es,
                           sa.n * es, (const char*)b, sb.b * es, sb.h * es, sb.n * es, partial, pl->tokens(), d,
                           pl->prob.heads);
    hipLaunchKernelGGL(sqerr_finish_kernel, dim3((n + 255) / 256), dim3(256), 0, s, partial, err, n);
    return launch_status("veda_output_sqerr");
}
