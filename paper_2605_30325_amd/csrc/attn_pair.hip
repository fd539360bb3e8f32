// Stage 4, bf16, query-tile-pair kernel (Eq. 2; Sec. 4.3 tile skipping; Alg. 1 "UnTile").
//
// A compute unit can pull K/V tiles from L2 into LDS at 64 bytes per clock at most, and a kept
// tile pair needs 32 KB of them for 512 matrix-pipe cycles of work: with one query tile per
// workgroup the loads, not the matrix cores, set the pace.  Neighbouring query tiles keep
// largely the same key tiles, so here one workgroup owns TWO neighbouring query tiles (partners
// along the axis in which the head's tile shape is thinnest: pair_tiles()) and walks the union
// of their two kept lists: a key tile kept by both is loaded once and used twice.  (Calls of few
// tiles, which leave room for a workgroup each, walk one list: plan.hip.)
//
// Four wavefronts of 32 query rows: two for each of the two tiles, or one for each of FOUR neighbouring thin tiles (32
// real rows or fewer, at the ragged edges of a grid: geometry.h, attn_items).  Every wave attends to all 64 slots of a
// key tile, so it needs no merge with another wave at the end.  A wave whose query tile does not keep the current key
// tile skips the step and only meets the others at the barrier; the matrix cores it leaves idle go to the
// second workgroup resident on the compute unit.
//
// Padding costs little: a query tile's real rows come first, so a wave beyond them idles, and a key tile
// with few real keys is a half step (attn_union.h).  The attention call alone, repeated, in turn on one box: on a
// 21 x 30 x 52 grid with 4x4x4 tiles, where 27 % of the tiles are such, 12 heads with every tile kept 7.9 -> 6.9 ms and
// with 10 % kept 0.98 -> 0.81; on 61 x 45 x 80, with few of them, 24 heads at 5 % kept 32.5 -> 32.15 ms.
// Thin tiles used to run two to a workgroup with half its waves idle.  Four together walk 1.3-2.0 times their list's length
// instead of 2 x 1.2-1.4, and their workgroups, the longest, start first and are spread evenly over the dies (left in
// raster order all of a head's last layer fell to one or two dies: 12 heads of 21x30x52 5 % slower than in twos).
// Whole calls, in turn on one box: 40 heads of 21x45x80 at 20 % kept (28 % of the tiles are thin) 33.0 -> 29.5 ms, of
// 21x30x52 at 5 % 2.05 -> 1.89; 12 heads of 21x30x52 at 10 % 0.943 -> 0.907, all kept 6.95 -> 6.44.
//
// The products are formed transposed (S^T = K Q^T, O^T = V^T P^T): a lane owns one query, its
// accumulator registers run over keys, P^T in registers already is the B operand of the second
// product.  K rows are loaded permuted by rho (bits 2,3 swapped) so that the eight keys a
// lane-half owns are contiguous in the channel-major V tile.  One step of one wave:
//     S^T block 0 (8 MFMA; in their shadow the wave's share of the NEXT tiles' global->LDS loads
//                  and the fetch of the step after next)
//     S^T block 1 (8 MFMA; in their shadow the row maximum of block 0 and, speculatively, the
//                  first 8 exponentials)
//     one comparison: need the reference move, has the tile padded slots?   (rarely: the slow path)
//     4 x [ 4 MFMA of O^T += V^T P^T ; the next 8 exponentials in their shadow ]   (at raised wave priority)
// K/V tiles are double buffered (2 x 32 KB at d = 128) and filled by direct global->LDS loads
// issued one step ahead.  Which key tile comes at which step is worked out before the loop, by all
// threads together, into a table in LDS (attn_union.h): a scalar-memory round trip inside the loop
// would make every wait for an LDS operand a wait for everything.
#include "attn_step.h"
#include "attn_union.h"

namespace veda {

// After the last step: normalise, transpose through LDS and scatter the real rows of the workgroup's four
// wavefronts to token order.  obuf: [4 wavefronts][32 rows][D] bf16, then lse_s; tok_s: token of each row, -1 = none.
template <int D>
__device__ __forceinline__ void finish_pair(const PairState<D>& st, const AttnArgs& a, const int* tok_s, char* smem,
                                            int head, int64_t b, int tid, int wave, int lq, int hh) {
    constexpr int kRowB = D * 2, kKChunks = kRowB / 16;
    const float l_all = st.l_run + __shfl_xor(st.l_run, 32);
    const float inv = l_all > 0.0f ? 1.0f / l_all : 0.0f;
    char* obuf = smem;
    float* lse_s = reinterpret_cast<float*>(smem + 4 * 32 * kRowB);   // [4][32]
    __syncthreads();
    {
        char* orow = obuf + (wave * 32 + lq) * kRowB;
#pragma unroll
        for (int nb = 0; nb < D / 32; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int d0 = 32 * nb + 8 * j + 4 * hh;
                typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
                bf16x4 pk;
#pragma unroll
                for (int t = 0; t < 4; ++t) pk[t] = (__bf16)(st.o[nb][4 * j + t] * inv);
                *reinterpret_cast<bf16x4*>(orow + d0 * 2) = pk;
            }
        if (hh == 0) lse_s[wave * 32 + lq] = (st.ref * st.resid + __log2f(l_all)) * kLn2;
    }
    __syncthreads();
    char* ob = a.out + b * a.so_b + head * a.so_h;
    for (int cid = tid; cid < 4 * 32 * kKChunks; cid += 256) {
        const int row = cid / kKChunks, ch = cid % kKChunks;
        const int n = tok_s[row];
        if (n >= 0)
            *reinterpret_cast<uint4*>(ob + (int64_t)n * a.so_n + ch * 16) =
                *reinterpret_cast<const uint4*>(obuf + row * kRowB + ch * 16);
    }
    if (a.lse && tid < 4 * 32) {
        const int n = tok_s[tid];
        if (n >= 0) a.lse[(b * a.n_heads + head) * a.tokens + n] = lse_s[tid];
    }
}

// One step of the merged walk over the kept lists of the two query tiles of a workgroup.
struct MergedStep {
    int j;         // key tile (head-local)
    int fl;        // bit 0: tile A keeps it, bit 1: tile B keeps it; the kind of step; 0 = past the end
    uint64_t vm;   // validity mask of key tile j; half steps: gathered mask | source chunks << 32
    int n0;        // K from token order: token index of its slot 0
};

// kGrouped: 128-token tiles.  The geometry in `a` is that of the 64-slot halves (tiles 2o, 2o+1
// of whole tile o): the workgroup's pair IS one whole query tile, both halves keep the same list
// (the CSR rows and entries count whole tiles), and every entry expands to its two halves.
// kTokK: K is read from token order (a.k_tok) instead of the tiled tensor: a key tile's rows
// are found at first-token + (lt*H + lh)*W + lw; the rows of padded slots are fetched from slot 0
// instead (any finite or non-finite value will do: their logits are overwritten with -inf).
// kTable: the steps come from a table in LDS built before the main loop (attn_union.h; heads of up
// to 16384 whole tiles); otherwise the lists are walked with scalar loads as the loop goes.
constexpr int kPairChunk = 128;   // step-table entries filled at a time

template <int D, bool kGrouped, bool kTokK, bool kExact, bool kTable>
__global__ __launch_bounds__(256, 2) void sparse_attn_bf16_pair_kernel(AttnArgs a) {
    constexpr int kRowB = D * 2;                 // bytes of one K row
    constexpr int kKBytes = kTile * kRowB;       // K tile
    constexpr int kVBytes = D * kTile * 2;       // V^T tile: D rows of 128 bytes
    constexpr int kSlot = kKBytes + kVBytes;     // one LDS slot: K tile then V^T tile
    constexpr int kKChunks = kRowB / 16;         // 16-byte chunks per K row
    constexpr int kLoads = kKBytes / 1024 / 4;   // direct-load instructions per wave per tile (K; same for V)
    constexpr int G = D / 16, NB = D / 32;
    constexpr int kLists = kGrouped ? 1 : kTable ? 4 : 2;   // kept lists of a workgroup, at most
    typedef UnionLds<kLists, kPairChunk> Table;
    extern __shared__ __align__(1024) char smem[];   // base bits 4-9 clear: see PairAddr

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, hh = lane >> 5;

    AttnItem it;
    if (!attn_work<kTable>(a, it)) return;
    const int head = it.head;
    const HeadGeom hg = a.heads[head];
    const int64_t b = blockIdx.y;
    const uint32_t place = it.waves >> (8 * wave);
    const int which = place & 3u, r = place & kItemSecond ? 1 : 0;
    const int qi = which == 0 ? it.tile[0] : which == 1 ? it.tile[1] : which == 2 ? it.tile[2] : it.tile[3];
    const int64_t row0 = kGrouped ? b * (a.total_tiles / 2) + hg.tile_off / 2 : b * a.total_tiles + hg.tile_off;
    const int lists = kGrouped ? 1 : it.n_tiles;
    int beg[kLists], cnt[kLists];
#pragma unroll
    for (int t = 0; t < kLists; ++t) {
        const int64_t row = row0 + (kGrouped ? it.tile[0] >> 1 : it.tile[t]);
        beg[t] = a.row_ptr[row];
        cnt[t] = t < lists ? a.row_ptr[row + 1] - beg[t] : 0;
    }
    // The kept lists and the validity masks are read-only for the whole launch and indexed
    // uniformly: reading them through the constant address space makes them scalar loads, so
    // no vector-memory counter waits of the compiler's own end up inside the main loop.
    typedef const __attribute__((address_space(4))) int32_t* const_i32_t;
    typedef const __attribute__((address_space(4))) uint64_t* const_u64_t;
    const const_i32_t colsA = (const_i32_t)(uintptr_t)(a.col_idx + beg[0]);
    const const_i32_t colsB = (const_i32_t)(uintptr_t)(a.col_idx + beg[kLists == 2 ? 1 : 0]);
    const int nA = cnt[0], nB = kLists == 2 ? cnt[kLists == 2 ? 1 : 0] : 0;   // walk mode
    const const_u64_t vmask = (const_u64_t)(uintptr_t)(a.valid_mask + hg.tile_off);
    const int64_t head_tile0 = b * a.total_tiles + hg.tile_off;
    const char* kt = kTokK ? a.k_tok + b * a.sk_b + head * a.sk_h : a.k + head_tile0 * kKBytes;
    const char* vt = a.v + head_tile0 * kVBytes;
    const const_i32_t n0s = (const_i32_t)(uintptr_t)(a.tile_n0 + hg.tile_off);

    const int list_range = kGrouped ? hg.n_tiles / 2 : hg.n_tiles;
    const uint64_t* vmask_g = a.valid_mask + hg.tile_off;
    const int32_t* n0s_g = a.tile_n0 + hg.tile_off;
    UnionEarly<kLists, 256, kGrouped> early;
    const int32_t* cols[kLists];
    if constexpr (kTable) {
#pragma unroll
        for (int t = 0; t < kLists; ++t) cols[t] = a.col_idx + beg[t];
        early.ask(cols, cnt, lists, list_range, vmask_g, n0s_g, tid);
        __builtin_amdgcn_sched_barrier(0);   // before Q's rows: loads return in order, and the table is what is waited for
    }

    // Q operand (B matrix of S^T = K Q^T): lane holds query row 32r+lq, channels 16t+8hh..+8.
    // Rows are the real slots of the query tile in order: with padding among its 64 slots a tile at a ragged
    // edge fills fewer rows, and a wave whose 32 rows are all beyond the real ones has nothing to compute.
    PairState<D> st;
    const uint64_t q_real = ((const_u64_t)(uintptr_t)(a.tile_real + hg.tile_off))[qi];
    const int q_rows = place & kItemIdle ? 0 : __popcll(q_real);
    int* tok_s = reinterpret_cast<int*>(smem + 2 * kSlot + (kTable ? sizeof(Table) : 0));   // [4][32] token of each row, -1 = none
    const bool real = 32 * r + lq < q_rows;
    {
        // from the tiled tensor, or straight from token order
        const char* qrow;
        int slot = 32 * r + lq;
        if (q_real != ~0ull) slot = real ? nth_bit(q_real, slot) : 0;
        const int n = real ? token_from(hg, n0s[qi], slot, a.H, a.W) : 0;
        if (hh == 0) tok_s[wave * 32 + lq] = real ? n : -1;
        if (a.q_tok) {
            qrow = a.q_tok + b * a.sq_b + head * a.sq_h + (int64_t)n * a.sq_n + 16 * hh;
        } else {
            qrow = a.q + (head_tile0 + qi) * kKBytes + slot * kRowB + 16 * hh;
        }
#pragma unroll
        for (int t = 0; t < G; ++t) st.qf[t] = *reinterpret_cast<const bf16x8*>(qrow + 32 * t);
    }
    auto scale_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < G; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                st.qf[t][e] = real ? (__bf16)((float)st.qf[t][e] * (kExact ? a.scale_pow2 : a.scale_log2)) : (__bf16)0.0f;
    };
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.o[nb][i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) st.start[i] = 0.0f;
    st.ref = st.l_run = 0.0f;
    st.resid = kExact ? a.scale_resid : 1.0f;
    st.started = false;

    // global -> LDS copy plan.  One wave instruction fills 1 KB of LDS, lane i at byte 16*i, so
    // the swizzle is applied on the global side: each lane fetches the chunk that belongs at
    // its fixed LDS position.  Wave w issues instructions w*kLoads .. w*kLoads+kLoads-1 of each
    // tile, all with one LDS base: instruction j carries the immediate offset 1024*j, which the
    // hardware adds to the LDS address AND to the global address, so every per-lane global offset
    // below is stored with 1024*j taken off again (plus kBias where it could go negative, the tile's
    // base address being lowered by the same amount).
    constexpr uint32_t kBias = kTokK ? 1024u * (kLoads - 1) : 0u;
    uint32_t k_src[kLoads], v_src[kLoads];
    uint32_t k_src0[kLoads];   // kTokK: the same chunk of the tile's anchor row
    int k_row[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int inst = wave * kLoads + j;
        const int krow = inst * (1024 / kRowB) + lane / kKChunks, kpos = lane % kKChunks;
        const uint32_t chunk = (uint32_t)((kpos ^ (rho(krow & 31) & (kKChunks - 1))) << 4);
        k_row[j] = krow;
        k_src0[j] = chunk + kBias - 1024u * j;
        if (kTokK) {   // byte offset of the row's token from the tile's anchor token (host checked: fits 32 bits)
            k_src[j] = (uint32_t)(token_from(hg, 0, krow, a.H, a.W) * a.sk_n) + chunk + kBias - 1024u * j;
        } else {
            k_src[j] = krow * kRowB + chunk - 1024u * j;
        }
        const int vrow = inst * 8 + (lane >> 3), vpos = lane & 7;
        v_src[j] = vrow * 128 + ((vpos ^ (((vrow >> 1) & 7) ^ ((vrow & 1) << 2))) << 4) - 1024u * j;
    }
    const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t wave_lds = smem_base + (uint32_t)wave * (kLoads * 1024);
    // Half steps: byte offset of slots 8, 16 and 32 from slot 0 (the extents of a tile are powers of two, so the
    // offset of any chunk of eight slots is the sum over the bits of its number), and this lane's V^T chunk:
    // chunk v_c in even instructions, v_c ^ 4 in odd ones.
    uint32_t k_chunk[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int sl = 8 << i;
        k_chunk[i] = kTokK ? (uint32_t)(token_from(hg, 0, sl, a.H, a.W) * a.sk_n) : (uint32_t)(sl * kRowB);
    }
    const int v_c = (lane & 7) ^ ((lane >> 4) & 3) ^ (((lane >> 3) & 1) << 2);
    auto chunk_off = [&](uint32_t c) __attribute__((always_inline)) {
        return ((c & 1u) ? k_chunk[0] : 0u) + ((c & 2u) ? k_chunk[1] : 0u) + ((c & 4u) ? k_chunk[2] : 0u);
    };
    // The K tile (what = 0) or the V^T tile (what = 1) of step e into LDS slot `sl`; nothing for an empty one or past the end.
    auto load_tile = [&](const MergedStep& e, int sl, int what) __attribute__((always_inline)) {
        uint32_t off[kLoads];
        if (what == 0) {
            const char* src = (kTokK ? kt + (int64_t)e.n0 * a.sk_n : kt + (int64_t)e.j * kKBytes) - kBias;
            const uint32_t dst = wave_lds + (uint32_t)sl * kSlot;
            if (__builtin_expect(e.fl & kStepWhole, 1)) {
                dma16_group_to_lds<kLoads>(dst, src, k_src);
            } else if (e.fl & kStepPart) {
                if (kTokK) {   // padded rows have no token
#pragma unroll
                    for (int j = 0; j < kLoads; ++j) off[j] = (e.vm >> k_row[j]) & 1ull ? k_src[j] : k_src0[j];
                    dma16_group_to_lds<kLoads>(dst, src, off);
                } else {
                    dma16_group_to_lds<kLoads>(dst, src, k_src);
                }
            } else if ((e.fl & kStepHalf) && wave < 2) {   // the first 32 rows, from the chunks that hold real tokens
                const uint32_t from = (uint32_t)(e.vm >> 32);
#pragma unroll
                for (int j = 0; j < kLoads; ++j) {
                    const int c = (wave * kLoads + j) * (1024 / kRowB) / 8;
                    const uint32_t moved = k_src[j] + chunk_off((from >> (8 * c)) & 255u) - chunk_off((uint32_t)c);
                    off[j] = !kTokK || (e.vm >> k_row[j]) & 1ull ? moved : k_src0[j];
                }
                dma16_group_to_lds<kLoads>(dst, src, off);
            }
        } else {
            const uint32_t dst = wave_lds + (uint32_t)sl * kSlot + kKBytes;
            const char* src = vt + (int64_t)e.j * kVBytes;
            if (__builtin_expect(e.fl & (kStepWhole | kStepPart), 1)) {
                dma16_group_to_lds<kLoads>(dst, src, v_src);
            } else if (e.fl & kStepHalf) {   // chunks 0-3 from where the real tokens are; chunks 4-7 are not read
                const uint32_t from = ((uint32_t)(e.vm >> 32) >> (8 * (v_c & 3))) & 255u;
                const uint32_t delta = (from - (uint32_t)(v_c & 3)) << 4;
#pragma unroll
                for (int j = 0; j < kLoads; ++j) off[j] = v_src[j] + (((v_c >> 2) & 1) == (j & 1) ? delta : 0u);
                dma16_group_to_lds<kLoads>(dst, src, off);
            }
        }
    };
    // All of this wave's LDS-bound loads have landed (vmcnt 0), then meet the other waves.
#define VEDA_LOADS_DONE_BARRIER()   \
    do {                            \
        wait_vmcnt<0>();            \
        __syncthreads();            \
    } while (0)

    PairAddr fa;
    fa.hh = hh;
    fa.k0 = smem_base + rho(lq) * kRowB + ((hh ^ (lq & (kKChunks - 1))) << 4);
    fa.v0 = smem_base + kKBytes + lq * 128 + ((hh ^ (((lq >> 1) & 7) ^ ((lq & 1) << 2))) << 4);

    // The steps: every key tile kept by at least one of the two query tiles, once; a key tile kept by
    // both is loaded once and used by both halves of the workgroup.
    // Table mode: the sequence is laid out in LDS before the loop (attn_union.h: ascending union,
    // whatever the order inside the lists) and the loop reads one entry per step, ahead of its use.
    // Walk mode: at every step take the smaller of the two list heads (ascending lists, as stage 3
    // writes them, share the most; any order stays correct).  The list heads are kept as (raw loaded
    // value, in-range flag) and only combined when the next step is formed, one step later: the scalar
    // loads get a whole step to return.  A step is formed in two halves (next_head: which tile and who
    // keeps it; next_advance: move the list positions and fetch the new heads) so that each fits the
    // shadow of one MFMA.  Everything of the walk is kept in 32-bit integers (flags as 0/1, never as
    // booleans) and the step's flags pass through readfirstlane: the walk then stays on the scalar
    // unit and the branches on it are scalar branches.
    constexpr int kEnd = 0x7fffffff;
    int ia = 0, ib = 0;
    int rawA = 0, rawB = 0, okA = 0, okB = 0;
    int gh = 0;         // grouped walk: which half of the current entry comes next
    int ta = 0, tb = 0; // this step consumes the head of list A / B
    // table mode: the raw entry read one step ahead of its use, the next entry to read, steps done
    Table& u = *reinterpret_cast<Table*>(smem + 2 * kSlot);
    const uint32_t tab_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)&u.tab[0];
    i32x4 raw_next = {0, 0, 0, 0};
    int s_read = 0, s_done = 0, total = 0;
    if constexpr (kTable) {
        total = union_table<kLists, 256, kPairChunk, kGrouped>(u, early, cols, cnt, lists, list_range, vmask_g, n0s_g, tid) * (kGrouped ? 2 : 1);
    } else {
        rawA = colsA[0];
        rawB = colsB[0];
        okA = nA > 0 ? 1 : 0;
        okB = nB > 0 ? 1 : 0;
    }
    auto next_head = [&](MergedStep& e) __attribute__((always_inline)) {
        if constexpr (kTable) {
            const UnionStep t = union_step(raw_next);
            e.j = t.j; e.fl = t.fl; e.vm = t.vm; e.n0 = t.n0;
            return;
        }
        int j, fl;
        if (kGrouped) {
            j = okA ? 2 * rawA + gh : 0;
            fl = okA ? 3 : 0;
            ta = gh;
        } else {
            const int headA = okA ? rawA : kEnd, headB = okB ? rawB : kEnd;
            const int jm = headA < headB ? headA : headB;
            const int live = jm != kEnd ? 1 : 0;
            ta = headA == jm ? live : 0;
            tb = headB == jm ? live : 0;
            j = live ? jm : 0;
            fl = ta | (tb << 1);
        }
        e.j = __builtin_amdgcn_readfirstlane(j);
        uint32_t lo, hi;
        const int kind = step_kind(vmask[e.j], lo, hi);
        e.fl = __builtin_amdgcn_readfirstlane(fl == 0 ? 0 : kind == kStepEmpty ? kind : fl | kind);
        e.vm = (uint64_t)hi << 32 | lo;
        e.n0 = kTokK ? n0s[e.j] : 0;
    };
    auto next_advance = [&]() __attribute__((always_inline)) {
        if constexpr (kTable) {
            raw_next = union_read<kPairChunk>(tab_lds, s_read);
            ++s_read;
            return;
        }
        ia += ta;
        okA = ia < nA ? 1 : 0;
        rawA = colsA[okA ? ia : 0];
        if (kGrouped) {
            gh ^= 1;
        } else {
            ib += tb;
            okB = ib < nB ? 1 : 0;
            rawB = colsB[okB ? ib : 0];
        }
    };
    // After the barrier that ends a step (table mode): when the loop has left one half of the
    // table's ring, that half is refilled with the steps that follow the other half's.
    auto step_done = [&]() __attribute__((always_inline)) {
        if constexpr (kTable) {
            ++s_done;
            if ((s_done & (kPairChunk - 1)) == 0)
                union_fill<kLists, 256, kPairChunk, kGrouped>(u, s_done + kPairChunk, total, list_range, vmask_g, n0s_g, tid);
        }
    };
    if constexpr (kTable) next_advance();   // entry 0 on its way

    // Step s (P = s & 1) computes on slot P while the tiles of step s+1 land in slot P^1.
    const int my_bit = 32 * r < q_rows ? (kGrouped ? 1 : 1 << which) : 128;   // 128: a bit no step has
    MergedStep e0, e1, e2;
    next_head(e0);
    next_advance();
    next_head(e1);
    next_advance();
    load_tile(e0, 0, 0);
    load_tile(e0, 0, 1);
    scale_q();
    VEDA_LOADS_DONE_BARRIER();   // also the Q loads: nothing vector-memory is pending below

    // One step.  A wave whose query tile keeps the current key tile does its housekeeping (loads of
    // the next tiles, next step of the walk) between the pieces of its step; a wave that skips the
    // step does it on its own.  (Two separate conditionals with an opaque flag rather than
    // if/else: with an else branch the register allocator keeps a second copy of the accumulators.)
#define VEDA_STEP(P)                                                                                     \
    do {                                                                                                 \
        int todo = 1;                                                                                    \
        if (__builtin_expect((e0.fl & (my_bit | kStepHalf)) == my_bit, 1)) {                             \
            PairStep<D, kExact> w;                                                                       \
            w.begin(fa, (uint32_t)((P) * kSlot));                                                        \
            w.template block0<0>(st);                                                                    \
            load_tile(e1, (P) ^ 1, 0);                                                                   \
            w.template block0<1>(st);                                                                    \
            load_tile(e1, (P) ^ 1, 1);                                                                   \
            w.template block0<2>(st);                                                                    \
            next_head(e2);                                                                               \
            w.template block0<3>(st);                                                                    \
            next_advance();                                                                              \
            w.finish(st, fa, e0.vm);                                                                     \
            todo = 0;                                                                                    \
        }                                                                                                \
        asm volatile("" : "+s"(todo));                                                                   \
        if (todo) {                                                                                      \
            load_tile(e1, (P) ^ 1, 0);                                                                   \
            load_tile(e1, (P) ^ 1, 1);                                                                   \
            next_head(e2);                                                                               \
            next_advance();                                                                              \
            if (e0.fl & my_bit) pair_half_step<D, kExact>(st, fa, (uint32_t)((P) * kSlot), (uint32_t)e0.vm); \
        }                                                                                                \
        e0 = e1; e1 = e2;                                                                                \
        VEDA_LOADS_DONE_BARRIER();                                                                       \
        step_done();                                                                                     \
    } while (0)
    while (e0.fl) {
        VEDA_STEP(0);
        if (!e0.fl) break;
        VEDA_STEP(1);
    }
#undef VEDA_STEP
#undef VEDA_LOADS_DONE_BARRIER

    finish_pair<D>(st, a, tok_s, smem, head, b, tid, wave, lq, hh);
}

// Two slots of (K tile + V^T tile), then the step table and the rows' tokens.
constexpr size_t pair_lds(int d, bool grouped, bool table) {
    const size_t tables = grouped ? sizeof(UnionLds<1, kPairChunk>) : sizeof(UnionLds<4, kPairChunk>);
    return (size_t)2 * 2 * kTile * d * 2 + (table ? tables : 0) + 4 * 32 * sizeof(int);
}
static_assert(2 * pair_lds(128, false, true) <= 160 * 1024, "two workgroups on a compute unit (launch bounds)");

veda_status launch_sparse_attn_bf16_pair(const veda_plan* pl, const AttnArgs& a, bool grouped, bool exact, bool walk,
                                         hipStream_t s) {
    const int d = pl->prob.head_dim;
    // the step table needs a bitmap over the tiles the lists may name
    bool table = !walk;
    for (const HeadGeom& g : pl->heads) table = table && (grouped ? g.n_tiles / 2 : g.n_tiles) <= kUnionMaxTiles;
    dim3 grid((unsigned)(table ? pl->attn_blocks : kXcd * pl->xcd_max_pairs), (unsigned)pl->prob.batch), block(256);
    const size_t smem = pair_lds(d, grouped, table);
#define VEDA_LAUNCH_PAIR_T(DD, GG, KK, EE, TT)                                                           \
    do {                                                                                                 \
        auto kern = sparse_attn_bf16_pair_kernel<DD, GG, KK, EE, TT>;                                    \
        if (smem > 64 * 1024)                                                                            \
            VEDA_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem)); \
        hipLaunchKernelGGL(kern, grid, block, smem, s, a);                                               \
    } while (0)
#define VEDA_LAUNCH_PAIR(DD, GG, KK)                                                                     \
    do {                                                                                                 \
        if (exact && table) VEDA_LAUNCH_PAIR_T(DD, GG, KK, true, true);                                  \
        else if (exact) VEDA_LAUNCH_PAIR_T(DD, GG, KK, true, false);                                     \
        else if (table) VEDA_LAUNCH_PAIR_T(DD, GG, KK, false, true);                                     \
        else VEDA_LAUNCH_PAIR_T(DD, GG, KK, false, false);                                               \
    } while (0)
    const int variant = (d == 128 ? 4 : 0) | (grouped ? 2 : 0) | (a.k_tok ? 1 : 0);
    switch (variant) {
        case 0: VEDA_LAUNCH_PAIR(64, false, false); break;
        case 1: VEDA_LAUNCH_PAIR(64, false, true); break;
        case 2: VEDA_LAUNCH_PAIR(64, true, false); break;
        case 3: VEDA_LAUNCH_PAIR(64, true, true); break;
        case 4: VEDA_LAUNCH_PAIR(128, false, false); break;
        case 5: VEDA_LAUNCH_PAIR(128, false, true); break;
        case 6: VEDA_LAUNCH_PAIR(128, true, false); break;
        default: VEDA_LAUNCH_PAIR(128, true, true); break;
    }
#undef VEDA_LAUNCH_PAIR
#undef VEDA_LAUNCH_PAIR_T
    return launch_status("sparse_attn_bf16_pair_kernel");
}

}  // namespace veda
