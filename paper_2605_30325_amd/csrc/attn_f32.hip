// Stage 4, fp32 (Eq. 2; Sec. 3.1 masked form; Sec. 4.3 tile skipping; Alg. 1 "UnTile"): the
// accuracy path (1e-4 against the double-precision definition), fp32 products on the bf16 matrix cores.
//
// Same work split as the bf16 kernel: a workgroup of four wavefronts of 32 rows owns one query tile, a pair of them
// or four thin ones, and walks the union of their kept lists (8 heads of 21x30x52, 10 % kept, thin tiles in fours instead of
// twos: whole call 3.44 -> 3.19 ms).  Partners in heads of more than kF32SplitTiles tiles share the form of their products and
// stay together (plan.hip); otherwise a tile's form is its own.  Padding is handled as in the bf16 kernel (real query rows first; half steps, attn_union.h).
// Every operand is split into three bf16 parts and a product is six bf16 ones (split_f32.h: why that is no less exact),
// 32 keys at a time:
//   S^T = K Q^T from the K planes, in the shadow of its last products V^T converted (landing area -> registers -> planes)
//   O^T += V^T P^T, in the shadow of its last products the next 32 keys' K converted
// with a barrier after each, so that one set of K planes and one of V^T planes serve (24 KB each at d = 128, 16 KB of
// landing area; 79 KB with the step table: two workgroups on a compute unit).  The query rows stay split in registers (96
// at d = 128, with 64 of O^T: this is why 32 keys, not 64).  K rows are read in the order rho, which leaves each lane eight
// consecutive keys of S^T as in the bf16 kernel.
// Measured, whole calls: 8 heads of 624 tiles, 10 % kept, 5.9 -> 3.3 ms (the products on fp32 matrix cores at 93 % of their
// rate before); 1.1 PFLOP/s of bf16 products, matrix pipes 52 % busy.  What is left: a fifth of the wave-steps belong
// to waves whose query tile does not keep the key tile, and two waves on a SIMD cover each other's
// softmax only so far.  d = 64 (168 registers) reloads one spilled fragment of Q per 32 keys, which waits for every load in
// flight; d = 128 spills nothing inside its steps since the two forms share one body of the chains.  Reading a group of products ahead gave 7 %, rounding pairs once 3 %, V^T rows on all banks 2 %;
// loads one phase earlier, priorities: 1-2 %.
//
// Long lists (AttnArgs::split_tiles) take v_mfma_f32_32x32x2_f32 instead, and numbers that are not finite come out of the
// split products as NaN: a tile that finds any in its results, or one too small for its parts (kF32Small), walks again
// that way, in heads of more than kF32SplitTiles tiles with its partner.  Which tiles share a workgroup otherwise leaves no trace in the
// results, nor do the other samples of the call or the way its steps are found.  There a lane owns one query (lane % 32) and one of the two terms of every instruction (h = lane / 32).  The pairing of the reduction index with h is free as long as both operands agree, and it is
// chosen so that one 16-byte LDS read feeds four instructions:
//   S^T, step (m, t):  h supplies channel 8m + 4h + t   (K row: float4 at channel 8m + 4h),
//   O^T, step (c, j, t): h supplies key 32c + 8j + 4h + t, which is exactly register 4j + t of the
//                        lane's S^T block c -- P^T needs no rearrangement at all.
// LDS rows are XOR-swizzled by 16-byte chunk (chunk ^ row) so that the 32 lanes reading the same
// chunk of 32 different rows spread over all banks; the swizzle is applied on the global side of
// the direct loads.  Online softmax, exp2 with log2(e) folded into Q in fp32.
#include "attn_common.h"
#include "attn_union.h"
#include "split_f32.h"

namespace veda {

constexpr int kF32Chunk = 128;   // step-table entries filled at a time
constexpr float kF32Slack = 8.0f;   // log2 units a row maximum may outgrow the softmax reference

// The split walk multiplies Q by 2^80 and V by 2^96, so that their parts hold every fp32 number (bf16 ends at 2^-133);
// what outgrows the range that leaves, |q| and |logit| of 2^48 and sums of 2^32, comes out not finite and walks again.
// Parts of K below 2^-133 move a logit by 2^-79 at most.  Those of a probability below 2^-102 are the rest: next to an
// output of 2^48 or more in this scale they are below 2^-25 of it for lists of a million keys; a smaller one that is not zero walks again.
constexpr float kF32QScale = 0x1p80f, kF32VScale = 0x1p96f, kF32Small = 0x1p48f;

// LDS: a K tile and a V^T tile, then the step table and the rows' tokens; at the end the output rows and their softmax sums
// lie over all but the tokens.
typedef UnionLds<4, kF32Chunk> F32Table;
template <int D, bool kTable>
constexpr size_t kF32Tokens = (size_t)2 * kTile * D * 4 + (kTable ? sizeof(F32Table) : 4 * 32 * sizeof(float));
template <int D, bool kTable> constexpr size_t kF32Lds = kF32Tokens<D, kTable> + 4 * 32 * sizeof(int);
static_assert(2 * kF32Lds<128, true> <= 160 * 1024 && 3 * kF32Lds<64, true> <= 160 * 1024, "workgroups on a compute unit (launch bounds)");

// kTable: the steps come from the table in LDS (attn_union.h), as in the bf16 kernel; otherwise the two
// lists are merged inside the loop (heads above 16384 tiles, VEDA_OPT_ATTN_LIST_WALK).
// d = 64: three workgroups on a compute unit (47 KB each); with two, 2 heads of 624 tiles, all kept, 7.34 instead of 7.14 ms.
template <int D, bool kTable>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void sparse_attn_f32_kernel(AttnArgs a) {
    constexpr int kKPitch = D * 4;               // bytes of one K row
    constexpr int kKBytes = kTile * kKPitch;     // K tile
    constexpr int kVPitch = kTile * 4;           // bytes of one V^T row (64 keys)
    constexpr int kVBytes = D * kVPitch;         // V^T tile (same size)
    constexpr int kKChunks = kKPitch / 16;       // 16-byte chunks per K row (32 or 16)
    constexpr int kLoads = kKBytes / 1024 / 4;   // direct loads per wave per tile: 8 (d = 128) or 4
    constexpr int kGroups = kLoads / 4;
    constexpr int NB = D / 32;                   // 32-channel blocks of O^T
    constexpr int kM = D / 8;                    // 16-byte K reads per key block and lane
    constexpr int kLists = kTable ? 4 : 2;       // kept lists of a workgroup, at most
    extern __shared__ __align__(1024) char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int idx = lane & 31, h = lane >> 5;

    AttnItem it;   // see the bf16 kernel
    if (!attn_work<kTable>(a, it)) return;
    const int head = it.head;
    const HeadGeom hg = a.heads[head];
    const int64_t b = blockIdx.y;
    const uint32_t place = it.waves >> (8 * wave);
    const int which = place & 3u, r = place & kItemSecond ? 1 : 0;
    const int qi = which == 0 ? it.tile[0] : which == 1 ? it.tile[1] : which == 2 ? it.tile[2] : it.tile[3];
    const int64_t head_tile0 = b * a.total_tiles + hg.tile_off;
    int beg[kLists], cnt[kLists];
#pragma unroll
    for (int t = 0; t < kLists; ++t) {
        beg[t] = a.row_ptr[head_tile0 + it.tile[t]];
        cnt[t] = t < it.n_tiles ? a.row_ptr[head_tile0 + it.tile[t] + 1] - beg[t] : 0;
    }
    typedef const __attribute__((address_space(4))) int32_t* const_i32_t;
    typedef const __attribute__((address_space(4))) uint64_t* const_u64_t;
    const const_i32_t colsA = (const_i32_t)(uintptr_t)(a.col_idx + beg[0]);
    const const_i32_t colsB = (const_i32_t)(uintptr_t)(a.col_idx + beg[1]);
    const int nA = cnt[0], nB = cnt[1];   // walk mode: two lists
    const const_u64_t vmask = (const_u64_t)(uintptr_t)(a.valid_mask + hg.tile_off);
    const char* kt = a.k + head_tile0 * kKBytes;
    const char* vt = a.v + head_tile0 * kVBytes;

    // Row 32r + idx is the tile's real slot of that rank; rows beyond the real slots read slot 0 and are not written.
    const uint64_t q_real = ((const_u64_t)(uintptr_t)(a.tile_real + hg.tile_off))[qi];
    const int q_rows = place & kItemIdle ? 0 : __popcll(q_real);
    const float* qrow;
    int* tok_s = reinterpret_cast<int*>(smem + kF32Tokens<D, kTable>);   // [4][32] token of each row, -1 = none
    {
        const bool real = 32 * r + idx < q_rows;
        int slot = 32 * r + idx;
        if (q_real != ~0ull) slot = real ? nth_bit(q_real, slot) : 0;
        if (h == 0) tok_s[wave * 32 + idx] = real ? token_from(hg, a.tile_n0[hg.tile_off + qi], slot, a.H, a.W) : -1;
        qrow = reinterpret_cast<const float*>(a.q + (head_tile0 + qi) * kKBytes + slot * kKPitch);
    }
    f32x16 o[NB];
    float m_run, l_run;
    auto begin_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[nb][i] = 0.0f;
        m_run = -INFINITY;
        l_run = 0.0f;
    };

    const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t wave_lds = smem_base + (uint32_t)wave * (kLoads * 1024);
    struct Step { int j, fl; uint64_t vm; };   // vm: the mask, or step_kind's lo | hi << 32 (half steps)
    constexpr int kKeepers = 15;
    // The steps: the union of the two kept lists.  Table mode: laid out in LDS before the loop; walk mode:
    // merged with scalar loads as the loop goes (32-bit integers on the scalar unit; see the bf16 kernel).
    constexpr int kEnd = 0x7fffffff;
    int ia = 0, ib = 0;
    int rawA = 0, rawB = 0, okA = 0, okB = 0;
    F32Table& u = *reinterpret_cast<F32Table*>(smem + kKBytes + kVBytes);
    const uint32_t tab_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)&u.tab[0];
    const uint64_t* vmask_g = a.valid_mask + hg.tile_off;
    const int32_t* n0s_g = a.tile_n0 + hg.tile_off;
    i32x4 raw_next = {0, 0, 0, 0};
    int s_read = 0, s_done = 0, total = 0;
    bool filled = false;   // the ring holds the first steps
    if constexpr (kTable) {
        const int32_t* cols[kLists];
#pragma unroll
        for (int t = 0; t < kLists; ++t) cols[t] = a.col_idx + beg[t];
        UnionEarly<kLists, 256, false> early;
        early.ask(cols, cnt, it.n_tiles, hg.n_tiles, vmask_g, n0s_g, tid);
        total = union_table<kLists, 256, kF32Chunk, false>(u, early, cols, cnt, it.n_tiles, hg.n_tiles, vmask_g, n0s_g, tid);
        filled = true;
    }
    // to the first step; ends with a barrier
    auto begin_walk = [&]() __attribute__((always_inline)) {
        s_done = 0;
        if constexpr (kTable) {
            if (!filled) {
                union_fill<4, 256, kF32Chunk, false, 2 * kF32Chunk>(u, 0, total, hg.n_tiles, vmask_g, n0s_g, tid);   // the whole ring
                __syncthreads();
            }
            filled = false;
            raw_next = union_read<kF32Chunk>(tab_lds, 0);
            s_read = 1;
        } else {
            ia = ib = 0;
            rawA = colsA[0];
            rawB = colsB[0];
            okA = nA > 0 ? 1 : 0;
            okB = nB > 0 ? 1 : 0;
            __syncthreads();
        }
    };
    auto next_step = [&](Step& e) __attribute__((always_inline)) {
        if constexpr (kTable) {
            const UnionStep t = union_step(raw_next);
            e.j = t.j; e.fl = t.fl; e.vm = t.vm;
            raw_next = union_read<kF32Chunk>(tab_lds, s_read);
            ++s_read;
            return;
        }
        const int headA = okA ? rawA : kEnd, headB = okB ? rawB : kEnd;
        const int jm = headA < headB ? headA : headB;
        const int live = jm != kEnd ? 1 : 0;
        const int ta = headA == jm ? live : 0, tb = headB == jm ? live : 0;
        e.j = __builtin_amdgcn_readfirstlane(live ? jm : 0);
        const int fl = ta | (tb << 1);
        uint32_t lo, hi;
        const int kind = step_kind(vmask[e.j], lo, hi);
        e.fl = __builtin_amdgcn_readfirstlane(fl == 0 ? 0 : kind == kStepEmpty ? kind : fl | kind);
        e.vm = (uint64_t)hi << 32 | lo;
        ia += ta;
        ib += tb;
        okA = ia < nA ? 1 : 0;
        okB = ib < nB ? 1 : 0;
        rawA = colsA[okA ? ia : 0];
        rawB = colsB[okB ? ib : 0];
    };

    const int my_bit = 32 * r < q_rows ? 1 << which : 128;   // 128: a bit no step has
    // The walk on bf16 matrix cores: every operand as the sum of three bf16 numbers, six products (see the head of the file).
    auto split_walk = [&](int walk_bit) __attribute__((always_inline)) {
        typedef SplitK<D> K;
        constexpr int G = D / 16, kI = K::kI;
        constexpr uint32_t kV = K::kPlanes, kRaw = 2 * K::kPlanes;   // V^T planes, landing area: 64 KB (d = 128) in all
        K ks;
        ks.init(smem_base, smem_base + kRaw, wave, lane);
        bf16x8 q[3][G];
        split_row<D>(qrow, h, a.scale_log2 * kF32QScale, q);
        struct Sub { int j, fl, c; uint32_t mask, hi, from; };   // 32 keys of a step: c-th half of key tile j, or a half step
        // K and V^T take turns in the landing area.  Past the end the loads go on, from key tile 0.
        auto load_k = [&](const Sub& e, int j) __attribute__((always_inline)) { ks.load(j, kt + (int64_t)e.j * kKBytes, e.from); };
        // V^T planes: [D][32], 16-byte chunk ^ row / 4 (any sixteen rows of a read on all banks); a wave has D / 4 rows
        const uint32_t v_lane = (uint32_t)(((D / 4) * wave + (lane >> 3)) * kVPitch + (lane & 1) * 16);
        auto load_v = [&](const Sub& e, int j) __attribute__((always_inline)) {
            const uint32_t chunk = (e.from >> (8 * ((lane >> 1) & 3))) & 255u;
            dma16_to_lds(ks.raw + 1024u * j, vt + (int64_t)e.j * kVBytes + 2048 * j, v_lane + chunk * 32u);
        };
        const int v_row = (D / 4) * wave + (lane >> 3), v_c = lane & 7;
        const uint32_t vw = smem_base + kV + v_row * 64 + (((v_c >> 1) ^ ((v_row >> 2) & 3)) << 4) + (v_c & 1) * 8;
        auto convert_v = [&](int j) __attribute__((always_inline)) { ks.put(j, (vw ^ (uint32_t)((j & 1) << 5)) + (uint32_t)(j * 8 * 64), kF32VScale); };
        const uint32_t vr = smem_base + kV + idx * 64 + ((h ^ ((idx >> 2) & 3)) << 4);
        auto of_step = [&](Sub& n) __attribute__((always_inline)) {
            Step e;
            next_step(e);
            n.j = e.j; n.fl = e.fl; n.c = 0;
            n.mask = (uint32_t)e.vm;
            n.hi = (uint32_t)(e.vm >> 32);
            n.from = e.fl & kStepHalf ? n.hi : 0x03020100u;
        };
        float thr = -INFINITY, ref = 0.0f;   // a row maximum above thr (in the products' scale) moves the reference
        begin_rows();
        begin_walk();
        Sub cur, nx;
        of_step(cur);
#pragma unroll
        for (int j = 0; j < kI; ++j) load_k(cur, j);
#pragma unroll
        for (int j = 0; j < kI; ++j) {
            ks.convert(j);
            load_v(cur, j);
        }
        K::meet();
        while (cur.fl) {
            const bool mine = (cur.fl & walk_bit) != 0;
            if (cur.c == 0 && (cur.fl & (kStepWhole | kStepPart))) {
                nx = cur;
                nx.c = 1;
                nx.mask = cur.hi;
                nx.from = 0x07060504u;
            } else {
                of_step(nx);
            }
            // S^T = K Q^T from the K planes, the V^T planes written
            // (two conditionals with an opaque flag rather than if / else: see the bf16 kernel)
            f32x16 s;
            int todo = 1;
            if (mine) {
                todo = 0;
                // d = 64 has registers for the small products in a sum of their own (the search's table, squares of
                // differences of outputs, 7.3e-9 -> 5.2e-9 from the 64-bit one; 1 % of the time)
                ks.template products<D == 64>(s, q, 0u, [&](int t) __attribute__((always_inline)) {
                    if (t >= G - kI) {
                        convert_v(t - (G - kI));
                        load_k(nx, t - (G - kI));
                    }
                });
            }
            asm volatile("" : "+s"(todo));
            if (todo) {
#pragma unroll
                for (int j = 0; j < kI; ++j) {
                    convert_v(j);
                    load_k(nx, j);
                }
            }
            K::meet();
            // O^T += V^T P^T, the next K planes written
            if (!todo) {
                bf16x8 vf[2][3];
#pragma unroll
                for (int u = 0; u < 3; ++u) vf[0][u] = K::frag(vr, u);
                __builtin_amdgcn_sched_barrier(0);
                if (cur.mask != ~0u) {   // register i is key 16*(i/8) + 8*h + i%8
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int bit = 16 * (i >> 3) + (i & 7);
                        const uint32_t lo = (uint32_t)((int)(cur.mask << (31 - bit)) >> 31), up = (uint32_t)((int)(cur.mask << (23 - bit)) >> 31);
                        s[i] = __builtin_amdgcn_inverse_ballot_w64((uint64_t)up << 32 | lo) ? s[i] : -INFINITY;
                    }
                }
                float mx = s[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
                if (__any(mx > thr)) {
                    asm volatile("" ::: "memory");
                    m_run = fmaxf(m_run, max_with_other_half(mx) * (1.0f / kF32QScale));
                    const float use = m_run == -INFINITY ? 0.0f : m_run;
                    const float alpha = thr == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ref - use);
                    ref = use;
                    thr = (m_run + kF32Slack) * kF32QScale;
                    l_run *= alpha;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[nb][i] *= alpha;
                }
                float psum = 0.0f;
                uint32_t pw[2][3][4];
                auto prob = [&](int kk, int e) __attribute__((always_inline)) {   // registers 8*kk + 2e, +1
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[8 * kk + 2 * e], 1.0f / kF32QScale, -ref));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(s[8 * kk + 2 * e + 1], 1.0f / kF32QScale, -ref));
                    psum += p0;
                    psum += p1;
                    uint32_t p[3];
                    split2(p0, p1, p);
#pragma unroll
                    for (int u = 0; u < 3; ++u) pw[kk][u][e] = p[u];
                };
#pragma unroll
                for (int e = 0; e < 4; ++e) prob(0, e);
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int g = 0; g < 2 * NB; ++g) {
                    const int kk = g / NB, nb = g % NB;
                    if (g + 1 < 2 * NB) {
#pragma unroll
                        for (int u = 0; u < 3; ++u) vf[(g + 1) & 1][u] = K::frag((vr ^ (uint32_t)(((g + 1) / NB) << 5)) + (uint32_t)(((g + 1) % NB) * 2048), u);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    const bf16x8 y0 = __builtin_bit_cast(bf16x8, u32x4{pw[kk][0][0], pw[kk][0][1], pw[kk][0][2], pw[kk][0][3]});
                    const bf16x8 y1 = __builtin_bit_cast(bf16x8, u32x4{pw[kk][1][0], pw[kk][1][1], pw[kk][1][2], pw[kk][1][3]});
                    const bf16x8 y2 = __builtin_bit_cast(bf16x8, u32x4{pw[kk][2][0], pw[kk][2][1], pw[kk][2][2], pw[kk][2][3]});
                    o[nb] = mul6(o[nb], vf[g & 1], y0, y1, y2);
                    if (kk == 0) {
#pragma unroll
                        for (int e = nb * 4 / NB; e < (nb + 1) * 4 / NB; ++e) prob(1, e);
                    } else {
#pragma unroll
                        for (int j = nb * kI / NB; j < (nb + 1) * kI / NB; ++j) {
                            ks.convert(j);
                            load_v(nx, j);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_s_setprio(0);
                l_run += psum;
            }
            asm volatile("" : "+s"(todo));
            if (todo) {
#pragma unroll
                for (int j = 0; j < kI; ++j) {
                    ks.convert(j);
                    load_v(nx, j);
                }
            }
            K::meet();
            if constexpr (kTable) {   // a step is done: the table's other half may have been left behind
                if (nx.c == 0) {
                    ++s_done;
                    if ((s_done & (kF32Chunk - 1)) == 0)
                        union_fill<4, 256, kF32Chunk, false>(u, s_done + kF32Chunk, total, hg.n_tiles, vmask_g, n0s_g, tid);
                }
            }
            cur = nx;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing lands any more
        __syncthreads();
    };

    // The walk on fp32 matrix cores, by the wavefronts that take part.
    auto exact_walk = [&](bool part) __attribute__((always_inline)) {
        const int walk_bit = part ? my_bit : 128;
        // Q operand: lane (query 32r + idx, half h) holds channels 8m + 4h + t, scaled by softmax_scale*log2(e).
        float qreg[D / 2];
#pragma unroll
        for (int m = 0; m < kM; ++m) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(qrow + 8 * m + 4 * h);
#pragma unroll
            for (int t = 0; t < 4; ++t) qreg[4 * m + t] = v[t] * a.scale_log2;
        }
        // global -> LDS copy plan (see the bf16 kernel): wave w issues instructions w*kLoads .. of each
        // tile, four to an M0 set-up, instruction j of a group with immediate offset 1024*(j%4), which
        // moves the LDS and the global address alike.
        uint32_t k_src[kLoads], v_src[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int inst = wave * kLoads + j;
            const int krow = inst * (1024 / kKPitch) + lane / kKChunks, kpos = lane % kKChunks;
            k_src[j] = krow * kKPitch + ((kpos ^ (krow & (kKChunks - 1))) << 4) - 1024u * (j % 4);
            const int vrow = inst * 4 + (lane >> 4), vpos = lane & 15;
            v_src[j] = vrow * kVPitch + ((vpos ^ (vrow & 15)) << 4) - 1024u * (j % 4);
        }
        auto load_k = [&](const Step& e) __attribute__((always_inline)) {
            if (!(e.fl & kKeepers)) return;
            uint32_t moved[2] = {0u, 0u};   // half: the chunks of this wave's first and last eight rows, moved
            if (e.fl & kStepHalf) {
                if (wave >= 2) return;      // only the first 32 rows are read
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = 2 * wave + u;
                    moved[u] = (((uint32_t)(e.vm >> (32 + 8 * c)) & 255u) - (uint32_t)c) * (8 * kKPitch);
                }
            }
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                uint32_t off[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) off[j] = k_src[4 * g + j] + moved[(4 * g + j) * 2 / kLoads];
                dma16_group_to_lds<4>(wave_lds + g * 4096, kt + (int64_t)e.j * kKBytes, off);
            }
        };
        const int v_c = (lane & 15) ^ (lane >> 4);   // this lane's 16-byte chunk (4 keys): v_c ^ 4*(j%4) in instruction j
        auto load_v = [&](const Step& e) __attribute__((always_inline)) {
            if (!(e.fl & kKeepers)) return;
            uint32_t moved[4] = {0u, 0u, 0u, 0u};
            if (e.fl & kStepHalf) {   // keys 0-31 from the chunks that hold real tokens; the others are not read
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t c = (uint32_t)(v_c ^ (4 * j));
                    const uint32_t from = (uint32_t)((e.vm >> 32) >> (8 * ((c >> 1) & 3))) & 255u;
                    moved[j] = c < 8 ? (from - (c >> 1)) * 32u : 0u;
                }
            }
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                uint32_t off[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) off[j] = v_src[4 * g + j] + moved[j];
                dma16_group_to_lds<4>(wave_lds + kKBytes + g * 4096, vt + (int64_t)e.j * kVBytes, off);
            }
        };
        // LDS addresses of this lane's first operand reads: the swizzle only touches bits the row offsets leave clear,
        // so K chunk 2m + h is at k0 ^ (m << 5), V^T chunk 2g + h at v0 ^ (g << 5).
        uint32_t k0 = smem_base + idx * kKPitch + (((uint32_t)h ^ (idx & (kKChunks - 1))) << 4);
        uint32_t v0 = smem_base + kKBytes + idx * kVPitch + (((uint32_t)h ^ (idx & 15)) << 4);

        // S^T block c = K Q^T: 32 keys x 32 queries
        auto logits = [&](f32x16& s, int c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.0f;
#pragma unroll
            for (int m = 0; m < kM; ++m) {
                const f32x4 kf = lds_read_f32x4((k0 ^ (uint32_t)(m << 5)) + (uint32_t)(32 * c * kKPitch));
#pragma unroll
                for (int t = 0; t < 4; ++t) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[t], qreg[4 * m + t], s, 0, 0, 0);
            }
        };
        // padded key slots: register i of a block is key 8*(i/4) + 4h + i%4
        auto mask_keys = [&](f32x16& s, uint32_t mask) __attribute__((always_inline)) {
            if (mask == ~0u) return;
            asm volatile("" ::: "memory");   // keeps this a branch
            const uint32_t half = mask >> (4 * h);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (!((half >> (8 * (i >> 2) + (i & 3))) & 1u)) s[i] = -INFINITY;
        };
        // O^T += V^T P^T over the 32 keys of block c
        auto outputs = [&](const f32x16& p, int c) __attribute__((always_inline)) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const f32x4 vf = lds_read_f32x4((v0 ^ (uint32_t)((4 * c + j) << 5)) + (uint32_t)(32 * nb * kVPitch));
#pragma unroll
                    for (int t = 0; t < 4; ++t) o[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[t], p[4 * j + t], o[nb], 0, 0, 0);
                }
            }
        };
        if (part) begin_rows();
        begin_walk();
        Step e0, e1;
        next_step(e0);
        load_k(e0);
        load_v(e0);
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the Q loads and the first tiles
        __syncthreads();

        while (e0.fl) {
            next_step(e1);
            asm volatile("" : "+v"(k0), "+v"(v0));   // the addresses of the reads are formed as they are needed: kept, they would spill
            const bool mine = (e0.fl & walk_bit) != 0, full = !(e0.fl & kStepHalf);
            f32x16 s0, s1;
            if (mine) {
                logits(s0, 0);
                mask_keys(s0, (uint32_t)e0.vm);
                if (full) {
                    logits(s1, 1);
                    mask_keys(s1, (uint32_t)(e0.vm >> 32));
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) s1[i] = -INFINITY;
                }
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's loads of V^T have landed
            __syncthreads();                      // everybody is done with K
            load_k(e1);
            if (mine) {
                float mx = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, fmaxf(s0[i], s1[i]));
                mx = max_with_other_half(mx);
                const float m_new = fmaxf(m_run, mx);
                const float m_use = m_new == -INFINITY ? 0.0f : m_new;
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);   // 0 on the first step (m_run = -inf)
                float psum = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    s0[i] = __builtin_amdgcn_exp2f(s0[i] - m_use);
                    psum += s0[i];
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    s1[i] = __builtin_amdgcn_exp2f(s1[i] - m_use);
                    psum += s1[i];
                }
                l_run = l_run * alpha + psum;
                m_run = m_new;
                if (__any(alpha != 1.0f)) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[nb][i] *= alpha;
                }
                outputs(s0, 0);
                if (full) outputs(s1, 1);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the next K tile
            __syncthreads();                      // everybody is done with V^T
            load_v(e1);
            e0 = e1;
            if constexpr (kTable) {   // the table's other half has been left behind: refill it
                ++s_done;
                if ((s_done & (kF32Chunk - 1)) == 0)
                    union_fill<4, 256, kF32Chunk, false>(u, s_done + kF32Chunk, total, hg.n_tiles, vmask_g, n0s_g, tid);
            }
        }

    };

    // Bit t of `again`: the tile in place t takes the chains, because its list or its partner's is too long or a result of either has to be
    // formed again.  (A flag beside the mask, and the splits for whatever is left: otherwise 26-35 spilled registers, not 8.)
    auto and_partner = [&](int t) __attribute__((always_inline)) { return (it.partners >> (t >> 1)) & 1 ? 3 << (t & 2) : 1 << t; };
    int again = 0, kept = 0;
#pragma unroll
    for (int t = 0; t < kLists; ++t) {
        if (cnt[t] > 0) kept |= 1 << t;
        if (cnt[t] > a.split_tiles) again |= and_partner(t);
    }
    bool chains = again != 0 && (kept & ~again) == 0;
    float unscale = 1.0f;
    if (!chains) {
        split_walk((again >> which) & 1 ? 128 : my_bit);
        float bad = l_run * 0.0f;   // NaN if anything is not finite
        uint32_t least = ~0u;       // 2 |o| - 1 in bits: zeros are the largest
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                bad = fmaf(o[nb][i], 0.0f, bad);
                least = min(least, (__float_as_uint(o[nb][i]) << 1) - 1u);
            }
        int* flag = reinterpret_cast<int*>(smem);   // the planes are done with
        const bool any_bad = __any(bad != 0.0f || least < (__float_as_uint(kF32Small) << 1) - 1u);
        if (lane == 0) flag[wave] = any_bad ? and_partner(which) : 0;
        __syncthreads();
        again |= __builtin_amdgcn_readfirstlane(flag[0] | flag[1] | flag[2] | flag[3]);
        chains = again != 0;
        unscale = 1.0f / kF32VScale;
        __syncthreads();
    }
    if (chains) {
        const bool part = ((again >> which) & 1) != 0;
        exact_walk(part);
        if (part) unscale = 1.0f;
    }

    // Normalise, transpose through LDS ([4 wavefronts][32 rows][D] fp32) and scatter the real rows.
    const float l_all = l_run + __shfl_xor(l_run, 32);
    const float inv = l_all > 0.0f ? unscale / l_all : 0.0f;
    __syncthreads();   // nobody fills the step table any more
    float* obuf = reinterpret_cast<float*>(smem);
    float* lse_s = obuf + 4 * 32 * D;
    {
        float* orow = obuf + (wave * 32 + idx) * D;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 v;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = o[nb][4 * j + t] * inv;
                *reinterpret_cast<f32x4*>(orow + 32 * nb + 8 * j + 4 * h) = v;
            }
        if (h == 0) lse_s[wave * 32 + idx] = (m_run + __log2f(l_all)) * kLn2;
    }
    __syncthreads();
    char* ob = a.out + b * a.so_b + head * a.so_h;
    for (int cid = tid; cid < 4 * 32 * kKChunks; cid += 256) {
        const int row = cid / kKChunks, ch = cid % kKChunks;
        const int n = tok_s[row];
        if (n >= 0)
            *reinterpret_cast<uint4*>(ob + (int64_t)n * a.so_n + ch * 16) =
                *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(obuf) + row * kKPitch + ch * 16);
    }
    if (a.lse && tid < 4 * 32) {
        const int n = tok_s[tid];
        if (n >= 0) a.lse[(b * a.n_heads + head) * a.tokens + n] = lse_s[tid];
    }
}

veda_status launch_sparse_attn_f32(const veda_plan* pl, const AttnArgs& a, bool walk, hipStream_t s) {
    const int d = pl->prob.head_dim;
    bool table = !walk;   // the step table's bitmaps cover 16384 tiles per head
    for (const HeadGeom& g : pl->heads) table = table && g.n_tiles <= kUnionMaxTiles;
    dim3 grid((unsigned)(table ? pl->attn_blocks : kXcd * pl->xcd_max_pairs), (unsigned)pl->prob.batch), block(256);
#define VEDA_LAUNCH_F32(DD, TT)                                                                          \
    do {                                                                                                 \
        auto kern = sparse_attn_f32_kernel<DD, TT>;                                                      \
        constexpr size_t smem = kF32Lds<DD, TT>;                                                         \
        if (smem > 64 * 1024)                                                                            \
            VEDA_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem)); \
        hipLaunchKernelGGL(kern, grid, block, smem, s, a);                                               \
    } while (0)
    if (d == 128) {
        if (table) VEDA_LAUNCH_F32(128, true); else VEDA_LAUNCH_F32(128, false);
    } else {
        if (table) VEDA_LAUNCH_F32(64, true); else VEDA_LAUNCH_F32(64, false);
    }
#undef VEDA_LAUNCH_F32
    return launch_status("sparse_attn_f32_kernel");
}

}  // namespace veda
