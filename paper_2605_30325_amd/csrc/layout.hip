// Stage 1 -- head-aware 3D tiling (Sec. 4.2: per-head pi = (p_t,p_h,p_w); Alg. 1 "Tiling";
// Alg. 2 "Tile"): gathers the tokens of every tile into one contiguous 64 x d block, zero
// fills padded slots and records which slots are real.  Pure byte movement, HBM bound:
// one workgroup per (tile, batch) moves 64 rows with 16-byte accesses.
#include "veda_internal.h"

namespace veda {

// out tile = [64][row_bytes]; each thread moves 16-byte chunks.
__global__ __launch_bounds__(256) void layout_token_major_kernel(
    const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head,
    const char* __restrict__ x, int64_t sb, int64_t sh, int64_t sn, char* __restrict__ out,
    int64_t total_tiles, int row_bytes, int T, int H, int W,
    uint64_t* __restrict__ valid_mask, int32_t* __restrict__ valid_cnt) {
    __shared__ int tok[kTile];
    const int g = blockIdx.x, b = blockIdx.y;
    const int head = tile_head[g];
    const HeadGeom hg = heads[head];
    const int i = g - hg.tile_off;
    if (threadIdx.x < kTile) {
        const int n = slot_token(hg, i, threadIdx.x, T, H, W);
        tok[threadIdx.x] = n;
        const uint64_t m = __ballot(n >= 0);
        if (threadIdx.x == 0 && b == 0) {
            if (valid_mask) valid_mask[g] = m;
            if (valid_cnt) valid_cnt[g] = __popcll(m);
        }
    }
    __syncthreads();
    const int cpr = row_bytes >> 4;  // 16-byte chunks per row
    const char* xb = x + b * sb + head * sh;
    char* ob = out + ((int64_t)b * total_tiles + g) * (int64_t)kTile * row_bytes;
    for (int c = threadIdx.x; c < kTile * cpr; c += 256) {
        const int l = c / cpr, ch = c - l * cpr;
        const int n = tok[l];
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (n >= 0) v = *reinterpret_cast<const uint4*>(xb + (int64_t)n * sn + ch * 16);
        *reinterpret_cast<uint4*>(ob + (int64_t)c * 16) = v;
    }
}

// out tile = [d][64] elements.  The tile is staged in LDS as [64][d] with one pad dword per
// row so that the column gathers spread over the banks.
template <typename E, int D> constexpr int kChannelMajorWords = kTile * (D * (int)sizeof(E) / 4 + 1);   // of the stage

// The plan's tables of the 64-slot tiles: what slot_token divides for.  With V's rows asked for together (channel_major_tile), whole calls
// before and after: 75 tiles (bf16, d = 64) 45.5 -> 44.5 us, 384 tiles 43.0 -> 41.9, 12 heads of 624 (d = 128) 560 -> 553.  Tried: all 64 rows
// of a tile asked for at once where few workgroups leave the registers, 1 % slower (longer code, fetched anew by every call).
struct TileTables {
    const int32_t* n0;       // anchor token
    const uint64_t* real;    // slots inside the grid
    __device__ __forceinline__ int token(const HeadGeom& hg, int64_t g, int l, int H, int W) const {
        return (real[g] >> l) & 1ull ? token_from(hg, n0[g], l, H, W) : -1;
    }
};

template <typename E, int D>
__device__ __forceinline__ void channel_major_tile(
    const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head, const TileTables tables,
    const char* __restrict__ x, int64_t sb, int64_t sh, int64_t sn, char* __restrict__ out,
    int64_t total_tiles, int H, int W,
    uint64_t* __restrict__ valid_mask, int32_t* __restrict__ valid_cnt, int g, int b, int* tok, uint32_t* stage) {
    constexpr int kRowBytes = D * (int)sizeof(E);
    constexpr int kRowWords = kRowBytes / 4;
    constexpr int kPitch = kRowWords + 1;   // dwords
    constexpr int kCpr = kRowBytes / 16;
    constexpr int kEpc = 16 / (int)sizeof(E);  // elements per 16-byte output chunk
    const int head = tile_head[g];
    const HeadGeom hg = heads[head];
    if (threadIdx.x < kTile) {
        const int n = tables.token(hg, g, threadIdx.x, H, W);
        tok[threadIdx.x] = n;
        const uint64_t m = __ballot(n >= 0);
        if (threadIdx.x == 0 && b == 0) {
            if (valid_mask) valid_mask[g] = m;
            if (valid_cnt) valid_cnt[g] = __popcll(m);
        }
    }
    __syncthreads();
    const char* xb = x + b * sb + head * sh;
    constexpr int kPer = kTile * kCpr / 256;   // 16-byte chunks of a thread, all asked for before the first is put down; padded rows read token 0
    uint4 v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int c = threadIdx.x + 256 * i, l = c / kCpr, ch = c - l * kCpr, n = tok[l];
        v[i] = *reinterpret_cast<const uint4*>(xb + (int64_t)(n >= 0 ? n : 0) * sn + ch * 16);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int c = threadIdx.x + 256 * i, l = c / kCpr, ch = c - l * kCpr;
        const bool real = tok[l] >= 0;
        uint32_t* s = stage + l * kPitch + ch * 4;
        s[0] = real ? v[i].x : 0u; s[1] = real ? v[i].y : 0u; s[2] = real ? v[i].z : 0u; s[3] = real ? v[i].w : 0u;
    }
    __syncthreads();
    const E* se = reinterpret_cast<const E*>(stage);
    constexpr int kPitchE = kPitch * 4 / (int)sizeof(E);
    constexpr int kChunksPerChannel = kTile / kEpc;
    char* ob = out + ((int64_t)b * total_tiles + g) * (int64_t)kTile * kRowBytes;
    for (int oc = threadIdx.x; oc < D * kChunksPerChannel; oc += 256) {
        const int ch = oc / kChunksPerChannel, l0 = (oc - ch * kChunksPerChannel) * kEpc;
        E tmp[kEpc];
#pragma unroll
        for (int j = 0; j < kEpc; ++j) tmp[j] = se[(l0 + j) * kPitchE + ch];
        *reinterpret_cast<uint4*>(ob + (int64_t)oc * 16) = *reinterpret_cast<const uint4*>(tmp);
    }
}

template <typename E, int D>
__global__ __launch_bounds__(256) void layout_channel_major_kernel(
    const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head, TileTables tables,
    const char* __restrict__ x, int64_t sb, int64_t sh, int64_t sn, char* __restrict__ out,
    int64_t total_tiles, int H, int W,
    uint64_t* __restrict__ valid_mask, int32_t* __restrict__ valid_cnt) {
    __shared__ int tok[kTile];
    __shared__ uint32_t stage[kChannelMajorWords<E, D>];
    channel_major_tile<E, D>(heads, tile_head, tables, x, sb, sh, sn, out, total_tiles, H, W, valid_mask, valid_cnt, blockIdx.x,
                             blockIdx.y, tok, stage);
}

// 128-token tiles: number of real tokens of a whole tile from the masks of its two halves.
__global__ void valid_cnt_pairs_kernel(const uint64_t* __restrict__ mask, int32_t* __restrict__ cnt, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cnt[i] = __popcll(mask[2 * i]) + __popcll(mask[2 * i + 1]);
}

// Token-major tiling with the TripPool descriptors (Eq. 4: Avg | Max | Min over the tile's real
// tokens, per channel) taken on the way, so the tiled tensor is not read back for them.
// One thread owns four channels of one tile and walks its 64 slots in order: the sum is the same
// slot-ascending fp32 chain the scoring stage uses, so the descriptors are bit-identical to the ones it
// derives from the tiled tensor.  A workgroup holds 256 / (D / 4) consecutive global tiles (they may belong
// to different heads).
// Bound by the latency of the loads on small inputs and by memory on large ones, so the rows of kBatch slots
// are requested before the first is used, padded ones included (from token 0), and four channels instead of
// eight bf16 ones make twice the wavefronts.  Measured, 8 slots at a time with 16-byte loads and now, calls repeated
// (inputs of up to 256 MB stay in the memory-side cache): 4 heads of 75 tiles, 2 samples (bf16, d = 64) 26 -> 11 us; 12
// heads of 624 tiles (bf16, d = 128) 39 -> 22, writing tiles 43 -> 39; 24 heads of 219,600 tokens 309 -> 277 us (1.49 GB,
// 5.4 TB/s), writing tiles 637 -> 540 (3.0 GB with the padding, 5.6 TB/s).  Single calls on inputs that have left the
// caches, from event to event: 51 -> 15, 72 -> 46 and 91 -> 73, 363 -> 331 and 660 -> 565.  Without the tiles half a
// batch is enough and makes more wavefronts: 22.3 us against 24.9 at 12 heads, 164 against 166 at 40 heads of 1440 tiles,
// alike on inputs that have left the caches.
// kWrite = false: descriptors (and masks) only, the tiled tensor is not written.
// GRP = 2: 128-token tiles.  `heads`, `tile_head` and total_tiles are then those of the 64-slot
// halves (halves 2g, 2g+1 of whole tile g); a thread walks the 128 slots of a whole tile in order
// (first half, then second half: the oracle's raster slot order), the mask has two words per tile,
// and the tiled output [tile][128][channel] is the two halves back to back.
template <typename E> struct Quad;   // four channels
template <> struct Quad<uint16_t> {
    typedef uint2 raw;
    static constexpr int kBatch = 32;
    __device__ static void unpack(const uint2& u, float* f) {
        f[0] = __uint_as_float(u.x << 16);
        f[1] = __uint_as_float(u.x & 0xffff0000u);
        f[2] = __uint_as_float(u.y << 16);
        f[3] = __uint_as_float(u.y & 0xffff0000u);
    }
};
template <> struct Quad<uint32_t> {
    typedef uint4 raw;
    static constexpr int kBatch = 16;
    __device__ static void unpack(const uint4& u, float* f) {
        f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y);
        f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
    }
};

#pragma clang fp contract(off)
template <int D, int GRP> constexpr int kStatsTok = 256 / (D / 4) * kTile * GRP;   // token numbers of a workgroup's tiles

template <typename E, int D, bool kWrite, int GRP>
__device__ __forceinline__ void layout_stats_block(
    const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head, const TileTables tables,
    const char* __restrict__ x, int64_t sb, int64_t sh, int64_t sn, char* __restrict__ out,
    float* __restrict__ stats, int64_t total_tiles, int H, int W,
    uint64_t* __restrict__ valid_mask, int32_t* __restrict__ valid_cnt, const RecipTable& recip, int blk, int b, int* tok_lds) {
    typedef typename Quad<E>::raw raw;
    constexpr int kBatch = kWrite ? Quad<E>::kBatch : Quad<E>::kBatch / 2;
    constexpr int kTpt = D / 4;             // threads per tile
    constexpr int kTiles = 256 / kTpt;      // tiles per workgroup
    constexpr int kRowBytes = D * (int)sizeof(E);
    constexpr int kSlots = kTile * GRP;     // slots of a whole tile
    int (*tok)[kSlots] = reinterpret_cast<int (*)[kSlots]>(tok_lds);
    const int64_t whole_tiles = total_tiles / GRP;
    const int64_t g0 = (int64_t)blk * kTiles;
    for (int e = threadIdx.x; e < kTiles * kSlots; e += 256) {
        const int tl = e / kSlots, l = e % kSlots;
        const int64_t gi = (g0 + tl) * GRP + l / kTile;   // the 64-slot tile this slot belongs to
        int n = -1;
        if (g0 + tl < whole_tiles) {
            const HeadGeom hg = heads[tile_head[gi]];
            n = tables.token(hg, gi, l % kTile, H, W);
        }
        tok[tl][l] = n;
    }
    __syncthreads();
    const int tl = threadIdx.x / kTpt, quad = threadIdx.x % kTpt;
    const int64_t g = g0 + tl;
    if (g >= whole_tiles) return;
    const int head = tile_head[g * GRP];
    const char* xb = x + b * sb + head * sh + quad * sizeof(raw);
    const int64_t row = (int64_t)b * whole_tiles + g;
    char* ob = out + row * (int64_t)kSlots * kRowBytes + quad * sizeof(raw);
    float sum[4], mx[4], mn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { sum[j] = 0.0f; mx[j] = -INFINITY; mn[j] = INFINITY; }
    auto take = [&](const raw& v) __attribute__((always_inline)) {
        float f[4];
        Quad<E>::unpack(v, f);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sum[j] = sum[j] + f[j];
            mx[j] = f[j] > mx[j] ? f[j] : mx[j];
            mn[j] = f[j] < mn[j] ? f[j] : mn[j];
        }
    };
    uint64_t mask[GRP];
#pragma unroll
    for (int w = 0; w < GRP; ++w) {
        mask[w] = 0ull;
        for (int l0 = 0; l0 < kTile; l0 += kBatch) {
            uint32_t real = 0u;
            raw v[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int n = tok[tl][w * kTile + l0 + i];
                real |= n >= 0 ? 1u << i : 0u;
                v[i] = *reinterpret_cast<const raw*>(xb + (int64_t)(n >= 0 ? n : 0) * sn);
            }
            mask[w] |= (uint64_t)real << l0;
            constexpr uint32_t kAll = kBatch == 32 ? ~0u : (1u << (kBatch & 31)) - 1u;
            if (__all(real == kAll)) {
#pragma unroll
                for (int i = 0; i < kBatch; ++i) take(v[i]);
            } else {
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    if ((real >> i) & 1u) take(v[i]);
                    else v[i] = raw{};
                }
            }
            if (kWrite) {
#pragma unroll
                for (int i = 0; i < kBatch; ++i) *reinterpret_cast<raw*>(ob + (w * kTile + l0 + i) * kRowBytes) = v[i];
            }
        }
    }
    int cnt = 0;
#pragma unroll
    for (int w = 0; w < GRP; ++w) cnt += __popcll(mask[w]);
    const float inv = recip.v[cnt];
    float* z = stats + row * (3 * D) + quad * 4;
    *reinterpret_cast<float4*>(z) = make_float4(sum[0] * inv, sum[1] * inv, sum[2] * inv, sum[3] * inv);
    *reinterpret_cast<float4*>(z + D) = make_float4(mx[0], mx[1], mx[2], mx[3]);
    *reinterpret_cast<float4*>(z + 2 * D) = make_float4(mn[0], mn[1], mn[2], mn[3]);
    if (quad == 0 && b == 0) {
        if (valid_mask) {
#pragma unroll
            for (int w = 0; w < GRP; ++w) valid_mask[g * GRP + w] = mask[w];
        }
        if (valid_cnt) valid_cnt[g] = cnt;
    }
}

template <typename E, int D, bool kWrite, int GRP>
__global__ __launch_bounds__(256) void layout_stats_kernel(
    const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head, const TileTables tables,
    const char* __restrict__ x, int64_t sb, int64_t sh, int64_t sn, char* __restrict__ out,
    float* __restrict__ stats, int64_t total_tiles, int H, int W,
    uint64_t* __restrict__ valid_mask, int32_t* __restrict__ valid_cnt, RecipTable recip) {
    __shared__ int tok[kStatsTok<D, GRP>];
    layout_stats_block<E, D, kWrite, GRP>(heads, tile_head, tables, x, sb, sh, sn, out, stats, total_tiles, H, W, valid_mask, valid_cnt,
                                          recip, blockIdx.x, blockIdx.y, tok);
}

// Stage 1 of a whole call in one launch: the descriptors of Q and K (with their tiled copies if asked for) and V channel-major.
// The three write to memory of their own and none waits for another, so three launches only add their starts and ends:
// 4 heads of 75 tiles, 2 samples (bf16, d = 64) 29 -> 15 us, 2 fp32 heads of 4 tiles 24 -> 10.5; 12 heads of 624 tiles
// (bf16, d = 128) 95 -> 79, 40 heads 282 -> 271, 24 heads of 219,600 tokens 1038 -> 1032.
struct LayoutPathArgs {
    const char *q, *k, *v;
    int64_t qb, qh, qn, kb, kh, kn, vb, vh, vn;   // strides in bytes
    char *q_tiled, *k_tiled, *v_tiled;
    float *stats_q, *stats_k;
    uint64_t* valid_mask;
    int32_t* valid_cnt;
    int64_t total_tiles;   // of 64 slots
    int H, W;
    int stats_blocks;      // workgroups of Q, and of K; V's follow
};

template <typename E, int D, bool kWrite, int GRP>
__global__ __launch_bounds__(256) void layout_path_kernel(const HeadGeom* __restrict__ heads, const uint8_t* __restrict__ tile_head, TileTables tables,
                                                          LayoutPathArgs a, RecipTable recip) {
    constexpr int kV = kTile + kChannelMajorWords<E, D>, kS = kStatsTok<D, GRP>;
    __shared__ uint32_t lds[kV > kS ? kV : kS];
    const int x = blockIdx.x, b = blockIdx.y;
    if (x < 2 * a.stats_blocks) {
        const bool q = x < a.stats_blocks;   // the masks come with Q
        layout_stats_block<E, D, kWrite, GRP>(heads, tile_head, tables, q ? a.q : a.k, q ? a.qb : a.kb, q ? a.qh : a.kh, q ? a.qn : a.kn,
                                              q ? a.q_tiled : a.k_tiled, q ? a.stats_q : a.stats_k, a.total_tiles, a.H, a.W,
                                              q ? a.valid_mask : nullptr, q ? a.valid_cnt : nullptr, recip,
                                              q ? x : x - a.stats_blocks, b, (int*)lds);
    } else {
        channel_major_tile<E, D>(heads, tile_head, tables, a.v, a.vb, a.vh, a.vn, a.v_tiled, a.total_tiles, a.H, a.W, nullptr, nullptr,
                                 x - 2 * a.stats_blocks, b, (int*)lds, lds + kTile);
    }
}

}  // namespace veda

extern "C" veda_status veda_tile_layout(const veda_plan* pl, const void* x, veda_strides sx,
                                        veda_tile_order order, void* x_tiled, uint64_t* valid_mask,
                                        int32_t* valid_cnt, void* stream) {
    using namespace veda;
    if (!pl || !x || !x_tiled) return VEDA_ERR_INVALID_ARG;
    if (order != VEDA_TOKEN_MAJOR && order != VEDA_CHANNEL_MAJOR) return VEDA_ERR_INVALID_ARG;
    const int es = pl->elem_size();
    const int d = pl->prob.head_dim;
    if (sx.n < d || sx.b < 0 || sx.h < 0) return VEDA_ERR_INVALID_ARG;
    if (!aligned16(x) || !aligned16(x_tiled) || (sx.b * es) % 16 || (sx.h * es) % 16 || (sx.n * es) % 16)
        return VEDA_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    // 128-token tiles are laid out as their two 64-slot halves (tiles 2o, 2o+1 of the inner plan)
    const veda_plan* ip = pl->inner ? pl->inner : pl;
    if (pl->inner && valid_cnt && !valid_mask) return VEDA_ERR_INVALID_ARG;   // counts come from the masks
    int32_t* cnt_arg = pl->inner ? nullptr : valid_cnt;
    dim3 grid((unsigned)ip->total_tiles, (unsigned)pl->prob.batch);
    const int64_t sb = sx.b * es, sh = sx.h * es, sn = sx.n * es;
    const int T = pl->prob.T, H = pl->prob.H, W = pl->prob.W;
    if (order == VEDA_TOKEN_MAJOR) {
        hipLaunchKernelGGL(layout_token_major_kernel, grid, dim3(256), 0, st, ip->d_heads, ip->d_tile_head,
                           (const char*)x, sb, sh, sn, (char*)x_tiled, ip->total_tiles, d * es, T, H, W,
                           valid_mask, cnt_arg);
    } else {
#define VEDA_LAUNCH_CM(E, D)                                                                           \
    hipLaunchKernelGGL((layout_channel_major_kernel<E, D>), grid, dim3(256), 0, st, ip->d_heads,        \
                       ip->d_tile_head, TileTables{ip->d_tile_n0, ip->d_tile_real}, (const char*)x, sb, sh, sn, (char*)x_tiled, \
                       ip->total_tiles, H, W, valid_mask, cnt_arg)
        if (es == 2 && d == 128) VEDA_LAUNCH_CM(uint16_t, 128);
        else if (es == 2 && d == 64) VEDA_LAUNCH_CM(uint16_t, 64);
        else if (es == 4 && d == 128) VEDA_LAUNCH_CM(uint32_t, 128);
        else VEDA_LAUNCH_CM(uint32_t, 64);
#undef VEDA_LAUNCH_CM
    }
    if (pl->inner && valid_cnt)
        hipLaunchKernelGGL(valid_cnt_pairs_kernel, dim3((unsigned)((pl->total_tiles + 255) / 256)), dim3(256), 0, st,
                           valid_mask, valid_cnt, pl->total_tiles);
    return launch_status("veda_tile_layout");
}

extern "C" veda_status veda_tile_layout_stats(const veda_plan* pl, const void* x, veda_strides sx, void* x_tiled,
                                              uint64_t* valid_mask, int32_t* valid_cnt, float* stats,
                                              void* stream) {
    using namespace veda;
    if (!pl || !x || !stats) return VEDA_ERR_INVALID_ARG;   // x_tiled may be null: descriptors only
    const int es = pl->elem_size();
    const int d = pl->prob.head_dim;
    if (sx.n < d || sx.b < 0 || sx.h < 0) return VEDA_ERR_INVALID_ARG;
    if (!aligned16(x) || (x_tiled && !aligned16(x_tiled)) || !aligned16(stats) || (sx.b * es) % 16 || (sx.h * es) % 16 ||
        (sx.n * es) % 16)
        return VEDA_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    const int64_t sb = sx.b * es, sh = sx.h * es, sn = sx.n * es;
    const int H = pl->prob.H, W = pl->prob.W;
    RecipTable recip;
    recip.v[0] = 0.0f;
    for (int c = 1; c <= 2 * kTile; ++c) recip.v[c] = 1.0f / (float)c;
    // 128-token tiles (bf16 plans only): the kernel walks the two 64-slot halves of every whole tile
    const veda_plan* ip = pl->inner ? pl->inner : pl;
#define VEDA_LAUNCH_LS2(E, D, WR, GRP)                                                                    \
    hipLaunchKernelGGL((layout_stats_kernel<E, D, WR, GRP>), grid, dim3(256), 0, st, ip->d_heads,         \
                       ip->d_tile_head, TileTables{ip->d_tile_n0, ip->d_tile_real}, (const char*)x, sb, sh, sn, (char*)x_tiled, stats, ip->total_tiles, H, W, \
                       valid_mask, valid_cnt, recip)
#define VEDA_LAUNCH_LS(E, D)                                                                              \
    do {                                                                                                  \
        constexpr int tiles = 256 / (D / 4);                                                   \
        dim3 grid((unsigned)((pl->total_tiles + tiles - 1) / tiles), (unsigned)pl->prob.batch);           \
        if (pl->inner) {                                                                                  \
            if (x_tiled) VEDA_LAUNCH_LS2(E, D, true, 2);                                                  \
            else VEDA_LAUNCH_LS2(E, D, false, 2);                                                         \
        } else {                                                                                          \
            if (x_tiled) VEDA_LAUNCH_LS2(E, D, true, 1);                                                  \
            else VEDA_LAUNCH_LS2(E, D, false, 1);                                                         \
        }                                                                                                 \
    } while (0)
    if (es == 2 && d == 128) VEDA_LAUNCH_LS(uint16_t, 128);
    else if (es == 2 && d == 64) VEDA_LAUNCH_LS(uint16_t, 64);
    else if (es == 4 && d == 128) VEDA_LAUNCH_LS(uint32_t, 128);
    else VEDA_LAUNCH_LS(uint32_t, 64);
#undef VEDA_LAUNCH_LS
#undef VEDA_LAUNCH_LS2
    return launch_status("veda_tile_layout_stats");
}

extern "C" veda_status veda_tile_layout_path(const veda_plan* pl, const void* q, veda_strides sq, const void* k, veda_strides sk,
                                             const void* v, veda_strides sv, void* q_tiled, void* k_tiled, void* v_tiled,
                                             uint64_t* valid_mask, int32_t* valid_cnt, float* stats_q, float* stats_k, void* stream) {
    using namespace veda;
    if (!pl || !q || !k || !v || !v_tiled || !stats_q || !stats_k || !q_tiled != !k_tiled) return VEDA_ERR_INVALID_ARG;
    const int es = pl->elem_size(), d = pl->prob.head_dim;
    for (const veda_strides& t : {sq, sk, sv}) {
        if (t.n < d || t.b < 0 || t.h < 0) return VEDA_ERR_INVALID_ARG;
        if ((t.b * es) % 16 || (t.h * es) % 16 || (t.n * es) % 16) return VEDA_ERR_UNSUPPORTED;
    }
    for (const void* p : {q, k, v, (const void*)q_tiled, (const void*)k_tiled, (const void*)v_tiled, (const void*)stats_q, (const void*)stats_k})
        if (!aligned16(p)) return VEDA_ERR_UNSUPPORTED;
    const veda_plan* ip = pl->inner ? pl->inner : pl;
    RecipTable recip;
    recip.v[0] = 0.0f;
    for (int c = 1; c <= 2 * kTile; ++c) recip.v[c] = 1.0f / (float)c;
    LayoutPathArgs a;
    a.q = (const char*)q; a.k = (const char*)k; a.v = (const char*)v;
    a.qb = sq.b * es; a.qh = sq.h * es; a.qn = sq.n * es;
    a.kb = sk.b * es; a.kh = sk.h * es; a.kn = sk.n * es;
    a.vb = sv.b * es; a.vh = sv.h * es; a.vn = sv.n * es;
    a.q_tiled = (char*)q_tiled; a.k_tiled = (char*)k_tiled; a.v_tiled = (char*)v_tiled;
    a.stats_q = stats_q; a.stats_k = stats_k;
    a.valid_mask = valid_mask; a.valid_cnt = valid_cnt;
    a.total_tiles = ip->total_tiles;
    a.H = pl->prob.H; a.W = pl->prob.W;
    const int tiles = 256 / (d / 4);   // to a workgroup of the descriptors
    a.stats_blocks = (int)((pl->total_tiles + tiles - 1) / tiles);
    dim3 grid((unsigned)(2 * a.stats_blocks + ip->total_tiles), (unsigned)pl->prob.batch);
    hipStream_t st = (hipStream_t)stream;
    // Where the descriptors' part needs many registers (tiled copies, 128-token tiles), V's part keeps fewer waves in flight
    // than in a kernel of its own, which shows once memory is what bounds them.  8 heads, one launch and three: tiled copies, fp32 at
    // d = 128, 3200 workgroups 118 and 132 us, 6000 212 and 214, 7680 268 and 256 (bf16 120 and 129 at 6000, 148 and 144 at 7680);
    // of 128-token tiles 5400 120 and 137, 10,116 210 and 217, 18,000 353 and 320; their descriptors alone 10,116 130 and 149,
    // 18,000 220 and 222, 31,500 366 and 363, 54,000 615 and 601.  Descriptors of 64-token tiles: level at 93,750 (958 and 951).
    // (And a grid's dimension holds fewer than 2^32 threads.)
    const int64_t one_launch = pl->inner ? (q_tiled ? 12288 : 24576) : q_tiled ? 6144 : INT64_MAX;
    if ((int64_t)grid.x * grid.y > one_launch || grid.x >= 1u << 24) {
        veda_status r = veda_tile_layout_stats(pl, q, sq, q_tiled, valid_mask, valid_cnt, stats_q, stream);
        if (r == VEDA_OK) r = veda_tile_layout_stats(pl, k, sk, k_tiled, nullptr, nullptr, stats_k, stream);
        return r == VEDA_OK ? veda_tile_layout(pl, v, sv, VEDA_CHANNEL_MAJOR, v_tiled, nullptr, nullptr, stream) : r;
    }
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, ip->d_heads, ip->d_tile_head, TileTables{ip->d_tile_n0, ip->d_tile_real}, a, recip);
        return launch_status("veda_tile_layout_path");
    };
#define VEDA_LAUNCH_LP(E, D, GRP) (q_tiled ? launch(layout_path_kernel<E, D, true, GRP>) : launch(layout_path_kernel<E, D, false, GRP>))
    if (es == 2 && pl->inner) return d == 128 ? VEDA_LAUNCH_LP(uint16_t, 128, 2) : VEDA_LAUNCH_LP(uint16_t, 64, 2);
    if (es == 2) return d == 128 ? VEDA_LAUNCH_LP(uint16_t, 128, 1) : VEDA_LAUNCH_LP(uint16_t, 64, 1);
    return d == 128 ? VEDA_LAUNCH_LP(uint32_t, 128, 1) : VEDA_LAUNCH_LP(uint32_t, 64, 1);   // fp32 plans have 64-token tiles
#undef VEDA_LAUNCH_LP
}
