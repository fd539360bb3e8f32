// Stage 2 -- statistics-aware tile scoring (Eq. 4 TripPool, Eq. 5 projections and score;
// Alg. 2 "Triplet Statistics Extraction" and "Projection & Score Estimation").
//
// The scores decide an integer (the top-k set), so every number here is produced by a fixed
// sequence of IEEE fp32 operations: this file is compiled with floating-point contraction
// off, every fused multiply-add is written as fmaf or issued as v_mfma_f32_32x32x2_f32 (which
// applies its two terms one after the other as fmas: see mlp_layer), and no chain is split or
// re-associated.
//   TripPool : sum over real slots in ascending slot order from +0; avg = sum * (1/count)
//              with 1/count rounded once on the host; max/min by plain comparisons.
//   phi      : per output, one fmaf chain over ascending input index started from the bias.
//   score    : per (i,j), one fmaf chain over ascending latent index from +0, then * scale.
#include <type_traits>

#include "direct_load.h"
#include "score_common.h"

#pragma clang fp contract(off)

namespace veda {

// One thread owns kN channels of one tile and walks its slots in order (kWords = 1: 64-token
// tiles; kWords = 2: 128-token tiles, stored as two consecutive 64-slot halves with one mask
// word each, so slot order is unchanged).
// grid = (ceil(rows / tiles_per_block), 2 tensors); rows = batch * total_tiles.
template <typename E, int D, int kWords>
__global__ __launch_bounds__(256) void trippool_kernel(const char* __restrict__ q_tiled,
                                                       const char* __restrict__ k_tiled,
                                                       const uint64_t* __restrict__ valid_mask,
                                                       float* __restrict__ zq, float* __restrict__ zk,
                                                       int64_t rows, int64_t total_tiles, RecipTable recip) {
    constexpr int kN = Chunk<E>::kN;
    constexpr int kTpt = D / kN;                 // threads per tile
    constexpr int kRowBytes = D * (int)sizeof(E);
    constexpr int kSlots = kWords * kTile;
    const int64_t row = (int64_t)blockIdx.x * (256 / kTpt) + threadIdx.x / kTpt;
    if (row >= rows) return;
    const int chunk = threadIdx.x % kTpt;
    const char* src = (blockIdx.y == 0 ? q_tiled : k_tiled) + row * (int64_t)kSlots * kRowBytes + chunk * 16;
    float* z = (blockIdx.y == 0 ? zq : zk) + row * (3 * D) + chunk * kN;
    uint64_t mask[kWords];
    bool full = true;
    int count = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
        mask[w] = valid_mask[(row % total_tiles) * kWords + w];
        full = full && mask[w] == ~0ull;
        count += __popcll(mask[w]);
    }
    float sum[kN], mx[kN], mn[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) { sum[j] = 0.0f; mx[j] = -INFINITY; mn[j] = INFINITY; }
    if (full) {
#pragma unroll 8
        for (int l = 0; l < kSlots; ++l) {
            float f[kN];
            Chunk<E>::unpack(*reinterpret_cast<const uint4*>(src + l * kRowBytes), f);
#pragma unroll
            for (int j = 0; j < kN; ++j) {
                sum[j] = sum[j] + f[j];
                mx[j] = f[j] > mx[j] ? f[j] : mx[j];
                mn[j] = f[j] < mn[j] ? f[j] : mn[j];
            }
        }
    } else {
#pragma unroll
        for (int w = 0; w < kWords; ++w) {
            for (int l = 0; l < kTile; ++l) {
                if (!((mask[w] >> l) & 1ull)) continue;
                float f[kN];
                Chunk<E>::unpack(*reinterpret_cast<const uint4*>(src + (w * kTile + l) * kRowBytes), f);
#pragma unroll
                for (int j = 0; j < kN; ++j) {
                    sum[j] = sum[j] + f[j];
                    mx[j] = f[j] > mx[j] ? f[j] : mx[j];
                    mn[j] = f[j] < mn[j] ? f[j] : mn[j];
                }
            }
        }
    }
    const float inv = recip.v[count];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
        z[j] = sum[j] * inv;
        z[D + j] = mx[j];
        z[2 * D + j] = mn[j];
    }
}

constexpr int kMlpRows = 64;       // tiles per workgroup
constexpr int kMlpCols = 128;      // output units per pass
constexpr int kMlpK = 16;          // reduction indices staged per step
constexpr int kMlpThreads = 256;
constexpr int kMlpXPitch = kMlpK + 4;   // floats; keeps every staged row 16-byte aligned
constexpr int kMlpWsFloats = kMlpK * kMlpCols;        // one weight stage
constexpr int kMlpXsFloats = kMlpRows * kMlpXPitch;   // one input stage

// One affine layer for the 64 rows of a workgroup:
//   out[r][n] = act(bias[n] + sum_k x[r][k] * w[k][n]),  one fmaf chain per (r,n), k ascending.
// The chains run on the matrix cores: v_mfma_f32_32x32x2_f32 adds its two products to the
// accumulator one after the other, each with its own rounding, in ascending k -- measured on
// gfx950 to give the bits of fmaf(x[k+1], w[k+1], fmaf(x[k], w[k], acc)) on 245,760 random chains
// of 64 terms, denormal sums and products included -- so a chain of these instructions over
// k = 0, 2, 4, ... started from the bias IS the chain above, at twice the rate of scalar fp32
// fma.  Wave w of the four owns output columns c0+32w..+31 for both 32-row halves (two 32x32
// accumulators); lane (col = lane%32, kh = lane/32) feeds x[row = col (+32)][k+kh] and
// w[k+kh][column] and holds rows (r%4) + 8(r/4) + 4kh of its column in register r.
// The weights of 16 reduction indices x 128 outputs are staged in LDS per step (ws, two buffers);
// the inputs come either from global memory, staged alongside (xs, two buffers), or from a
// resident LDS array (x_lds).  The global loads of step s+1 are in flight while step s is
// computed; one barrier per step.  Results go to an LDS array (y_lds, pitch ldy) or to global
// rows (y_glb, pitch N).
typedef __attribute__((ext_vector_type(16))) float mlp_f32x16;

template <bool kXGlobal, bool kYLds>
__device__ __forceinline__ void mlp_layer(const float* __restrict__ x_glb, const float* x_lds, int ldx, int rows,
                                          int K, const float* __restrict__ w, const float* __restrict__ bias,
                                          int N, bool relu, float* y_lds, int ldy, float* __restrict__ y_glb,
                                          float* xs, float* ws) {
    constexpr int kWPer = kMlpWsFloats / kMlpThreads;   // staged weights per thread and step (8)
    static_assert(kMlpRows * (kMlpK / 4) == kMlpThreads, "one float4 of the inputs per thread and step");
    static_assert(kMlpRows == 64 && kMlpCols == 128 && kMlpThreads == 256, "four waves x (2 x 32 rows) x 32 columns");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, kh = lane >> 5;
    const int xr = threadIdx.x / (kMlpK / 4), xi = (threadIdx.x % (kMlpK / 4)) * 4;   // staged input float4
    for (int c0 = 0; c0 < N; c0 += kMlpCols) {
        // 64 columns or fewer left (the second layer of the usual estimators): four waves x 32 rows x 32 columns, so
        // that no wave sits idle and each has half the instructions (stages 2+3 of 4 blocks of 64 rows, 192 -> 64 -> 32:
        // 33.2 -> 29.5 us; of 24 heads of 219,600 tokens, 384 -> 128 -> 64: 1125 -> 1116 us)
        const bool narrow = N - c0 <= kMlpCols / 2;
        const int half = narrow ? wave >> 1 : 0, wcol = 32 * (narrow ? wave & 1 : wave);   // first row half, first column
        const int n = c0 + wcol + col;
        const float bv = n < N ? bias[n] : 0.0f;
        mlp_f32x16 acc[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = bv;
        float wreg[kWPer];
        float4 xreg = make_float4(0.f, 0.f, 0.f, 0.f);
        auto fetch = [&](int k0) {
            const int kc = K - k0 < kMlpK ? K - k0 : kMlpK;
#pragma unroll
            for (int u = 0; u < kWPer; ++u) {
                const int t = threadIdx.x + u * kMlpThreads, i = t / kMlpCols, c = t % kMlpCols;
                wreg[u] = (i < kc && c0 + c < N) ? w[(int64_t)(k0 + i) * N + c0 + c] : 0.0f;
            }
            if (kXGlobal) {   // K is a multiple of 4 here
                xreg = (xr < rows && xi < kc) ? *reinterpret_cast<const float4*>(x_glb + (int64_t)xr * K + k0 + xi)
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        };
        auto stash = [&](int buf) {
#pragma unroll
            for (int u = 0; u < kWPer; ++u) ws[buf * kMlpWsFloats + threadIdx.x + u * kMlpThreads] = wreg[u];
            if (kXGlobal) *reinterpret_cast<float4*>(xs + buf * kMlpXsFloats + xr * kMlpXPitch + xi) = xreg;
        };
        __syncthreads();   // the previous pass (or layer) is done with both stages
        fetch(0);
        stash(0);
        __syncthreads();
        int buf = 0;
        for (int k0 = 0; k0 < K; k0 += kMlpK, buf ^= 1) {
            const int kc = K - k0 < kMlpK ? K - k0 : kMlpK;
            const bool more = k0 + kMlpK < K;
            if (more) fetch(k0 + kMlpK);
            const float* wb = ws + buf * kMlpWsFloats + wcol + col + kh * kMlpCols;
            const int xp = kXGlobal ? kMlpXPitch : ldx;
            const float* xb = (kXGlobal ? xs + buf * kMlpXsFloats : x_lds + k0) + (32 * half + col) * xp + kh;
            if (kc == kMlpK && narrow) {
#pragma unroll
                for (int kk = 0; kk < kMlpK; kk += 2)
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[kk], wb[kk * kMlpCols], acc[0], 0, 0, 0);
            } else if (kc == kMlpK) {
#pragma unroll
                for (int kk = 0; kk < kMlpK; kk += 2) {
                    const float b = wb[kk * kMlpCols];
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[kk], b, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[32 * xp + kk], b, acc[1], 0, 0, 0);
                }
            } else {
                const int other = narrow ? 0 : 32 * xp;   // narrow: the second accumulator is not used
                int kk = 0;
                for (; kk + 2 <= kc; kk += 2) {
                    const float b = wb[kk * kMlpCols];
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[kk], b, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[other + kk], b, acc[1], 0, 0, 0);
                }
                if (kk < kc) {
                    // odd reduction length: the instruction's second term is made -0 * +0 = -0, the one
                    // addend that leaves every accumulator value, signed zeros included, as it is
                    const float b = kh ? 0.0f : wb[kk * kMlpCols];
                    const float a0 = kh ? -0.0f : xb[kk], a1 = kh ? -0.0f : xb[other + kk];
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b, acc[1], 0, 0, 0);
                }
            }
            if (more) stash(buf ^ 1);
            __syncthreads();
        }
        if (n < N) {
            // one running pointer, advanced store by store: 32 precomputed 64-bit addresses would
            // not fit beside the accumulators
            int row = 32 * half + 4 * kh;
            float* yp = kYLds ? y_lds + row * ldy + n : y_glb + (int64_t)row * N + n;
            const int pitch = kYLds ? ldy : N;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                if (rb == 1 && narrow) break;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float v = (relu && !(acc[rb][r] > 0.0f)) ? 0.0f : acc[rb][r];
                    if (kYLds || row < rows) *yp = v;
                    // next row: +1 inside a group of four, +5 to the next group (rows 8g..8g+3 of this lane half)
                    const int step = (r & 3) == 3 ? 5 : 1;
                    yp += (int64_t)step * pitch;
                    row += step;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
}

// One workgroup projects up to 64 consecutive tiles of one head (Eq. 5, phi_q or phi_k).
// row_blk[x] = head << 24 | index of the 64-tile block inside that head.
// grid = (row blocks of all heads, 2 estimators, batch); dynamic LDS = staging + hidden layer.
__global__ __launch_bounds__(kMlpThreads, 3) void mlp_kernel(const HeadGeom* __restrict__ heads,
                                                         const int32_t* __restrict__ row_blk,
                                                         const float* __restrict__ zq, const float* __restrict__ zk,
                                                         float* __restrict__ yq, float* __restrict__ yk,
                                                         MlpDev pq, MlpDev pk, int64_t total_tiles,
                                                         float* __restrict__ hq, float* __restrict__ hk) {
    extern __shared__ __align__(16) float smem[];
    const MlpDev p = blockIdx.y == 0 ? pq : pk;
    float* hglb = blockIdx.y == 0 ? hq : hk;   // hidden layer kept in global scratch instead of LDS, if given
    const float* z = blockIdx.y == 0 ? zq : zk;
    float* y = blockIdx.y == 0 ? yq : yk;
    float* ws = smem;                                   // 2 x [16][128]
    float* xs = ws + 2 * kMlpWsFloats;                  // 2 x [64][20]
    float* hs = xs + 2 * kMlpXsFloats;                  // [64][ldh]
    const int32_t code = row_blk[blockIdx.x];
    const int head = code >> 24, blk = code & 0xffffff;
    const HeadGeom hg = heads[head];
    const int rows = hg.n_tiles - blk * kMlpRows < kMlpRows ? hg.n_tiles - blk * kMlpRows : kMlpRows;
    const int64_t row0 = (int64_t)blockIdx.z * total_tiles + hg.tile_off + (int64_t)blk * kMlpRows;
    const float* x = z + row0 * p.in_dim;
    float* out = y + row0 * p.out_dim;
    if (p.hidden && hglb) {
        // The 64 x hidden intermediate goes through global memory (it stays in L2): without it in
        // LDS more workgroups fit on a compute unit (three instead of two).  The barrier that opens the second
        // layer also orders these stores before its loads (same workgroup).
        float* hrow = hglb + row0 * p.hidden;
        mlp_layer<true, false>(x, nullptr, 0, rows, p.in_dim, p.w1 + (int64_t)head * p.in_dim * p.hidden,
                  p.b1 + (int64_t)head * p.hidden, p.hidden, p.relu != 0, nullptr, 0, hrow, xs, ws);
        mlp_layer<true, false>(hrow, nullptr, 0, rows, p.hidden, p.w2 + (int64_t)head * p.hidden * p.out_dim,
                  p.b2 + (int64_t)head * p.out_dim, p.out_dim, false, nullptr, 0, out, xs, ws);
    } else if (p.hidden) {
        const int ldh = (p.hidden + 3) & ~3;
        mlp_layer<true, true>(x, nullptr, 0, rows, p.in_dim, p.w1 + (int64_t)head * p.in_dim * p.hidden,
                  p.b1 + (int64_t)head * p.hidden, p.hidden, p.relu != 0, hs, ldh, nullptr, xs, ws);
        mlp_layer<false, false>(nullptr, hs, ldh, rows, p.hidden, p.w2 + (int64_t)head * p.hidden * p.out_dim,
                  p.b2 + (int64_t)head * p.out_dim, p.out_dim, false, nullptr, 0, out, xs, ws);
    } else {
        mlp_layer<true, false>(x, nullptr, 0, rows, p.in_dim, p.w1 + (int64_t)head * p.in_dim * p.out_dim,
                  p.b1 + (int64_t)head * p.out_dim, p.out_dim, false, nullptr, 0, out, xs, ws);
    }
}

// The same projections for the usual sizes (hidden 128 or 64, in_dim a multiple of 16): 16 reduction indices of weights and
// inputs at a time through a ring of kDepth stages in LDS, filled by direct loads two stages ahead, one barrier per stage.
// Bound by the matrix pipe where there are many blocks and by the chain of a block where there are few, so a workgroup
// takes as few rows as give its four waves a 32 x 32 block each: 32 of 128 outputs (half the chain of the kernel above, and
// twice the workgroups: 40 heads of 624 tiles were 800 workgroups on 768 places, a second round for 32 of them), 64 of 64.
// The hidden layer stays in LDS, over the first layer's stages.
// Measured, kernel above and this one, between the other kernels of a call: 4 heads of 75 tiles, 2 samples (192 -> 64 -> 32)
// 22 -> 13 us; 384 -> 128 -> 64: 12 heads of 624 tiles 51 -> 32, 40 heads 130 -> 87, 24 heads of 219,600 tokens 282 -> 232 us
// (88 TFLOP/s).  A block's 32 stages take 1700 cycles each where two share a SIMD, 1024 of them products.
// LDS stages: weights [16][N] as they lie in memory, odd rows with the 128-byte halves of each 256 bytes exchanged (lanes
// 0-31 read row k, lanes 32-63 row k + 1); inputs [rows][16], 16-byte chunk ^ row / 4.
template <int N> struct MlpStage {
    static constexpr int kBytes = 16 * N * 4, kLoads = kBytes / 1024, kRowChunks = N / 4;
    static constexpr int kPer = kLoads >= 4 ? kLoads / 4 : 1;   // loads per wave; two loads: waves 2, 3 repeat those of 0, 1
    static __device__ __forceinline__ uint32_t lane_offset(int lane) {
        const int row = lane / kRowChunks, c = lane % kRowChunks;
        return (uint32_t)(row * kRowChunks + (N % 64 == 0 ? c ^ ((row & 1) << 3) : c)) * 16u;
    }
    // rows k .. k + 15 of w, k = 16 * stage
    static __device__ __forceinline__ void load(const float* w, int stage, uint32_t lds, int wave, uint32_t lane_off) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int q = kLoads >= 4 ? wave * kPer + i : wave & 1;
            dma16_to_lds(lds + 1024u * q, (const char*)w + (int64_t)stage * kBytes + 1024 * q, lane_off);
        }
    }
};

// Stages of the ring: four, 40 KB for 128 outputs (three: 215 instead of 210 us for stages 2+3 of 40 heads of 624 tiles, six: 237).
constexpr int kMlpDepth = 4;

template <int N1, int N2, int kRows>
__global__ __launch_bounds__(256) void mlp_staged_kernel(const HeadGeom* __restrict__ heads, const int32_t* __restrict__ row_blk,
                                                            const float* __restrict__ zq, const float* __restrict__ zk,
                                                            float* __restrict__ yq, float* __restrict__ yk, MlpDev pq, MlpDev pk,
                                                            int64_t total_tiles) {
    typedef MlpStage<N1> W1;
    typedef MlpStage<N2> W2;
    constexpr int kXLoads = kRows / 16;                         // 1024-byte loads of a stage's inputs: 2 or 4
    constexpr int kStage = W1::kBytes + kXLoads * 1024, kDepth = kMlpDepth;
    constexpr int kC1 = W1::kPer + 1, kC2 = W2::kPer;           // loads per wave and stage
    constexpr int kPitchB = (N1 + 4) * 4;                       // of the hidden layer: rows on all banks
    // The hidden rows lie in the first three stages, behind what the second layer's stages take of them.
    constexpr int kPieceRows = (kStage - W2::kBytes) / kPitchB;
    static_assert(kDepth >= 3 && 3 * kPieceRows >= kRows, "room for the hidden layer");
    auto hidden_row = [](int r) { return (uint32_t)(r / kPieceRows * kStage + W2::kBytes + r % kPieceRows * kPitchB); };
    constexpr int kSub = kLatentRows / kRows;                   // workgroups to an entry of the row-block table
    static_assert((kRows / 32) * (N1 / 32) == 4, "a 32 x 32 block for each wave");
    extern __shared__ __align__(1024) float smem[];
    const MlpDev p = blockIdx.y == 0 ? pq : pk;
    const int32_t code = row_blk[blockIdx.x / kSub];
    const int head = code >> 24, first = (code & 0xffffff) * kLatentRows + (int)(blockIdx.x % kSub) * kRows;
    const HeadGeom hg = heads[head];
    const int rows = hg.n_tiles - first < kRows ? hg.n_tiles - first : kRows;
    if (rows <= 0) return;
    const int64_t row0 = (int64_t)blockIdx.z * total_tiles + hg.tile_off + first;
    const int K = p.in_dim, n1 = K / 16;
    constexpr int n2 = N1 / 16;
    const char* x = (const char*)((blockIdx.y == 0 ? zq : zk) + row0 * K);
    float* y = (blockIdx.y == 0 ? yq : yk) + row0 * N2;
    const float* w1 = p.w1 + (int64_t)head * K * N1;
    const float* w2 = p.w2 + (int64_t)head * N1 * N2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), col = lane & 31, kh = lane >> 5;
    const int rb = wave / (N1 / 32), cb = wave % (N1 / 32);     // this wave's block of the hidden layer
    const int rb2 = wave / (N2 / 32), cb2 = wave % (N2 / 32);   // and of the output, if it has one
    float b1 = p.b1[head * N1 + 32 * cb + col], b2 = p.b2[head * N2 + 32 * cb2 + col];
    asm volatile("" : "+v"(b1), "+v"(b2));   // have arrived before the loads that are counted
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t off1 = W1::lane_offset(lane), off2 = W2::lane_offset(lane);
    const int xq = wave % kXLoads;
    uint32_t xoff;
    {
        const int row = 16 * xq + lane / 4, real = row < rows ? row : rows - 1;
        xoff = (uint32_t)(real * K * 4 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
    }
    // stages 0 .. n1 - 1 are the first layer's, those after them the second's
    auto load = [&](int s) __attribute__((always_inline)) {
        const uint32_t at = base + (uint32_t)(s % kDepth) * kStage;
        if (s < n1) {
            W1::load(w1, s, at, wave, off1);
            dma16_to_lds(at + W1::kBytes + 1024u * xq, x + 64 * s, xoff);
        } else if (s < n1 + n2) {
            W2::load(w2, s - n1, at, wave, off2);
        }
    };
    auto meet = []() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    typedef const __attribute__((address_space(3))) float* lds_f32_ptr;
    typedef __attribute__((address_space(3))) float* lds_f32_wptr;
    typedef __attribute__((ext_vector_type(4))) float f4;
    typedef const __attribute__((address_space(3))) f4* lds_f4_ptr;
    // 16 terms of the chains: x(m) gives the four inputs 4m .. 4m + 3 of this lane's row
    auto chain = [&](mlp_f32x16 acc, uint32_t w, int n, int c, auto xs) __attribute__((always_inline)) {
        const uint32_t wl = w + (uint32_t)(kh * n + ((32 * c + col) ^ (n % 64 == 0 ? kh << 5 : 0))) * 4u;
        f4 a[4];
        float b[8];
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] = xs(m);
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = *(lds_f32_ptr)(uintptr_t)(wl + (uint32_t)(2 * i * n * 4));
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float even = a[i >> 1][2 * (i & 1)], odd = a[i >> 1][2 * (i & 1) + 1];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(kh ? odd : even, b[i], acc, 0, 0, 0);
        }
        return acc;
    };
#pragma unroll
    for (int s = 0; s < kDepth - 1; ++s) load(s);
    mlp_f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = b1;
    const int xrow = 32 * rb + col;
    for (int s = 0; s < n1; ++s) {
        // stage s has landed: only the loads of the kDepth - 2 stages after it are on their way, of which the second layer's
        // have fewer
        if (s + kDepth - 2 < n1) wait_vmcnt<(kDepth - 2) * kC1>(); else wait_vmcnt<(kDepth - 2) * kC2>();
        meet();
        load(s + kDepth - 1);   // into the place that everybody has left
        const uint32_t at = base + (uint32_t)(s % kDepth) * kStage;
        acc = chain(acc, at, N1, cb, [&](int m) __attribute__((always_inline)) {
            return *(lds_f4_ptr)(uintptr_t)(at + W1::kBytes + xrow * 64 + ((m ^ ((xrow >> 2) & 3)) << 4));
        });
    }
    meet();   // the first layer's stages have been read
    const bool relu = p.relu != 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float v = (relu && !(acc[r] > 0.0f)) ? 0.0f : acc[r];
        *(lds_f32_wptr)(uintptr_t)(base + hidden_row(32 * rb + (r & 3) + 8 * (r >> 2) + 4 * kh) + (uint32_t)(32 * cb + col) * 4u) = v;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = b2;
    const bool has_block = 32 * rb2 < kRows;
    const uint32_t hrow = base + hidden_row(has_block ? 32 * rb2 + col : 0);
    for (int s = n1; s < n1 + n2; ++s) {
        if (s + kDepth - 2 < n1 + n2) wait_vmcnt<(kDepth - 2) * kC2>(); else wait_vmcnt<0>();
        meet();
        load(s + kDepth - 1);
        if (has_block)
            acc = chain(acc, base + (uint32_t)(s % kDepth) * kStage, N2, cb2, [&](int m) __attribute__((always_inline)) {
                return *(lds_f4_ptr)(uintptr_t)(hrow + (uint32_t)(16 * (s - n1) + 4 * m) * 4u);
            });
    }
    if (has_block) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 32 * rb2 + (r & 3) + 8 * (r >> 2) + 4 * kh;
            if (row < rows) y[(int64_t)row * N2 + 32 * cb2 + col] = acc[r];
        }
    }
}

// The same for few rows, where the time is that of one workgroup's chain: v_mfma_f32_16x16x4_f32 takes four terms of a chain in
// 32 cycles where the 32 x 32 form takes two in 64 (the same bits: chain_probe_kernel), so a workgroup has 16 rows, its wavefronts
// a quarter of the columns each, and a stage's operands are read behind the products of the one before.
// LDS stages: weights [16][N], the 64-byte blocks of row k exchanged by k % 4 (N = 32: by k / 2 % 2), so that the four rows an
// instruction takes lie on all banks; inputs [16][16], 16-byte chunk ^ row / 4.  The hidden layer has a place of its own.
template <int N> struct MlpStage16 {
    static constexpr int kBytes = 16 * N * 4, kLoads = kBytes / 1024, kRowChunks = N / 4;
    static constexpr int kPer = kLoads >= 4 ? kLoads / 4 : 1;   // loads per wave; two loads: waves 2, 3 repeat those of 0, 1
    static_assert(N == 128 || N == 64 || N == 32, "rows to a load, loads to a wave");
    static __device__ __forceinline__ uint32_t lane_offset(int lane) {
        const int row = lane / kRowChunks, c = lane % kRowChunks;
        return (uint32_t)(row * kRowChunks + (c ^ (N == 32 ? (row >> 1 & 1) << 2 : (row & 3) << 2))) * 16u;
    }
    static __device__ __forceinline__ void load(const float* w, int stage, uint32_t lds, int wave, uint32_t lane_off) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int q = kLoads >= 4 ? wave * kPer + i : wave & 1;
            // N = 128: two rows to a load, every second load the rows 2 and 3 of four
            dma16_to_lds(lds + 1024u * q, (const char*)w + (int64_t)stage * kBytes + 1024 * q, N == 128 && (i & 1) ? lane_off ^ 128u : lane_off);
        }
    }
    // of row 4i + h, columns 16c .. 16c + 15
    static __device__ __forceinline__ uint32_t at(int i, int h, int c) {
        return (uint32_t)((4 * i + h) * N * 4 + (c ^ (N == 32 ? h >> 1 : h)) * 64);
    }
};

// Measured, whole calls with the kernel above and this one: 75 tiles (192 -> 64 -> 32) 50.1 -> 45.4 us, 4 heads of 75, 2 samples
// 76.4 -> 71.8; 3 heads of 64 (384 -> 128 -> 64) 52.5 -> 48.3, 8 heads of 624 403 -> 398, 12 heads of 624 892 -> 899 (936
// workgroups; at 192 -> 64 -> 32 384 -> 381), 40 heads of 624 1911 -> 1923: this one up to as many workgroups as are resident.
constexpr int64_t kRows16Most = 768;   // three to a compute unit (45 KB)

template <int N1, int N2>
constexpr int kMlp16Lds = kMlpDepth * (MlpStage16<N1>::kBytes + 1024) + 16 * (N1 + 4) * 4;

template <int N1, int N2>
__global__ __launch_bounds__(256) void mlp_rows16_kernel(const HeadGeom* __restrict__ heads, const int32_t* __restrict__ row_blk,
                                                            const float* __restrict__ zq, const float* __restrict__ zk,
                                                            float* __restrict__ yq, float* __restrict__ yk, MlpDev pq, MlpDev pk,
                                                            int64_t total_tiles) {
    typedef MlpStage16<N1> W1;
    typedef MlpStage16<N2> W2;
    constexpr int kRows = 16, kSub = kLatentRows / kRows, kDepth = kMlpDepth;
    constexpr int kStage = W1::kBytes + 1024, kHidden = kDepth * kStage, kPitchB = (N1 + 4) * 4;
    constexpr int kC1 = W1::kPer + 1, kC2 = W2::kPer;   // loads per wave and stage
    static_assert(kDepth == 4 && kC2 <= kC1, "the waits below");
    constexpr int kCols = N1 / 64;                      // blocks of 16 columns of a wavefront
    extern __shared__ __align__(1024) float smem[];
    const MlpDev p = blockIdx.y == 0 ? pq : pk;
    const int32_t code = row_blk[blockIdx.x / kSub];
    const int head = code >> 24, first = (code & 0xffffff) * kLatentRows + (int)(blockIdx.x % kSub) * kRows;
    const HeadGeom hg = heads[head];
    const int rows = hg.n_tiles - first < kRows ? hg.n_tiles - first : kRows;
    if (rows <= 0) return;
    const int64_t row0 = (int64_t)blockIdx.z * total_tiles + hg.tile_off + first;
    const int K = p.in_dim, n1 = K / 16;
    constexpr int n2 = N1 / 16;
    const char* x = (const char*)((blockIdx.y == 0 ? zq : zk) + row0 * K);
    float* y = (blockIdx.y == 0 ? yq : yk) + row0 * N2;
    const float* w1 = p.w1 + (int64_t)head * K * N1;
    const float* w2 = p.w2 + (int64_t)head * N1 * N2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), col = lane & 15, h = lane >> 4;
    const bool has_block = 16 * wave < N2;              // of the output
    float b1[kCols], b2 = p.b2[head * N2 + (has_block ? 16 * wave : 0) + col];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
        b1[c] = p.b1[head * N1 + 16 * (kCols * wave + c) + col];
        asm volatile("" : "+v"(b1[c]));   // have arrived before the loads that are counted
    }
    asm volatile("" : "+v"(b2));
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t off1 = W1::lane_offset(lane), off2 = W2::lane_offset(lane);
    uint32_t xoff;
    {
        const int row = lane / 4, real = row < rows ? row : rows - 1;
        xoff = (uint32_t)(real * K * 4 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
    }
    // stages 0 .. n1 - 1 are the first layer's, those after them the second's
    auto load = [&](int s) __attribute__((always_inline)) {
        const uint32_t at = base + (uint32_t)(s % kDepth) * kStage;
        if (s < n1) {
            W1::load(w1, s, at, wave, off1);
            dma16_to_lds(at + W1::kBytes, x + 64 * s, xoff);   // by all four: the same count for each
        } else if (s < n1 + n2) {
            W2::load(w2, s - n1, at, wave, off2);
        }
    };
    // Stage s has landed everywhere: of the loads only those of the two stages after it are on their way (the second layer's are fewer).
    auto landed = [&](int s) __attribute__((always_inline)) {
        if (s + 2 < n1) wait_vmcnt<2 * kC1>();
        else if (s + 2 < n1 + n2) wait_vmcnt<2 * kC2>();
        else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    typedef const __attribute__((address_space(3))) float* lds_f32_ptr;
    typedef __attribute__((address_space(3))) float* lds_f32_wptr;
    typedef __attribute__((ext_vector_type(4))) float f4;
    struct Frag { float a[4], b[kCols][4]; };   // term 4i + h of this lane's row, and of its columns
    auto read1 = [&](Frag& f, int s) __attribute__((always_inline)) {
        const uint32_t at = base + (uint32_t)(s % kDepth) * kStage, xr = at + W1::kBytes + (uint32_t)(col * 64 + h * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f.a[i] = *(lds_f32_ptr)(uintptr_t)(xr + (uint32_t)((i ^ (col >> 2)) << 4));
#pragma unroll
            for (int c = 0; c < kCols; ++c) f.b[c][i] = *(lds_f32_ptr)(uintptr_t)(at + W1::at(i, h, kCols * wave + c) + col * 4u);
        }
    };
    auto read2 = [&](Frag& f, int s) __attribute__((always_inline)) {
        const uint32_t at = base + (uint32_t)(s % kDepth) * kStage, hr = base + kHidden + (uint32_t)(col * kPitchB + (16 * (s - n1) + h) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f.a[i] = *(lds_f32_ptr)(uintptr_t)(hr + 16u * i);
            f.b[0][i] = *(lds_f32_ptr)(uintptr_t)(at + W2::at(i, h, has_block ? wave : 0) + col * 4u);
        }
    };
#pragma unroll
    for (int s = 0; s < kDepth - 1; ++s) load(s);
    f4 acc[kCols];
#pragma unroll
    for (int c = 0; c < kCols; ++c) acc[c] = f4{b1[c], b1[c], b1[c], b1[c]};
    Frag f, next;
    landed(0);
    read1(f, 0);
    for (int s = 0; s < n1; ++s) {
        load(s + kDepth - 1);   // into the place of stage s - 1, read before everybody met for stage s
        if (s + 1 < n1) {
            landed(s + 1);
            read1(next, s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < kCols; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[i], f.b[c][i], acc[c], 0, 0, 0);
        f = next;
    }
    const bool relu = p.relu != 0;
#pragma unroll
    for (int c = 0; c < kCols; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float v = (relu && !(acc[c][r] > 0.0f)) ? 0.0f : acc[c][r];
            *(lds_f32_wptr)(uintptr_t)(base + kHidden + (uint32_t)((4 * h + r) * kPitchB + (16 * (kCols * wave + c) + col) * 4)) = v;
        }
    f4 out = {b2, b2, b2, b2};
    landed(n1);   // and the hidden layer is written
    read2(f, n1);
    for (int s = n1; s < n1 + n2; ++s) {
        load(s + kDepth - 1);
        if (s + 1 < n1 + n2) {
            landed(s + 1);
            read2(next, s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (has_block) {
#pragma unroll
            for (int i = 0; i < 4; ++i) out = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[i], f.b[0][i], out, 0, 0, 0);
        }
        f = next;
    }
    if (has_block) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * h + r < rows) y[(int64_t)(4 * h + r) * N2 + 16 * wave + col] = out[r];
    }
}

// Both estimators alike in size, and one of the sizes above.
template <int N1, int N2> static bool staged_sizes(const MlpDev& q, const MlpDev& k, const float* zq, const float* zk) {
    auto fits = [](const MlpDev& p) {
        return p.hidden == N1 && p.out_dim == N2 && p.in_dim % 16 == 0 && aligned16(p.w1) && aligned16(p.w2);
    };
    return fits(q) && fits(k) && q.in_dim == k.in_dim && aligned16(zq) && aligned16(zk);
}

constexpr int kSB = 128;      // score block edge
constexpr int kSC = 32;       // latent coordinates staged per step
constexpr int kSPitch = 36;   // LDS pitch of one staged latent row (floats): rows stay 16-byte
                              // aligned and 8 consecutive rows start in 8 different bank groups

// A 128x128 block (bi, bj) of one head's score matrix (Eq. 5) by one workgroup.  Every score is
// one fma chain over ascending latent coordinate from +0, run on the matrix cores like the
// projections' (see mlp_layer: v_mfma_f32_32x32x2_f32 over the coordinate pairs gives the bits of
// the fmaf chain).  Wave w holds rows 32w..32w+31 x all 128 columns in four 32x32 accumulators:
// register r of lane (col = lane%32, kh = lane/32) is row (r%4) + 8(r/4) + 4kh, column 32cb + col.
// Latent rows are staged row-major in LDS, 32 coordinates at a time.
// Rows and columns past the head's last tile are not multiplied, 32 at a time: a short row's time is that of its own
// products.  Loading the second 32 coordinates behind the first's products spills (20 -> 24..40 us for 12 heads of 624 tiles).
__device__ __forceinline__ void score_block_128(const HeadGeom& hg, int bi, int bj, int64_t b, float* qs, float* ks,
                                                const float* __restrict__ yq, const float* __restrict__ yk,
                                                float* __restrict__ scores, int dp, float scale,
                                                int64_t total_tiles, int64_t score_elems) {
    const int nT = hg.n_tiles;
    const float* qbase = yq + (b * total_tiles + hg.tile_off) * dp;
    const float* kbase = yk + (b * total_tiles + hg.tile_off) * dp;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, kh = lane >> 5;
    mlp_f32x16 acc[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
    constexpr int kPer = kSB * (kSC / 4) / 256;   // float4s of each side per thread and stage
    float4 qv[kPer], kv[kPer];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = threadIdx.x + 256 * u, r = t / (kSC / 4), c4 = (t % (kSC / 4)) * 4;
            qv[u] = kv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c0 + c4 < dp) {   // dp is a multiple of 4
                if (bi * kSB + r < nT) qv[u] = *reinterpret_cast<const float4*>(qbase + (int64_t)(bi * kSB + r) * dp + c0 + c4);
                if (bj * kSB + r < nT) kv[u] = *reinterpret_cast<const float4*>(kbase + (int64_t)(bj * kSB + r) * dp + c0 + c4);
            }
        }
    };
    const float* qa = qs + (32 * wave + col) * kSPitch + kh;   // A: q[row = col][c + kh]
    const float* kb = ks + col * kSPitch + kh;                  // B: k[column = col][c + kh]
    auto products = [&](auto blocks, int cn) {
        auto step = [&](int c) {
            const float a = qa[c];
#pragma unroll
            for (int cb = 0; cb < decltype(blocks)::value; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, kb[32 * cb * kSPitch + c], acc[cb], 0, 0, 0);
        };
        if (cn == kSC) {
#pragma unroll
            for (int c = 0; c < kSC; c += 2) step(c);
        } else {
            for (int c = 0; c < cn; c += 2) step(c);
        }
    };
    const int first_row = __builtin_amdgcn_readfirstlane(bi * kSB + 32 * wave);
    const int col_blocks = first_row < nT ? (nT - bj * kSB + 31) / 32 : 0;   // that hold any column
    for (int c0 = 0; c0 < dp; c0 += kSC) {
        const int cn = dp - c0 < kSC ? dp - c0 : kSC;
        fetch(c0);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int t = threadIdx.x + 256 * u, r = t / (kSC / 4), c4 = (t % (kSC / 4)) * 4;
            *reinterpret_cast<float4*>(qs + r * kSPitch + c4) = qv[u];
            *reinterpret_cast<float4*>(ks + r * kSPitch + c4) = kv[u];
        }
        __syncthreads();
        if (col_blocks >= 4) products(std::integral_constant<int, 4>(), cn);
        else if (col_blocks == 3) products(std::integral_constant<int, 3>(), cn);
        else if (col_blocks == 2) products(std::integral_constant<int, 2>(), cn);
        else if (col_blocks == 1) products(std::integral_constant<int, 1>(), cn);
    }
    float* sbase = scores + b * score_elems + hg.score_off;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = bi * kSB + 32 * wave + (r & 3) + 8 * (r >> 2) + 4 * kh;
        if (i >= nT) continue;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int j = bj * kSB + 32 * cb + col;
            if (j < nT) sbase[(int64_t)i * nT + j] = acc[cb][r] * scale;
        }
    }
}

// All score blocks, one workgroup each.
// The head is counted with one load per 64 heads; a search was six, each waiting for the one before.  With that and the blocks
// left out: 2 heads of 4 tiles 5.0 -> 3.9 us, 4 of 75 (2 samples) 7.7 -> 6.9, 12 of 624 20.7 -> 19.3, 40 of 624 51.5 -> 47.0.
__global__ __launch_bounds__(256, 3) void score_kernel(const HeadGeom* __restrict__ heads, int n_heads,
                                                    const float* __restrict__ yq, const float* __restrict__ yk,
                                                    float* __restrict__ scores, int dp, float scale,
                                                    int64_t total_tiles, int64_t score_elems) {
    __shared__ __align__(16) float qs[kSB * kSPitch];
    __shared__ __align__(16) float ks[kSB * kSPitch];
    int head = -1;   // the last head whose first block is <= blockIdx.x
    for (int h0 = 0; h0 < n_heads; h0 += 64) {
        const int h = h0 + (threadIdx.x & 63);
        head += __popcll(__ballot(h < n_heads && (int)blockIdx.x >= heads[h < n_heads ? h : 0].score_blk_off));
    }
    const HeadGeom hg = heads[head];
    const int blk = blockIdx.x - hg.score_blk_off;
    const int bi = blk / hg.score_blk_dim, bj = blk - bi * hg.score_blk_dim;
    score_block_128(hg, bi, bj, blockIdx.y, qs, ks, yq, yk, scores, dp, scale, total_tiles, score_elems);
}

// Only the score rows somebody asked for: one workgroup per 128 rows of a head (the even
// entries of the 64-row table), which leaves at once unless one of the marks of its rows is set
// (marks: one per 128 consecutive rows of the latents, row >> 7) and otherwise forms all the
// blocks of its rows.
__global__ __launch_bounds__(256, 2) void score_marked_rows_kernel(const HeadGeom* __restrict__ heads,
                                                                const int32_t* __restrict__ row_blk,
                                                                const float* __restrict__ yq,
                                                                const float* __restrict__ yk,
                                                                float* __restrict__ scores, int dp, float scale,
                                                                int64_t total_tiles, int64_t score_elems,
                                                                const int32_t* __restrict__ marks) {
    __shared__ __align__(16) float qs[kSB * kSPitch];
    __shared__ __align__(16) float ks[kSB * kSPitch];
    const int32_t code = row_blk[blockIdx.x];
    if (code & 1) return;
    const HeadGeom hg = heads[code >> 24];
    const int bi = (code & 0xffffff) >> 1, nT = hg.n_tiles;
    const int64_t b = blockIdx.y;
    const int64_t g0 = b * total_tiles + hg.tile_off + (int64_t)bi * kSB;
    const int last = nT - 1 - bi * kSB < kSB - 1 ? nT - 1 - bi * kSB : kSB - 1;
    if (!(marks[g0 >> 7] | marks[(g0 + last) >> 7])) return;
    for (int bj = 0; bj < hg.score_blk_dim; ++bj)
        score_block_128(hg, bi, bj, b, qs, ks, yq, yk, scores, dp, scale, total_tiles, score_elems);
}

veda_status check_mlp(const veda_plan* pl, const veda_mlp* m) {
    if (!m || !m->w1 || !m->b1) return VEDA_ERR_INVALID_ARG;
    if (m->in_dim != 3 * pl->prob.head_dim) return VEDA_ERR_INVALID_ARG;
    if (m->hidden < 0 || m->out_dim < 1) return VEDA_ERR_INVALID_ARG;
    if (m->hidden > 0 && (!m->w2 || !m->b2)) return VEDA_ERR_INVALID_ARG;
    if (m->act != VEDA_ACT_IDENTITY && m->act != VEDA_ACT_RELU) return VEDA_ERR_INVALID_ARG;
    if (m->hidden > 512 || m->out_dim > 256 || (m->out_dim & 3)) return VEDA_ERR_UNSUPPORTED;
    return VEDA_OK;
}

static void fill_recip(RecipTable& recip) {
    recip.v[0] = 0.0f;
    for (int c = 1; c <= 2 * kTile; ++c) recip.v[c] = 1.0f / (float)c;
}

// TripPool (Eq. 4) of the tiled Q and K into zq, zk.
void launch_trippool(const veda_plan* pl, const void* q_tiled, const void* k_tiled, const uint64_t* valid_mask,
                            float* zq, float* zk, hipStream_t s) {
    const int d = pl->prob.head_dim;
    const int64_t total = pl->total_tiles, rows = total * pl->prob.batch;
    RecipTable recip;
    fill_recip(recip);

    const bool bf16 = pl->prob.dtype == VEDA_BF16;
#define VEDA_LAUNCH_TP(E, D)                                                                               \
    do {                                                                                                   \
        constexpr int tpb = 256 / (D / Chunk<E>::kN);                                                      \
        dim3 grid((unsigned)((rows + tpb - 1) / tpb), 2);                                                  \
        if (pl->inner)                                                                                     \
            hipLaunchKernelGGL((trippool_kernel<E, D, 2>), grid, dim3(256), 0, s, (const char*)q_tiled,    \
                               (const char*)k_tiled, valid_mask, zq, zk, rows, total, recip);              \
        else                                                                                               \
            hipLaunchKernelGGL((trippool_kernel<E, D, 1>), grid, dim3(256), 0, s, (const char*)q_tiled,    \
                               (const char*)k_tiled, valid_mask, zq, zk, rows, total, recip);              \
    } while (0)
    if (bf16 && d == 128) VEDA_LAUNCH_TP(uint16_t, 128);
    else if (bf16) VEDA_LAUNCH_TP(uint16_t, 64);
    else if (d == 128) VEDA_LAUNCH_TP(uint32_t, 128);
    else VEDA_LAUNCH_TP(uint32_t, 64);
#undef VEDA_LAUNCH_TP
}

// Weight-free scorer (App. A.3): latent y = [avg | root_lambda * sqrt(max(0, (max-avg)(avg-min)))] per tile,
// whose plain dot product is the mean product plus lambda times the dispersion product.
__global__ __launch_bounds__(256) void closed_form_latent_kernel(const float* __restrict__ zq, const float* __restrict__ zk,
                                                                 float* __restrict__ yq, float* __restrict__ yk,
                                                                 int64_t rows, int d, float root_lambda) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= rows * d) return;
    const int64_t i = e / d;
    const int c = (int)(e - i * d);
    const float* z = (blockIdx.y == 0 ? zq : zk) + i * 3 * d;
    float* y = (blockIdx.y == 0 ? yq : yk) + i * 2 * d;
    const float mu = z[c], mx = z[d + c], mn = z[2 * d + c];
    const float up = mx - mu, dn = mu - mn;
    float p = up * dn;
    p = p > 0.0f ? p : 0.0f;
    y[c] = mu;
    y[d + c] = root_lambda * sqrtf(p);
}

// Projections (Eq. 5 phi_q, phi_k) of the descriptors zq, zk into the latents yq, yk.
veda_status launch_projections(const veda_plan* pl, const veda_mlp* phi_q, const veda_mlp* phi_k, const float* zq,
                               const float* zk, float* yq, float* yk, float* hq, float* hk, hipStream_t s) {
    MlpDev pq{phi_q->in_dim, phi_q->hidden, phi_q->out_dim, phi_q->act == VEDA_ACT_RELU, phi_q->w1, phi_q->b1, phi_q->w2, phi_q->b2};
    MlpDev pk{phi_k->in_dim, phi_k->hidden, phi_k->out_dim, phi_k->act == VEDA_ACT_RELU, phi_k->w1, phi_k->b1, phi_k->w2, phi_k->b2};
    if (pl->chain_unit() == VEDA_CHAINS_VECTOR) return launch_projections_vector(pl, pq, pk, zq, zk, yq, yk, s);
    int64_t blocks16 = 0;   // workgroups of 16 rows
    for (const HeadGeom& g : pl->heads) blocks16 += (g.n_tiles + 15) / 16;
    const bool rows16 = 2 * blocks16 * pl->prob.batch <= kRows16Most;
#define VEDA_TRY_STAGED(N1, N2, ROWS)                                                                    \
    if (staged_sizes<N1, N2>(pq, pk, zq, zk)) {                                                          \
        dim3 sgrid((unsigned)(pl->row_blocks * (kLatentRows / (ROWS))), 2, (unsigned)pl->prob.batch);    \
        if (rows16) {                                                                                    \
            hipLaunchKernelGGL((mlp_rows16_kernel<N1, N2>), dim3((unsigned)(pl->row_blocks * (kLatentRows / 16)), 2, (unsigned)pl->prob.batch), \
                               dim3(256), (kMlp16Lds<N1, N2>), s, pl->d_heads, pl->d_row_blk, zq, zk, yq, yk, pq, pk, pl->total_tiles); \
            return launch_status("mlp_rows16_kernel");                                                   \
        }                                                                                                \
        hipLaunchKernelGGL((mlp_staged_kernel<N1, N2, ROWS>), sgrid, dim3(256), kMlpDepth * (16 * (N1) * 4 + (ROWS) * 64), s, \
                           pl->d_heads, pl->d_row_blk, zq, zk, yq, yk, pq, pk, pl->total_tiles);         \
        return launch_status("mlp_staged_kernel");                                                       \
    }
    VEDA_TRY_STAGED(128, 64, 32)
    VEDA_TRY_STAGED(64, 32, 64)
#undef VEDA_TRY_STAGED
    const int max_hidden = phi_q->hidden > phi_k->hidden ? phi_q->hidden : phi_k->hidden;
    // the global route reads the hidden layer back as float4 rows
    if (!hq || !hk || (phi_q->hidden & 3) || (phi_k->hidden & 3)) hq = hk = nullptr;
    const size_t smem = sizeof(float) * ((size_t)2 * kMlpWsFloats + (size_t)2 * kMlpXsFloats +
                                         (hq ? 0 : (size_t)kMlpRows * (size_t)((max_hidden + 3) & ~3)));
    if (smem > 64 * 1024)
        VEDA_HIP_TRY(hipFuncSetAttribute((const void*)mlp_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    dim3 mgrid((unsigned)pl->row_blocks, 2, (unsigned)pl->prob.batch);
    hipLaunchKernelGGL(mlp_kernel, mgrid, dim3(kMlpThreads), smem, s, pl->d_heads, pl->d_row_blk, zq, zk, yq,
                       yk, pq, pk, pl->total_tiles, hq, hk);
    return launch_status("mlp_kernel");
}

// The score blocks of all heads (Eq. 5) from latents of dp coordinates.  marks != nullptr: one
// mark per 128 consecutive rows of the latents (row >> 7); only the score rows of 128-row blocks
// that touch a marked group are formed.
veda_status launch_score_blocks(const veda_plan* pl, const float* yq, const float* yk, float* scores, int dp,
                                float scale, const int32_t* marks, hipStream_t s) {
    if (pl->chain_unit() == VEDA_CHAINS_VECTOR) return launch_score_blocks_vector(pl, yq, yk, scores, dp, scale, marks, s);
    if (marks) {
        dim3 rgrid((unsigned)pl->row_blocks, (unsigned)pl->prob.batch);
        hipLaunchKernelGGL(score_marked_rows_kernel, rgrid, dim3(256), 0, s, pl->d_heads, pl->d_row_blk, yq, yk, scores,
                           dp, scale, pl->total_tiles, pl->score_elems, marks);
        return launch_status("score_marked_rows_kernel");
    }
    dim3 sgrid((unsigned)pl->score_blocks, (unsigned)pl->prob.batch);
    hipLaunchKernelGGL(score_kernel, sgrid, dim3(256), 0, s, pl->d_heads, pl->prob.heads, yq, yk, scores, dp,
                       scale, pl->total_tiles, pl->score_elems);
    return launch_status("score_kernel");
}

// hq, hk: scratch for the hidden layers, or null.
static veda_status project_and_score(const veda_plan* pl, const veda_mlp* phi_q, const veda_mlp* phi_k, float scale,
                                     const float* zq, const float* zk, float* yq, float* yk, float* hq, float* hk,
                                     float* scores, hipStream_t s) {
    const veda_status st = launch_projections(pl, phi_q, phi_k, zq, zk, yq, yk, hq, hk, s);
    if (st != VEDA_OK) return st;
    return launch_score_blocks(pl, yq, yk, scores, phi_q->out_dim, scale, nullptr, s);
}

}  // namespace veda

extern "C" veda_status veda_plan_workspace_layout(const veda_plan* pl, const veda_mlp* phi_q, const veda_mlp* phi_k,
                                                  veda_workspace_layout* out) {
    if (!pl || !phi_q || !phi_k || !out || phi_q->out_dim != phi_k->out_dim) return VEDA_ERR_INVALID_ARG;
    const int64_t rows = pl->total_tiles * pl->prob.batch, d = pl->prob.head_dim, dp = phi_q->out_dim;
    out->stats_q = 0;                       // the order veda_tile_score carves its workspace in
    out->stats_k = rows * 3 * d;
    out->latent_q = 2 * rows * 3 * d;
    out->latent_k = 2 * rows * 3 * d + rows * dp;
    return VEDA_OK;
}

extern "C" veda_status veda_tile_score(const veda_plan* pl, const void* q_tiled, const void* k_tiled,
                                       const uint64_t* valid_mask, const veda_mlp* phi_q,
                                       const veda_mlp* phi_k, float scale, float* scores, void* workspace,
                                       size_t workspace_bytes, void* stream) {
    using namespace veda;
    if (!pl || !q_tiled || !k_tiled || !valid_mask || !scores) return VEDA_ERR_INVALID_ARG;
    veda_status st = check_mlp(pl, phi_q);
    if (st == VEDA_OK) st = check_mlp(pl, phi_k);
    if (st != VEDA_OK) return st;
    if (phi_q->out_dim != phi_k->out_dim) return VEDA_ERR_INVALID_ARG;
    if (!aligned16(q_tiled) || !aligned16(k_tiled) || !aligned16(workspace)) return VEDA_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < veda_plan_workspace_bytes(pl, phi_q, phi_k)) return VEDA_ERR_WORKSPACE;

    const int dp = phi_q->out_dim;
    const int64_t total = pl->total_tiles, rows = total * pl->prob.batch;
    veda_workspace_layout lay;
    (void)veda_plan_workspace_layout(pl, phi_q, phi_k, &lay);
    float* zq = (float*)workspace + lay.stats_q;
    float* zk = (float*)workspace + lay.stats_k;
    float* yq = (float*)workspace + lay.latent_q;
    float* yk = (float*)workspace + lay.latent_k;
    float* hq = yk + rows * dp;               // the plan's workspace size has room for both hidden layers
    float* hk = hq + rows * (phi_q->hidden > 0 ? phi_q->hidden : 0);
    hipStream_t s = (hipStream_t)stream;

    launch_trippool(pl, q_tiled, k_tiled, valid_mask, zq, zk, s);
    st = launch_status("trippool_kernel");
    if (st != VEDA_OK) return st;

    return project_and_score(pl, phi_q, phi_k, scale, zq, zk, yq, yk, hq, hk, scores, s);
}

extern "C" veda_status veda_tile_score_stats(const veda_plan* pl, const float* stats_q, const float* stats_k,
                                             const veda_mlp* phi_q, const veda_mlp* phi_k, float scale,
                                             float* scores, void* workspace, size_t workspace_bytes,
                                             void* stream) {
    using namespace veda;
    if (!pl || !stats_q || !stats_k || !scores) return VEDA_ERR_INVALID_ARG;
    veda_status st = check_mlp(pl, phi_q);
    if (st == VEDA_OK) st = check_mlp(pl, phi_k);
    if (st != VEDA_OK) return st;
    if (phi_q->out_dim != phi_k->out_dim) return VEDA_ERR_INVALID_ARG;
    if (!aligned16(stats_q) || !aligned16(stats_k) || !aligned16(workspace)) return VEDA_ERR_UNSUPPORTED;
    const int64_t rows = pl->total_tiles * pl->prob.batch;
    const int dp = phi_q->out_dim;
    if (!workspace || workspace_bytes < sizeof(float) * (size_t)rows * 2 * (size_t)dp) return VEDA_ERR_WORKSPACE;
    float* yq = (float*)workspace;
    float* yk = yq + rows * dp;
    // with room for them the hidden layers go through the workspace too (twice the workgroups per
    // compute unit); the results are the same either way
    const size_t hid = (size_t)(phi_q->hidden > 0 ? phi_q->hidden : 0) + (size_t)(phi_k->hidden > 0 ? phi_k->hidden : 0);
    const bool roomy = workspace_bytes >= sizeof(float) * (size_t)rows * (2 * (size_t)dp + hid);
    float* hq = roomy ? yk + rows * dp : nullptr;
    float* hk = roomy ? hq + rows * (phi_q->hidden > 0 ? phi_q->hidden : 0) : nullptr;
    return project_and_score(pl, phi_q, phi_k, scale, stats_q, stats_k, yq, yk, hq, hk, scores, (hipStream_t)stream);
}

extern "C" veda_status veda_tile_score_closed_form(const veda_plan* pl, const void* q_tiled, const void* k_tiled,
                                                   const uint64_t* valid_mask, float lambda, float* scores,
                                                   void* workspace, size_t workspace_bytes, void* stream) {
    using namespace veda;
    if (!pl || !q_tiled || !k_tiled || !valid_mask || !scores) return VEDA_ERR_INVALID_ARG;
    if (!(lambda >= 0.0f) || !(lambda < INFINITY)) return VEDA_ERR_INVALID_ARG;
    if (!aligned16(q_tiled) || !aligned16(k_tiled) || !aligned16(workspace)) return VEDA_ERR_UNSUPPORTED;
    const int d = pl->prob.head_dim;
    const int64_t rows = pl->total_tiles * pl->prob.batch;
    if (!workspace || workspace_bytes < sizeof(float) * (size_t)rows * 10 * (size_t)d) return VEDA_ERR_WORKSPACE;
    float* zq = (float*)workspace;
    float* zk = zq + rows * 3 * d;
    float* yq = zk + rows * 3 * d;
    float* yk = yq + rows * 2 * d;
    hipStream_t s = (hipStream_t)stream;
    launch_trippool(pl, q_tiled, k_tiled, valid_mask, zq, zk, s);
    veda_status st = launch_status("trippool_kernel");
    if (st != VEDA_OK) return st;
    dim3 lgrid((unsigned)((rows * d + 255) / 256), 2);
    hipLaunchKernelGGL(closed_form_latent_kernel, lgrid, dim3(256), 0, s, zq, zk, yq, yk, rows, d, sqrtf(lambda));
    st = launch_status("closed_form_latent_kernel");
    if (st != VEDA_OK) return st;
    return launch_score_blocks(pl, yq, yk, scores, 2 * d, 1.0f, nullptr, s);
}
