// fp32 products on the bf16 matrix cores, for the fp32 attention kernel.  (The target scores keep the fp32 chains: a
// score that moves in its last bits can change places with another in the top-k, and with it the kept lists.)
//
// A number is split into three bf16 numbers, each the rounding of what is left: 3 x 8 bits hold fp32's 24, so the sum
// is exact of what is finite and not below 2^-109 (there up to 2^-134, half of bf16's smallest subnormal, is lost: the kernel
// scales its operands away from it, see kF32QScale).  Of the nine products of two split operands the six largest
// are formed, each by v_mfma_f32_32x32x16_bf16 with fp32 accumulation; the three left out are below 2^-26 of the
// product, an eighth of its rounding to fp32.  Six such instructions take 192 cycles where v_mfma_f32_32x32x2_f32 takes
// 512 for the same 16 terms, and they round the running sum 6 times where it rounds 16: dot products of 64 to 32768
// terms, normal, uniform and log-normal operands, came out 2 to 76 % nearer to the 64-bit result (relative 2-norm; 128
// normal terms 2.0e-7 -> 1.6e-7).
// What is not finite does not survive (an infinity's remainder is NaN, and its products with remainders of either
// sign cancel): every such product is NaN; the kernel finds that in its results and forms them again on fp32 matrix cores.
#pragma once

#include "attn_common.h"

namespace veda {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef const __attribute__((address_space(3))) f32x4* lds_f32x4_ptr;
__device__ __forceinline__ f32x4 lds_read_f32x4(uint32_t addr) { return *(lds_f32x4_ptr)(uintptr_t)addr; }

// x0, x1 -> p[0] + p[1] + p[2], two bf16 to a register.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t (&p)[3]) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const bf16x2 t = {(__bf16)x0, (__bf16)x1};
        p[u] = __builtin_bit_cast(uint32_t, t);
        asm("" : "+v"(p[u]));   // or each half is rounded once more for the difference
        if (u < 2) {
            x0 -= __uint_as_float(p[u] << 16);
            x1 -= __uint_as_float(p[u] & 0xffff0000u);
        }
    }
}

// A lane's part of a query row of D channels, times `scale`: q[u][t] holds channels 16t + 8h .. + 7.
template <int D> __device__ __forceinline__ void split_row(const float* row, int h, float scale, bf16x8 (&q)[3][D / 16]) {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        uint32_t w[3][4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(row + 16 * t + 8 * h + 4 * e);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                uint32_t p[3];
                split2(x[2 * c] * scale, x[2 * c + 1] * scale, p);
#pragma unroll
                for (int u = 0; u < 3; ++u) w[u][2 * e + c] = p[u];
            }
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) q[u][t] = __builtin_bit_cast(bf16x8, u32x4{w[u][0], w[u][1], w[u][2], w[u][3]});
    }
}

// c + x y without the product of the largest parts.
__device__ __forceinline__ f32x16 mul5(f32x16 c, const bf16x8 (&x)[3], const bf16x8& y0, const bf16x8& y1, const bf16x8& y2) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], y0, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y2, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y1, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y0, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y1, c, 0, 0, 0);
}
// c + x y, the small products first.
__device__ __forceinline__ f32x16 mul6(f32x16 c, const bf16x8 (&x)[3], const bf16x8& y0, const bf16x8& y1, const bf16x8& y2) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y0, mul5(c, x, y0, y1, y2), 0, 0, 0);
}

// 32 rows of K as three bf16 planes in LDS, [32][D] each, 16-byte chunk ^ rho(row): a read takes one chunk of rows
// rho(0..31), which then lie on all banks.  A wave fetches eight rows by direct loads into a landing area of its own,
// splits what it fetched and writes it to the planes.  The landing area's places are converted in turn and asked for
// again at once: one phase of products lies between.
template <int D> struct SplitK {
    static constexpr int kRowB = D * 4, kRowChunks = kRowB / 16, kPc = D * 2 / 16;
    static constexpr int kPlane = 32 * D * 2, kPlanes = 3 * kPlane;
    static constexpr int kI = 32 * kRowB / 4096;      // loads per wave: 4 (d = 128) or 2
    static constexpr int kLanding = 4 * kI * 1024;    // bytes, all waves
    uint32_t raw, raw_lane, kw, kr;                   // this wave's landing area, this lane in it; its place in a plane; its reads
    int wave;

    __device__ __forceinline__ void init(uint32_t planes, uint32_t landing, int wave_, int lane) {
        wave = wave_;
        raw = landing + (uint32_t)wave * (kI * 1024);
        raw_lane = raw + 16u * lane;
        const int row = 8 * wave + lane / kRowChunks, c = lane % kRowChunks;
        kw = planes + row * (D * 2) + (((c >> 1) ^ (rho(row) & (kPc - 1))) << 4) + (c & 1) * 8;
        kr = planes + rho(lane & 31) * (D * 2) + (((lane >> 5) ^ (lane & (kPc - 1))) << 4);
    }
    // The j-th load: rows of the 32 are those of the tile's eight-row chunks from & 255, (from >> 8) & 255, ...
    __device__ __forceinline__ void load(int j, const char* tile, uint32_t from) const {
        dma16_to_lds(raw + 1024u * j, tile + ((from >> (8 * wave)) & 255u) * (8 * kRowB) + 1024 * j, raw_lane - raw);
    }
    // The place at hand has landed when the kI - 1 loads after it are left: load() is called without exception.
    static __device__ __forceinline__ void landed() {
        if constexpr (kI == 4) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
        static_assert(kI == 4 || kI == 2, "the counts above");
    }
    // Four numbers of the j-th load, times `scale`, to their places in three planes at `to`.
    __device__ __forceinline__ void put(int j, uint32_t to, float scale) const {
        landed();
        const f32x4 x = lds_read_f32x4(raw_lane + 1024u * j);
        uint32_t p0[3], p1[3];
        split2(x[0] * scale, x[1] * scale, p0);
        split2(x[2] * scale, x[3] * scale, p1);
        typedef __attribute__((address_space(3))) u32x2* lds_u32x2_ptr;
#pragma unroll
        for (int u = 0; u < 3; ++u) *(lds_u32x2_ptr)(uintptr_t)(to + u * kPlane) = u32x2{p0[u], p1[u]};
    }
    __device__ __forceinline__ void convert(int j, uint32_t planes = 0u) const {
        constexpr int kRows = 1024 / kRowB;   // rows of a load
        put(j, planes + (kw ^ (uint32_t)((rho(j * kRows) & (kPc - 1)) << 4)) + (uint32_t)(j * kRows * D * 2), 1.0f);
    }
    static __device__ __forceinline__ bf16x8 frag(uint32_t at, int u) {
        typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8_ptr;
        return *(lds_bf16x8_ptr)(uintptr_t)(at + (uint32_t)(u * kPlane));
    }
    // K rows rho(0..31) times the wave's split query rows; at(t) comes behind the products of channel step t.
    // kApart: the small products in a sum of their own (16 more registers).
    template <bool kApart, typename At>
    __device__ __forceinline__ void products(f32x16& s, const bf16x8 (&q)[3][D / 16], uint32_t planes, At at) const {
        constexpr int G = D / 16;
        bf16x8 kf[2][3];
        f32x16 small;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = small[i] = 0.0f;
#pragma unroll
        for (int u = 0; u < 3; ++u) kf[0][u] = frag(kr + planes, u);
#pragma unroll
        for (int t = 0; t < G; ++t) {
            if (t + 1 < G) {
#pragma unroll
                for (int u = 0; u < 3; ++u) kf[(t + 1) & 1][u] = frag((kr ^ (uint32_t)((t + 1) << 5)) + planes, u);
            }
            __builtin_amdgcn_sched_barrier(0);   // read a whole group of products ahead
            if constexpr (kApart) {
                small = mul5(small, kf[t & 1], q[0][t], q[1][t], q[2][t]);
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t & 1][0], q[0][t], s, 0, 0, 0);
                if (t == G - 1) s += small;
            } else {
                s = mul6(s, kf[t & 1], q[0][t], q[1][t], q[2][t]);
            }
            at(t);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // LDS reads and writes of this wave done, then meet the others; loads into the wave's own landing area go on.
    static __device__ __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
};

}  // namespace veda
