// Decode attention without a plan: out[i,h,:] = softmax(q K^T * scale) V (Section 2.1) for batches whose
// histories are so short, or so few, that detecting aliases, cutting the work and merging pieces would cost
// more than it saves.  A block that several requests alias is read once per request, out of L2 after the
// first (workgroups are numbered so that, with 8 KV heads, those of one KV head share an XCD).
//
// One workgroup per (request, row tile of 16 query heads, KV head) and, where these are too few to fill the
// chip, per piece of the history: the pieces take the request's tiles in turn and leave partial rows, which the workgroup
// that comes last folds.  A wave takes every (waves x pieces)-th tile of 32 tokens (16 for float32 from head_dim 128 on),
// each on the matrix cores, straight from global memory into the operand registers:
//     S^T = K Q^T     lane (n, kg) = (lane % 16, lane / 16) holds K rows as 16-byte chunks 4 j + kg of token
//                     row n, and q's chunks alike: any order of the head dims serves, as long as both agree
//     O^T += V^T P^T  the scores' accumulator layout (head n, tokens 4 kg + r) is the B operand as it stands;
//                     V is read as whole token rows 4 kg + r.  float32 (16x16x4 products, one k-slot per lane
//                     group): row element 4 n + i of the A operand of product i, no data movement; bfloat16
//                     (16x16x32): an 8x8 transpose in registers.
// Accumulation is float32: float32 caches use the float32 matrix instructions, and with bfloat16 caches the
// softmax weights enter the second product as the sum of two bfloat16 numbers (the weight rounded, and what that
// left over, rounded: 2^-17 of the weight is lost), the denominator as unrounded float32.  Against weights in
// float32, over 56 shapes of 33 to 2000 tokens: the same error against float64 to within 2e-6 of it.
//
// Bound: latency (the chain length, table row and q -> K -> V -> fold over the waves) for short histories, 6 to 8 us
// in all; then memory, at 5.0 to 5.9 TB/s where the chip is full (8 and more where what requests share sits in L2; a compute
// unit fetches 53 GB/s at most); with float32, more than four query heads and few workgroups the matrix cores' float32 rate (a
// block of 16 tokens is 64 instructions of 32 cycles at head_dim 128, whatever part of the 16 query rows is real).  Measured
// against the vector-unit kernel it replaces: float32 8/2/64, 4 requests of 320 tokens 11.6 -> 9.1 us a call; float32
// 32/8/128, 16 requests of 1152 to 2048 tokens 78.7 -> 34.6; against plan, sweep and merge: bf16 28/4/128, 8 requests of 90
// to 700 tokens 23.6 -> 9.1.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "../../include/fea.h"
#include "fea_plan.h"

namespace fea {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ uint32_t bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Sums, maxima and exchanges across the halves and the rows of 16 lanes of a wave, without a detour through LDS.
struct Pair { float a, b; };
__device__ __forceinline__ Pair swap32(float x, float y) {   // the upper half of x against the lower half of y
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair swap16(float x, float y) {   // the odd rows of x against the even rows of y
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
template <int CTRL> __device__ __forceinline__ float lanes_moved(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float max_over_kg(float x) {
    const Pair p = swap32(x, x);
    x = fmaxf(p.a, p.b);
    const Pair q = swap16(x, x);
    return fmaxf(q.a, q.b);
}
__device__ __forceinline__ float sum_over_kg(float x) {
    const Pair p = swap32(x, x);
    x = p.a + p.b;
    const Pair q = swap16(x, x);
    return q.a + q.b;
}

// A lane's registers of one tile, and the two products, for row tiles of R query heads.  A lane works out the weights of
// PN tokens for one head.
template <typename T, int D, int R> struct Tile;

template <int D> struct Tile<float, D, 16> {
    static constexpr int TB = D >= 128 ? 1 : 2;            // blocks per tile
    static constexpr int PN = 4 * TB;
    static constexpr int KC = D / 16;                      // chunks of a K row per lane
    static constexpr int VH = D >= 64 ? D / 64 : 1;        // chunks of a V row per lane
    static constexpr int NI = 4 * VH;                      // output products (head_dim 32: half of their rows count)
    static constexpr int ES = 4;
    f32x4 k[TB][KC], v[TB][4][VH], q[KC];

    __device__ __forceinline__ void load_q(const char* rows, int nh, int n, int kg) {
        const char* row = rows + min(n, nh - 1) * (D * ES);
#pragma unroll
        for (int j = 0; j < KC; ++j) q[j] = n < nh ? *reinterpret_cast<const f32x4*>(row + (4 * j + kg) * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void load_k(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int j = 0; j < KC; ++j) k[b][j] = *reinterpret_cast<const f32x4*>(blk + (uint32_t)(n * (D * 4) + kg * 16 + j * 64));
    }
    __device__ __forceinline__ void load_v(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < VH; ++h)
                v[b][r][h] = *reinterpret_cast<const f32x4*>(blk + (uint32_t)((4 * kg + r) * (D * 4) + (D >= 64 ? n : n & 7) * 16 + h * 256));
    }
    __device__ __forceinline__ void mask(float (&p)[PN], int rest, int, int kg) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * b + 4 * kg + r >= rest) {
                    p[4 * b + r] = -INFINITY;
#pragma unroll
                    for (int h = 0; h < VH; ++h) v[b][r][h] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
    }
    __device__ __forceinline__ void scores(float (&p)[PN]) {
        // Partial sums of 8 products, added up in pairs: a single chain over the head dims would be one rounding after
        // another, which doubles the error of the scores.
        constexpr int GC = KC < 4 ? KC : 4, Y = D == 256 ? 1 : GC / 2;    // chunks taken together, partial sums over them (head_dim 256: 16 products each, 8 spill registers)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int j0 = 0; j0 < KC; j0 += GC) {
                f32x4 c[Y][4];
#pragma unroll
                for (int x = 0; x < GC / Y; ++x)
#pragma unroll
                    for (int y = 0; y < Y; ++y)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            c[y][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[b][j0 + x * Y + y][e], q[j0 + x * Y + y][e],
                                                                           x == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : c[y][e], 0, 0, 0);
                if constexpr (Y == 2) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[0][e] += c[1][e];
                }
                const f32x4 part = (c[0][0] + c[0][1]) + (c[0][2] + c[0][3]);
#pragma unroll
                for (int r = 0; r < 4; ++r) p[4 * b + r] = j0 == 0 ? part[r] : p[4 * b + r] + part[r];
            }
    }
    __device__ __forceinline__ void accumulate(const float (&p)[PN], f32x4 (&o)[NI], int) {
        // The sums over a block start at zero and are added to the running ones: a short chain of products, and a chain
        // of one addition per block (the error grows with the length of a chain).
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int h = 0; h < VH; ++h) {
                f32x4 c[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        c[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[b][r][h][e], p[4 * b + r], r == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : c[e], 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[4 * h + e] += c[e];
            }
    }
    static __device__ __forceinline__ int head(int n) { return n; }
    static __device__ __forceinline__ bool one_of_row(int, int kg) { return kg == 0; }   // (of the lanes that hold a row's sums)
    static __device__ __forceinline__ float row_max(float x) { return max_over_kg(x); }
    static __device__ __forceinline__ float row_sum(float x) { return sum_over_kg(x); }
    static __device__ __forceinline__ void rescale(f32x4 (&o)[NI], float al) {
#pragma unroll
        for (int i = 0; i < NI; ++i) o[i] *= al;
    }
    // product i = 4 h + e, output row m = 4 kg + r: dim 64 h + 4 m + e
    template <int PAD> static __device__ __forceinline__ void to_lds(float (*rows)[PAD], const f32x4 (&o)[NI], int nh, int n, int kg) {
        if (n >= nh) return;
        float* row = rows[n];
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (D >= 64 || kg < 2)
                    *reinterpret_cast<f32x4*>(row + 64 * h + 4 * (4 * kg + r)) = f32x4{o[4 * h][r], o[4 * h + 1][r], o[4 * h + 2][r], o[4 * h + 3][r]};
    }
};

template <int D> struct Tile<bf16_t, D, 16> {
    static constexpr int TB = 2, PN = 8;
    static constexpr int KC = D / 32;
    static constexpr int VH = D == 256 ? 2 : 1;
    static constexpr int NI = D / 16;
    static constexpr int ES = 2;
    u32x4 k[TB][KC], v[TB][4][VH], q[KC];

    __device__ __forceinline__ void load_q(const char* rows, int nh, int n, int kg) {
        const char* row = rows + min(n, nh - 1) * (D * ES);
#pragma unroll
        for (int j = 0; j < KC; ++j) q[j] = n < nh ? ld16(row + (4 * j + kg) * 16) : u32x4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void load_k(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int j = 0; j < KC; ++j) k[b][j] = ld16(blk + (uint32_t)(n * (D * 2) + kg * 16 + j * 64));
    }
    __device__ __forceinline__ void load_v(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < VH; ++h) v[b][r][h] = ld16(blk + (uint32_t)((4 * kg + r) * (D * 2) + (D >= 128 ? n : n & 7) * 16 + h * 256));
    }
    __device__ __forceinline__ void mask(float (&p)[PN], int rest, int, int kg) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * b + 4 * kg + r >= rest) {
                    p[4 * b + r] = -INFINITY;
#pragma unroll
                    for (int h = 0; h < VH; ++h) v[b][r][h] = u32x4{0u, 0u, 0u, 0u};
                }
    }
    __device__ __forceinline__ void scores(float (&p)[PN]) {
        f32x4 s[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KC; ++j)
#pragma unroll
            for (int b = 0; b < TB; ++b)
                s[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[b][j]), __builtin_bit_cast(bf16x8, q[j]), s[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) p[4 * b + r] = s[b][r];
    }
    __device__ __forceinline__ void accumulate(const float (&p)[PN], f32x4 (&o)[NI], int n) {
        bf16x8 hi, lo;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            hi[x] = (__bf16)p[x];
            lo[x] = (__bf16)(p[x] - (float)hi[x]);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            u32x4 t;
            if constexpr (D >= 128) {
                const int h = i >> 3, e = i & 7;
                const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int j0 = 2 * w, j1 = 2 * w + 1;
                    t[w] = __builtin_amdgcn_perm(v[j1 >> 2][j1 & 3][h][e >> 1], v[j0 >> 2][j0 & 3][h][e >> 1], sel);
                }
            } else {
                // lanes n and n + 8 hold the same chunk: lane n < 8 hands over its elements 0..3, lane n >= 8 elements 4..7
                const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int j0 = 2 * w, j1 = 2 * w + 1;
                    const uint32_t a1 = n < 8 ? v[j1 >> 2][j1 & 3][0][i >> 1] : v[j1 >> 2][j1 & 3][0][2 + (i >> 1)];
                    const uint32_t a0 = n < 8 ? v[j0 >> 2][j0 & 3][0][i >> 1] : v[j0 >> 2][j0 & 3][0][2 + (i >> 1)];
                    t[w] = __builtin_amdgcn_perm(a1, a0, sel);
                }
            }
            const bf16x8 a = __builtin_bit_cast(bf16x8, t);
            o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hi, o[i], 0, 0, 0);
            o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, lo, o[i], 0, 0, 0);
        }
    }
    static __device__ __forceinline__ int head(int n) { return n; }
    static __device__ __forceinline__ bool one_of_row(int, int kg) { return kg == 0; }
    static __device__ __forceinline__ float row_max(float x) { return max_over_kg(x); }
    static __device__ __forceinline__ float row_sum(float x) { return sum_over_kg(x); }
    static __device__ __forceinline__ void rescale(f32x4 (&o)[NI], float al) {
#pragma unroll
        for (int i = 0; i < NI; ++i) o[i] *= al;
    }
    // product i, output row m = 4 kg + r: dim 128 (i / 8) + 8 m + i % 8; head_dim 64: 8 m + i, or 8 (m - 8) + 4 + i
    template <int PAD> static __device__ __forceinline__ void to_lds(float (*rows)[PAD], const f32x4 (&o)[NI], int nh, int n, int kg) {
        if (n >= nh) return;
        float* row = rows[n];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * kg + r;
            if constexpr (D >= 128) {
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int e = 0; e < 8; e += 4)
                        *reinterpret_cast<f32x4*>(row + 128 * h + 8 * m + e) =
                            f32x4{o[8 * h + e][r], o[8 * h + e + 1][r], o[8 * h + e + 2][r], o[8 * h + e + 3][r]};
            } else {
                *reinterpret_cast<f32x4*>(row + (m < 8 ? 8 * m : 8 * (m - 8) + 4)) = f32x4{o[0][r], o[1][r], o[2][r], o[3][r]};
            }
        }
    }
};

// float32, query groups of up to four heads: products of 4x4, sixteen of them to an instruction of 8 cycles.  A 16x16 product
// of four real rows does four times the work, and its 32 cycles bound the batches that L2 serves.  Measured against it, over
// 180 shapes: 0.86 of the time in the mean (0.63 to 1.03); 32/8/128, 16 requests of 1152 to 2048 tokens 34.6 -> 31.1 us,
// 32/8/32, 200 requests of 1600 tokens, 90 % shared, 94 -> 57.  Not with two such sets for five to eight heads: 1.06 of the
// time (0.87 to 1.34: twice the registers for q, and short histories wait for its loads).
//     S = K Q^T      product (tq, kg) = lane / 4: token rows 4 tq .. 4 tq + 3 of a block (lane n = 4 tq + row), chunks 4 j + kg;
//                    its four sums over kg are exchanged so that lane (n, kg) ends with token 4 tq + kg and head n % 4
//     O += P V       one token's weights are one product's A operand, handed to all products whose lanes hold that token's V
//                    row: a load of 16 bytes a lane covers 64 / LR rows, and instruction x takes, for each of them, the weights
//                    of the x-th of the products in their lanes (the row's token follows from that: token_of).
template <int CB, int X> __device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CB, X, 0);
}
template <int D> struct Tile<float, D, 4> {
    static constexpr int TB = D >= 128 ? 1 : 2, PN = TB;   // blocks per tile; a lane has one token of each
    static constexpr int KC = D / 16, NI = 4, ES = 4;
    static constexpr int LR = D / 4;                       // lanes that a V row takes
    static constexpr int NX = LR / 4;                      // loads of V per block, products per V row
    static constexpr int CB = NX == 2 ? 1 : NX == 4 ? 2 : NX == 8 ? 3 : 4;
    f32x4 k[TB][KC], v[TB][NX], q[KC];

    static __device__ __forceinline__ int token_of(int x, int n, int kg) {   // of the V row that this lane holds of load x
        const int from = (n + 16 * kg) / LR * NX + x;      // the product whose weights it meets
        return 4 * (from & 3) + (from >> 2);
    }
    __device__ __forceinline__ void load_q(const char* rows, int nh, int n, int kg) {
        const char* row = rows + min(head(n), nh - 1) * (D * ES);
#pragma unroll
        for (int j = 0; j < KC; ++j) q[j] = head(n) < nh ? *reinterpret_cast<const f32x4*>(row + (4 * j + kg) * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void load_k(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int j = 0; j < KC; ++j) k[b][j] = *reinterpret_cast<const f32x4*>(blk + (uint32_t)(n * (D * 4) + kg * 16 + j * 64));
    }
    __device__ __forceinline__ void load_v(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int x = 0; x < NX; ++x)
            v[b][x] = *reinterpret_cast<const f32x4*>(blk + (uint32_t)(token_of(x, n, kg) * (D * 4) + (n + 16 * kg) % LR * 16));
    }
    __device__ __forceinline__ void mask(float (&p)[PN], int rest, int n, int kg) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            if (16 * b + (n & ~3) + kg >= rest) p[b] = -INFINITY;
#pragma unroll
            for (int x = 0; x < NX; ++x)
                if (16 * b + token_of(x, n, kg) >= rest) v[b][x] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __device__ __forceinline__ void scores(float (&p)[PN]) {
        constexpr int GC = KC < 8 ? KC : 8;                // products in one chain
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            f32x4 s;
#pragma unroll
            for (int j0 = 0; j0 < KC; j0 += GC) {
                f32x4 c[4];
#pragma unroll
                for (int j = j0; j < j0 + GC; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[e] = mfma4<0, 0>(k[b][j][e], q[j][e], j == j0 ? f32x4{0.f, 0.f, 0.f, 0.f} : c[e]);
                const f32x4 part = (c[0] + c[1]) + (c[2] + c[3]);
                s = j0 == 0 ? part : s + part;
            }
            const Pair even = swap32(s[0], s[2]), odd = swap32(s[1], s[3]);   // lower half: tokens 0 and 1, upper: 2 and 3
            const Pair all = swap16(even.a + even.b, odd.a + odd.b);
            p[b] = all.a + all.b;
        }
    }
    template <int X> __device__ __forceinline__ void take(int b, float w, f32x4 (&c)[4]) {
        if constexpr (X < NX) {
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = mfma4<CB, X>(w, v[b][X][e], X == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : c[e]);
            take<X + 1>(b, w, c);
        }
    }
    __device__ __forceinline__ void accumulate(const float (&p)[PN], f32x4 (&o)[NI], int) {
        // (chains as short as above: a block's sums start at zero)
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            f32x4 c[4];
            take<0>(b, p[b], c);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] += c[e];
        }
    }
    static __device__ __forceinline__ int head(int n) { return n & 3; }
    static __device__ __forceinline__ bool one_of_row(int n, int kg) { return n < 4 && kg == 0; }
    static __device__ __forceinline__ float row_max(float x) {
        x = fmaxf(x, lanes_moved<0x124>(x));               // rotated by 4 and by 8 within 16 lanes
        x = fmaxf(x, lanes_moved<0x128>(x));
        return max_over_kg(x);
    }
    static __device__ __forceinline__ float row_sum(float x) {
        x += lanes_moved<0x124>(x);
        x += lanes_moved<0x128>(x);
        return sum_over_kg(x);
    }
    static __device__ __forceinline__ void rescale(f32x4 (&o)[NI], float al) {
        const f32x4 f = {lanes_moved<0x00>(al), lanes_moved<0x55>(al), lanes_moved<0xAA>(al), lanes_moved<0xFF>(al)};   // of heads 0..3
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] *= f;
    }
    // o[e][r]: head r, dim 4 (lane % LR) + e; the 64 / LR groups of lanes hold sums over tokens of their own
    template <int PAD> static __device__ __forceinline__ void to_lds(float (*rows)[PAD], const f32x4 (&o)[NI], int, int n, int kg) {
        const int at = 4 * ((n + 16 * kg) % LR);
        if constexpr (LR == 64) {
#pragma unroll
            for (int r = 0; r < 4; ++r) *reinterpret_cast<f32x4*>(&rows[r][at]) = f32x4{o[0][r], o[1][r], o[2][r], o[3][r]};
        } else {
            f32x4 x, y;                                    // lower half: heads 0 and 1, upper: 2 and 3
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const Pair a = swap32(o[e][0], o[e][2]), b = swap32(o[e][1], o[e][3]);
                x[e] = a.a + a.b;
                y[e] = b.a + b.b;
            }
            if constexpr (LR == 32) {
                *reinterpret_cast<f32x4*>(&rows[kg & 2][at]) = x;
                *reinterpret_cast<f32x4*>(&rows[(kg & 2) + 1][at]) = y;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {              // row kg of lanes: head kg
                    const Pair a = swap16(x[e], y[e]);
                    x[e] = a.a + a.b;
                    if constexpr (LR == 8) x[e] += lanes_moved<0x128>(x[e]);
                }
                if (LR == 16 || n < 8) *reinterpret_cast<f32x4*>(&rows[kg][at]) = x;
            }
        }
    }
};

// x mod d, and x becomes x / d; the divisors are mostly powers of two (1 among them), and a true division is 40 dependent instructions.
__device__ __forceinline__ int take_digit(int& x, int d) {
    const int v = x;
    if ((d & (d - 1)) == 0) { x = v >> (31 - __clz(d)); return v & (d - 1); }
    x = v / d;
    return v - x * d;
}

// Waves of a workgroup: eight, two to a SIMD (a lane holds a whole tile: up to 256 registers); at head_dim 256 four.  Two
// where the table has no more than two tiles: the others would only hold registers, of which a workgroup of eight takes
// all that a compute unit has (bf16 32/8/128, 2000 requests of one block 185 -> 61 us; float32 64/1/64, 250 of one block
// 18.9 -> 6.9, the vector-unit kernel before 13.2; four requests of one block 4.98 -> 4.68).
template <int D> constexpr int direct_waves() { return D == 256 ? 4 : 8; }
// log2 of the largest softmax weight before a row's reference exponent is raised.  float32: any score above it raises it
// (the rounding of score - reference grows with its size, so the largest weights want theirs near zero).
template <typename T> constexpr float direct_slack() { return sizeof(T) == 4 ? 0.f : 24.f; }

// Partial rows of the pieces of a history, handed from the workgroups that make them to the one that folds them: written past
// the caches and read past them (device scope), since the workgroups may sit on different XCDs.
__device__ __forceinline__ void put_pair(float* p, float x, float y) {
    const unsigned long long v = (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get_pair(const float* p) {
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// Counts an arrival of `of` (at most 128) at *p; true for the last, which leaves zero.  Nobody clears the workspace: a counter is
// one whose upper 56 bits are the key, and any other word counts as zero.  (An addition to such a word counts nobody; whoever
// sees one is counted by the exchange, so everyone is counted once.)
__device__ __forceinline__ bool arrives_last(unsigned long long* p, int of) {
    constexpr unsigned long long kKey = 0xFEA5D1A2C37E6B00ull;
    unsigned long long old = __hip_atomic_fetch_add(p, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (((old ^ kKey) >> 8) != 0) {
        unsigned long long cur = old + 1, next;
        do next = ((cur ^ kKey) >> 8) != 0 ? kKey | 1 : cur + 1;
        while (!__hip_atomic_compare_exchange_strong(p, &cur, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        old = next - 1;
    }
    if ((int)(old & 255) + 1 < of) return false;
    __hip_atomic_store(p, kKey, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

template <typename T> __device__ __forceinline__ void store4(char* dst, float x0, float x1, float x2, float x3) {
    if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4*>(dst) = f32x4{x0, x1, x2, x3};
    else *reinterpret_cast<uint2*>(dst) = make_uint2(bf16_rne(x0) | (bf16_rne(x1) << 16), bf16_rne(x2) | (bf16_rne(x3) << 16));
}

template <typename T, int D, int R, int W>
__global__ __launch_bounds__(64 * W) void decode_direct_kernel(SweepArgs a, int row_tiles, int pieces) {
    using TileT = Tile<T, D, R>;
    constexpr int TB = TileT::TB, NI = TileT::NI, ES = TileT::ES, PN = TileT::PN;
    constexpr int BLK = kBlock * D * ES;           // bytes of one (block, KV head)
    constexpr int PAD = D + 4;                     // floats between the rows of the fold buffer (16 rows written side by side)
    __shared__ __attribute__((aligned(16))) float s_acc[W][R][PAD];
    __shared__ float2 s_ml[W][R];
    __shared__ bool s_last;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    int i = blockIdx.x;
    const int g = take_digit(i, a.Hkv), rt = take_digit(i, row_tiles), pc = take_digit(i, pieces);
    const int nh = min(16, a.G - 16 * rt);         // query heads of this row tile

    // The length, the ids of this wave's blocks and the query rows are requested together (the ids without
    // knowing the length: every address is inside the request's table row; entries past the length are not used).
    const int32_t* row = a.bt + (size_t)i * a.stride;
    const int first = pc * W + wave, step = W * pieces;   // tiles of this wave: first, first + step, ...
    auto ids_from = [&](int t0) {                         // lane TB x + b: block b of the x-th tile from t0 on
        const int col = TB * (t0 + (lane / TB) * step) + lane % TB;
        return row[min(max(col, 0), a.stride - 1)];
    };
    const int raw_len = a.seq_lens[i];
    int ids = a.stride > 0 ? ids_from(first) : 0;
    TileT tile;
    tile.load_q(static_cast<const char*>(a.q) + ((size_t)i * a.Hq + g * a.G + 16 * rt) * (D * ES), nh, n, kg);
    const int L = __builtin_amdgcn_readfirstlane(min(max(raw_len, 0), a.stride * kBlock));
    const int nb = (L + kBlock - 1) / kBlock, ntiles = (nb + TB - 1) / TB;

    f32x4 o[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = kLowest, l = 0.f;                    // of the lane's head: reference exponent (alike in all its lanes), this lane's part of the denominator
    const char* kb[TB];
    const char* vb[TB];
    auto locate = [&](int t, int at) {             // the blocks of tile t, whose ids sit in lanes TB at + b
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            // (a negative entry inside a request's length - the caller's error - must not become a read before the cache)
            const int blk = max(__builtin_amdgcn_readlane(ids, TB * at + (TB * t + b < nb ? b : 0)), 0);
            const size_t off = ((size_t)blk * a.Hkv + g) * BLK;
            kb[b] = static_cast<const char*>(a.k_cache) + off;
            vb[b] = static_cast<const char*>(a.v_cache) + off;
        }
    };
    // Scores to weights.  (bfloat16: the reference is raised to the row maximum only when a score outgrows it by 2^24, which
    // the float32 sums absorb without loss; the first score above -inf always does)
    auto weigh = [&](float (&p)[PN]) {
        float mx = p[0];
#pragma unroll
        for (int y = 1; y < PN; ++y) mx = fmaxf(mx, p[y]);
        mx *= a.scale_log2;
        if (__any(mx > m + direct_slack<T>())) {
            const float mn = fmaxf(m, TileT::row_max(mx));
            const float al = exp2_fast(m - mn);    // (0 where the reference was the lowest number)
            l *= al;
            TileT::rescale(o, al);
            m = mn;
        }
#pragma unroll
        for (int y = 0; y < PN; ++y) {
            p[y] = exp2_fast(fmaf(p[y], a.scale_log2, -m));
            l += p[y];
        }
    };
    // K of the next tile is asked for when this one's has been read, V likewise, and each is waited for where it is read: only
    // if the compiler leaves the loads where they stand.  The two empty statements, unlike one another, keep it from moving
    // those of V - the same before the loop and at its end - to the loop's head, behind the wait for K.  (float32 32/8/128, 16
    // requests of 1152 to 2048 tokens 31.1 -> 29.4 us, bf16 28/4/128, 8 of 90 to 700 tokens 8.8 -> 8.5; 244 bf16 shapes 0.98 of
    // the time in the mean.)
    if (first < ntiles) {
        locate(first, 0);
#pragma unroll
        for (int b = 0; b < TB; ++b) tile.load_k(b, kb[b], n, kg);
#pragma unroll
        for (int b = 0; b < TB; ++b) tile.load_v(b, vb[b], n, kg);
        asm volatile("; first tile asked for" ::: "memory");
        float p[PN];
        int t = first;
        for (int at = 0; t + step < ntiles; t += step) {
            tile.scores(p);
            if (++at == 64 / TB) {
                ids = ids_from(t + step);
                asm volatile("" : "+v"(ids));      // waited for here, once in 64 blocks, and not wherever ids are read
                at = 0;
            }
            locate(t + step, at);
#pragma unroll
            for (int b = 0; b < TB; ++b) tile.load_k(b, kb[b], n, kg);
            weigh(p);
            tile.accumulate(p, o, n);
#pragma unroll
            for (int b = 0; b < TB; ++b) tile.load_v(b, vb[b], n, kg);
            asm volatile("; next tile asked for" ::: "memory");
        }
        tile.scores(p);
        const int rest = L - t * (TB * kBlock);
        // tokens past the end: weight 0, and whatever their V rows hold is left out
        if (rest < TB * kBlock) tile.mask(p, rest, n, kg);
        weigh(p);
        tile.accumulate(p, o, n);
    }
    TileT::template to_lds<PAD>(s_acc[wave], o, nh, n, kg);
    l = TileT::row_sum(l);
    if (TileT::one_of_row(n, kg)) s_ml[wave][TileT::head(n)] = make_float2(m, l);
    __syncthreads();

    // fold the waves (fixed order) at the common reference exponent
    float* const acc = reinterpret_cast<float*>(a.ws + a.lay.acc);
    float* const mls = reinterpret_cast<float*>(a.ws + a.lay.ml);
    const size_t row0 = (size_t)(i * a.Hkv + g) * pieces * a.G + 16 * rt;   // of piece p and the tile's head h: partial row row0 + p G + h
    char* const out = static_cast<char*>(a.out) + ((size_t)i * a.Hq + g * a.G + 16 * rt) * (D * ES);
    for (int y = tid; y < nh * (D / 8); y += 64 * W) {
        const int h = y / (D / 8), c = y - h * (D / 8);
        float M = kLowest;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, s_ml[w][h].x);
        float den = 0.f, num[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) num[e] = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float2 ml = s_ml[w][h];
            const float f = exp2_fast(ml.x - M);   // (a wave that had no tile, or no score above -inf, has sums of 0)
            den = fmaf(f, ml.y, den);
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(&s_acc[w][h][8 * c]), a1 = *reinterpret_cast<const f32x4*>(&s_acc[w][h][8 * c + 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) { num[e] = fmaf(f, a0[e], num[e]); num[4 + e] = fmaf(f, a1[e], num[4 + e]); }
        }
        if (pieces > 1) {
            const size_t r = row0 + (size_t)pc * a.G + h;
#pragma unroll
            for (int e = 0; e < 8; e += 2) put_pair(acc + r * D + 8 * c + e, num[e], num[e + 1]);
            if (c == 0) put_pair(mls + 2 * r, M, den);
        } else {
            const float inv = L == 0 ? 0.f : 1.f / den;   // an empty history gives a zero row, one of scores of -inf alone 0/0
#pragma unroll
            for (int e = 0; e < 8; e += 4) store4<T>(out + (h * D + 8 * c + e) * ES, num[e] * inv, num[e + 1] * inv, num[e + 2] * inv, num[e + 3] * inv);
        }
    }
    // The workgroup that comes last to a history (of a KV head and row tile) folds its pieces, in their order: the result does
    // not depend on who comes last.  About 3 us, where a launch of its own takes 5 (float32 32/8/128, 16 requests of 1152 to
    // 2048 tokens in two pieces each 29.4 -> 27.3 us a call).
    if (pieces > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial rows have arrived
        __syncthreads();
        if (tid == 0) s_last = arrives_last(reinterpret_cast<unsigned long long*>(a.ws + a.lay.pre) + (i * a.Hkv + g) * row_tiles + rt, pieces);
        __syncthreads();
        if (s_last) {
            for (int y = tid; y < nh * (D / 4); y += 64 * W) {
                const int h = y / (D / 4), c = y - h * (D / 4);
                float M = kLowest, den = 0.f;
                f32x4 num = {0.f, 0.f, 0.f, 0.f};
                constexpr int kAtOnce = 8;
                for (int p0 = 0; p0 < pieces; p0 += kAtOnce) {
                    float2 v[kAtOnce], x0[kAtOnce], x1[kAtOnce];
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k) {
                        const size_t r = row0 + (size_t)min(p0 + k, pieces - 1) * a.G + h;
                        v[k] = get_pair(mls + 2 * r);
                        x0[k] = get_pair(acc + r * D + 4 * c);
                        x1[k] = get_pair(acc + r * D + 4 * c + 2);
                    }
                    float Mn = M;
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k) Mn = fmaxf(Mn, v[k].x);   // (where there is none left: the last piece's)
                    const float f0 = exp2_fast(M - Mn);
                    M = Mn;
                    den *= f0;
                    num *= f0;
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k) {
                        if (p0 + k < pieces) {
                            const float f = exp2_fast(v[k].x - M);
                            den = fmaf(f, v[k].y, den);
                            num[0] = fmaf(f, x0[k].x, num[0]);
                            num[1] = fmaf(f, x0[k].y, num[1]);
                            num[2] = fmaf(f, x1[k].x, num[2]);
                            num[3] = fmaf(f, x1[k].y, num[3]);
                        }
                    }
                }
                const float inv = L == 0 ? 0.f : 1.f / den;
                store4<T>(out + (h * D + 4 * c) * ES, num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv);
            }
        }
    }
    // What a later look at the workspace finds: no plan, this kernel.
    if (blockIdx.x == 0 && tid < H_WORDS)
        reinterpret_cast<int*>(a.ws)[tid] = tid == H_VARIANT ? 2 : tid == H_WAVES ? (int)gridDim.x * W : 0;
}

template <typename T, int D, int R, int W>
void launch_waves(const SweepArgs& a, int pieces, const Launch& L) {
    const int row_tiles = (a.G + 15) / 16;
    hipExtLaunchKernelGGL((decode_direct_kernel<T, D, R, W>), dim3((unsigned)(a.B * a.Hkv * row_tiles * pieces)), dim3(64 * W), 0,
                          static_cast<hipStream_t>(L.stream), static_cast<hipEvent_t>(L.ev_start), static_cast<hipEvent_t>(L.ev_stop), 0,
                          a, row_tiles, pieces);
}

template <typename T, int D, int R>
void launch_rows(const SweepArgs& a, int pieces, const Launch& L) {
    if (a.stride <= 2 * Tile<T, D, R>::TB) launch_waves<T, D, R, 2>(a, pieces, L);
    else launch_waves<T, D, R, direct_waves<D>()>(a, pieces, L);
}

template <typename T, int D>
void launch(const SweepArgs& a, int pieces, const Launch& L) {
    if constexpr (sizeof(T) == 4) {
        if (a.G <= 4) return launch_rows<T, D, 4>(a, pieces, L);
    }
    launch_rows<T, D, 16>(a, pieces, L);
}

}  // namespace

void launch_decode_direct(const SweepArgs& a, int dtype, int head_dim, int pieces, const Launch& L) {
    if (dtype == FEA_DTYPE_F32) {
        switch (head_dim) {
            case 32: launch<float, 32>(a, pieces, L); break;
            case 64: launch<float, 64>(a, pieces, L); break;
            case 128: launch<float, 128>(a, pieces, L); break;
            case 256: launch<float, 256>(a, pieces, L); break;
            default: break;
        }
    } else {
        switch (head_dim) {
            case 64: launch<bf16_t, 64>(a, pieces, L); break;
            case 128: launch<bf16_t, 128>(a, pieces, L); break;
            case 256: launch<bf16_t, 256>(a, pieces, L); break;
            default: break;
        }
    }
}

}  // namespace fea
