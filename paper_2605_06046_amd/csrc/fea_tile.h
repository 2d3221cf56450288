// A tile of a history in a wave's registers - K and V straight from global memory into the operands of the matrix cores' two
// products, scores and weights, the sums over the tiles - for the kernels that read every history on its own: the one without
// a plan (fea_direct.hip, which says how the operands lie) and the sweep of a batch that shares nothing (fea_sweep_mfma.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "fea_device.h"
#include "fea_plan.h"

namespace fea {
namespace tile {

struct bf16_t { uint16_t bits; };


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

// bfloat16, K of a block in a 16-row product: lane (n, kg) has row n, chunks (of 16 bytes) k_chunk(j, kg), j < KC; q likewise.  It is
// not loaded so - a load then takes 16 bytes of a row for each of four neighbouring lanes - but four lanes read a row's 64 bytes in
// one piece, four rows one after the other, and hand each other what is theirs (rows of 128 bytes: two lanes, two rows): 64
// instructions for four chunks a lane.  Measured against rows in neighbouring lanes: 16 requests on a prefix of 1500, 32/8/128, 14.9 ->
// 11.6 us, 24 on one of 500, 64/8/128, 11.4 -> 9.2, 60 in two groups, 32/2/128, 17.1 -> 15.2, 8 of 90 to 700 tokens, 28/4/128, 8.0 ->
// 7.2, 40 on 1500, 8/2/64, 9.7 -> 8.7; five others 0.97 to 1.00 of the time.  float32 groups of more than four heads, which the
// products bind, take 1.02 to 1.07 of the time so; and where a wave has a tile or two in all it waits for the moves as well, see the
// plan-free kernel's rule.  (Conditional moves that take the partner's register through their own exchange, by
// hand, are half as many instructions and took 1.00 to 1.05 of the time.)
template <int KC> __device__ __forceinline__ int k_chunk(int j, int kg) { return KC == 2 ? 2 * kg + j : 16 * (j >> 2) + 4 * kg + (j & 3); }
template <int KC> __device__ __forceinline__ uint32_t k_offset(int j, int n, int kg) {    // of load j, from the block's start
    return KC == 2 ? (uint32_t)((2 * (n >> 1) + j) * 128 + (2 * kg + (n & 1)) * 16)
                   : (uint32_t)((4 * (n >> 2) + (j & 3)) * (KC * 64) + (16 * (j >> 2) + 4 * kg + (n & 3)) * 16);
}
template <int CTRL> __device__ __forceinline__ u32x4 chunk_moved(u32x4 x) {
#pragma unroll
    for (int w = 0; w < 4; ++w) x[w] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[w], CTRL, 0xF, 0xF, true);
    return x;
}
template <int CTRL> __device__ __forceinline__ void swap_chunks(bool upper, u32x4& x, u32x4& y) {   // the lower lane's y against the upper one's x
    const u32x4 from_y = chunk_moved<CTRL>(y), from_x = chunk_moved<CTRL>(x);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        x[w] = upper ? from_y[w] : x[w];
        y[w] = upper ? y[w] : from_x[w];
    }
}
template <int KC> __device__ __forceinline__ void to_rows(u32x4 (&x)[KC]) {
    const int n = threadIdx.x & 15;
#pragma unroll
    for (int j = 0; j < KC; j += 2) swap_chunks<0xB1>(n & 1, x[j], x[j + 1]);
    if constexpr (KC > 2) {
#pragma unroll
        for (int j = 0; j < KC; j += 4) {
            swap_chunks<0x4E>(n & 2, x[j], x[j + 2]);
            swap_chunks<0x4E>(n & 2, x[j + 1], x[j + 3]);
        }
    }
}

// A lane's registers of one tile, and the two products, for row tiles of R query heads.  A lane works out the weights of
// PN tokens for one head.  ONCE: its bytes are read once and pass by the caches.  PIECES: K rows are loaded in pieces; whole histories
// keep them in neighbouring lanes (with pieces 64 requests of 4224 to 5120 tokens, 32/8/128, 202 -> 207 us, 512 of 512 to 4096,
// 64/8/128, 744 -> 747; 256 of 512 to 1024 138.4 -> 132.9).
template <typename T, int D, int R, bool ONCE = false, bool PIECES = !ONCE> struct Tile;

template <int D> struct Tile<float, D, 16, false, true> {
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

template <int D, bool ONCE, bool PIECES> struct Tile<bf16_t, D, 16, ONCE, PIECES> {
    static constexpr int TB = 2, PN = 8;
    static constexpr int KC = D / 32;
    static constexpr int VH = D == 256 ? 2 : 1;
    static constexpr int NI = D / 16;
    static constexpr int ES = 2;
    u32x4 k[TB][KC], v[TB][4][VH], q[KC];

    __device__ __forceinline__ void load_q(const char* rows, int nh, int n, int kg) {
        const char* row = rows + min(n, nh - 1) * (D * ES);
#pragma unroll
        for (int j = 0; j < KC; ++j) q[j] = n < nh ? ld16(row + (PIECES ? k_chunk<KC>(j, kg) : 4 * j + kg) * 16) : u32x4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void load_k(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int j = 0; j < KC; ++j) k[b][j] = ld16<ONCE>(blk + (PIECES ? k_offset<KC>(j, n, kg) : (uint32_t)(n * (D * 2) + kg * 16 + j * 64)));
    }
    __device__ __forceinline__ void load_v(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < VH; ++h) v[b][r][h] = ld16<ONCE>(blk + (uint32_t)((4 * kg + r) * (D * 2) + (D >= 128 ? n : n & 7) * 16 + h * 256));
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
        if constexpr (PIECES) {
#pragma unroll
            for (int b = 0; b < TB; ++b) to_rows(k[b]);
        }
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
    // (APART: what is left of a weight meets zeros where V is infinite or NaN: the rounded weight has made that product, and
    // zero or a negative rest times infinity would make the sum NaN)
    template <bool APART = false> __device__ __forceinline__ void accumulate(const float (&p)[PN], f32x4 (&o)[NI], int n) {
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
            if constexpr (APART) {
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    t[w] &= ((t[w] & 0x7F80u) == 0x7F80u ? 0u : 0xFFFFu) | ((t[w] & 0x7F800000u) == 0x7F800000u ? 0u : 0xFFFF0000u);
            }
            o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t), lo, o[i], 0, 0, 0);
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
    // product i, output row m = 4 kg + r
    static __device__ __forceinline__ int dim_of(int i, int m) {
        if constexpr (D >= 128) return 128 * (i >> 3) + 8 * m + (i & 7);
        else return m < 8 ? 8 * m + i : 8 * (m - 8) + 4 + i;
    }
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
//     S = K Q^T      on the vector unit: 16 lanes side by side read 256 bytes of a K row, four rows 4 t + kg a load, and each lane
//                    multiplies its chunks with those of the four heads; the 16 lanes' sums are halved among them from step to
//                    step, so that lane (n, kg) ends with token 4 (n / 4) + kg and head n % 4.  A product's operand would be four
//                    rows in four neighbouring lanes, and that a load then hands out 16 bytes of every row is what bound the
//                    kernel: 32/8/128, 16 requests of 1152 to 2048 tokens 28.2 -> 23.6 us, 40 of 300 to 2000 94.6 -> 86.8,
//                    16/4/256, 20 of 1124 to 1824 32.9 -> 26.9, 32/8/64, 60 on one prefix of 2048 50.7 -> 41.8; eight others
//                    0.87 to 0.96 of the time.
//     O += P V       one token's weights are one product's A operand, handed to all products whose lanes hold that token's V
//                    row: a load of 16 bytes a lane covers 64 / LR rows, and instruction x takes, for each of them, the weights
//                    of the x-th of the products in their lanes (the row's token follows from that: token_of).
template <int CB, int X> __device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CB, X, 0);
}
template <int D> struct Tile<float, D, 4, false, true> {
    static constexpr int TB = D >= 128 ? 1 : 2, PN = TB;   // blocks per tile; a lane has one token of each
    static constexpr int KC = D / 16, NI = 4, ES = 4;
    static constexpr int CC = D >= 64 ? D / 64 : 1;        // chunks of a K row per lane
    static constexpr int RR = KC / CC;                     // rows per lane and block: 4 (head_dim 32: 2, 8 lanes a row)
    static constexpr int LR = D / 4;                       // lanes that a V row takes
    static constexpr int NX = LR / 4;                      // loads of V per block, products per V row
    static constexpr int CB = NX == 2 ? 1 : NX == 4 ? 2 : NX == 8 ? 3 : 4;
    f32x4 k[TB][KC], v[TB][NX], q[4 * CC];

    static __device__ __forceinline__ int token_of(int x, int n, int kg) {   // of the V row that this lane holds of load x
        const int from = (n + 16 * kg) / LR * NX + x;      // the product whose weights it meets
        return 4 * (from & 3) + (from >> 2);
    }
    __device__ __forceinline__ void load_q(const char* rows, int nh, int n, int) {
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int c = 0; c < CC; ++c)
                q[h * CC + c] = h < nh ? *reinterpret_cast<const f32x4*>(rows + h * (D * ES) + (D >= 64 ? n + 16 * c : n & 7) * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void load_k(int b, const char* blk, int n, int kg) {
#pragma unroll
        for (int t = 0; t < RR; ++t)
#pragma unroll
            for (int c = 0; c < CC; ++c)
                k[b][t * CC + c] = *reinterpret_cast<const f32x4*>(blk + (uint32_t)((D >= 64 ? 4 * t + kg : 4 * t + 8 * (n >> 3) + kg) * (D * ES) +
                                                                                    (D >= 64 ? n + 16 * c : n & 7) * 16));
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
        const int n = threadIdx.x & 15;
        auto halve = [](bool upper, float x, float y, auto moved) {    // the lower lanes' x, the upper ones' y, with the partner's
            return (upper ? y : x) + moved(upper ? x : y);
        };
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            float s[RR][4];
#pragma unroll
            for (int t = 0; t < RR; ++t)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    float even = 0.f, odd = 0.f;           // (two chains: half the error of one, and half the wait)
#pragma unroll
                    for (int c = 0; c < CC; ++c) {
                        const f32x4 x = k[b][t * CC + c], y = q[h * CC + c];
                        even = c == 0 ? x[0] * y[0] : fmaf(x[0], y[0], even);
                        odd = c == 0 ? x[1] * y[1] : fmaf(x[1], y[1], odd);
                        even = fmaf(x[2], y[2], even);
                        odd = fmaf(x[3], y[3], odd);
                    }
                    s[t][h] = even + odd;
                }
            if constexpr (RR == 4) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int h = 0; h < 4; ++h) s[t][h] = halve(n & 8, s[t][h], s[2 + t][h], lanes_moved<0x128>);      // rotated by 8
            }
#pragma unroll
            for (int h = 0; h < 4; ++h) s[0][h] = halve(n & 4, s[0][h], s[1][h], lanes_moved<0x141>);                  // mirrored in 8
#pragma unroll
            for (int h = 0; h < 2; ++h) s[0][h] = halve(n & 2, s[0][h], s[0][2 + h], lanes_moved<0x4E>);
            p[b] = halve(n & 1, s[0][0], s[0][1], lanes_moved<0xB1>);
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

// log2 of the largest softmax weight before a row's reference exponent is raised.  float32: any score above it raises it
// (the rounding of score - reference grows with its size, so the largest weights want theirs near zero).
template <typename T> constexpr float direct_slack() { return sizeof(T) == 4 ? 0.f : 24.f; }

// Scores to weights: o, the sums over the tiles so far, m and l, the reference exponent of the lane's head (alike in all its
// lanes) and this lane's part of the denominator.  (bfloat16: the reference is raised to the row maximum only when a score
// outgrows it by 2^24, which the float32 sums absorb without loss; the first score above -inf always does)
template <class TileT, typename T>
__device__ __forceinline__ void weigh(float (&p)[TileT::PN], f32x4 (&o)[TileT::NI], float& m, float& l, float scale_log2) {
    float mx = p[0];
#pragma unroll
    for (int y = 1; y < TileT::PN; ++y) mx = fmaxf(mx, p[y]);
    mx *= scale_log2;
    if (__any(mx > m + direct_slack<T>())) {
        const float mn = fmaxf(m, TileT::row_max(mx));
        const float al = exp2_fast(m - mn);        // (0 where the reference was the lowest number)
        l *= al;
        TileT::rescale(o, al);
        m = mn;
    }
#pragma unroll
    for (int y = 0; y < TileT::PN; ++y) {
        p[y] = exp2_fast(fmaf(p[y], scale_log2, -m));
        l += p[y];
    }
}

// Elements 8 c .. 8 c + 7 of head h's row, folded over the waves of a workgroup (in fixed order) at their common reference
// exponent M.  A wave that had no tile, or no score above -inf, has sums of 0.
template <int W, int R, int PAD> __device__ __forceinline__ void fold_waves(const float (&acc)[W][R][PAD], const float2 (&ml)[W][R], int h, int c,
                                                                            float& M, float& den, float (&num)[8]) {
    M = kLowest;
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, ml[w][h].x);
    den = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) num[e] = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const float f = exp2_fast(ml[w][h].x - M);
        den = fmaf(f, ml[w][h].y, den);
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(&acc[w][h][8 * c]), a1 = *reinterpret_cast<const f32x4*>(&acc[w][h][8 * c + 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) { num[e] = fmaf(f, a0[e], num[e]); num[4 + e] = fmaf(f, a1[e], num[4 + e]); }
    }
}

// Whether one of a lane's sums is NaN.  (The maximum that hands NaN on takes two of them an instruction.)
__device__ __forceinline__ bool any_nan(const float (&x)[8]) {
    float y = x[0];
#pragma unroll
    for (int e = 1; e < 7; e += 2) y = __builtin_elementwise_maximum(__builtin_elementwise_maximum(y, x[e]), x[e + 1]);
    y = __builtin_elementwise_maximum(y, x[7]);
    return y != y;
}
template <int NI> __device__ __forceinline__ bool any_nan(const f32x4 (&o)[NI]) {
    static_assert(NI % 2 == 0, "two at a time, and the first and the last");
    f32x4 x = o[0];
#pragma unroll
    for (int i = 1; i + 1 < NI; i += 2)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x[r], o[i][r]), o[i + 1][r]);
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = __builtin_elementwise_maximum(x[r], o[NI - 1][r]);
    const float y = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x[0], x[1]), __builtin_elementwise_maximum(x[2], x[3]));
    return y != y;
}

// bfloat16, where a sum is NaN: V holds infinities or NaN then, or the scores do, and of a weight only the rounded part may meet an
// infinity of V.  The tiles are read once more, `group` of them from `first` on and so every `step`, one after the other: nothing
// waits for such a row.  Sums over the tiles of before, in their order, that were not NaN come out as they were.
template <class TileT, int D>
__device__ __forceinline__ void sweep_apart(TileT& tile, f32x4 (&o)[TileT::NI], float& m, float& l, const SweepArgs& a, const int32_t* row, int g, int L,
                                            int first, int group, int step, int n, int kg) {
    constexpr int TB = TileT::TB, PN = TileT::PN, BLK = kBlock * D * TileT::ES;
    const int nb = (L + kBlock - 1) / kBlock, ntiles = (nb + TB - 1) / TB;
#pragma unroll
    for (int j = 0; j < TileT::NI; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    m = kLowest;
    l = 0.f;
#pragma unroll 1
    for (int t0 = first; t0 < ntiles; t0 += step)
#pragma unroll 1
        for (int t = t0; t < min(t0 + group, ntiles); ++t) {
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const int blk = max(__builtin_amdgcn_readfirstlane(row[TB * t + (TB * t + b < nb ? b : 0)]), 0);
                const size_t off = ((size_t)blk * a.Hkv + g) * BLK;
                tile.load_k(b, static_cast<const char*>(a.k_cache) + off, n, kg);
                tile.load_v(b, static_cast<const char*>(a.v_cache) + off, n, kg);
            }
            float p[PN];
            tile.scores(p);
            const int rest = L - t * (TB * kBlock);
            if (rest < TB * kBlock) tile.mask(p, rest, n, kg);
            weigh<TileT, bf16_t>(p, o, m, l, a.scale_log2);
            tile.template accumulate<true>(p, o, n);
        }
}

}  // namespace tile
}  // namespace fea
