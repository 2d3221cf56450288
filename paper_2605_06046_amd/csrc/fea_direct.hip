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
// in all; then memory, at 5.0 to 5.9 TB/s where the chip is full (8 and more where what requests share sits in L2); with float32, more than four query heads and few workgroups the matrix cores' float32 rate (a
// block of 16 tokens is 64 instructions of 32 cycles at head_dim 128, whatever part of the 16 query rows is real).  Measured
// against the vector-unit kernel it replaces: float32 8/2/64, 4 requests of 320 tokens 11.6 -> 6.0 us a call; float32
// 32/8/128, 16 requests of 1152 to 2048 tokens 78.7 -> 22.7; against plan, sweep and merge: bf16 28/4/128, 8 requests of 90
// to 700 tokens 23.6 -> 6.7.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "../../include/fea.h"
#include "fea_plan.h"
#include "fea_tile.h"

namespace fea {
namespace {

using namespace tile;

// Waves of a workgroup: eight, two to a SIMD (a lane holds a whole tile: up to 256 registers); at head_dim 256 four.  Two
// where the table has no more than two tiles: the others would only hold registers, of which a workgroup of eight takes
// all that a compute unit has (bf16 32/8/128, 2000 requests of one block 185 -> 61 us; float32 64/1/64, 250 of one block
// 18.9 -> 6.9, the vector-unit kernel before 13.2; four requests of one block 4.98 -> 4.68).
template <int D> constexpr int direct_waves() { return D == 256 ? 4 : 8; }
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

template <typename T, int D, int R, int W, bool PIECES>
__global__ __launch_bounds__(64 * W) void decode_direct_kernel(SweepArgs a, int row_tiles, int pieces) {
    using TileT = Tile<T, D, R, false, PIECES>;
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
    float m = kLowest, l = 0.f;
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
    auto weigh_tile = [&](float (&p)[PN]) { weigh<TileT, T>(p, o, m, l, a.scale_log2); };
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
            weigh_tile(p);
            tile.accumulate(p, o, n);
#pragma unroll
            for (int b = 0; b < TB; ++b) tile.load_v(b, vb[b], n, kg);
            asm volatile("; next tile asked for" ::: "memory");
        }
        tile.scores(p);
        const int rest = L - t * (TB * kBlock);
        // tokens past the end: weight 0, and whatever their V rows hold is left out
        if (rest < TB * kBlock) tile.mask(p, rest, n, kg);
        weigh_tile(p);
        tile.accumulate(p, o, n);
    }
    TileT::template to_lds<PAD>(s_acc[wave], o, nh, n, kg);
    l = TileT::row_sum(l);
    if (TileT::one_of_row(n, kg)) s_ml[wave][TileT::head(n)] = make_float2(m, l);
    __syncthreads();

    // fold the waves
    float* const acc = reinterpret_cast<float*>(a.ws + a.lay.acc);
    float* const mls = reinterpret_cast<float*>(a.ws + a.lay.ml);
    const size_t row0 = (size_t)(i * a.Hkv + g) * pieces * a.G + 16 * rt;   // of piece p and the tile's head h: partial row row0 + p G + h
    char* const out = static_cast<char*>(a.out) + ((size_t)i * a.Hq + g * a.G + 16 * rt) * (D * ES);
    bool nan = false;
    for (int y = tid; y < nh * (D / 8); y += 64 * W) {
        const int h = y / (D / 8), c = y - h * (D / 8);
        float M, den, num[8];
        fold_waves(s_acc, s_ml, h, c, M, den, num);
        if constexpr (sizeof(T) == 2) nan |= any_nan(num);
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
    // Sums that are NaN: the wave that has folded them reads the workgroup's tiles again for the infinities among them.  (Looked for
    // here and not in every wave's own sums: +0.8 instead of +2.0 % of a call's time over 36 shapes of 3 to 30 us.)
    if constexpr (sizeof(T) == 2) {
        if (__builtin_expect(__any(nan), 0)) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the same elements are written once more)
            tile.load_q(static_cast<const char*>(a.q) + ((size_t)i * a.Hq + g * a.G + 16 * rt) * (D * ES), nh, n, kg);
            sweep_apart<TileT, D>(tile, o, m, l, a, row, g, L, pc * W, W, step, n, kg);
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int dim = TileT::dim_of(j, 4 * kg + r);
                    if (n >= nh || __builtin_isfinite(o[j][r]) || (n * (D / 8) + dim / 8) / 64 % W != wave) continue;   // (no such head; as it was; another wave's)
                    if (pieces > 1) __hip_atomic_store(acc + (row0 + (size_t)pc * a.G + n) * D + dim, o[j][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else *reinterpret_cast<uint16_t*>(out + (n * D + dim) * ES) = (uint16_t)bf16_rne(o[j][r]);
                }
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
                    const float f0 = exp2f(M - Mn);   // (exp2f: pieces whose weights lie below 2^-126 count, as in a merge)
                    M = Mn;
                    den *= f0;
                    num *= f0;
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k) {
                        if (p0 + k < pieces) {
                            const float f = exp2f(v[k].x - M);
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
        reinterpret_cast<int*>(a.ws)[tid] = tid == H_VARIANT ? kNoPlan : tid == H_WAVES ? (int)gridDim.x * W : 0;
}

template <typename T, int D, int R, int W, bool PIECES = true>
void launch_waves(const SweepArgs& a, int pieces, const Launch& L) {
    const int row_tiles = (a.G + 15) / 16;
    hipExtLaunchKernelGGL((decode_direct_kernel<T, D, R, W, PIECES>), dim3((unsigned)(a.B * a.Hkv * row_tiles * pieces)), dim3(64 * W), 0,
                          static_cast<hipStream_t>(L.stream), static_cast<hipEvent_t>(L.ev_start), static_cast<hipEvent_t>(L.ev_stop), 0,
                          a, row_tiles, pieces);
}

// bfloat16 K rows come in pieces (fea_tile.h) where that saves more than the moves behind the loads cost.  Not at head_dim 256 in
// tables of two rounds of a workgroup's tiles, 16 blocks: 32/8/256, 100 requests of 32 tokens 16.4 us with pieces, 14.6 without, 55 of
// 60 to 140 14.9 and 14.2, 30 of 130 to 190 8.9 and 8.4 (10.4 and 9.7 with four sets of caches in turn).  Beyond, 0.92 to 0.94 of the time
// with pieces for 16 of 180 to 260 (in turn 0.99), 1.05 for 30 of 160 to 220.  Nor at head_dim 128 in tables of two tiles: 64/8/128, 180
// of 32 tokens 7.8 and 7.4 (up to 100 requests 0.98 to 1.01).  In wider ones 0.89 to 1.01 with pieces from 33 tokens on, 1.03 to 1.06 for
// 100 requests and more of one or two blocks.  Head_dim 64, of whose chunks half as many move: 0.97 to 1.00.
template <typename T, int D, int R>
void launch_rows(const SweepArgs& a, int pieces, const Launch& L) {
    constexpr int TB = Tile<T, D, R>::TB, W = direct_waves<D>();
    constexpr bool kShortApart = sizeof(T) == 2 && D >= 128;
    if (a.stride <= 2 * TB) return launch_waves<T, D, R, 2, !kShortApart>(a, pieces, L);
    if constexpr (kShortApart && D == 256) {
        if (a.stride <= 2 * TB * W) return launch_waves<T, D, R, W, false>(a, pieces, L);
    }
    launch_waves<T, D, R, W>(a, pieces, L);
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
