// Cumulative chunk hashes on the device: the chunk-parallel formulation of the
// prefix hash computation (appendix "Prefix Hash Computation", Algorithm 2).
// Every 16-token chunk is hashed on its own into a leaf (the parallel phase, one
// thread per chunk), then the leaves of a request are chained in order (the
// sequential phase, O(C) per request, one wave).  One workgroup per request;
// leaves pass through LDS in slabs: one wave chains a slab while the others make
// the leaves of the next.  The arithmetic is the one documented at
// fea_chunk_hashes; the host function and this kernel must agree bit for bit.
#include <hip/hip_runtime.h>

#include "../../include/fea.h"
#include "fea_internal.h"

namespace fea {

namespace {

constexpr unsigned long long kGammaD = 0x9E3779B97F4A7C15ull;
constexpr unsigned long long kH0D = 0x243F6A8885A308D3ull;
constexpr int kChunk = FEA_BLOCK_TOKENS;
constexpr int kSlab = 256;          // leaves made at a time

__device__ __forceinline__ unsigned long long mixd(unsigned long long x) {
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

struct HashArgs {
    const int32_t* tokens;
    const int64_t* tok_offsets;
    const int64_t* hash_offsets;
    unsigned long long* hashes;
    int64_t n_tokens, n_hashes;
};

// h + gamma, wave-uniform, and lane C of (lo, hi) = h.  Whichever unit wrote h: the scalar unit's reads of it are ordered by
// the hardware, and a value the vector unit has just written wants two wait states before another vector instruction reads
// it, which the two scalar additions are.
template <int C> __device__ __forceinline__ unsigned long long put_lane(int& lo, int& hi, unsigned long long h, unsigned long long gamma) {
    uint32_t nl, nh;
    asm volatile("s_add_u32 %0, %4, %6\n\ts_addc_u32 %1, %5, %7\n\tv_writelane_b32 %2, %4, %8\n\tv_writelane_b32 %3, %5, %8"
        : "=&s"(nl), "=&s"(nh), "+v"(lo), "+v"(hi)
        : "s"((uint32_t)h), "s"((uint32_t)(h >> 32)), "s"((uint32_t)gamma), "s"((uint32_t)(gamma >> 32)), "n"(C) : "scc");
    return (unsigned long long)nl | ((unsigned long long)nh << 32);
}

// The multipliers of a mixing step and the chain's increment, kept in scalar registers: as literals they would make two
// words of an instruction, and one wave alone waits for what it fetches.
struct MixConsts { unsigned long long m1, m2, gamma; };
__device__ __forceinline__ unsigned long long low64(unsigned long long x, unsigned long long m) {
    const uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), ml = (uint32_t)m, mh = (uint32_t)(m >> 32);
    const uint32_t hi = __umulhi(xl, ml) + xl * mh + xh * ml;
    return (unsigned long long)(xl * ml) | ((unsigned long long)hi << 32);
}
__device__ __forceinline__ unsigned long long mixs(unsigned long long x, const MixConsts& k) {
    x = low64(x ^ (x >> 30), k.m1);
    x = low64(x ^ (x >> 27), k.m2);
    return x ^ (x >> 31);
}

// Leaves in lanes FROM .. FROM + 7, moved to scalar registers side by side: eight cycles a chunk, where a lane read on its own
// among scalar instructions holds up the next of them, 23 cycles a chunk (of 197).
template <int FROM> __device__ __forceinline__ void take_leaves(unsigned long long (&x)[8], int lo, int hi) {
    asm volatile(
        "v_readlane_b32 s64, %8, %10\n\tv_readlane_b32 s65, %9, %10\n\tv_readlane_b32 s66, %8, %11\n\tv_readlane_b32 s67, %9, %11\n\t"
        "v_readlane_b32 s68, %8, %12\n\tv_readlane_b32 s69, %9, %12\n\tv_readlane_b32 s70, %8, %13\n\tv_readlane_b32 s71, %9, %13\n\t"
        "v_readlane_b32 s72, %8, %14\n\tv_readlane_b32 s73, %9, %14\n\tv_readlane_b32 s74, %8, %15\n\tv_readlane_b32 s75, %9, %15\n\t"
        "v_readlane_b32 s76, %8, %16\n\tv_readlane_b32 s77, %9, %16\n\tv_readlane_b32 s78, %8, %17\n\tv_readlane_b32 s79, %9, %17"
        : "={s[64:65]}"(x[0]), "={s[66:67]}"(x[1]), "={s[68:69]}"(x[2]), "={s[70:71]}"(x[3]), "={s[72:73]}"(x[4]), "={s[74:75]}"(x[5]),
          "={s[76:77]}"(x[6]), "={s[78:79]}"(x[7])
        : "v"(lo), "v"(hi), "n"(FROM), "n"(FROM + 1), "n"(FROM + 2), "n"(FROM + 3), "n"(FROM + 4), "n"(FROM + 5), "n"(FROM + 6), "n"(FROM + 7));
}

// Chunks C .. 15 of a batch: leaves and hashes in lanes 0 .. 15; hg: the last hash + gamma.
constexpr int kBatch = 16;
template <int C, bool SHORT> __device__ __forceinline__ void chain(unsigned long long& hg, const MixConsts& k, int left, int leaf_lo, int leaf_hi,
                                                                   unsigned long long (&x)[8], int& out_lo, int& out_hi) {
    if constexpr (C < kBatch) {
        if (SHORT && C >= left) return;
        if constexpr (C % 8 == 0) take_leaves<C>(x, leaf_lo, leaf_hi);
        hg = put_lane<C>(out_lo, out_hi, mixs(mixs(hg, k) ^ x[C % 8], k), k.gamma);
        chain<C + 1, SHORT>(hg, k, left, leaf_lo, leaf_hi, x, out_lo, out_hi);
    }
}

// Four neighbouring tokens, loadable from any 4-byte boundary.
struct __attribute__((packed, aligned(4))) Tok4 { uint32_t t[4]; };

// Bound: the chain, two mixing steps per chunk one after the other: 43 instructions of one wave, which issues one every four
// cycles; 190 cycles a chunk, 165 of them the 39 scalar instructions of the two steps.  It runs in scalar registers (a 64-bit
// product is six scalar instructions of 4 bytes; on the vector unit it is four, but of 8 bytes, and a wave alone waits for what it
// fetches: 36 instructions a chunk take 153 cycles on some compute units and 202 on others).  Leaves are handed over and hashes
// collected in batches of 16 lanes, whose numbers are then part of the instructions, and the constants sit in registers.  Only the
// first slab's leaves stand in line with the chain, one wave of them to a SIMD.  64 requests of 4224 to 5120 tokens: 48.1 us with
// the chain in vector registers and through LDS, 31.1 with a lane read before each leaf's use and 2048 leaves before the chain
// (five waves of them), 29.9 in slabs, 28.3 with the lane reads side by side; one of 100000 tokens 542, 530 and 495.
constexpr int kHashThreads = 256;
static_assert(kHashThreads == kSlab && kSlab % kBatch == 0, "a thread per leaf of the first slab; whole batches");
__global__ __launch_bounds__(kHashThreads) void chunk_hash_kernel(HashArgs a) {
    __shared__ unsigned long long s_leaf[2][kSlab];
    const int i = blockIdx.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = a.tok_offsets[i], t1 = a.tok_offsets[i + 1];
    if (t0 < 0 || t1 < t0 || t1 > a.n_tokens) return;            // inconsistent offsets: the row is skipped
    const int64_t T = t1 - t0, C = (T + kChunk - 1) / kChunk;
    const int64_t h0 = a.hash_offsets[i];
    if (h0 < 0 || h0 + C > a.n_hashes) return;
    const int32_t* tok = a.tokens + t0;
    auto make_leaf = [&](int64_t c) -> unsigned long long {      // parallel phase: independent leaves
        const int64_t first = c * kChunk;
        const int len = (int)(T - first < kChunk ? T - first : kChunk);
        unsigned long long x = mixd(kGammaD ^ (unsigned long long)len);
        if (len == kChunk) {
            Tok4 w[kChunk / 4];
#pragma unroll
            for (int j = 0; j < kChunk / 4; ++j) w[j] = *reinterpret_cast<const Tok4*>(tok + first + 4 * j);
#pragma unroll
            for (int j = 0; j < kChunk; ++j) x = mixd(x ^ (unsigned long long)w[j >> 2].t[j & 3]);
        } else {
            for (int j = 0; j < len; ++j) x = mixd(x ^ (unsigned long long)(uint32_t)tok[first + j]);
        }
        return x;
    };
    if (tid < C) s_leaf[0][tid] = make_leaf(tid);
    __syncthreads();
    unsigned long long hg = kH0D + kGammaD;                       // carried by the first wave across slabs
    int buf = 0;
    for (int64_t base = 0; base < C; base += kSlab, buf ^= 1) {
        const int n = __builtin_amdgcn_readfirstlane((int)(C - base < kSlab ? C - base : kSlab));
        if (wave == 0) {                                          // sequential phase: the chain
            hg = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)hg) |
                 ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(hg >> 32)) << 32);
            MixConsts k = {0xBF58476D1CE4E5B9ull, 0x94D049BB133111EBull, kGammaD};
            asm("" : "+s"(k.m1), "+s"(k.m2), "+s"(k.gamma));
            const unsigned long long* leaves = s_leaf[buf];
            const int at = tid & (kBatch - 1);
            unsigned long long leaf = leaves[at];                 // (past the end: anything, which nothing is made of)
            for (int c0 = 0; c0 < n; c0 += kBatch) {
                const int leaf_lo = (int)(uint32_t)leaf, leaf_hi = (int)(uint32_t)(leaf >> 32);
                leaf = leaves[min(c0 + kBatch, kSlab - kBatch) + at];
                int out_lo = 0, out_hi = 0;
                unsigned long long x[8];
                if (n - c0 >= kBatch) chain<0, false>(hg, k, kBatch, leaf_lo, leaf_hi, x, out_lo, out_hi);
                else chain<0, true>(hg, k, n - c0, leaf_lo, leaf_hi, x, out_lo, out_hi);
                if (tid < kBatch && c0 + tid < n)
                    a.hashes[h0 + base + c0 + tid] = (unsigned long long)(uint32_t)out_lo | ((unsigned long long)(uint32_t)out_hi << 32);
            }
        } else {
            for (int x = tid - 64; x < kSlab && base + kSlab + x < C; x += kHashThreads - 64) s_leaf[buf ^ 1][x] = make_leaf(base + kSlab + x);
        }
        __syncthreads();
    }
}

}  // namespace
}  // namespace fea

using namespace fea;

extern "C" int32_t fea_chunk_hashes_device(const int32_t* tokens, int64_t n_tokens, const int64_t* tok_offsets,
                                           int32_t B, const int64_t* hash_offsets, uint64_t* hashes,
                                           int64_t n_hashes, void* hip_stream) {
    if (B < 0 || n_tokens < 0 || n_hashes < 0) return fail(FEA_EINVAL, "fea_chunk_hashes_device: negative size");
    if (B == 0) return FEA_OK;
    if (!tok_offsets || !hash_offsets || (n_tokens > 0 && !tokens) || (n_hashes > 0 && !hashes))
        return fail(FEA_EINVAL, "fea_chunk_hashes_device: NULL device pointer");
    HashArgs a;
    a.tokens = tokens;
    a.tok_offsets = tok_offsets;
    a.hash_offsets = hash_offsets;
    a.hashes = reinterpret_cast<unsigned long long*>(hashes);
    a.n_tokens = n_tokens;
    a.n_hashes = n_hashes;
    hipLaunchKernelGGL(chunk_hash_kernel, dim3((unsigned)B), dim3(kHashThreads), 0, static_cast<hipStream_t>(hip_stream), a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FEA_EHIP, "fea_chunk_hashes_device: launch failed: %s", hipGetErrorString(e));
    return FEA_OK;
}
