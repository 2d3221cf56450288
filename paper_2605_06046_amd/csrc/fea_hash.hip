// Cumulative chunk hashes on the device: the chunk-parallel formulation of the
// prefix hash computation (appendix "Prefix Hash Computation", Algorithm 2).
// Every 16-token chunk is hashed on its own into a leaf (the parallel phase, one
// thread per chunk), then the leaves of a request are chained in order (the
// sequential phase, O(C) per request, one wave).  One workgroup per request;
// leaves pass through LDS in tiles so the chaining wave never waits on global
// memory.  The arithmetic is the one documented at fea_chunk_hashes; the host
// function and this kernel must agree bit for bit.
#include <hip/hip_runtime.h>

#include "../../include/fea.h"
#include "fea_internal.h"

namespace fea {

namespace {

constexpr unsigned long long kGammaD = 0x9E3779B97F4A7C15ull;
constexpr unsigned long long kH0D = 0x243F6A8885A308D3ull;
constexpr int kChunk = FEA_BLOCK_TOKENS;
constexpr int kLeafTile = 2048;     // leaves staged per pass: 16 KB of LDS

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

// Lane c of (lo, hi) = x; x and c are wave-uniform.  Whichever unit wrote their registers: the scalar unit reads c (the lane
// must be in M0, two scalar sources are one too many), which the hardware orders, and a value the vector unit has just
// written wants two wait states before another vector instruction reads it, which the write of M0 and the s_nop are.
__device__ __forceinline__ void put_lane(int& lo, int& hi, unsigned long long x, int c) {
    asm("s_mov_b32 m0, %4\n\ts_nop 0\n\tv_writelane_b32 %0, %2, m0\n\tv_writelane_b32 %1, %3, m0"
        : "+v"(lo), "+v"(hi) : "s"((uint32_t)x), "s"((uint32_t)(x >> 32)), "s"(c) : "m0");
}

// Four neighbouring tokens, loadable from any 4-byte boundary.
struct __attribute__((packed, aligned(4))) Tok4 { uint32_t t[4]; };

// Bound: the chain, two mixing steps per chunk one after the other.  One wave runs it in scalar registers (a 64-bit
// product is six scalar instructions of one issue slot each; on the vector unit its multiplications take four slots
// each): a wave's worth of leaves is handed over lane by lane, the hashes are collected lane by lane and stored
// together.  64 requests of 4224 to 5120 tokens: 48.1 us with the chain in vector registers and through LDS, 34.0 now
// (87 ns a chunk; launch, tokens and leaves are the other 6 us).
constexpr int kHashThreads = 512;
__global__ __launch_bounds__(kHashThreads) void chunk_hash_kernel(HashArgs a) {
    __shared__ unsigned long long s_leaf[kLeafTile];
    const int i = blockIdx.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = a.tok_offsets[i], t1 = a.tok_offsets[i + 1];
    if (t0 < 0 || t1 < t0 || t1 > a.n_tokens) return;            // inconsistent offsets: the row is skipped
    const int64_t T = t1 - t0, C = (T + kChunk - 1) / kChunk;
    const int64_t h0 = a.hash_offsets[i];
    if (h0 < 0 || h0 + C > a.n_hashes) return;
    const int32_t* tok = a.tokens + t0;
    unsigned long long h = kH0D;                                  // carried by the first wave across tiles
    for (int64_t base = 0; base < C; base += kLeafTile) {
        const int n = __builtin_amdgcn_readfirstlane((int)(C - base < kLeafTile ? C - base : kLeafTile));
        for (int c = tid; c < n; c += kHashThreads) {             // parallel phase: independent leaves
            const int64_t first = (base + c) * kChunk;
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
            s_leaf[c] = x;
        }
        __syncthreads();
        if (wave == 0) {                                          // sequential phase: the chain
            h = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)h) |
                ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(h >> 32)) << 32);
            for (int c0 = 0; c0 < n; c0 += 64) {
                const unsigned long long leaf = c0 + tid < n ? s_leaf[c0 + tid] : 0ull;
                const int leaf_lo = (int)(uint32_t)leaf, leaf_hi = (int)(uint32_t)(leaf >> 32);
                int out_lo = 0, out_hi = 0;
                const int m = n - c0 < 64 ? n - c0 : 64;
                auto link = [&](int c) {
                    const unsigned long long x = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane(leaf_lo, c) |
                                                 ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane(leaf_hi, c) << 32);
                    h = mixd(mixd(h + kGammaD) ^ x);
                    put_lane(out_lo, out_hi, h, c);
                };
                if (m == 64) {
#pragma unroll 8
                    for (int c = 0; c < 64; ++c) link(c);
                } else {
                    for (int c = 0; c < m; ++c) link(c);
                }
                if (tid < m) a.hashes[h0 + base + c0 + tid] = (unsigned long long)(uint32_t)out_lo | ((unsigned long long)(uint32_t)out_hi << 32);
            }
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
