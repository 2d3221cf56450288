// Alias detection and work-list construction on the device (one workgroup).
//
// Reads only the block tables and lengths.  Requests whose table rows start with
// the same run of block ids form a group (the device-side sibling of the shared
// prefix tip of Section 4.2: the deepest level all members agree on); the run is
// swept once for the whole group, the remaining columns of each request are swept
// on their own.  A group is only a way to save KV reads: membership requires
// nothing but equal block ids over the run and full blocks for every member, so
// the result is the same attention whatever the tables look like.
//
// The sweeps are then laid end to end as one stream of 32-token tiles (shared
// runs first) and the stream is cut into equal shares, one per sweep wave, so
// that every wave moves the same number of KV bytes; a cut inside a segment just
// adds one partial result to it.  With an explicit split size the segments are
// cut every `split` blocks instead and the pieces dealt out in equal numbers.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <type_traits>

#include "fea_device.h"
#include "fea_plan.h"

namespace fea {

__device__ __forceinline__ int cdiv(int a, int b) { return (a + b - 1) / b; }

// Integer division by a run-time divisor without the ~40-instruction expansion:
// exact for 0 <= x < 2^24 and 1 <= d (row and request counts are far below that).
struct FastDiv {
    int d;
    float rcp;
    __device__ explicit FastDiv(int dd) : d(dd), rcp(1.0f / (float)dd) {}
    __device__ __forceinline__ int div(int x) const {
        int q = (int)((float)x * rcp);
        const int r = x - q * d;
        if (r >= d) ++q;
        if (r < 0) --q;
        return q;
    }
    __device__ __forceinline__ int cdiv(int x) const { return div(x + d - 1); }
};

// The same through double precision: exact for 0 <= x < 2^31 (tile positions).
struct WideDiv {
    int d;
    double rcp;
    __device__ explicit WideDiv(int dd) : d(dd), rcp(1.0 / (double)dd) {}
    __device__ __forceinline__ int div(int x) const {
        int q = (int)((double)x * rcp);
        const long long r = (long long)x - (long long)q * d;
        if (r >= d) ++q;
        if (r < 0) --q;
        return q;
    }
};

// floor(x / d) for 0 <= x < 2^52 and d >= 1 through double precision: the 64-bit
// integer division expands to hundreds of dependent instructions, which is felt in
// the serial stretches of a single-workgroup kernel.
__device__ __forceinline__ long long ddiv(long long x, int d) {
    long long q = (long long)((double)x / (double)d);
    const long long r = x - q * d;
    if (r >= d) ++q;
    if (r < 0) --q;
    return q;
}

// Sums and minima over the lanes of a wave in the vector unit's own lane shifts (a shift within a row of 16 lanes, then
// the last lane of a row, and of the lower half, handed on): a handful of instructions, where a shuffle through LDS would
// be a round trip per step.
template <int CTRL, int ROWS> __device__ __forceinline__ int lane_shift(int v, int other) {
    return __builtin_amdgcn_update_dpp(other, v, CTRL, ROWS, 0xF, false);   // lanes without a source: `other`
}
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += lane_shift<0x111, 0xF>(v, 0);
    v += lane_shift<0x112, 0xF>(v, 0);
    v += lane_shift<0x114, 0xF>(v, 0);
    v += lane_shift<0x118, 0xF>(v, 0);
    v += lane_shift<0x142, 0xA>(v, 0);
    v += lane_shift<0x143, 0xC>(v, 0);
    return v;
}
__device__ __forceinline__ float wave_sum(float x) {
    auto shifted = [](float v, auto ctrl, auto rows) {
        return __int_as_float(lane_shift<decltype(ctrl)::value, decltype(rows)::value>(__float_as_int(v), 0));
    };
    using std::integral_constant;
    x += shifted(x, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});
    x += shifted(x, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    x += shifted(x, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    x += shifted(x, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    x += shifted(x, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});
    x += shifted(x, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan_incl(v), 63); }
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    constexpr int kNone = -1;   // the largest value
    int v = (int)x;
    auto least = [](int p, int q) { return (int)min((uint32_t)p, (uint32_t)q); };
    v = least(v, lane_shift<0x111, 0xF>(v, kNone));
    v = least(v, lane_shift<0x112, 0xF>(v, kNone));
    v = least(v, lane_shift<0x114, 0xF>(v, kNone));
    v = least(v, lane_shift<0x118, 0xF>(v, kNone));
    v = least(v, lane_shift<0x142, 0xA>(v, kNone));
    v = least(v, lane_shift<0x143, 0xC>(v, kNone));
    return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}

// Prefix sums over the block in two levels: a wave's total into s_sums[wave] and, after a barrier, what the waves before this
// one have and what all have - the 16 totals once more by lane shifts, in the 16 lanes of a row (added up by every thread on
// its own they were 50 instructions, of all 16 waves).
__device__ __forceinline__ int waves_before(const int* s_sums, int& total) {
    static_assert(kPlanThreads / 64 == 16, "one total per lane of a row");
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int v = s_sums[threadIdx.x & 15];
    v += lane_shift<0x111, 0xF>(v, 0);
    v += lane_shift<0x112, 0xF>(v, 0);
    v += lane_shift<0x114, 0xF>(v, 0);
    v += lane_shift<0x118, 0xF>(v, 0);
    total = __builtin_amdgcn_readlane(v, 15);
    return wave == 0 ? 0 : __builtin_amdgcn_readlane(v, wave - 1);
}
// Exclusive prefix sum of one int per thread over the block, with one barrier.  `s_sums` must not be in use by another scan.
__device__ __forceinline__ int block_scan_excl(int v, int* s_sums, int& total) {
    const int x = wave_scan_incl(v);
    if ((threadIdx.x & 63) == 63) s_sums[threadIdx.x >> 6] = x;
    __syncthreads();
    return waves_before(s_sums, total) + x - v;
}

// Four neighbouring table columns, loadable from any 4-byte boundary.
struct __attribute__((packed, aligned(4))) Cols4 { int32_t c[4]; };

// Hash slots for n keys: 16 each up to 256 keys (a probe more is a serial round trip to LDS for a whole wave; with four each
// 1.3 us were lost where 120 keys are looked up; not all 4096 for a few keys, since all are cleared), then 4096 in all, which
// come down to two each at the limit of 2048.
__device__ __forceinline__ int slots_for(int n) {
    int slots = 512;
    while (slots < 16 * n && slots < kHashSlots) slots <<= 1;
    return slots;
}
__device__ __forceinline__ uint32_t slot_of(int key) { return ((uint32_t)key * 2654435761u) >> 20; }  // 12 bits

__device__ __forceinline__ void write_item(Item* it, int who, int g, int nrows, int mlist_off, int c0, int c1,
                                           int pbase, int tok_end) {
    int4* p = reinterpret_cast<int4*>(it);
    p[0] = make_int4(who, g, nrows, mlist_off);
    p[1] = make_int4(c0, c1, pbase, tok_end);
}

// Leaders and common runs for large tables, on many workgroups (the planner's one
// workgroup would pull every follower's and leader's row through a single CU: 71 of its
// 105 us for 800 requests of 10K tokens).  Every workgroup finds the leaders for itself
// (smallest request index per first block; a few thousand LDS operations), then its waves
// take followers in turn: 64 lanes x 4 columns per step, the first differing column and the
// follower's block there picked from the lowest lane that saw a difference.
__global__ __launch_bounds__(kRunThreads) void run_kernel(PlanArgs a) {
    __shared__ int keys[kHashSlots], vals[kHashSlots];
    __shared__ int s_len[kGroupReqMax];
    __shared__ short s_lead[kGroupReqMax];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nG = a.grouping ? min(a.B, kGroupReqMax) : 0;
    const int maxL = a.stride * kBlock;
    constexpr int kPer = kGroupReqMax / kRunThreads;
    const int slots = slots_for(nG);
    const uint32_t slot_mask = (uint32_t)slots - 1;
    int my_key[kPer], my_len[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {       // lengths and first blocks are on their way while the table is cleared
        const int i = tid + k * kRunThreads;
        my_len[k] = 0;
        my_key[k] = -1;
        if (i < nG && maxL > 0) {
            my_len[k] = a.seq_lens[i];
            my_key[k] = a.bt[(size_t)i * a.stride];
        }
    }
    for (int s = tid; s < slots; s += kRunThreads) { keys[s] = -1; vals[s] = INT_MAX; }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = tid + k * kRunThreads;
        if (i < nG) {
            const int L = max(0, min(my_len[k], maxL));
            s_len[i] = L;
            if (L < kBlock) my_key[k] = -1;
            const int key = my_key[k];
            if (key >= 0) {
                uint32_t s = slot_of(key) & slot_mask;
                for (;;) {
                    const int old = atomicCAS(&keys[s], -1, key);
                    if (old == -1 || old == key) { atomicMin(&vals[s], i); break; }
                    s = (s + 1) & slot_mask;
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = tid + k * kRunThreads;
        if (i < nG) {
            int lead = -1;
            const int key = my_key[k];
            if (key >= 0) {
                uint32_t s = slot_of(key) & slot_mask;
                while (keys[s] != key) s = (s + 1) & slot_mask;
                lead = vals[s];
            }
            s_lead[i] = (short)lead;
        }
    }
    __syncthreads();
    unsigned long long* pre = reinterpret_cast<unsigned long long*>(a.ws + a.lay.pre);
    int* pre_lead = reinterpret_cast<int*>(pre + kGroupReqMax);
    const int waves = gridDim.x * (kRunThreads / 64);
    for (int i = blockIdx.x * (kRunThreads / 64) + (tid >> 6); i < nG; i += waves) {
        const int lead = s_lead[i];
        const int cp = lead >= 0 ? min(s_len[i], s_len[lead]) / kBlock : 0;
        unsigned long long res = ((unsigned long long)(uint32_t)cp << 32) | 0xFFFFFFFFull;
        if (lead >= 0 && lead != i) {
            const int32_t* ri = a.bt + (size_t)i * a.stride;
            const int32_t* rl = a.bt + (size_t)lead * a.stride;
            constexpr int kWin = 4;   // column windows (64 lanes x 4 columns) requested together
            bool done = false;
            for (int c0 = 0; c0 < cp && !done; c0 += 256 * kWin) {
                int4 x[kWin], y[kWin];
#pragma unroll
                for (int u = 0; u < kWin; ++u) {
                    const int c = c0 + u * 256 + lane * 4;
                    x[u] = y[u] = make_int4(0, 0, 0, 0);
                    if (c < cp) {
                        if (c + 4 <= a.stride) {
                            const Cols4 xv = *reinterpret_cast<const Cols4*>(ri + c), yv = *reinterpret_cast<const Cols4*>(rl + c);
                            x[u] = make_int4(xv.c[0], xv.c[1], xv.c[2], xv.c[3]);
                            y[u] = make_int4(yv.c[0], yv.c[1], yv.c[2], yv.c[3]);
                        } else {
                            const bool two = c + 1 < a.stride, three = c + 2 < a.stride;
                            x[u] = make_int4(ri[c], two ? ri[c + 1] : 0, three ? ri[c + 2] : 0, 0);
                            y[u] = make_int4(rl[c], two ? rl[c + 1] : 0, three ? rl[c + 2] : 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < kWin; ++u) {
                    const int c = c0 + u * 256 + lane * 4;
                    int first = INT_MAX, mine = 0;
                    if (x[u].w != y[u].w) { first = c + 3; mine = x[u].w; }
                    if (x[u].z != y[u].z) { first = c + 2; mine = x[u].z; }
                    if (x[u].y != y[u].y) { first = c + 1; mine = x[u].y; }
                    if (x[u].x != y[u].x) { first = c; mine = x[u].x; }
                    const unsigned long long seen = __ballot(!done && first < cp);
                    if (seen) {   // lanes hold rising columns: the lowest lane has the first difference
                        const int src = __ffsll((long long)seen) - 1;
                        const int f0 = __shfl(first, src), m0 = __shfl(mine, src);
                        res = ((unsigned long long)(uint32_t)f0 << 32) | (uint32_t)m0;
                        done = true;
                    }
                }
            }
        }
        if (lane == 0) { pre[i] = res; pre_lead[i] = lead; }
    }
}

// What the planner's launch does besides: its workgroup keeps one compute unit busy, and next to nothing of the memory, for 13 us
// and more.  Others meanwhile read the ends of the histories - the part that is hardly ever shared, which the sweep therefore
// takes from memory - and throw away what they read: the sweep then finds it nearer.  Whole tiles of every history, as many as come
// nearest to 28 MB (where there are tiles small enough to choose: 16 MB gain half as much, 48 no more, and take longer than the planner
// where it is quick).  One tile of a large batch is up to 56 MB: 300 to 420 requests of 8 KV heads, or 600 to 840 of 4, take 0.957 to 0.983
// of a call's time with it (16 shapes of head_dim 128), 500 to 840 of 8 at head_dim 64 0.964 to 1.001 (9).  The launch ends, and the
// sweep starts, when all of them have; they write nothing but a word of the header.
//  - Half of the compute units do it: 1.00 of a call's time where there is nothing to read (all of them 1.003, 0.1 to 0.5 us for
//    their start), and as much gained.
//  - They wait 2400 cycles first: the planner reads its tables then, and waits for them.
//  - They do it if half of the requests that share a run with one of theirs (of 32 looked at) have `own` columns and more behind what
//    they share, 60 MB in all if they are alike: where much less is read for the first time by the sweep, or nothing is shared (the
//    planner is done at once then, 64 requests of 4224 to 5120 tokens 229 -> 234 us), there is little to gain.
// 64 requests on one prefix of 4096, 32/8/128: 50.1 -> 48.1 us a call; 128 of head_dim 64 in 8 groups 49.7 -> 47.3, 32 on one of 32K
// 67.0 -> 64.0; after run_kernel 256 in 8 groups on 4096 155.1 -> 151.5, 240 of 16/2/128 73.2 -> 70.0, 400 of 8/2/64 the same.  80
// drawn shapes that share runs, while the sweep's own loads stayed in the caches: 0.986 of the time (nine sets of caches in turn 0.97).
constexpr int kAheadMB = 28, kOwnMB = 60, kAheadSample = 32;
__device__ __forceinline__ void read_ahead(const PlanArgs& a) {
    __shared__ int s_go;
    constexpr int kWaves = kPlanThreads / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    __builtin_amdgcn_s_sleep(38);          // (of 64 cycles)
    if (wave == 0) {
        const int i = blockIdx.x % a.B, other = (i + 1 + (lane % kAheadSample)) % a.B;
        const int32_t* row = a.bt + (size_t)i * a.stride;
        const int32_t* peer = a.bt + (size_t)other * a.stride;
        const int L = max(0, min(a.seq_lens[other], a.stride * kBlock)), at = (L + kBlock - 1) / kBlock - 1 - a.own;
        const bool shares = lane < kAheadSample && other != i && peer[0] == row[0], apart = shares && at >= 1 && peer[max(at, 0)] != row[max(at, 0)];
        const int all = __popcll(__ballot(shares)), n = __popcll(__ballot(apart));
        if (lane == 0) s_go = all > 0 && 2 * n >= all;
    }
    __syncthreads();
    if (!s_go) return;
    if (threadIdx.x == 0) reinterpret_cast<int*>(a.ws)[H_AHEAD] = a.ahead;
    const int units = a.B * a.Hkv;
    for (int w = (blockIdx.x - 1) * kWaves + wave; w < units * a.ahead; w += (gridDim.x - 1) * kWaves) {
        const int t = w / units, u = w - t * units, i = u / a.Hkv, g = u - i * a.Hkv;
        const int32_t* row = a.bt + (size_t)i * a.stride;
        const int L = max(0, min(a.seq_lens[i], a.stride * kBlock)), c1 = (L + kBlock - 1) / kBlock - 1 - 2 * t;
        if (c1 < 1) continue;
        const size_t at0 = ((size_t)max(row[c1 - 1], 0) * a.Hkv + g) * a.block_bytes, at1 = ((size_t)max(row[c1], 0) * a.Hkv + g) * a.block_bytes;
        const char* k = static_cast<const char*>(a.k_cache);
        const char* v = static_cast<const char*>(a.v_cache);
        const char* from[4] = {k + at0, k + at1, v + at0, v + at1};
        for (int at = 0; at < a.block_bytes; at += 2048) {     // (head_dim 64: 2 KB a block)
            u32x4 x[4][2];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int j = 0; j < 2; ++j) x[b][j] = ld16(from[b] + at + 1024 * j + 16 * lane);
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int j = 0; j < 2; ++j) asm volatile("" :: "v"(x[b][j]));
        }
    }
}

constexpr int kSegmentTiles = 1;              // tiles that a further segment of a share costs
constexpr int kGroupMax = kGroupReqMax / 2;   // a group has at least two members

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(PlanArgs a) {
    static_assert(kHashSlots == 4096, "slot_of() yields 12 bits");
    __shared__ union {
        struct { int keys[kHashSlots]; int vals[kHashSlots]; } h;                     // leader finding only
        struct { int run[kGroupReqMax]; int cnt[kGroupReqMax]; int moff[kGroupReqMax];
                 int gseg[kGroupMax]; } c;                                            // afterwards
    } u;
    __shared__ struct { int keys[kHashSlots]; int vals[kHashSlots]; } h2;             // subgroup leaders (nested runs)
    __shared__ unsigned short s_r1[kGroupReqMax];
    __shared__ unsigned long long s_lcpv[kGroupReqMax];   // round one: (common run << 32) | the follower's block where it ends
    __shared__ short s_lead[kGroupReqMax];      // request ids fit 16 bits (kGroupReqMax <= 32767)
    __shared__ int s_len[kGroupReqMax];
    __shared__ union {
        struct { int lcp[kGroupReqMax]; short lead2[kGroupReqMax]; } x;   // until the group runs are known
        struct { int npc[kGroupMax]; int ibase[kGroupMax]; int rbase[kGroupMax]; } g;   // then the cut of each group
    } v;
    __shared__ union {
        unsigned short flw[kGroupReqMax];       // followers (grouped, not leader), for the run detection
        unsigned short glist[kGroupMax];        // then the list of viable leaders
    } w;
    __shared__ __attribute__((aligned(16))) int s_sums[4][kPlanThreads / 64];
    __shared__ int s_ngroups, s_ngrouped, s_shared_blocks, s_nflw, s_nest, s_adopt, s_alike, s_longest[kPlanThreads / 64];

    if (blockIdx.x > 0) { read_ahead(a); return; }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int* hdr = reinterpret_cast<int*>(a.ws);
    ReqDesc* req = reinterpret_cast<ReqDesc*>(a.ws + a.lay.req);
    GroupDesc* grp = reinterpret_cast<GroupDesc*>(a.ws + a.lay.grp);
    int* members = reinterpret_cast<int*>(a.ws + a.lay.members);
    SegDesc* segs = reinterpret_cast<SegDesc*>(a.ws + a.lay.segs);
    int* wave_first = reinterpret_cast<int*>(a.ws + a.lay.wave_first);
    Item* items = reinterpret_cast<Item*>(a.ws + a.lay.items);

    const int B = a.B, Hkv = a.Hkv;
    const int nG = a.grouping ? min(B, kGroupReqMax) : 0;
    const int maxL = a.stride * kBlock;
    auto clampL = [&](int L) { return max(0, min(L, maxL)); };

    int my_key[kGroupReqMax / kPlanThreads], my_longest = 0;
    const int slots = slots_for(nG);
    const uint32_t slot_mask = (uint32_t)slots - 1;
    int my_len[kGroupReqMax / kPlanThreads];
    if (!a.pre) {   // lengths and first blocks are on their way while the tables are cleared
#pragma unroll
        for (int k = 0; k < kGroupReqMax / kPlanThreads; ++k) {
            const int i = tid + k * kPlanThreads;
            my_len[k] = 0;
            my_key[k] = -1;
            if (i < nG && maxL > 0) {
                my_len[k] = a.seq_lens[i];
                my_key[k] = a.bt[(size_t)i * a.stride];
            }
        }
    }
    for (int s = tid; s < slots; s += kPlanThreads) { h2.keys[s] = -1; h2.vals[s] = INT_MAX; }
    if (tid == 0) { s_ngroups = 0; s_ngrouped = 0; s_shared_blocks = 0; s_nflw = 0; s_alike = 0; }
    if (a.pre) {
        __syncthreads();   // (s_nflw is zero)
        // ---- leaders and common runs were found by run_kernel
        const unsigned long long* pre = reinterpret_cast<const unsigned long long*>(a.ws + a.lay.pre);
        const int* pre_lead = reinterpret_cast<const int*>(pre + kGroupReqMax);
        for (int i = tid; i < nG; i += kPlanThreads) {
            s_len[i] = clampL(a.seq_lens[i]);
            s_lead[i] = (short)pre_lead[i];
            s_lcpv[i] = pre[i];
            if (pre_lead[i] >= 0 && pre_lead[i] != i) s_nflw = 1;   // (here only whether there is any)
        }
        __syncthreads();
    } else {
        // ---- leaders: smallest request index among those with the same first block
        for (int s = tid; s < slots; s += kPlanThreads) { u.h.keys[s] = -1; u.h.vals[s] = INT_MAX; }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kGroupReqMax / kPlanThreads; ++k) {
            const int i = tid + k * kPlanThreads;
            if (i < nG) {
                const int L = clampL(my_len[k]);
                s_len[i] = L;
                my_longest = max(my_longest, L);
                if (L < kBlock) my_key[k] = -1;
                const int key = my_key[k];
                if (key >= 0) {
                    uint32_t s = slot_of(key) & slot_mask;
                    for (;;) {
                        const int old = atomicCAS(&u.h.keys[s], -1, key);
                        if (old == -1 || old == key) { atomicMin(&u.h.vals[s], i); break; }
                        s = (s + 1) & slot_mask;
                    }
                }
            }
        }
        my_longest = ~(int)wave_min(~(uint32_t)my_longest);
        if (lane == 0) s_longest[wave] = my_longest;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kGroupReqMax / kPlanThreads; ++k) {
            const int i = tid + k * kPlanThreads;
            if (i < nG) {
                int lead = -1, lcp = 0;
                const int key = my_key[k];
                if (key >= 0) {
                    uint32_t s = slot_of(key) & slot_mask;
                    while (u.h.keys[s] != key) s = (s + 1) & slot_mask;
                    lead = u.h.vals[s];
                    lcp = min(s_len[i], s_len[lead]) / kBlock;
                    if (lead != i) w.flw[atomicAdd(&s_nflw, 1)] = (unsigned short)i;
                }
                s_lead[i] = (short)lead;
                s_lcpv[i] = ((unsigned long long)(uint32_t)lcp << 32) | 0xFFFFFFFFull;
            }
        }
        __syncthreads();   // the hash table is dead from here on; its memory becomes run/cnt/moff/...
    }
    // ---- nothing shared (no two requests with the same first block), and much of it: no plan.  The sweep reads whole histories,
    // a workgroup one at a time, longest first, and whoever is done takes the next: shares cut beforehand end as far apart as
    // the XCDs' rates differ (10 %).  Needs no order among equals, so the requests are put into 64 classes of length.
    if (__builtin_expect(a.histories > 0 && s_nflw == 0, 0)) {
        __shared__ int s_class[64];
        if (tid < 64) s_class[tid] = 0;
        int longest = 0, tiles = 0;
        for (int i = tid; i < B; i += kPlanThreads) {
            longest = max(longest, s_len[i]);
            tiles += (s_len[i] + 2 * kBlock - 1) / (2 * kBlock);
        }
        longest = ~(int)wave_min(~(uint32_t)longest);
        tiles = wave_sum(tiles);
        if (lane == 0) { s_sums[0][wave] = longest; s_sums[1][wave] = tiles; }
        __syncthreads();
        longest = ~(int)wave_min(~(uint32_t)s_sums[0][lane & 15]);
        waves_before(s_sums[1], tiles);
        // (enough for every wave, no history that alone takes longer than everything does on average, and none so short that
        // its start - 6 us until its first tile is there - counts)
        if ((long long)tiles * Hkv >= max((long long)a.histories, (long long)((longest + 2 * kBlock - 1) / (2 * kBlock)) * (a.tune.n_waves / 4)) &&
            tiles >= (long long)a.histories_each * B) {
            const float per_class = 64.f / (float)(longest + 1);
            int cls[kGroupReqMax / kPlanThreads], at[kGroupReqMax / kPlanThreads];
#pragma unroll
            for (int k = 0; k < kGroupReqMax / kPlanThreads; ++k) {
                const int i = tid + k * kPlanThreads;
                if (i < B) {
                    cls[k] = 63 - min(63, (int)((float)s_len[i] * per_class));
                    at[k] = atomicAdd(&s_class[cls[k]], 1);
                }
            }
            __syncthreads();
            const int mine = s_class[lane], before = wave_scan_incl(mine) - mine;   // (of class `lane`, in every wave)
            __shared__ int s_first[64];
            if (wave == 0) s_first[lane] = before;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kGroupReqMax / kPlanThreads; ++k) {
                const int i = tid + k * kPlanThreads;
                if (i < B) members[s_first[cls[k]] + at[k]] = i;
            }
            if (tid < H_WORDS) {
                const int units = B * Hkv;
                hdr[tid] = tid == H_ITEMS ? units : tid == H_SPLIT ? (longest + kBlock - 1) / kBlock : tid == H_VARIANT ? kHistories
                         : tid == H_WAVES ? a.tune.n_waves : tid == H_CAPACITY ? a.lay.max_items : tid == H_HISTORIES ? 1 : 0;
            }
            return;
        }
    }
    auto reset_groups = [&](int moff0) {
        for (int i = tid; i < nG; i += kPlanThreads) { u.c.run[i] = INT_MAX; u.c.cnt[i] = 0; u.c.moff[i] = moff0; }
    };
    reset_groups(0);
    // (where the runs are already known no other barrier stands between what is read and written above - whether anything is
    // shared, which thread 0 clears below, and the groups' words, which the first round below counts in - and there)
    if (a.pre) __syncthreads();

    // ---- longest common run of block ids with the leader's row.  All (follower,
    // column group) pairs are spread flat over the threads, six at a time so that
    // their loads are in flight together; a mismatch lowers the follower's run with
    // an LDS atomic.  Columns below from(i) are known to agree and are not read, and columns past the
    // longest history are not looked at (a table is often as wide as the longest history that is allowed) - but
    // where run_kernel has found the runs, the search for nested ones goes over the table's width.
    int columns = a.stride;
    if (!a.pre) {
        columns = ~(int)wave_min(~(uint32_t)s_longest[lane & 15]) / kBlock;
    }
    auto lcp_pass = [&](int nflw, const short* lead_of, auto&& from, auto&& hit) {
        constexpr int cpe = 4;                             // columns per element
        const int epr = cdiv(columns, cpe);                // elements per row (the last one may be short)
        const FastDiv by_epr(max(epr, 1));
        const int total = nflw * epr;
        constexpr int kBatch = 6;
        for (int e0 = tid; e0 < total; e0 += kBatch * kPlanThreads) {
            int4 xs[kBatch], ys[kBatch];
            int who[kBatch], col[kBatch], cap[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int e = e0 + q * kPlanThreads;
                who[q] = -1;
                if (e < total) {
                    const int f = by_epr.div(e);
                    const int i = w.flw[f];
                    const int lead = lead_of[i];
                    const int c = (e - f * epr) * cpe;
                    const int cp = min(s_len[i], s_len[lead]) / kBlock;   // the starting value of lcp[i]
                    if (c < cp && c + cpe > from(i)) {
                        who[q] = i; col[q] = c; cap[q] = cp;
                        const int32_t* ri = a.bt + (size_t)i * a.stride + c;
                        const int32_t* rl = a.bt + (size_t)lead * a.stride + c;
                        if (c + cpe <= a.stride) {          // rows need not start on 16-byte boundaries
                            const Cols4 x = *reinterpret_cast<const Cols4*>(ri), y = *reinterpret_cast<const Cols4*>(rl);
                            xs[q] = make_int4(x.c[0], x.c[1], x.c[2], x.c[3]);
                            ys[q] = make_int4(y.c[0], y.c[1], y.c[2], y.c[3]);
                        } else {                            // the row's last, short element
                            const bool two = c + 1 < a.stride, three = c + 2 < a.stride;
                            xs[q] = make_int4(ri[0], two ? ri[1] : 0, three ? ri[2] : 0, 0);
                            ys[q] = make_int4(rl[0], two ? rl[1] : 0, three ? rl[2] : 0, 0);
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                if (who[q] >= 0) {
                    int first = INT_MAX, mine = 0;
                    if (xs[q].w != ys[q].w) { first = col[q] + 3; mine = xs[q].w; }
                    if (xs[q].z != ys[q].z) { first = col[q] + 2; mine = xs[q].z; }
                    if (xs[q].y != ys[q].y) { first = col[q] + 1; mine = xs[q].y; }
                    if (xs[q].x != ys[q].x) { first = col[q]; mine = xs[q].x; }
                    if (first < cap[q]) hit(who[q], first, mine);
                }
            }
        }
    };
    auto note_run_end = [&](int who, int first, int mine) {   // the run and the follower's block that ends it
        atomicMin(&s_lcpv[who], ((unsigned long long)(uint32_t)first << 32) | (uint32_t)mine);
    };
    if (!a.pre) {
        lcp_pass(s_nflw, s_lead, [](int) { return 0; }, note_run_end);
        __syncthreads();
    }

    // A 32-token tile costs a wave more the more query rows ride on it: weights in
    // sixteenths of a 16-row tile's sweep.
    const int w32 = a.tune.weights & 255, w64 = (a.tune.weights >> 8) & 255;
    auto tile_weight = [&](int rows) { return rows <= 16 ? 16 : (rows <= 32 ? w32 : w64); };
    const FastDiv by_mpt(a.mpt);
    bool split_off = false;   // groups have split off groups, which sweep the outer run again
    // Row tiles of one piece of a shared run read the same KV bytes.  On the matrix-core path the sweep
    // runs them as a team of 2 or 4 waves of one workgroup that fetches every tile once; for that the
    // row tiles of a piece sit on neighbouring shares, in slots of 1, 2 or a multiple of 4 (the slots
    // past the last row tile hold waves that only help fetching), and every group starts on a multiple of 4.
    const bool teams = a.teams != 0 && a.split_user == 0;   // (with a fixed split a share holds several items: no teams)
    auto tiles_padded = [&](int tiles_r) { return (!teams || tiles_r <= 2) ? tiles_r : ((tiles_r + 3) & ~3); };
    auto items_padded = [&](int n) { return teams ? ((n + 3) & ~3) : n; };
    // cost of one 32-token tile of a shared run per wave that sweeps it, for a group of cnt members: a team
    // fetches the tile once for all its row tiles and overlaps the two products, which makes the tile far
    // cheaper for a wave than a tile it streams and sweeps alone
    // (a team of 2 fetches half of every tile per wave, a team of 4 a quarter.  Both 12 sixteenths.  With 10 for a team of 4 the
    // cuts move and with them what weights are rounded against: outputs of 64 requests on 4096, 32/8/128, differ by 0.003, as far
    // from float64 as before, in the same time - 48.6 to 49.3 us, 48.6 to 49.9 with 12 -, 240 of 16/2/128 in 4 groups 72.0 -> 69.6,
    // 500 on one of 10240 167 to 173, 165 to 173 with 12)
    const int w_team = (a.tune.weights >> 16) & 255, w_team2 = (a.tune.weights >> 24) & 127;
    auto group_weight = [&](int cnt) {
        const int tiles_r = by_mpt.cdiv(cnt);
        return (teams && tiles_r >= 2) ? (tiles_r == 2 ? w_team2 : w_team) : tile_weight(min(a.mpt, cnt) * a.G);
    };
    // ... and what a piece costs the two waves of a small team besides its tiles: they fill the table of block ids
    // and the ring before the first tile, and drain it after the last, with half the lanes a team of 4 has for it
    // (measured: 32 requests on one 4096-token prefix 26.2 -> 24.6 us; with the same charge on teams of 4, whose
    // pieces it shortens as well, the 64-request batch lost 0.5 us to the merge of the extra pieces)
    auto group_fixed = [&](int cnt) { return (teams && by_mpt.cdiv(cnt) == 2) ? a.tune.team_fixed : 0; };

    // ---- nested prefixes.  Members of a group may go on sharing blocks past the group's
    // run (a common system prompt, then a few conversations: the radix patterns of
    // Section 3).  A second round finds, inside every group, the members that carry the
    // same block in the first column after the run, and their common run from there.
    // Such a subgroup becomes a group of its own (run measured from column 0, so it sweeps
    // the outer run again) when that saves more sweep cost than it adds, by the tile weights;
    // the members left behind keep the outer run under the smallest index among them.
    //
    // A follower agrees with its leader over lcp >= run columns.  If lcp > run it is in the
    // leader's subgroup and its run there is lcp itself; if lcp == run, the block that
    // tells its subgroup sits in column lcp - the very entry the run detection stopped at,
    // which it hands over together with the column (no further memory round trip).
    // Stage by stage: (1) runs, sizes (and, the first time, ranks) of the groups as they
    // are; (2) keys into a hash table of their own; (3) subgroup leaders.  With nothing
    // nested that is all (two barriers more than without this stage) and the results of
    // (1) stand.  Otherwise the subgroups' runs are measured and the ones that pay split
    // off; those are looked at again (a further level of sharing), kMaxLevels times at most.
    // Members left behind, and subgroups that stay, are final.
    constexpr int kPer = kGroupReqMax / kPlanThreads;
    constexpr int kMaxLevels = 4;
    int my_rank[kPer];
    {
        int lead1[kPer];
        bool act[kPer];          // still part of a group that may split further
        bool regroup = false;    // groups changed after the first stage (1): stats and ranks are redone
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + k * kPlanThreads;
            lead1[k] = i < nG ? (int)s_lead[i] : -1;
            act[k] = lead1[k] >= 0;
            my_rank[k] = 0;
        }
        for (int level = 0; level < kMaxLevels; ++level) {
            int r1[kPer], lcp1[kPer];
            bool in[kPer];
            if (tid == 0) { s_nflw = 0; s_nest = 0; s_adopt = 0; }
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int i = tid + k * kPlanThreads;
                lcp1[k] = 0;
                my_key[k] = -1;
                if (act[k]) {
                    const unsigned long long lv = s_lcpv[i];
                    lcp1[k] = (int)(lv >> 32);
                    v.x.lcp[i] = lcp1[k];
                    if (lead1[k] != i && lcp1[k] < s_len[i] / kBlock) {
                        // the block in the column where the follower left its leader: the run detection saw
                        // it, unless the leader's row simply ended there
                        my_key[k] = (uint32_t)lv != 0xFFFFFFFFu ? (int)(uint32_t)lv : a.bt[(size_t)i * a.stride + lcp1[k]];
                    }
                    atomicMin(&u.c.run[lead1[k]], lcp1[k]);
                    const int rank = atomicAdd(&u.c.cnt[lead1[k]], 1);
                    if (level == 0) my_rank[k] = rank;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                in[k] = act[k] && u.c.cnt[lead1[k]] >= 2 && u.c.run[lead1[k]] >= a.tune.min_run;
                r1[k] = in[k] ? u.c.run[lead1[k]] : 0;
                if (!in[k] || lcp1[k] > r1[k]) my_key[k] = -1;      // only the members that leave the leader at the run
                const int key = my_key[k];
                if (key >= 0) {
                    uint32_t s = slot_of(key) & slot_mask;
                    for (;;) {
                        const int old = atomicCAS(&h2.keys[s], -1, key);
                        if (old == -1 || old == key) { atomicMin(&h2.vals[s], tid + k * kPlanThreads); break; }
                        s = (s + 1) & slot_mask;
                    }
                }
            }
            __syncthreads();
            int lead2[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int i = tid + k * kPlanThreads;
                lead2[k] = -1;
                const int key = my_key[k];
                if (key >= 0) {
                    uint32_t s = slot_of(key) & slot_mask;
                    while (h2.keys[s] != key) s = (s + 1) & slot_mask;
                    const int cand = h2.vals[s];
                    lead2[k] = s_lead[cand] == lead1[k] ? cand : i;     // only within the same outer group
                    s_lcpv[i] = ((unsigned long long)(uint32_t)(min(s_len[i], s_len[lead2[k]]) / kBlock) << 32) | 0xFFFFFFFFull;
                    if (lead2[k] != i) w.flw[atomicAdd(&s_nflw, 1)] = (unsigned short)i;
                } else if (in[k] && (lead1[k] == i || lcp1[k] > r1[k])) {
                    lead2[k] = lead1[k];                                // the leader's own subgroup: runs are known
                    if (lead1[k] != i) atomicAdd(&s_nest, 1);
                }
                if (i < nG) { v.x.lead2[i] = (short)lead2[k]; s_r1[i] = (unsigned short)min(r1[k], 65535); }
            }
            __syncthreads();
            const int nflw2 = s_nflw;
            if (nflw2 + s_nest == 0) break;            // uniform: nothing (more) is nested
            regroup = true;
            if (nflw2 > 0) {
                lcp_pass(nflw2, v.x.lead2, [&](int i) { return (int)s_r1[i]; }, note_run_end);
                __syncthreads();
            }
            reset_groups(INT_MAX);
            __syncthreads();
            int lcp2[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {           // runs and sizes of the subgroups
                const int i = tid + k * kPlanThreads;
                lcp2[k] = 0;
                if (lead2[k] >= 0) {
                    lcp2[k] = (int)(s_lcpv[i] >> 32);
                    atomicMin(&u.c.run[lead2[k]], lcp2[k]);
                    atomicAdd(&u.c.cnt[lead2[k]], 1);
                }
            }
            __syncthreads();
            bool adopt[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                adopt[k] = false;
                if (lead2[k] >= 0) {
                    const int c2 = u.c.cnt[lead2[k]], run2 = u.c.run[lead2[k]];
                    // private sweeps saved plus the outer group's relief against the subgroup's own sweep
                    const long long gain = 16ll * c2 * (run2 - r1[k]) + (long long)r1[k] * group_weight(2 * a.mpt) * by_mpt.div(c2);
                    const long long cost = (long long)run2 * group_weight(c2) * by_mpt.cdiv(c2);
                    adopt[k] = c2 >= 2 && gain > cost;
                    if (adopt[k] && lead2[k] == tid + k * kPlanThreads) atomicAdd(&s_adopt, 1);
                    if (!adopt[k] && c2 >= 2 && run2 > r1[k]) s_alike = 1;   // (of their own columns some are the same)
                }
                if (in[k] && !adopt[k]) atomicMin(&u.c.moff[lead1[k]], tid + k * kPlanThreads);   // who leads the rest
            }
            __syncthreads();
            int lead_f[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) lead_f[k] = adopt[k] ? lead2[k] : (in[k] ? u.c.moff[lead1[k]] : lead1[k]);
            const bool again = s_adopt > 0 && level + 1 < kMaxLevels;
            split_off = split_off || s_adopt > 0;
            if (s_adopt > 0 && level + 1 == kMaxLevels && tid == 0) s_alike = 1;   // (not looked at)
            __syncthreads();                           // every leader is read before any changes
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int i = tid + k * kPlanThreads;
                if (in[k]) {
                    s_lead[i] = (short)lead_f[k];
                    v.x.lcp[i] = adopt[k] ? lcp2[k] : r1[k];
                }
                lead1[k] = lead_f[k];
                act[k] = adopt[k];
            }
            if (!again) break;                         // uniform
            // the groups that split off are looked at again, with clean tables
            for (int s = tid; s < slots; s += kPlanThreads) { h2.keys[s] = -1; h2.vals[s] = INT_MAX; }
            reset_groups(0);   // every thread changed only its own requests' entries above
            __syncthreads();
        }
        if (regroup) {
            __syncthreads();
            reset_groups(0);
            __syncthreads();
            // runs, sizes and ranks of the groups as they are now
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int i = tid + k * kPlanThreads;
                my_rank[k] = 0;
                if (i < nG) {
                    const int lead = s_lead[i];
                    if (lead >= 0) {
                        atomicMin(&u.c.run[lead], v.x.lcp[i]);
                        my_rank[k] = atomicAdd(&u.c.cnt[lead], 1);
                    }
                }
            }
            __syncthreads();
        }
    }
    // lcp[] and flw[] are dead from here on; run/cnt hold every group's run (the shortest
    // common run over its members) and size, my_rank the arrival at the group's counter
    // A run swept by teams is cut to an even number of columns (tiles are two columns; a piece with a column left
    // over is not taken by a team, and the waves that sweep it on their own hold up the team they share a
    // workgroup with).  The members read the column left over with their own ones, out of L2 after the first.
    if (teams) {
        for (int i = tid; i < nG; i += kPlanThreads)
            if (s_lead[i] == i && u.c.cnt[i] > a.mpt) u.c.run[i] &= ~1;
        __syncthreads();
    }
    auto viable = [&](int i) { return s_lead[i] == i && u.c.cnt[i] >= 2 && u.c.run[i] >= a.tune.min_run; };

    // ---- member-list offsets (exclusive scan over leaders) and the list of groups; and, for the cost model below, the
    // private stream: request i owns Hkv * priv_units(i) consecutive units (its tiles and its charge), KV head by KV head.  Its segments (request,
    // KV head) are the entries the threads share out, so that a batch of few requests still spreads over many lanes.
    auto run_of = [&](int i) {   // shared columns of request i (0 if ungrouped)
        if (i >= nG) return 0;
        const int lead = s_lead[i];
        return (lead >= 0 && viable(lead)) ? u.c.run[lead] : 0;
    };
    auto len_of = [&](int i) { return i < nG ? s_len[i] : clampL(a.seq_lens[i]); };
    // What a segment is to the wave that sweeps it, in tiles (per KV head): its tiles, and the change to another request
    // (query rows, the first tile's way through the pipeline, the partial rows).  Measured, per segment more in a share:
    // 1.2 us at head_dim 64 and 128, 2.4 at 256, where a tile takes 0.9, 1.5 to 1.9 and 1.65.  Shares cut by tiles alone
    // ended that much apart (22 to 32 us in a batch of head_dim 64, 22 to 27 since), and the batch ends with the last.
    // One tile charged against none, attention under a reused plan, mean over 1500 shapes: head_dim 64 0.95 of the time
    // where something is shared and 0.99 where nothing is, 256 0.93 and 0.99, 128 0.98 and 0.99.  Not charged
    //  - at head_dim 128 where the requests share runs and have less than a tile of their own for every wave: the shares of the
    //    runs, which teams sweep, come out longer for the sake of private ones that hardly count (up to 1.24 times the time, in
    //    the mean the same);
    //  - where nothing is shared and every wave has 24 tiles or more: memory binds such a stream whatever the shares (0.995 in
    //    the mean), and even ones do better (sweep of 64 requests of 4224 to 5120 tokens, 32/8/128, 236 against 231 us; 512 of
    //    512 to 4096, 64/8/128, 897 against 890; with 4 to 8 tiles to a wave the charge takes 0.98 of the time).
    auto priv_tiles = [&](int i) { return ((((len_of(i) + kBlock - 1) / kBlock) - run_of(i)) + 1) >> 1; };
    const int NE = B * Hkv;
    const int per = (NE + kPlanThreads - 1) / kPlanThreads;
    const int e0 = tid * per, e1 = min(NE, e0 + per);
    const FastDiv by_hkv(Hkv);
    int T_pr, tbase, segs_pr, per_seg;    // units of the private stream, those before the thread's first segment, segments that have any, a segment's charge
    {
        const int per_lead = (nG + kPlanThreads - 1) / kPlanThreads;   // 0, 1 or 2
        const int i0 = tid * per_lead, i1 = min(nG, i0 + per_lead);
        int local = 0, lt = 0, ls = 0;
        for (int i = i0; i < i1; ++i)
            if (viable(i)) local += u.c.cnt[i];
        for (int e = e0, seen = -1, t = 0; e < e1; ++e) {     // (neighbouring segments mostly are one request's)
            const int i = by_hkv.div(e);
            if (i != seen) { seen = i; t = priv_tiles(i); }
            lt += t;
            ls += t > 0 ? 1 : 0;
        }
        const int tiles_in_wave = wave_scan_incl(lt), segs_in_wave = wave_scan_incl(ls);   // (the scans share the one barrier)
        if (lane == 63) { s_sums[1][wave] = tiles_in_wave; s_sums[3][wave] = segs_in_wave; }
        int total;
        int base = block_scan_excl(local, s_sums[0], total);
        const int sbase = segs_in_wave - ls + waves_before(s_sums[3], segs_pr);
        tbase = tiles_in_wave - lt + waves_before(s_sums[1], T_pr);
        const bool few_own = teams && total > 0 && T_pr < a.tune.n_waves, long_own = total == 0 && T_pr / 24 >= a.tune.n_waves;
        per_seg = a.variant == 1 && a.split_user == 0 && !few_own && !long_own ? kSegmentTiles : 0;
        tbase += per_seg * sbase;
        T_pr += per_seg * segs_pr;
        for (int i = i0; i < i1; ++i)
            if (viable(i)) {
                u.c.moff[i] = base;
                base += u.c.cnt[i];
                const int gi = atomicAdd(&s_ngroups, 1);
                w.glist[gi] = (unsigned short)i;
                s_r1[i] = (unsigned short)gi;      // (what it held is dead: now where a leader's group stands in the list)
                atomicAdd(&s_shared_blocks, u.c.run[i]);
            }
        if (tid == 0) s_ngrouped = total;
    }
    __syncthreads();
    const int n_groups = s_ngroups;

    // ---- cost model (tile weights as above).  Shared runs are cut into
    // equal pieces per segment, one piece per wave (a "share"); the private columns of
    // all requests form one stream of tiles that is cut into equal shares for the
    // remaining waves.  Both kinds of share are sized to the same cost.
    //
    // shared side: wave 0 sizes the shares, lanes over the groups
    __shared__ int s_plan[8];
    // Quotients from the hardware's reciprocal (this stretch is serial, a true division a dozen dependent steps): exact up to
    // quotients of 2^22, where the product is less than one off; idiv takes a second step and is exact for every x >= 0.
    auto near_div = [](int x, int d, float rcp) {
        const int qq = (int)((float)x * rcp), r = x - qq * d;
        return qq + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
    };
    auto idiv = [&](int x, int d) {
        const float rcp = __builtin_amdgcn_rcpf((float)d);
        const int qq = (int)((float)x * rcp), r = x - qq * d, q2 = (int)((float)r * rcp), r2 = r - q2 * d;
        return qq + q2 + (r2 >= d ? 1 : 0) - (r2 < 0 ? 1 : 0);
    };
    if (wave == 0) {
        auto scan_excl = [&](int v, int& total) {
            const int x = wave_scan_incl(v);
            total = __builtin_amdgcn_readlane(x, 63);
            return x - v;
        };
        const int fixed_tiles = a.split_user > 0 ? a.split_user >> 1 : 0;   // split_user is even
        // group gi's leader, members and run: the lane keeps those of group `lane` in registers
        // (every pass below starts there, and there are rarely more than 64 groups)
        int my_ld = 0, my_cnt = 0, my_run = 0;
        if (lane < n_groups) { my_ld = w.glist[lane]; my_cnt = u.c.cnt[my_ld]; my_run = u.c.run[my_ld]; }
        auto group = [&](int gi, int& ld, int& cnt, int& run) {
            if (gi == lane) { ld = my_ld; cnt = my_cnt; run = my_run; }
            else { ld = w.glist[gi]; cnt = u.c.cnt[ld]; run = u.c.run[ld]; }
        };
        // (sums over the groups in float, exact up to 2^24: they only say where the search below starts, and how few waves a small
        // batch gets.  The quotient of the two is rounded up exactly: one more than that is a tile more in every share of a
        // batch whose shares are as short as they may be.)
        float u_loc = 0.f, t_loc = 0.f;
        for (int gi = lane; gi < n_groups; gi += 64) {
            int ld, cnt, run;
            group(gi, ld, cnt, run);
            const float t = (float)(Hkv * by_mpt.cdiv(cnt)) * (float)((run + 1) >> 1);
            u_loc += t * (float)group_weight(cnt);
            t_loc += t;
        }
        const long long U = 16ll * T_pr + (long long)wave_sum(u_loc);
        const float total_tiles = (float)(T_pr - per_seg * segs_pr) + wave_sum(t_loc);   // (tiles to sweep: what a segment is charged is none)
        const int n_act = max(1, (int)fminf((float)a.tune.n_waves, total_tiles * __builtin_amdgcn_rcpf((float)max(a.tune.min_piece, 1))));
        // Pieces of a group's run of T_seg tiles when a share may cost Q.
        auto pieces = [&](int cnt, int T_seg, int Q) {
            const int want = fixed_tiles > 0 ? fixed_tiles : max(1, idiv(max(Q - group_fixed(cnt), 0), group_weight(cnt)));
            return idiv(T_seg + want - 1, want);
        };
        // shares of the private stream at cost Q per share, and their tiles
        auto own_shares = [&](int Q, int& q) {
            const int n_pr = max(1, (int)ddiv(16ll * T_pr + Q - 1, Q));   // (only where nothing fitted the waves, below)
            q = max(1, idiv(T_pr + n_pr - 1, n_pr));
            return idiv(T_pr + q - 1, q);
        };
        int Q = U + n_act <= INT_MAX ? idiv((int)U + n_act - 1, n_act) : (int)min(1ll << 25, ddiv(U + n_act - 1, n_act));   // the even split
        Q = min(1 << 25, max(16, Q));
        int q = 1, n_sh = 0;
        bool searched = false;
        if (fixed_tiles == 0 && n_groups > 0 && n_groups <= 32) {
            // Shares are whole tiles and pieces whole fractions of a run, so the even split rarely fits the waves,
            // and which cost near it does is a matter of rounding.  Every lane tries one cost for the shared
            // pieces, from 3/4 of the even split to 7/4 of it; the waves the pieces leave over share the private
            // stream; the lane whose longest share (shared piece or private share) costs least wins.
            const int Qc = Q - (Q >> 2) + (int)(((long long)Q * lane) >> 6);
            // (What a group brings to it is worked out by the lane that holds the group.  The tiles a share may hold are
            // exact, and the pieces wherever they fit the waves, so what is chosen here is what is laid out below.)
            const int my_slots = Hkv * tiles_padded(by_mpt.cdiv(my_cnt)), my_w = group_weight(max(my_cnt, 1)), my_fixed = group_fixed(my_cnt);
            int slots = 0, longest = 0;
            for (int gi = 0; gi < n_groups; ++gi) {
                const int T_seg = (__builtin_amdgcn_readlane(my_run, gi) + 1) >> 1, wt = __builtin_amdgcn_readlane(my_w, gi);
                const int fixed = __builtin_amdgcn_readlane(my_fixed, gi);
                const int want = max(1, idiv(max(Qc - fixed, 0), wt));
                const int n_pc = near_div(T_seg + want - 1, want, __builtin_amdgcn_rcpf((float)want));
                slots += items_padded(__builtin_amdgcn_readlane(my_slots, gi) * n_pc);
                longest = max(longest, near_div(T_seg + n_pc - 1, n_pc, __builtin_amdgcn_rcpf((float)n_pc)) * wt + fixed);
            }
            int qq = 0;
            if (T_pr > 0) {
                const int n_own = min(n_act - slots, idiv(T_pr + a.tune.min_piece - 1, max(a.tune.min_piece, 1)));
                qq = n_own >= 1 ? idiv(T_pr + n_own - 1, n_own) : -1;
                if (qq > (1 << 26)) qq = -1;
            }
            const bool fits = slots <= n_act && qq >= 0;
            // least cost; among equals the largest Qc (fewest pieces), which the lane number in the low bits says
            const uint32_t cost = fits ? min((uint32_t)max(longest, 16 * qq), (1u << 25) - 2u) : (1u << 25) - 1u;
            const uint32_t best = wave_min((cost << 6) | (uint32_t)(63 - lane));
            if (best >> 6 != (1u << 25) - 1u) {
                const int who = 63 - (int)(best & 63u);
                Q = __builtin_amdgcn_readlane(Qc, who);
                q = max(1, __builtin_amdgcn_readlane(qq, who));
                searched = true;
            }
        }
        // Otherwise (very many groups, or nothing fitted): start from the even split and grow the cost until
        // shared pieces plus private shares fit the waves (a wave with two shares would be the tail).
        for (int round = 0; round < 4; ++round) {
            int loc = 0;
            for (int gi = lane; gi < n_groups; gi += 64) {
                int ld, cnt, run;
                group(gi, ld, cnt, run);
                const int n_pc = pieces(cnt, (run + 1) >> 1, Q);
                v.g.npc[gi] = n_pc;
                loc += items_padded(Hkv * tiles_padded(by_mpt.cdiv(cnt)) * n_pc);
            }
            n_sh = wave_sum(loc);
            if (fixed_tiles > 0 || searched) break;
            const int shares = n_sh + own_shares(Q, q);
            if (shares <= n_act) break;
            Q = (int)min(1ll << 25, ddiv((long long)Q * shares + n_act - 1, n_act) + 1);
        }
        // bases of the groups in list order: shares/items, segments, partial rows
        int ib = 0, sb = 0, rb = 0;
        for (int g0 = 0; g0 < n_groups; g0 += 64) {
            const int gi = g0 + lane;
            int ni = 0, nsg = 0, nr = 0;
            if (gi < n_groups) {
                int ld, cnt, run;
                group(gi, ld, cnt, run);
                nsg = Hkv * by_mpt.cdiv(cnt);
                ni = items_padded(Hkv * tiles_padded(by_mpt.cdiv(cnt)) * v.g.npc[gi]);
                nr = Hkv * v.g.npc[gi] * cnt * a.G;
            }
            int ti, ts, tr;
            const int xi = scan_excl(ni, ti), xs = scan_excl(nsg, ts), xr = scan_excl(nr, tr);
            if (gi < n_groups) {
                v.g.ibase[gi] = ib + xi;
                u.c.gseg[gi] = sb + xs;
                v.g.rbase[gi] = rb + xr;
            }
            ib += ti; sb += ts; rb += tr;
        }
        if (lane == 0) {
            s_plan[0] = fixed_tiles;
            s_plan[1] = q = max(q, 1 + per_seg);
            s_plan[2] = n_sh;
            s_plan[3] = rb;
        }
    }
    __syncthreads();
    const int fixed_tiles = s_plan[0], q = s_plan[1], n_sh = s_plan[2], rows_sh = s_plan[3];

    auto priv_units = [&](int i) {
        const int t = priv_tiles(i);
        return t > 0 ? t + per_seg : 0;
    };

    // Cutting one segment of `units` into pieces, walking along the stream: `rem` units of share `k` are used up
    // at the segment's start.  Calls f(jb, je, starts_share, k) for every piece of tiles, in order, and moves (k, rem)
    // to the segment's end.  (The units before the first tile may be all a share has left: that makes no piece.  A
    // share holds more than those, so its first units always make one.)
    auto for_pieces = [&](int units, int& k, int& rem, auto&& f) {
        if (units == 0) return;
        const int tiles = units - per_seg;
        if (fixed_tiles > 0) {
            for (int j = 0; j < tiles; j += fixed_tiles) f(j, min(tiles, j + fixed_tiles), false, k);
            return;
        }
        int room = q - rem - per_seg;
        bool starts = rem == 0;
        if (room == 0) { room = q; starts = true; ++k; }
        for (int j = 0;;) {
            const int take = min(tiles - j, room);
            f(j, j + take, starts, k);
            j += take;
            room -= take;
            if (j >= tiles) break;
            room = q;
            starts = true;
            ++k;
        }
        rem = q - room;
        if (rem == q) { rem = 0; ++k; }
    };
    // Columns that one item alone reads are marked: the sweep has them pass by the caches.  Not marked are a request's own columns
    // where others may have the same ones (nothing was looked for, a request has no place among those that were compared, or a
    // subgroup was found and left as it was, one of them for the whole batch), and runs with more than one row tile, or, in a batch where
    // any group has split off, that subgroups may sweep too.  Nor is anything in a
    // batch of less than 32 MB: the memory-side cache (256 MB) holds what eight layers of it read from one step to the next.
    const bool far = a.variant == 1 && T_pr - per_seg * segs_pr + Hkv * (s_shared_blocks >> 1) >= a.far_tiles;
    const int own_once = far && a.grouping && B <= kGroupReqMax && s_alike == 0 ? kOnce : 0;
    const WideDiv by_q(max(q, 1));
    const int k_start = by_q.div(tbase), rem_start = tbase - k_start * q;

    // ---- item counts of the thread's segments, scanned in stream order.  The pieces are not walked for that (a batch of few
    // long histories has hundreds to a segment, one thread's): a segment has a piece for the share it starts in - unless its
    // charge is all that is left there - and one for every share it reaches into.
    int li = 0;
    {
        const float rcp_q = __builtin_amdgcn_rcpf((float)q);
        int rem = rem_start;
        for (int e = e0, seen = -1, t = 0; e < e1; ++e) {
            const int i = by_hkv.div(e);
            if (i != seen) { seen = i; t = priv_units(i); }
            if (t == 0) continue;
            if (fixed_tiles > 0) {
                li += idiv(t + fixed_tiles - 1, fixed_tiles);
            } else {
                const int end = rem + t, last = near_div(end - 1, q, rcp_q);   // (end < 2^31: a share's units and a segment's; at most as many shares as waves)
                li += last + (q - rem > per_seg ? 1 : 0);
                rem = end - last * q;
                if (rem == q) rem = 0;
            }
        }
    }
    int priv_items;
    const int ibase = n_sh + block_scan_excl(li, s_sums[2], priv_items);
    const int total_items = n_sh + priv_items, total_rows = rows_sh + priv_items * a.G;
    const bool overflow = total_items > a.lay.max_items || total_rows > a.lay.max_rows;

    // shares: a shared piece each, then the cuts of the private stream; with a fixed
    // split all items are dealt out in equal numbers instead
    const int n_shares = overflow ? 0 : (fixed_tiles > 0 ? min(a.tune.n_waves, total_items) : n_sh + (T_pr + q - 1) / q);
    // first item of every share: a shared piece is its own share, the private shares'
    // entries are written by whoever emits their first item (below); with a fixed split
    // the items are dealt out evenly; then the end marks
    for (int x = tid; x <= n_shares; x += kPlanThreads) {
        if (x == n_shares) wave_first[x] = overflow ? 0 : total_items;
        else if (fixed_tiles > 0) wave_first[x] = (int)ddiv((long long)x * total_items, n_shares);
        else if (x < n_sh) wave_first[x] = x;
    }
    if (tid == 0) wave_first[a.lay.max_items] = overflow ? 0 : total_items;

    // ---- descriptors and items of the requests' own columns
    {
        int k = k_start, rem = rem_start, idx = ibase;
        int seen = -1, L = 0, nb = 0, c0 = 0, units = 0;
        for (int e = e0; e < e1; ++e) {
            const int i = by_hkv.div(e), g = e - i * Hkv;
            if (i != seen) { seen = i; L = len_of(i); nb = (L + kBlock - 1) / kBlock; c0 = run_of(i); units = priv_units(i); }
            const int seg_first = idx;
            if (!overflow) {
                for_pieces(units, k, rem, [&](int jb, int je, bool starts, int kk) {
                    const int cs = c0 + 2 * jb, ce = min(nb, c0 + 2 * je);
                    // (the piece that ends at the request's last column is marked: it grows with the request, see refresh_kernel)
                    write_item(&items[idx], i, g | own_once, a.G, ce == nb ? kOpenEnded : -1, cs, ce, rows_sh + (idx - n_sh) * a.G, min(L, ce * kBlock));
                    if (starts) wave_first[n_sh + kk] = idx;
                    ++idx;
                });
            }
            SegDesc sd;
            sd.pbase = rows_sh + (seg_first - n_sh) * a.G;
            sd.npieces = idx - seg_first;
            segs[e] = sd;
        }
    }
    // ---- member lists of the groups (the rank lives with the thread that drew it), and the requests' descriptors, with where a
    // member of a group finds the partials of the shared run (its rank is its position in the member list).  Nothing from here
    // on reads what another thread has stored to memory: a barrier would wait for all of those stores (members and group
    // descriptors after one took 1.5 us more where a batch has 250 requests, 3.9 where it has 500).
    for (int i = tid, k = 0; i < B; i += kPlanThreads, ++k) {
        const int L = len_of(i), lead = i < nG ? (int)s_lead[i] : -1;
        const bool grouped = lead >= 0 && viable(lead);
        int4 shared = make_int4(0, 0, 0, 0);
        int run = 0;
        if (grouped) {
            const int gi = s_r1[lead], cnt = u.c.cnt[lead], n_pc = v.g.npc[gi];
            const int rank = k == 0 ? my_rank[0] : my_rank[kPer - 1];
            const int tau = by_mpt.div(rank), full_rows = a.mpt * a.G;
            run = u.c.run[lead];
            members[u.c.moff[lead] + rank] = i;
            shared.x = n_pc;
            shared.y = v.g.rbase[gi] + n_pc * tau * full_rows + (rank - tau * a.mpt) * a.G;
            shared.z = n_pc * cnt * a.G;
            shared.w = (tau + 1) * a.mpt >= cnt ? (cnt - tau * a.mpt) * a.G : full_rows;
        }
        int4* rd = reinterpret_cast<int4*>(&req[i]);
        rd[0] = shared;
        rd[1] = make_int4((L + kBlock - 1) / kBlock, L, grouped ? lead : -1, run);
    }
    // ---- descriptors and items of the groups: one team of waves per group, its lanes
    // over the group's items (the fewer groups, the bigger the teams).
    // Order: KV head, piece, row tile - the row tiles of one piece read the same KV bytes
    // and sit on neighbouring shares, which the sweep maps to one XCD.
    if (!overflow) {
        int team = kPlanThreads / 64;   // waves per team: the largest power of two with teams >= groups (at least 1)
        while (team > 1 && (kPlanThreads / 64) / team < n_groups) team >>= 1;
        const int lstep = team * 64, l0 = tid & (lstep - 1), n_teams = kPlanThreads / lstep;
        for (int gi = tid / lstep; gi < n_groups; gi += n_teams) {
            const int ld = w.glist[gi];
            const int cnt = u.c.cnt[ld], run = u.c.run[ld];
            const int tiles_r = by_mpt.cdiv(cnt), T_seg = (run + 1) >> 1;
            const int n_pc = v.g.npc[gi];
            // tiles per piece: the fixed split's, or the run's tiles dealt out evenly (the first `extra` pieces hold one
            // more).  A short last piece would not be worth a team, and the pair of waves sweeping it on their own
            // would sit in a workgroup with a team: its barriers wait for every wave of the workgroup that is still
            // running, so that team would start only when those two had finished.
            const int ps = fixed_tiles > 0 ? fixed_tiles : T_seg / n_pc;
            const int extra = fixed_tiles > 0 ? 0 : T_seg - ps * n_pc;
            if (l0 == 0) {
                GroupDesc gd;
                gd.leader = ld;
                gd.members = cnt;
                gd.run = run;
                gd.member_off = u.c.moff[ld];
                gd.tiles = tiles_r;
                gd.seg_base = u.c.gseg[gi];
                gd.pad[0] = gd.pad[1] = 0;
                grp[ld] = gd;
            }
            const int tiles_p = tiles_padded(tiles_r);
            const int team = (teams && tiles_r >= 2) ? (tiles_r == 2 ? 2 : 4) : 0;
            const int once = far && tiles_r == 1 && !split_off ? kOnce : 0;
            const FastDiv by_tp(tiles_p), by_pc(n_pc);
            const int n = Hkv * n_pc * tiles_p, n_slots = items_padded(n);
            const int full_rows = a.mpt * a.G, last_rows = (cnt - (tiles_r - 1) * a.mpt) * a.G;
            // partial rows of segment (g, tau): pieces p = 0 .. n_pc-1, rows(tau) each; segments in (g, tau) order
            const int rows_per_head = cnt * a.G;
            for (int k = l0; k < n_slots; k += lstep) {
                Item* dst = &items[v.g.ibase[gi] + k];
                if (k >= n) {                          // filler up to the next multiple of 4: nothing to sweep
                    write_item(dst, 0, 0, 0, -1, 0, 0, 0, 0);
                    continue;
                }
                const int rest = by_tp.div(k), tau = k - rest * tiles_p;
                const int g = by_pc.div(rest), pc = rest - g * n_pc;
                const int cs = 2 * (pc * ps + min(pc, extra)), ce = min(run, cs + 2 * (ps + (pc < extra ? 1 : 0)));
                const int g_team = g | once | (team << 16) | ((team ? (tau & (team - 1)) : 0) << 20);   // KV head, team size, rank in the team
                if (tau >= tiles_r) {                  // no rows of its own: a team member that only fetches
                    write_item(dst, ld, g_team, 0, -1, cs, ce, 0, ce * kBlock);
                    continue;
                }
                const int rows = tau == tiles_r - 1 ? last_rows : full_rows;
                const int seg_pbase = v.g.rbase[gi] + n_pc * (g * rows_per_head + tau * full_rows);
                write_item(dst, ld, g_team, rows, u.c.moff[ld] + tau * a.mpt, cs, ce, seg_pbase + pc * rows, ce * kBlock);
                if (pc == 0) {
                    SegDesc sd;
                    sd.pbase = seg_pbase;
                    sd.npieces = n_pc;
                    segs[(size_t)B * Hkv + u.c.gseg[gi] + g * tiles_r + tau] = sd;
                }
            }
        }
    }
    if (tid == 0) {
        hdr[H_ITEMS] = overflow ? 0 : total_items;
        hdr[H_QUEUE] = 0;
        hdr[H_GROUPS] = n_groups;
        hdr[H_GROUPED] = s_ngrouped;
        hdr[H_SPLIT] = fixed_tiles > 0 ? 2 * fixed_tiles : 2 * q;
        hdr[H_ROWS] = total_rows;
        hdr[H_SHARED_BLOCKS] = s_shared_blocks;
        hdr[H_VARIANT] = a.variant;
        hdr[H_OVERFLOW] = overflow ? 1 : 0;
        hdr[H_WAVES] = n_shares;
        hdr[H_CAPACITY] = a.lay.max_items;
        hdr[H_HISTORIES] = 0;
    }
}

// What a refresh does where the workspace holds no plan (the calls before it needed none, and the table has since grown
// past what is done without one), or one whose sections lie elsewhere (with a fixed split they follow from the table's
// width, and the table has grown): every (request, KV head) history cut evenly into pieces of its own, nothing looked for
// that requests share.  Every piece is a share: (slots past a short history's pieces hold none, which only a share of its
// own may).  The header is written by the workgroup that comes last, when all have seen that there is no plan.
__device__ __forceinline__ void plain_split(const PlanArgs& a) {
    int* hdr = reinterpret_cast<int*>(a.ws);
    ReqDesc* req = reinterpret_cast<ReqDesc*>(a.ws + a.lay.req);
    SegDesc* segs = reinterpret_cast<SegDesc*>(a.ws + a.lay.segs);
    int* wave_first = reinterpret_cast<int*>(a.ws + a.lay.wave_first);
    Item* items = reinterpret_cast<Item*>(a.ws + a.lay.items);
    const int NE = a.B * a.Hkv, min_piece = max(a.tune.min_piece, 1);
    const int pieces = max(1, min(a.tune.n_waves / NE, min(a.lay.max_items / NE, a.lay.max_rows / (NE * a.G))));
    const int n_items = NE * pieces;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < n_items; x += gridDim.x * blockDim.x) {
        const int e = x / pieces, p = x - e * pieces, i = e / a.Hkv, g = e - i * a.Hkv;
        const int L = max(0, min(a.seq_lens[i], a.stride * kBlock)), nb = cdiv(L, kBlock), tiles = (nb + 1) >> 1;
        const int np = min(pieces, cdiv(tiles, min_piece));
        if (p < np) {
            const int each = tiles / np, extra = tiles - each * np, jb = p * each + min(p, extra), je = jb + each + (p < extra ? 1 : 0);
            const int ce = min(nb, 2 * je);
            write_item(&items[x], i, g, a.G, ce == nb ? kOpenEnded : -1, 2 * jb, ce, x * a.G, min(L, ce * kBlock));
        } else {
            write_item(&items[x], 0, 0, 0, -1, 0, 0, 0, 0);
        }
        wave_first[x] = x;
        if (p == 0) {
            SegDesc sd;
            sd.pbase = x * a.G;
            sd.npieces = np;
            segs[e] = sd;
            if (g == 0) {
                ReqDesc rd;
                rd.ns_sh = rd.sh_base0 = rd.sh_gstride = rd.sh_pstride = 0;
                rd.nb = nb;
                rd.L = L;
                rd.group = -1;
                rd.priv_c0 = 0;
                req[i] = rd;
            }
        }
        if (x == n_items - 1) wave_first[n_items] = wave_first[a.lay.max_items] = n_items;
    }
    __syncthreads();   // (the whole workgroup has read the header)
    if (threadIdx.x == 0 && atomicAdd(&hdr[H_QUEUE], 1) == (int)gridDim.x - 1) {
        hdr[H_QUEUE] = hdr[H_GROUPS] = hdr[H_GROUPED] = hdr[H_SHARED_BLOCKS] = hdr[H_OVERFLOW] = 0;
        hdr[H_ITEMS] = hdr[H_WAVES] = n_items;
        hdr[H_SPLIT] = 2 * cdiv((a.stride + 1) >> 1, pieces);
        hdr[H_ROWS] = n_items * a.G;
        hdr[H_VARIANT] = a.variant;
        hdr[H_CAPACITY] = a.lay.max_items;
        hdr[H_HISTORIES] = 0;
    }
}

// A plan made for shorter histories: the requests have grown since (decode steps append tokens, tables got
// new columns at their ends), nothing else changed.  The split of the work stays; the last piece of every
// request's own columns is stretched to the request's length now.  (Lengths that shrank would leave the plan
// wrong - attention over rows that no longer count - but never out of bounds: a piece keeps at least one tile.)
__global__ __launch_bounds__(256) void refresh_kernel(PlanArgs a) {
    const int* hdr = reinterpret_cast<const int*>(a.ws);
    int capacity = hdr[H_CAPACITY];
    const int variant = hdr[H_VARIANT], made = hdr[H_ITEMS];
    FEA_TOGETHER(capacity, variant, made, a.lay.items);   // (one round trip for the header's words)
    if (capacity != a.lay.max_items) { plain_split(a); return; }
    if (variant == kHistories) return;   // whole histories are read at their lengths of now
    Item* items = reinterpret_cast<Item*>(a.ws + a.lay.items);
    const int n_items = min(made, a.lay.max_items);
    const int maxL = a.stride * kBlock;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_items; i += gridDim.x * blockDim.x) {
        const int4 w0 = reinterpret_cast<const int4*>(&items[i])[0];
        if (w0.w != kOpenEnded) continue;
        const int who = w0.x;
        if (who < 0 || who >= a.B) continue;
        int4 w1 = reinterpret_cast<const int4*>(&items[i])[1];
        const int L = max(0, min(a.seq_lens[who], maxL));
        w1.y = max((L + kBlock - 1) / kBlock, w1.x + 1);      // c1
        w1.w = max(L, w1.x * kBlock + 1);                     // tok_end
        reinterpret_cast<int4*>(&items[i])[1] = w1;
    }
    // a request that had no columns of its own then (empty, or every block shared) has no piece to stretch
    const ReqDesc* req = reinterpret_cast<const ReqDesc*>(a.ws + a.lay.req);
    const SegDesc* segs = reinterpret_cast<const SegDesc*>(a.ws + a.lay.segs);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.B; i += gridDim.x * blockDim.x)
        if (segs[(size_t)i * a.Hkv].npieces == 0 && min(a.seq_lens[i], maxL) > req[i].L)
            atomicOr(reinterpret_cast<int*>(a.ws) + H_OVERFLOW, 2);
}

void launch_refresh(const PlanArgs& a, const Launch& L) {
    hipExtLaunchKernelGGL(refresh_kernel, dim3(32), dim3(256), 0, static_cast<hipStream_t>(L.stream),
                          static_cast<hipEvent_t>(L.ev_start), static_cast<hipEvent_t>(L.ev_stop), 0, a);
}

void set_read_ahead(PlanArgs& a, const void* k_cache, const void* v_cache, int head_dim, int cus) {
    a.k_cache = k_cache;
    a.v_cache = v_cache;
    a.block_bytes = kBlock * head_dim * 2;
    a.ahead_grid = cus / 2;
    const int64_t column = (int64_t)a.B * a.Hkv * 2 * a.block_bytes;       // bytes of K and V of a column of every request
    a.ahead = a.ahead_grid > 1 ? (int32_t)std::min<int64_t>(a.stride / 4, (kAheadMB * 1000000ll + column) / (2 * column)) : 0;
    a.own = (int32_t)(kOwnMB * 1000000ll / column);
}

void launch_plan(const PlanArgs& a, const Launch& L) {
    hipStream_t st = static_cast<hipStream_t>(L.stream);
    hipEvent_t e0 = static_cast<hipEvent_t>(L.ev_start), e1 = static_cast<hipEvent_t>(L.ev_stop);
    if (a.pre) {   // each dispatch gets a whole pair of events; the step runs from the first start to the last stop
        hipExtLaunchKernelGGL(run_kernel, dim3(a.pre_grid), dim3(kRunThreads), 0, st, e0,
                              static_cast<hipEvent_t>(L.ev_mid[0]), 0, a);
        hipExtLaunchKernelGGL(plan_kernel, dim3(a.ahead > 0 ? a.ahead_grid : 1), dim3(kPlanThreads), 0, st, static_cast<hipEvent_t>(L.ev_mid[1]), e1, 0, a);
    } else {
        hipExtLaunchKernelGGL(plan_kernel, dim3(a.ahead > 0 ? a.ahead_grid : 1), dim3(kPlanThreads), 0, st, e0, e1, 0, a);
    }
}

}  // namespace fea
