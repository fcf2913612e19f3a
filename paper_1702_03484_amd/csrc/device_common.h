// Device helpers shared by the gfx950 kernels: wave64 scans, block scans and
// the status words of single-pass decoupled look-back.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define MQ_WAVE 64
#define MQ_BLOCK 256
#define MQ_WAVES (MQ_BLOCK / MQ_WAVE)

#include "mail.h"

namespace mq {

// Posts the words the calling thread has stored to m.data (its wave's, when
// every lane of the wave calls the fence first): the host sees them once it
// sees the flag.
__device__ __forceinline__ void mail_post(const Mail& m) {
    __threadfence_system();
    __hip_atomic_store(m.flag, m.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Bounds-checked build (-DMQ_DEBUG; `python -m paper_1702_03484_amd.build
// --debug` writes libmapsq_debug.so, loaded when MAPSQ_LIB=debug): every
// data-dependent store index of the sort, segment, materialisation and
// compaction kernels is checked against the extent of what it writes; an
// index outside it is printed with its file and line and the store is
// skipped, so a wrong index shows up as a message instead of a memory fault.
// In the normal build the check is the constant true and costs nothing.
#ifdef MQ_DEBUG
__device__ __noinline__ inline bool dbg_in_bounds(uint64_t i, uint64_t n, const char* file, int line) {
    if (i < n) return true;
    printf("mapsq bounds check: %s:%d index %llu outside [0, %llu)\n", file, line, (unsigned long long)i,
           (unsigned long long)n);
    return false;
}
#define MQ_IN_BOUNDS(i, n) ::mq::dbg_in_bounds((uint64_t)(i), (uint64_t)(n), __FILE__, __LINE__)
#else
#define MQ_IN_BOUNDS(i, n) true
#endif

__device__ __forceinline__ uint32_t lane() { return __lane_id(); }
__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << __lane_id()) - 1ull; }

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
#pragma unroll
    for (int o = 1; o < MQ_WAVE; o <<= 1) {
        T t = __shfl_up(v, o, MQ_WAVE);
        if ((int)lane() >= o) v += t;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = MQ_WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, MQ_WAVE);
    return v;
}

// lane - 1's value; lane 0 gets `first` (DPP: the wave shifted right by one)
// every lane must be active: a lane whose neighbour is not gets `first` as well
__device__ __forceinline__ uint32_t wave_prev(uint32_t v, uint32_t first) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xf, 0xf, false);
}

// inclusive wave sum by DPP: within rows of 16, then across them
__device__ __forceinline__ uint32_t wave_incl_u32(uint32_t x) {
#define MQ_DPP_ADD(ctrl, rows) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false)
    MQ_DPP_ADD(0x111, 0xf);  // row_shr 1, 2, 4, 8
    MQ_DPP_ADD(0x112, 0xf);
    MQ_DPP_ADD(0x114, 0xf);
    MQ_DPP_ADD(0x118, 0xf);
    MQ_DPP_ADD(0x142, 0xa);  // row_bcast 15 into rows 1 and 3
    MQ_DPP_ADD(0x143, 0xc);  // row_bcast 31 into rows 2 and 3
#undef MQ_DPP_ADD
    return x;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
#define MQ_DPP_MAX(ctrl, rows) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false))
    MQ_DPP_MAX(0x111, 0xf);
    MQ_DPP_MAX(0x112, 0xf);
    MQ_DPP_MAX(0x114, 0xf);
    MQ_DPP_MAX(0x118, 0xf);
    MQ_DPP_MAX(0x142, 0xa);
    MQ_DPP_MAX(0x143, 0xc);
#undef MQ_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)x, MQ_WAVE - 1);
}

__device__ __forceinline__ uint32_t last_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, MQ_WAVE - 1);
}

// Exclusive scan over the block (MQ_BLOCK threads).  `tmp` is MQ_WAVES
// entries of LDS.  Returns the exclusive prefix; *total gets the block sum.
// Contains __syncthreads(); every thread of the block must call it.
template <typename T>
__device__ __forceinline__ T block_excl_scan(T v, T* tmp, T* total) {
    T inc = wave_incl_scan(v);
    const uint32_t w = threadIdx.x / MQ_WAVE;
    if (lane() == MQ_WAVE - 1) tmp[w] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < MQ_WAVES; i++) {
        T x = tmp[i];
        if ((uint32_t)i < w) before += x;
        all += x;
    }
    *total = all;
    __syncthreads();
    return before + inc - v;
}

// ---- decoupled look-back status words ------------------------------------
// 64-bit word: [63:42] epoch (22 bits), [41:40] flag, [39:0] value.  A word
// whose epoch differs from the running pass's epoch counts as "not yet
// published", so the status array is never cleared between passes.
constexpr uint32_t ST_AGG = 1;  // the tile's own aggregate
constexpr uint32_t ST_INC = 2;  // inclusive prefix up to and including the tile
constexpr uint64_t ST_VAL_MASK = (1ull << 40) - 1ull;
constexpr uint64_t SAT40 = ST_VAL_MASK;  // saturation cap of 40-bit sums

__device__ __forceinline__ uint64_t st_pack(uint32_t epoch, uint32_t flag, uint64_t v) {
    return ((uint64_t)epoch << 42) | ((uint64_t)flag << 40) | (v & ST_VAL_MASK);
}
__device__ __forceinline__ void st_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t st_load(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t sat_add(uint64_t a, uint64_t b) {
    uint64_t s = a + b;
    return s > SAT40 ? SAT40 : s;
}

// Exclusive prefix of tile `tile` over tiles [first_tile, tile) for one
// status column; `stride` is the distance between consecutive tiles' words.
// Reads up to 4 predecessors per round so their load latencies overlap;
// spins until predecessors publish.  Sums saturate at 2^40 - 1.  (Windows of
// 8 and 16 were slower on a 16M + 16M-record sort, 0.81 and 1.13 against
// 0.79 ms: every poll is a device-scope load, and wider polls add traffic
// the spinning waves compete for.)
__device__ __forceinline__ uint64_t lookback(const uint64_t* status, uint32_t tile, uint32_t first_tile,
                                             uint32_t stride, uint32_t epoch) {
    constexpr int WIN = 4;
    uint64_t excl = 0;
    int64_t t = (int64_t)tile - 1;
    while (t >= (int64_t)first_tile) {
        uint64_t w[WIN];
#pragma unroll
        for (int k = 0; k < WIN; k++)
            w[k] = (t - k >= (int64_t)first_tile) ? st_load(status + (uint64_t)(t - k) * stride) : 0ull;
        int k = 0;
        bool done = false;
        for (; k < WIN && t - k >= (int64_t)first_tile; k++) {
            const uint32_t flag = (uint32_t)(w[k] >> 40) & 3u;
            if ((uint32_t)(w[k] >> 42) != epoch || flag == 0) break;  // not yet published: retry from here
            excl = sat_add(excl, w[k] & ST_VAL_MASK);
            if (flag == ST_INC) {
                done = true;
                break;
            }
        }
        if (done) break;
        if (k == 0) __builtin_amdgcn_s_sleep(1);
        t -= k;
    }
    return excl;
}

// Wave-parallel look-back over one status column (stride 1): each probe
// reads the LB_PER_LANE * 64 predecessors below `top` at once (lane L the
// LB_PER_LANE nearest after those of lanes < L) and stops at the nearest
// inclusive prefix.  One word per lane was the fastest window on the
// 512-join batched launch (67.9 ms, against 69.4 with 2 words per lane,
// 71.0 with 4 and 72.8 with 8): a wider probe shortens the walk over
// aggregates but every word is a device-scope load.  Every lane of the
// calling wave must call it; all lanes return the exclusive prefix of `tile`
// (saturating at 2^40 - 1).
constexpr int LB_PER_LANE = 1;

__device__ __forceinline__ uint64_t wave_lookback(const uint64_t* status, uint32_t tile, uint32_t first_tile,
                                                  uint32_t epoch) {
    constexpr int64_t WIN = (int64_t)LB_PER_LANE * MQ_WAVE;
    uint64_t excl = 0;
    int64_t top = (int64_t)tile - 1;
    while (top >= (int64_t)first_tile) {
        uint64_t w[LB_PER_LANE];
        bool inr[LB_PER_LANE];
#pragma unroll
        for (int j = 0; j < LB_PER_LANE; j++) {
            const int64_t t = top - (int64_t)lane() * LB_PER_LANE - j;
            inr[j] = t >= (int64_t)first_tile;
            w[j] = inr[j] ? st_load(status + t) : 0ull;
        }
        // this lane: the first of its words that is an inclusive prefix (or
        // out of range), and whether any word before it is unpublished
        int jinc = LB_PER_LANE;
        bool pending = false;
#pragma unroll
        for (int j = LB_PER_LANE - 1; j >= 0; j--) {
            const uint32_t flag = (uint32_t)(w[j] >> 40) & 3u;
            const bool valid = !inr[j] || ((uint32_t)(w[j] >> 42) == epoch && flag != 0);
            const bool inc = !inr[j] || (valid && flag == ST_INC);
            if (inc) jinc = j;
        }
#pragma unroll
        for (int j = 0; j < LB_PER_LANE; j++) {
            const uint32_t flag = (uint32_t)(w[j] >> 40) & 3u;
            const bool valid = !inr[j] || ((uint32_t)(w[j] >> 42) == epoch && flag != 0);
            if (j <= jinc && !valid) pending = true;
        }
        const uint64_t incm = __ballot(jinc < LB_PER_LANE);
        const uint32_t stop = incm ? (uint32_t)__builtin_ctzll(incm) : 64u;  // lanes 0..stop count
        const uint64_t need = stop >= 63 ? ~0ull : ((2ull << stop) - 1ull);
        if (__ballot(pending) & need) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        uint64_t v = 0;
        if (lane() <= stop) {
#pragma unroll
            for (int j = 0; j < LB_PER_LANE; j++)
                if (inr[j] && (lane() < stop || j <= jinc)) v += w[j] & ST_VAL_MASK;
        }
        v = wave_sum(v);  // at most 256 * 2^40: no overflow
        excl = sat_add(excl, v > SAT40 ? SAT40 : v);
        if (stop < 64) break;
        top -= WIN;
    }
    return excl;
}

// Publish a tile aggregate and resolve its exclusive prefix over tiles
// [first_tile, tile) with one wave (all 64 lanes of that wave call it).
// Returns the exclusive prefix in every lane of the wave.
__device__ __forceinline__ uint64_t tile_prefix_wave(uint64_t* status, uint32_t tile, uint32_t first_tile,
                                                     uint32_t epoch, uint64_t agg) {
    agg = agg > SAT40 ? SAT40 : agg;
    if (tile == first_tile) {
        if (lane() == 0) st_store(status + tile, st_pack(epoch, ST_INC, agg));
        return 0;
    }
    if (lane() == 0) st_store(status + tile, st_pack(epoch, ST_AGG, agg));
    const uint64_t ex = wave_lookback(status, tile, first_tile, epoch);
    if (lane() == 0) st_store(status + tile, st_pack(epoch, ST_INC, sat_add(ex, agg)));
    return ex;
}

__device__ __forceinline__ uint64_t tile_prefix_wave0(uint64_t* status, uint32_t tile, uint32_t epoch, uint64_t agg) {
    return tile_prefix_wave(status, tile, 0, epoch, agg);
}

// Both bounds of v in the ascending c[lo, hi): the first element >= v and the
// first > v, by a group of G consecutive lanes (all with the same arguments):
// one probe of G evenly spaced elements a level, for both bounds while they lie
// in one bracket, then half of the group for each.  A level costs one memory
// round trip and leaves 1/G of the bracket.
template <int G, class Pos>
__device__ __forceinline__ void group_bounds(const int32_t* __restrict__ c, Pos lo, Pos hi, int32_t v, Pos& lower,
                                             Pos& upper) {
    static_assert(G >= 4 && G <= MQ_WAVE && (G & (G - 1)) == 0, "group of lanes");
    constexpr int LOG = __builtin_ctz(G);
    const uint32_t gl = lane() % G, g0 = lane() - gl;
    const uint64_t gmask = G == MQ_WAVE ? ~0ull : (1ull << (G % MQ_WAVE)) - 1ull;
    Pos l0 = lo, l1 = hi, u0 = lo, u1 = hi;
    while (l0 < l1 || u0 < u1) {
        const bool one = l0 == u0 && l1 == u1;
        const bool up = !one && gl >= G / 2;  // this lane probes for the upper bound only
        const Pos p0 = up ? u0 : l0, p1 = up ? u1 : l1;
        const int sh = one ? LOG : LOG - 1;  // 2^sh probes a bound
        const uint32_t at = one ? gl : gl % (G / 2);
        const Pos up1 = ((Pos)1 << sh) - 1, step = (p1 - p0 + up1) >> sh;
        const Pos pos = p0 + (Pos)at * step;
        const bool in = pos < p1;
        const int32_t x = in ? c[pos] : 0;
        const uint64_t below = __ballot(in && x < v) >> g0 & gmask;      // probes before the lower bound (a prefix)
        const uint64_t upto = __ballot(in && x <= v) >> g0 & gmask;      // before the upper bound
        constexpr uint64_t LOW = (1ull << (G / 2)) - 1ull;
        const uint32_t nl = (uint32_t)__popcll(one ? below : below & LOW);
        const uint32_t nu = (uint32_t)__popcll(one ? upto : upto >> (G / 2));
        const Pos sl = (l1 - l0 + up1) >> sh, su = (u1 - u0 + up1) >> sh;
        if (l0 < l1) {
            l1 = nl == 0 ? l0 : min(l1, l0 + (Pos)nl * sl);
            l0 = nl == 0 ? l0 : l0 + (Pos)(nl - 1) * sl + 1;
        }
        if (u0 < u1) {
            u1 = nu == 0 ? u0 : min(u1, u0 + (Pos)nu * su);
            u0 = nu == 0 ? u0 : u0 + (Pos)(nu - 1) * su + 1;
        }
    }
    lower = l0;
    upper = u0;
}

// Next dynamic tile id from a counter (thread 0), broadcast through LDS.
// takes > 0: the ids the whole launch will take; whoever takes the last one
// sets the counter back to 0, so it needs no clearing before the next launch.
__device__ __forceinline__ uint32_t next_tile(uint32_t* counter, uint32_t* s_slot, uint32_t takes = 0) {
    if (threadIdx.x == 0) {
        const uint32_t t = atomicAdd(counter, 1u);
        if (t + 1 == takes) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_slot = t;
    }
    __syncthreads();
    uint32_t t = *s_slot;
    __syncthreads();
    return t;
}

}  // namespace mq
