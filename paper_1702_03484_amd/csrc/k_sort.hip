// The Shuffle step of Algorithm 1 (both sides' records grouped by key):
// stable LSD radix sort of (u32 key, u32 payload) pairs for gfx950.
//
// One histogram launch counts the digits of every pass at once; each pass is
// then one launch that ranks a tile in LDS and scatters it to its final
// place, the tile's global offsets coming from a decoupled look-back over
// per-digit status words.  Ranking is stable: within a wave64 the peers of a
// digit are found with one __ballot per digit bit, waves own consecutive
// slices of the tile, and tiles take dynamic ids in input order.
//
// First-pass ("gen") mode reads the keys of two input segments (the LEFT
// then the RIGHT partial-match table of a join), subtracts a base and
// generates the payload as the record's position in that concatenation, or
// reads it from the record's one value column (the side then rides in the
// key's low bit), so the intermediate records are never written out before
// the first scatter.
#include "device_common.h"
#include "kernels.h"
#include "tile_ops.h"

#include <algorithm>

namespace mq {

// Cell idx of the concatenation c0 (n0 cells) ++ c1.  Callers clamp idx
// into range and load unconditionally, then transform: a load (or its use)
// inside a divergent branch makes every load wait for the one before.
__device__ __forceinline__ int32_t src_load(const int32_t* c0, const int32_t* c1, uint32_t n0, uint32_t idx) {
    const bool right = idx >= n0;
    return (right ? c1 : c0)[right ? idx - n0 : idx];
}

__device__ __forceinline__ uint32_t src_key_of(const SortSrc& s, int32_t raw, uint32_t idx) {
    const uint32_t rel = ((uint32_t)raw - (uint32_t)s.base) & s.mask;
    return s.carry ? rel << 1 | (idx >= s.n0 ? 1u : 0u) : rel;
}

// Digit histograms of every pass in two launches: each block counts its
// keys into LDS (all loads of a tile in flight at once, one atomic per run
// of equal digits) and stores its counts to its own row of a partial table;
// a second kernel sums the rows.
// No device-wide atomics: they serialise on the few hundred counters.
constexpr int HIST_IPT = 16;
constexpr uint32_t HIST_BLOCKS = 512;
// from here on blocks of 1,024 threads, two to a CU: 32M keys of two columns
// 34 us, with 256 46, and 67 with a key a load; fewer keys need the blocks
constexpr uint32_t HIST_BIG = 1u << 22;

template <int RB, bool GEN, uint32_t NT>
__global__ __launch_bounds__(NT) void radix_hist_kernel(SortSrc src, const uint32_t* __restrict__ keys,
                                                              uint32_t n, int shift0, int passes,
                                                              uint32_t* __restrict__ part) {
    using R = Radix<RB>;
    __shared__ uint32_t sh[R::MAXP * R::BUCKETS];
    for (int i = threadIdx.x; i < R::MAXP * R::BUCKETS; i += NT) sh[i] = 0;
    __syncthreads();
    constexpr uint32_t TILE = NT * HIST_IPT;
    const uint32_t ntiles = (n - 1) / TILE + 1;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        // a whole tile of one side on a 16-byte boundary: four keys a load,
        // neighbouring lanes on neighbouring addresses; else a thread's 16
        // consecutive keys one by one (4 bytes of every line per load).  Runs of
        // one digit (index-ordered keys have long ones) cost one LDS atomic.
        const uint32_t base = t * TILE;
        const bool right = GEN && base >= src.n0;
        const uint32_t* from = GEN ? reinterpret_cast<const uint32_t*>(right ? src.k1 + (base - src.n0) : src.k0 + base)
                                   : keys + base;
        const bool vec = (GEN && !right ? min(n, src.n0) : n) - base >= TILE &&
                         reinterpret_cast<uintptr_t>(from) % 16 == 0;
        uint32_t k[HIST_IPT];
        if (vec) {
            const uint4* f4 = reinterpret_cast<const uint4*>(from);
#pragma unroll
            for (int i = 0; i < HIST_IPT; i += 4) {
                const uint4 q = f4[i / 4 * NT + threadIdx.x];
                k[i] = q.x;
                k[i + 1] = q.y;
                k[i + 2] = q.z;
                k[i + 3] = q.w;
            }
            if (GEN) {
#pragma unroll
                for (int i = 0; i < HIST_IPT; i++) k[i] = src_key_of(src, (int32_t)k[i], base);  // one side
            }
        }
        const uint32_t first = base + threadIdx.x * HIST_IPT;
        if (!vec) {
#pragma unroll
            for (int i = 0; i < HIST_IPT; i++) {
                const uint32_t idx = min(first + i, n - 1);
                k[i] = GEN ? (uint32_t)src_load(src.k0, src.k1, src.n0, idx) : keys[idx];
            }
            if (GEN) {
#pragma unroll
                for (int i = 0; i < HIST_IPT; i++) k[i] = src_key_of(src, (int32_t)k[i], first + i);
            }
        }
        const int cnt = vec ? HIST_IPT : first >= n ? 0 : (int)min((uint32_t)HIST_IPT, n - first);
        for (int p = 0; p < passes; p++) {
            const int sh_p = shift0 + p * RB;
            uint32_t cur = (k[0] >> sh_p) & R::MASK, run = 0;
#pragma unroll
            for (int i = 0; i < HIST_IPT; i++) {
                if (i < cnt) {
                    const uint32_t d = (k[i] >> sh_p) & R::MASK;
                    if (d != cur) {
                        atomicAdd(&sh[p * R::BUCKETS + cur], run);
                        cur = d;
                        run = 0;
                    }
                    run++;
                }
            }
            if (run) atomicAdd(&sh[p * R::BUCKETS + cur], run);
        }
    }
    __syncthreads();
    uint32_t* row = part + (uint64_t)blockIdx.x * passes * R::BUCKETS;
    for (int i = threadIdx.x; i < passes * R::BUCKETS; i += NT) row[i] = sh[i];
}

// hist[c] = sum over the partial rows.  A block of 16 waves owns 64
// counters: lane L of wave w adds rows w, w + 16, ... of counter c0 + L
// (coalesced 256-byte row slices, four loads in flight per lane), and the
// 16 partial sums meet in LDS.
constexpr int HRED_WAVES = 16;

__global__ __launch_bounds__(HRED_WAVES * MQ_WAVE) void hist_reduce_kernel(const uint32_t* __restrict__ part,
                                                                           uint32_t rows, uint32_t width,
                                                                           uint32_t* __restrict__ hist) {
    __shared__ uint32_t sh[HRED_WAVES][MQ_WAVE];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t c = blockIdx.x * MQ_WAVE + lane();
    uint32_t s = 0;
    if (c < width) {
        uint32_t r = w;
        for (; r + 3 * HRED_WAVES < rows; r += 4 * HRED_WAVES) {
            const uint32_t a0 = part[(uint64_t)r * width + c];
            const uint32_t a1 = part[(uint64_t)(r + HRED_WAVES) * width + c];
            const uint32_t a2 = part[(uint64_t)(r + 2 * HRED_WAVES) * width + c];
            const uint32_t a3 = part[(uint64_t)(r + 3 * HRED_WAVES) * width + c];
            s += (a0 + a1) + (a2 + a3);
        }
        for (; r < rows; r += HRED_WAVES) s += part[(uint64_t)r * width + c];
    }
    sh[w][lane()] = s;
    __syncthreads();
    if (w == 0 && c < width) {
        uint32_t t = 0;
#pragma unroll
        for (int k = 0; k < HRED_WAVES; k++) t += sh[k][lane()];
        hist[c] = t;
    }
}

hipError_t launch_hist_reduce(const uint32_t* part, uint32_t rows, uint32_t width, uint32_t* hist,
                              hipStream_t stream) {
    hist_reduce_kernel<<<(width + MQ_WAVE - 1) / MQ_WAVE, HRED_WAVES * MQ_WAVE, 0, stream>>>(part, rows, width, hist);
    return hipGetLastError();
}

uint32_t radix_hist_part_words(int rb, int passes) { return HIST_BLOCKS * (uint32_t)passes << rb; }

// Shape of a radix pass.  Digits of up to 8 bits at 16 keys per thread run in
// 16-wave blocks, two to a CU within 64 VGPRs and 75 KB of LDS each, tiles of
// 16,384 records (32M records, carried pass: 148 us, against 181 us in 8-wave
// blocks of half the tile, four to a CU: a pass pays for tiles in look-backs).
// Carried passes of 2^24.6 records and more take 32 keys per thread, tiles of
// 32,768 records in 137 KB: 133 us at 32M records, but 93 against 88 us for one
// at 20M, where 610 tiles fill 256 CUs unevenly.  (Whole sorts of 24-bit keys,
// 32 against 16 keys: 12.6M records 0.197 and 0.206 ms, 16.8M 0.233 and 0.249,
// 21M 0.297 and 0.300, 25M 0.330 and 0.348, 33.6M 0.431 and 0.456, so the line
// could lie lower.)  The first pass (its keys come from two columns) stays at
// 16: 132 us, against 148.  Everything else, small sorts and wide digits, runs
// in 4-wave blocks.
constexpr uint32_t SORT_BIG = 3u << 23;
__host__ __device__ constexpr bool sort_wide(int rb, int kpt) { return rb <= 8 && kpt == 16; }
__host__ __device__ constexpr int sort_waves(int rb, int kpt) { return sort_wide(rb, kpt) ? 16 : 4; }

// One tile: wave-striped slices, element i of a lane is base + (w*KPT + i)*64 +
// lane; loads are unconditional (FULL: whole tiles; else clamped into range)
// and all in flight at once.
template <int RB, int KPT, bool GEN, int NW, bool FULL>
__device__ __forceinline__ void radix_tile(SplitSmem<RB, KPT, NW>& sm, const SortSrc& src,
                                           const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                           uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t n,
                                           uint32_t base, uint32_t valid_n, int shift,
                                           const uint32_t* __restrict__ ghist, uint64_t* __restrict__ status,
                                           uint32_t tile, uint32_t epoch) {
    constexpr uint32_t TILE = NW * MQ_WAVE * KPT;
    const uint32_t o0 = threadIdx.x / MQ_WAVE * KPT * MQ_WAVE + lane();
    // a first-pass tile on one side of the join loads from a uniform base
    const bool right = GEN && base >= src.n0;
    const bool one = GEN && (right || src.n0 - base >= TILE);
    uint32_t key[KPT];
    if (GEN) {
        int32_t raw[KPT];
        if (one) {
            const int32_t* kt = right ? src.k1 + (base - src.n0) : src.k0 + base;
#pragma unroll
            for (int i = 0; i < KPT; i++) raw[i] = kt[FULL ? o0 + i * MQ_WAVE : min(o0 + i * MQ_WAVE, valid_n - 1)];
        } else {
#pragma unroll
            for (int i = 0; i < KPT; i++)
                raw[i] = src_load(src.k0, src.k1, src.n0, base + min(o0 + i * MQ_WAVE, valid_n - 1));
        }
#pragma unroll
        for (int i = 0; i < KPT; i++) {
            key[i] = src_key_of(src, raw[i], base + o0 + i * MQ_WAVE);
            if (!FULL && o0 + i * MQ_WAVE >= valid_n) key[i] = 0xffffffffu;
        }
    } else {
        const uint32_t* kt = kin + base;
#pragma unroll
        for (int i = 0; i < KPT; i++) {
            key[i] = kt[FULL ? o0 + i * MQ_WAVE : min(o0 + i * MQ_WAVE, valid_n - 1)];
            if (!FULL && o0 + i * MQ_WAVE >= valid_n) key[i] = 0xffffffffu;
        }
    }
    const uint32_t* vt = GEN ? nullptr : vin + base;
    const int32_t* gt = GEN && src.carry && one ? (right ? src.v1 + (base - src.n0) : src.v0 + base) : nullptr;
    auto load_vals = [&](int, uint32_t(&val)[KPT]) {
        if (!GEN) {
#pragma unroll
            for (int i = 0; i < KPT; i++) val[i] = vt[FULL ? o0 + i * MQ_WAVE : min(o0 + i * MQ_WAVE, valid_n - 1)];
        } else if (!src.carry) {
#pragma unroll
            for (int i = 0; i < KPT; i++) val[i] = base + o0 + i * MQ_WAVE;
        } else if (one) {
#pragma unroll
            for (int i = 0; i < KPT; i++)
                val[i] = (uint32_t)gt[FULL ? o0 + i * MQ_WAVE : min(o0 + i * MQ_WAVE, valid_n - 1)];
        } else {
#pragma unroll
            for (int i = 0; i < KPT; i++)
                val[i] = (uint32_t)src_load(src.v0, src.v1, src.n0, base + min(o0 + i * MQ_WAVE, valid_n - 1));
        }
    };
    sort_tile_split<RB, KPT, NW, FULL>(sm, key, valid_n, shift, ghist, status, tile, 0, epoch, kout, n, 1, load_vals,
                                       [&](int) { return vout; });
}

template <int RB, int KPT, bool GEN, int NW>
__global__ __launch_bounds__(NW * MQ_WAVE, NW == 16 && KPT == 16 ? 8 : 4) void radix_pass_kernel(
    SortSrc src, const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, uint32_t n, int shift, const uint32_t* __restrict__ ghist,
    uint64_t* __restrict__ status, uint32_t* __restrict__ tile_ctr, uint32_t epoch) {
    constexpr uint32_t TILE = NW * MQ_WAVE * KPT;
    __shared__ SplitSmem<RB, KPT, NW> sm;
    __shared__ uint32_t s_tile;
    const uint32_t tile = uni(next_tile(tile_ctr, &s_tile, gridDim.x));
    const uint32_t base = tile * TILE;
    const uint32_t valid_n = min(TILE, n - base);
    if (valid_n == TILE)
        radix_tile<RB, KPT, GEN, NW, true>(sm, src, kin, vin, kout, vout, n, base, TILE, shift, ghist, status, tile,
                                           epoch);
    else
        radix_tile<RB, KPT, GEN, NW, false>(sm, src, kin, vin, kout, vout, n, base, valid_n, shift, ghist, status,
                                            tile, epoch);
}

#define MQ_RB_LIST(X) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11)

hipError_t launch_radix_hist(const SortSrc& src, const uint32_t* keys, uint32_t n, int rb, int shift0, int passes,
                             uint32_t* part, uint32_t* hist, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (shift0 < 0 || passes < 1 || shift0 + (passes - 1) * rb > 31) return hipErrorInvalidValue;
    const uint32_t nt = n >= HIST_BIG ? 1024u : (uint32_t)MQ_BLOCK;
    const uint32_t blocks = std::min((n - 1) / (nt * HIST_IPT) + 1, HIST_BLOCKS);
    bool gen = keys == nullptr;
#define MQ_HG(B, G)                                                                                     \
    if (nt == 1024)                                                                                     \
        radix_hist_kernel<B, G, 1024><<<blocks, nt, 0, stream>>>(src, keys, n, shift0, passes, part);   \
    else                                                                                                \
        radix_hist_kernel<B, G, MQ_BLOCK><<<blocks, nt, 0, stream>>>(src, keys, n, shift0, passes, part)
#define MQ_H(B)            \
    case B:                \
        if (gen) {         \
            MQ_HG(B, true);  \
        } else {           \
            MQ_HG(B, false); \
        }                  \
        break;
    switch (rb) {
        MQ_RB_LIST(MQ_H)
        default: return hipErrorInvalidValue;
    }
#undef MQ_HG
#undef MQ_H
    const uint32_t width = (uint32_t)passes << rb;
    return launch_hist_reduce(part, blocks, width, hist, stream);
}

hipError_t launch_radix_pass(int rb, int kpt, const SortSrc& src, const uint32_t* kin, const uint32_t* vin,
                             uint32_t* kout, uint32_t* vout, uint32_t n, int shift, const uint32_t* hist_pass,
                             uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (shift < 0 || shift > 31) return hipErrorInvalidValue;
    bool gen = kin == nullptr;
#define MQ_P(B, K, KE, G)                                                                                \
    radix_pass_kernel<B, KE, G, sort_waves(B, K)><<<radix_tiles(n, K, B, G), sort_waves(B, K) * MQ_WAVE, 0, stream>>>( \
        src, kin, vin, kout, vout, n, shift, hist_pass, status, tile_ctr, epoch)
    const bool big = n >= SORT_BIG;
#define MQ_PK(B)                                                  \
    case B:                                                       \
        if (kpt == 8) {                                           \
            if (gen) MQ_P(B, 8, 8, true);                         \
            else MQ_P(B, 8, 8, false);                            \
        } else if (gen) {                                         \
            MQ_P(B, 16, 16, true);                                \
        } else if (sort_wide(B, 16) && big) {                     \
            MQ_P(B, 16, (sort_wide(B, 16) ? 32 : 16), false);     \
        } else {                                                  \
            MQ_P(B, 16, 16, false);                               \
        }                                                         \
        break;
    switch (rb) {
        MQ_RB_LIST(MQ_PK)
        default: return hipErrorInvalidValue;
    }
#undef MQ_PK
#undef MQ_P
    return hipGetLastError();
}

uint32_t radix_tiles(uint32_t n, int kpt, int rb, bool gen) {
    const uint32_t per = sort_wide(rb, kpt) && !gen && n >= SORT_BIG ? 32u : (uint32_t)kpt;
    const uint32_t tile = (uint32_t)(sort_waves(rb, kpt) * MQ_WAVE) * per;
    return n ? (n - 1) / tile + 1 : 0u;
}

}  // namespace mq
