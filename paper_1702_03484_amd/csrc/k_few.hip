// The Shuffle step for a join whose LEFT side holds few distinct keys (an
// intermediate result that grew from a small table: tens of millions of rows,
// hundreds of keys).  Sorting such a side on all bits of its keys takes three
// passes and then a gather per value column.  Here the keys both sides share
// are numbered in ascending order through a bitmap, each side is grouped by
// that number in one counting pass that moves the value columns themselves,
// and the segments follow from the two histograms: the rows come out exactly
// as from the sort (keys ascending, input order inside a key).
//
// 59M rows of 475 keys with two value columns: histogram and pass are bound by
// memory (each key read twice, each value read and written once).
#include "device_common.h"
#include "kernels.h"
#include "tile_ops.h"

#include <algorithm>

namespace mq {

// ---- the numbering ----------------------------------------------------------
constexpr int FT_IPT = 16;
constexpr uint32_t FT_TILE = MQ_BLOCK * FT_IPT;  // bitmap words per tile

__global__ __launch_bounds__(MQ_BLOCK) void few_table_kernel(const uint32_t* __restrict__ bm, uint32_t words,
                                                             int32_t base, FewEntry* __restrict__ table,
                                                             int32_t* __restrict__ keys, uint64_t* __restrict__ status,
                                                             uint32_t* __restrict__ tile_ctr, uint32_t epoch,
                                                             Mail mail) {
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_scan[MQ_WAVES];
    __shared__ uint64_t s_excl;
    const uint32_t tile = next_tile(tile_ctr, &s_tile, gridDim.x);
    const uint32_t first = tile * FT_TILE + threadIdx.x * FT_IPT;
    uint32_t b[FT_IPT], sum = 0;
#pragma unroll
    for (int i = 0; i < FT_IPT; i++) {
        b[i] = first + i < words ? bm[first + i] : 0u;
        sum += (uint32_t)__popc(b[i]);
    }
    uint32_t all;
    uint32_t at = block_excl_scan<uint32_t>(sum, s_scan, &all);
    if (threadIdx.x < MQ_WAVE) {
        const uint64_t ex = tile_prefix_wave0(status, tile, epoch, all);
        if (lane() == 0) {
            s_excl = ex;
            if (tile == gridDim.x - 1) {
                mail.data[0] = (uint32_t)(ex + all);
                mail.data[1] = (uint32_t)((ex + all) >> 32);
                mail_post(mail);
            }
        }
    }
    __syncthreads();
    at += (uint32_t)s_excl;
#pragma unroll
    for (int i = 0; i < FT_IPT; i++) {
        if (first + i >= words) break;
        table[first + i] = FewEntry{b[i], at};
        uint32_t r = at;
        for (uint32_t left = b[i]; left && r < FEW_KEYS; left &= left - 1, r++)
            keys[r] = (int32_t)((uint32_t)base + (first + i) * 32u + (uint32_t)__builtin_ctz(left));
        at += (uint32_t)__popc(b[i]);
    }
}

// rank of a relative key, or `none`
__device__ __forceinline__ uint32_t few_rank(const FewSide& s, uint32_t k, uint32_t none) {
    const bool in = k < s.range;
    const FewEntry e = s.table[in ? k >> 5 : 0u];
    const uint32_t bit = k & 31u;
    const uint32_t rank = e.before + (uint32_t)__popc(e.bits & ((1u << bit) - 1u));
    return in && (e.bits >> bit & 1u) ? min(rank, none) : none;
}

// ---- rows per key -----------------------------------------------------------
constexpr int FH_IPT = 16;
constexpr uint32_t FH_BLOCKS = 1024;

// A wave reads 64 consecutive keys at a time; rows of one key mostly come in
// runs (the join before wrote them key by key), so 64 equal ranks are one LDS
// atomic.
template <int RB>
__global__ __launch_bounds__(MQ_BLOCK) void few_hist_kernel(FewSide s, uint32_t* __restrict__ part) {
    constexpr uint32_t B = 1u << RB, NONE = B - 1;
    constexpr uint32_t TILE = MQ_BLOCK * FH_IPT;
    __shared__ uint32_t sh[B];
    for (uint32_t i = threadIdx.x; i < B; i += MQ_BLOCK) sh[i] = 0;
    __syncthreads();
    const uint32_t ntiles = (s.n + TILE - 1) / TILE;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const uint32_t first = t * TILE + threadIdx.x / MQ_WAVE * (FH_IPT * MQ_WAVE) + lane();
        uint32_t d[FH_IPT];
#pragma unroll
        for (int i = 0; i < FH_IPT; i++) d[i] = (uint32_t)s.keys[min(first + i * MQ_WAVE, s.n - 1)];
#pragma unroll
        for (int i = 0; i < FH_IPT; i++) {
            d[i] = few_rank(s, d[i] - (uint32_t)s.base, NONE);
            if (first + i * MQ_WAVE >= s.n) d[i] = NONE;
        }
#pragma unroll
        for (int i = 0; i < FH_IPT; i++) {
            const uint32_t d0 = uni(d[i]);
            if (__ballot(d[i] != d0) == 0ull) {
                if (lane() == 0) atomicAdd(&sh[d0], (uint32_t)MQ_WAVE);
            } else if (d[i] != NONE) {
                atomicAdd(&sh[d[i]], 1u);
            }
        }
    }
    __syncthreads();
    uint32_t* row = part + (uint64_t)blockIdx.x * B;
    for (uint32_t i = threadIdx.x; i < B; i += MQ_BLOCK) row[i] = i == NONE ? 0u : sh[i];
}

// ---- segments ---------------------------------------------------------------
// one block, one key per thread
__global__ __launch_bounds__(1024) void few_segments_kernel(const uint32_t* __restrict__ lhist,
                                                            const uint32_t* __restrict__ rhist,
                                                            const int32_t* __restrict__ keys, uint32_t nkeys,
                                                            uint32_t* __restrict__ seg_ls, uint32_t* __restrict__ seg_lc,
                                                            uint32_t* __restrict__ seg_rs, uint32_t* __restrict__ seg_rc,
                                                            uint64_t* __restrict__ seg_off, uint32_t* __restrict__ nseg,
                                                            int32_t* __restrict__ lkey, Mail mail) {
    constexpr int W = 1024 / MQ_WAVE;
    __shared__ uint32_t s_l[W], s_r[W];
    __shared__ uint64_t s_p[W];
    const uint32_t d = threadIdx.x, w = d / MQ_WAVE;
    const uint32_t cl = d < nkeys ? lhist[d] : 0u, cr = d < nkeys ? rhist[d] : 0u;
    const uint64_t pairs = min((uint64_t)cl * cr, SAT40);  // 1,024 of them stay far below 2^64
    const uint32_t il = wave_incl_scan(cl), ir = wave_incl_scan(cr);
    const uint64_t ip = wave_incl_scan(pairs);
    if (lane() == MQ_WAVE - 1) {
        s_l[w] = il;
        s_r[w] = ir;
        s_p[w] = ip;
    }
    __syncthreads();
    uint32_t el = il - cl, er = ir - cr;
    uint64_t ep = ip - pairs, total = 0;
    uint32_t rows_l = 0;
    for (uint32_t i = 0; i < W; i++) {
        rows_l += s_l[i];
        if (i < w) {
            el += s_l[i];
            er += s_r[i];
            ep += s_p[i];
        }
        total += s_p[i];
    }
    if (d < nkeys) {
        seg_ls[d] = el;
        seg_lc[d] = cl;
        seg_rs[d] = er;
        seg_rc[d] = cr;
        seg_off[d] = min(ep, SAT40);
        lkey[el] = keys[d];
    }
    if (d == 0) {
        total = min(total, SAT40);
        *nseg = nkeys;
        mail.data[0] = nkeys;
        mail.data[2] = (uint32_t)total;
        mail.data[3] = (uint32_t)(total >> 32);
        mail.data[4] = rows_l;
        mail_post(mail);
    }
}

// ---- the pass ---------------------------------------------------------------
// 8 keys per thread in 16-wave blocks, two to a CU, for every digit width: 59M
// rows, 8 bits, two value columns: 270 us (2.8 TB/s of the other 1.2 GB).  With
// 16 keys the loads of the next column spill at 64 VGPRs (413 us), and blocks
// with more registers are too few (300-310).
constexpr int FP_KPT = 8;
constexpr int FP_LOOKUPS = 4;
constexpr int FP_WAVES = 16;

template <int RB, int NW, bool FULL>
__device__ __forceinline__ void few_tile(SplitSmem<RB, FP_KPT, NW>& sm, const FewSide& s, uint32_t base,
                                         uint32_t valid_n, const uint32_t* __restrict__ hist, uint32_t n_out,
                                         uint64_t* __restrict__ status, uint32_t tile, uint32_t epoch) {
    constexpr uint32_t NONE = (1u << RB) - 1;
    const uint32_t o0 = threadIdx.x / MQ_WAVE * FP_KPT * MQ_WAVE + lane();
    uint32_t key[FP_KPT];
    const int32_t* kt = s.keys + base;
#pragma unroll
    for (int i = 0; i < FP_KPT; i++) key[i] = (uint32_t)kt[FULL ? o0 + i * MQ_WAVE : min(o0 + i * MQ_WAVE, valid_n - 1)];
#pragma unroll
    for (int i = 0; i < FP_KPT; i++) {
        key[i] = few_rank(s, key[i] - (uint32_t)s.base, NONE);
        if (!FULL && o0 + i * MQ_WAVE >= valid_n) key[i] = 0xffffffffu;
        if (i % FP_LOOKUPS == FP_LOOKUPS - 1) __builtin_amdgcn_sched_barrier(0);
    }
    auto load_vals = [&](int c, uint32_t(&val)[FP_KPT]) {
        const int32_t* in = s.in[c];
        uint32_t o = o0;
        asm volatile("" : "+v"(o));  // the places are computed again, not kept over the ranking
        if (s.ids) {
            const uint32_t* it = s.ids + base;
#pragma unroll
            for (int i = 0; i < FP_KPT; i++) val[i] = it[FULL ? o + i * MQ_WAVE : min(o + i * MQ_WAVE, valid_n - 1)];
#pragma unroll
            for (int i = 0; i < FP_KPT; i++) {
                val[i] = (uint32_t)in[val[i]];
                if (i % FP_LOOKUPS == FP_LOOKUPS - 1) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            in += base;
#pragma unroll
            for (int i = 0; i < FP_KPT; i++)
                val[i] = (uint32_t)in[FULL ? o + i * MQ_WAVE : min(o + i * MQ_WAVE, valid_n - 1)];
        }
    };
    sort_tile_split<RB, FP_KPT, NW, FULL, false>(sm, key, valid_n, 0, hist, status, tile, 0, epoch, nullptr, n_out, s.nv,
                                                 load_vals,
                                                 [&](int c) { return reinterpret_cast<uint32_t*>(s.out[c]); });
}

template <int RB, int NW>
__global__ __launch_bounds__(NW * MQ_WAVE, 8) void few_pass_kernel(
    FewSide s, const uint32_t* __restrict__ hist, uint32_t n_out, uint64_t* __restrict__ status,
    uint32_t* __restrict__ tile_ctr, uint32_t epoch) {
    constexpr uint32_t TILE = NW * MQ_WAVE * FP_KPT;
    __shared__ SplitSmem<RB, FP_KPT, NW> sm;
    __shared__ uint32_t s_tile;
    const uint32_t tile = uni(next_tile(tile_ctr, &s_tile, gridDim.x));
    const uint32_t base = tile * TILE;
    const uint32_t valid_n = min(TILE, s.n - base);
    if (valid_n == TILE)
        few_tile<RB, NW, true>(sm, s, base, TILE, hist, n_out, status, tile, epoch);
    else
        few_tile<RB, NW, false>(sm, s, base, valid_n, hist, n_out, status, tile, epoch);
}

uint32_t few_table_tiles(uint64_t range) { return (uint32_t)(((range + 31) / 32 + FT_TILE - 1) / FT_TILE); }

hipError_t launch_few_table(const uint32_t* bm, uint64_t range, int32_t base, FewEntry* table, int32_t* keys,
                            uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, Mail mail, hipStream_t stream) {
    if (range == 0) return hipErrorInvalidValue;
    few_table_kernel<<<few_table_tiles(range), MQ_BLOCK, 0, stream>>>(bm, (uint32_t)((range + 31) / 32), base, table,
                                                                      keys, status, tile_ctr, epoch, mail);
    return hipGetLastError();
}

int few_bits(uint32_t nkeys) { return nkeys < 64 ? 6 : nkeys < 256 ? 8 : nkeys < 512 ? 9 : 10; }

static uint32_t few_hist_blocks(uint32_t n) {
    return std::min((n + MQ_BLOCK * FH_IPT - 1) / (MQ_BLOCK * FH_IPT), FH_BLOCKS);
}
uint32_t few_part_words(int rb) { return FH_BLOCKS << rb; }

hipError_t launch_few_hist(const FewSide& s, int rb, uint32_t* part, uint32_t* hist, hipStream_t stream) {
    if (s.n == 0) return hipErrorInvalidValue;
    const uint32_t blocks = few_hist_blocks(s.n);
#define MQ_F(B)                                                                 \
    case B: few_hist_kernel<B><<<blocks, MQ_BLOCK, 0, stream>>>(s, part); break;
    switch (rb) {
        MQ_F(6) MQ_F(8) MQ_F(9) MQ_F(10)
        default: return hipErrorInvalidValue;
    }
#undef MQ_F
    return launch_hist_reduce(part, blocks, 1u << rb, hist, stream);
}

hipError_t launch_few_segments(const uint32_t* lhist, const uint32_t* rhist, const int32_t* keys, uint32_t nkeys,
                               uint32_t* seg_ls, uint32_t* seg_lc, uint32_t* seg_rs, uint32_t* seg_rc,
                               uint64_t* seg_off, uint32_t* nseg, int32_t* lkey, Mail mail, hipStream_t stream) {
    if (nkeys == 0 || nkeys > FEW_KEYS) return hipErrorInvalidValue;
    few_segments_kernel<<<1, 1024, 0, stream>>>(lhist, rhist, keys, nkeys, seg_ls, seg_lc, seg_rs, seg_rc, seg_off,
                                                nseg, lkey, mail);
    return hipGetLastError();
}

static uint32_t few_tiles(uint32_t n) {
    constexpr uint32_t tile = FP_WAVES * MQ_WAVE * FP_KPT;
    return (n + tile - 1) / tile;
}
size_t few_status_words(uint32_t n, int rb) { return (size_t)few_tiles(n) << rb; }

hipError_t launch_few_pass(const FewSide& s, int rb, const uint32_t* hist, uint32_t n_out, uint64_t* status,
                           uint32_t* tile_ctr, uint32_t epoch, hipStream_t stream) {
    if (s.n == 0 || s.nv < 1 || s.nv > FEW_COLS) return hipErrorInvalidValue;
#define MQ_F(B)                                                                                             \
    case B:                                                                                                 \
        few_pass_kernel<B, FP_WAVES><<<few_tiles(s.n), FP_WAVES * MQ_WAVE, 0, stream>>>(         \
            s, hist, n_out, status, tile_ctr, epoch);                                                       \
        break;
    switch (rb) {
        MQ_F(6) MQ_F(8) MQ_F(9) MQ_F(10)
        default: return hipErrorInvalidValue;
    }
#undef MQ_F
    return hipGetLastError();
}

}  // namespace mq
