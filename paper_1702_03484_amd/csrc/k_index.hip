// Loading and indexing a store on gfx950: one pass that copies, checks and
// bounds the triples, and the packing of triples into 64-bit words that the
// radix passes sort whole.
//
// A triple is the word (p - pmin | first | second), `second` in the low so
// bits, held as two 32-bit halves; the sort passes carry one half as the key
// and the other as the payload, so both columns of an index come out of the
// last pass in order and nothing is gathered through a permutation.  (Sorting
// a permutation instead and gathering four columns through it per order took
// 2.8 of the 6.0 ms of a 20M-triple load: every gathered cell fetched a cache
// line of its own.)
#include "device_common.h"
#include "kernels.h"

#include <algorithm>

namespace mq {

constexpr uint32_t IX_THREADS = 256;

static uint32_t ix_grid(uint64_t items, uint64_t per_block, uint32_t cap) {
    const uint64_t b = (items + per_block - 1) / per_block;
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(b, cap));
}

// ---- ingest ----------------------------------------------------------------
__global__ void ingest_init_kernel(IngestOut* out) {
    if (threadIdx.x == 0) *out = IngestOut{INT32_MAX, INT32_MIN, INT32_MAX, INT32_MIN, 0u, 0u};
}

struct IngestAcc {
    int32_t so_lo = INT32_MAX, so_hi = INT32_MIN, p_lo = INT32_MAX, p_hi = INT32_MIN;
    uint32_t bad = 0;
    __device__ __forceinline__ void take(int32_t s, int32_t p, int32_t o) {
        so_lo = min(so_lo, min(s, o));
        so_hi = max(so_hi, max(s, o));
        p_lo = min(p_lo, p);
        p_hi = max(p_hi, p);
        bad += (s < 0 || s == INT32_MAX) + (p < 0 || p == INT32_MAX) + (o < 0 || o == INT32_MAX);
    }
};

// HBM-bound: reads 12 B and (COPY) writes 12 B per triple, once.  VEC: every
// column is 16-byte aligned, four triples per load.  One block-level
// reduction and five atomics per block.  20M triples: 0.26 ms as three
// copies, three check passes and two bound passes, 0.13 ms (3.8 TB/s) as
// this pass.
template <bool COPY, bool VEC>
__global__ __launch_bounds__(IX_THREADS) void ingest_kernel(const int32_t* __restrict__ s, const int32_t* __restrict__ p,
                                                            const int32_t* __restrict__ o, int32_t* __restrict__ ds,
                                                            int32_t* __restrict__ dp, int32_t* __restrict__ dq,
                                                            uint64_t n, IngestOut* __restrict__ out) {
    IngestAcc a;
    const uint64_t t0 = blockIdx.x * (uint64_t)IX_THREADS + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * IX_THREADS;
    uint64_t tail = 0;
    if (VEC) {
        const uint64_t n4 = n / 4;
        const int4* s4 = reinterpret_cast<const int4*>(s);
        const int4* p4 = reinterpret_cast<const int4*>(p);
        const int4* o4 = reinterpret_cast<const int4*>(o);
        for (uint64_t i = t0; i < n4; i += stride) {
            const int4 x = s4[i], y = p4[i], z = o4[i];
            a.take(x.x, y.x, z.x);
            a.take(x.y, y.y, z.y);
            a.take(x.z, y.z, z.z);
            a.take(x.w, y.w, z.w);
            if (COPY) {
                reinterpret_cast<int4*>(ds)[i] = x;
                reinterpret_cast<int4*>(dp)[i] = y;
                reinterpret_cast<int4*>(dq)[i] = z;
            }
        }
        tail = n4 * 4;
    }
    for (uint64_t i = tail + t0; i < n; i += stride) {
        const int32_t x = s[i], y = p[i], z = o[i];
        a.take(x, y, z);
        if (COPY) {
            ds[i] = x;
            dp[i] = y;
            dq[i] = z;
        }
    }
#pragma unroll
    for (int d = MQ_WAVE / 2; d > 0; d >>= 1) {
        a.so_lo = min(a.so_lo, __shfl_xor(a.so_lo, d));
        a.so_hi = max(a.so_hi, __shfl_xor(a.so_hi, d));
        a.p_lo = min(a.p_lo, __shfl_xor(a.p_lo, d));
        a.p_hi = max(a.p_hi, __shfl_xor(a.p_hi, d));
        a.bad += __shfl_xor(a.bad, d);
    }
    __shared__ IngestOut sh[IX_THREADS / MQ_WAVE];
    if (lane() == 0) sh[threadIdx.x / MQ_WAVE] = IngestOut{a.so_lo, a.so_hi, a.p_lo, a.p_hi, a.bad, 0u};
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < IX_THREADS / MQ_WAVE; w++) {
            a.so_lo = min(a.so_lo, sh[w].so_min);
            a.so_hi = max(a.so_hi, sh[w].so_max);
            a.p_lo = min(a.p_lo, sh[w].p_min);
            a.p_hi = max(a.p_hi, sh[w].p_max);
            a.bad += sh[w].bad;
        }
        atomicMin(&out->so_min, a.so_lo);
        atomicMax(&out->so_max, a.so_hi);
        atomicMin(&out->p_min, a.p_lo);
        atomicMax(&out->p_max, a.p_hi);
        if (a.bad) atomicAdd(&out->bad, a.bad);
    }
}

hipError_t launch_ingest(const int32_t* s, const int32_t* p, const int32_t* o, int32_t* ds, int32_t* dp, int32_t* dq,
                         uint64_t n, IngestOut* out, hipStream_t stream) {
    ingest_init_kernel<<<1, MQ_WAVE, 0, stream>>>(out);
    if (n == 0) return hipGetLastError();
    const bool copy = ds != s;
    uintptr_t any = 0;
    for (const void* q : {(const void*)s, (const void*)p, (const void*)o, (const void*)ds, (const void*)dp, (const void*)dq})
        any |= reinterpret_cast<uintptr_t>(q);
    const bool vec = any % 16 == 0;
    const uint32_t blocks = ix_grid(n, IX_THREADS * (vec ? 8 : 4), 2048);
    if (copy && vec)
        ingest_kernel<true, true><<<blocks, IX_THREADS, 0, stream>>>(s, p, o, ds, dp, dq, n, out);
    else if (copy)
        ingest_kernel<true, false><<<blocks, IX_THREADS, 0, stream>>>(s, p, o, ds, dp, dq, n, out);
    else if (vec)
        ingest_kernel<false, true><<<blocks, IX_THREADS, 0, stream>>>(s, p, o, ds, dp, dq, n, out);
    else
        ingest_kernel<false, false><<<blocks, IX_THREADS, 0, stream>>>(s, p, o, ds, dp, dq, n, out);
    return hipGetLastError();
}

// ---- packed triples --------------------------------------------------------
// every array below is a 256-byte-aligned arena column: four elements per
// 16-byte access, the last n mod 4 one by one

__device__ __forceinline__ uint64_t triple_word(uint32_t p, uint32_t first, uint32_t second, int so) {
    return (uint64_t)p << (2 * so) | (uint64_t)first << so | second;
}

// reads 12 B, writes 8 B per triple
__global__ __launch_bounds__(IX_THREADS) void pack_triples_kernel(const int32_t* __restrict__ s,
                                                                  const int32_t* __restrict__ p,
                                                                  const int32_t* __restrict__ o, uint64_t n,
                                                                  int32_t pmin, int so, uint32_t* __restrict__ w0,
                                                                  uint32_t* __restrict__ w1) {
    const uint64_t t0 = blockIdx.x * (uint64_t)IX_THREADS + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * IX_THREADS;
    const uint64_t n4 = n / 4;
    auto word = [&](int32_t a, int32_t b, int32_t c) {
        return triple_word((uint32_t)(b - pmin), (uint32_t)a, (uint32_t)c, so);
    };
    for (uint64_t i = t0; i < n4; i += stride) {
        const int4 x = reinterpret_cast<const int4*>(s)[i], y = reinterpret_cast<const int4*>(p)[i],
                   z = reinterpret_cast<const int4*>(o)[i];
        const uint64_t a = word(x.x, y.x, z.x), b = word(x.y, y.y, z.y), c = word(x.z, y.z, z.z),
                       d = word(x.w, y.w, z.w);
        reinterpret_cast<uint4*>(w0)[i] = make_uint4((uint32_t)a, (uint32_t)b, (uint32_t)c, (uint32_t)d);
        reinterpret_cast<uint4*>(w1)[i] =
            make_uint4((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), (uint32_t)(d >> 32));
    }
    for (uint64_t i = n4 * 4 + t0; i < n; i += stride) {
        const uint64_t a = word(s[i], p[i], o[i]);
        w0[i] = (uint32_t)a;
        w1[i] = (uint32_t)(a >> 32);
    }
}

// The sorted words back to the index's two columns.  REPACK (the PSO order):
// the same triples as (p | second | first) words, the input of the POS sort
// (which then only has to sort by second and p: inside those, the order so
// far is by first), and the first position of every predicate.
template <bool REPACK>
__global__ __launch_bounds__(IX_THREADS) void unpack_triples_kernel(
    const uint32_t* __restrict__ w0, const uint32_t* __restrict__ w1, uint64_t n, int so, int32_t* __restrict__ first, int32_t* __restrict__ second, uint32_t* __restrict__ r0, uint32_t* __restrict__ r1,
    int32_t* __restrict__ pred, int64_t* __restrict__ pred_pos, uint32_t* __restrict__ npred, uint32_t cap) {
    const uint64_t t0 = blockIdx.x * (uint64_t)IX_THREADS + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * IX_THREADS;
    const uint32_t mask = (uint32_t)((1ull << so) - 1ull);
    const uint64_t groups = (n + 3) / 4;
    for (uint64_t g = t0; g < groups; g += stride) {
        const uint64_t i0 = 4 * g;
        const bool whole = i0 + 4 <= n;
        uint32_t lo[4], hi[4], f[4], c[4], p[4];
        if (whole) {
            const uint4 a = reinterpret_cast<const uint4*>(w0)[g], b = reinterpret_cast<const uint4*>(w1)[g];
            lo[0] = a.x, lo[1] = a.y, lo[2] = a.z, lo[3] = a.w;
            hi[0] = b.x, hi[1] = b.y, hi[2] = b.z, hi[3] = b.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                lo[k] = i0 + k < n ? w0[i0 + k] : 0u;
                hi[k] = i0 + k < n ? w1[i0 + k] : 0u;
            }
        }
        uint64_t r[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint64_t w = (uint64_t)hi[k] << 32 | lo[k];
            p[k] = (uint32_t)(w >> so >> so);
            f[k] = (uint32_t)(w >> so) & mask;
            c[k] = (uint32_t)w & mask;
            r[k] = REPACK ? triple_word(p[k], c[k], f[k], so) : 0ull;
        }
        if (whole) {
            reinterpret_cast<int4*>(first)[g] = make_int4(f[0], f[1], f[2], f[3]);
            reinterpret_cast<int4*>(second)[g] = make_int4(c[0], c[1], c[2], c[3]);
            if (REPACK) {
                reinterpret_cast<uint4*>(r0)[g] =
                    make_uint4((uint32_t)r[0], (uint32_t)r[1], (uint32_t)r[2], (uint32_t)r[3]);
                reinterpret_cast<uint4*>(r1)[g] = make_uint4((uint32_t)(r[0] >> 32), (uint32_t)(r[1] >> 32),
                                                             (uint32_t)(r[2] >> 32), (uint32_t)(r[3] >> 32));
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (i0 + k < n) {
                    first[i0 + k] = (int32_t)f[k];
                    second[i0 + k] = (int32_t)c[k];
                    if (REPACK) {
                        r0[i0 + k] = (uint32_t)r[k];
                        r1[i0 + k] = (uint32_t)(r[k] >> 32);
                    }
                }
        }
        if (REPACK) {
            uint32_t prev = p[0];
            if (i0) prev = (uint32_t)(((uint64_t)w1[i0 - 1] << 32 | w0[i0 - 1]) >> so >> so);
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (i0 + k < n) {
                    if (i0 + k == 0 || p[k] != prev) {
                        const uint32_t at = atomicAdd(npred, 1u);
                        if (at < cap) {
                            pred[at] = (int32_t)p[k];
                            pred_pos[at] = (int64_t)(i0 + k);
                        }
                    }
                    prev = p[k];
                }
        }
    }
}

hipError_t launch_pack_triples(const int32_t* s, const int32_t* p, const int32_t* o, uint64_t n, int32_t pmin, int so,
                               uint32_t* w0, uint32_t* w1, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (so < 0 || so > 31) return hipErrorInvalidValue;
    pack_triples_kernel<<<ix_grid(n, IX_THREADS * 8, 4096), IX_THREADS, 0, stream>>>(s, p, o, n, pmin, so, w0, w1);
    return hipGetLastError();
}

hipError_t launch_unpack_pso(const uint32_t* w0, const uint32_t* w1, uint64_t n, int so, int32_t* first, int32_t* second,
                             uint32_t* r0, uint32_t* r1, int32_t* pred, int64_t* pred_pos,
                             uint32_t* npred, uint32_t cap, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (so < 0 || so > 31) return hipErrorInvalidValue;
    unpack_triples_kernel<true><<<ix_grid(n, IX_THREADS * 8, 4096), IX_THREADS, 0, stream>>>(
        w0, w1, n, so, first, second, r0, r1, pred, pred_pos, npred, cap);
    return hipGetLastError();
}

hipError_t launch_unpack_pos(const uint32_t* w0, const uint32_t* w1, uint64_t n, int so, int32_t* first,
                             int32_t* second, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (so < 0 || so > 31) return hipErrorInvalidValue;
    unpack_triples_kernel<false><<<ix_grid(n, IX_THREADS * 8, 4096), IX_THREADS, 0, stream>>>(
        w0, w1, n, so, first, second, nullptr, nullptr, nullptr, nullptr, nullptr, 0);
    return hipGetLastError();
}

// ---- distinct values per predicate -----------------------------------------
// cnt[q] = runs of equal values in col over the rows of predicate q (its rows
// are [off[q], off[q + 1])), for the PSO subject column (blockIdx.y 0) and the
// POS object column (1).  A wave owns DIST_IPT * 64 consecutive rows: each row
// is read once (its neighbour comes from the next lane), the heads are kept as
// bit words and counted per predicate under a mask (where many predicates meet
// in a wave's rows, every head finds its predicate by itself), and the block's
// counts meet in LDS before one add per predicate, unless its rows hold more
// predicates than there is room for.  20M triples, 15 predicates: 53 us; 100
// with the row before fetched again and every head tested against the
// predicate's bounds, 627 as two launches per predicate.  Where a block of a
// small store holds several predicates, adding its heads to memory one by one
// queues them on a few words: 158,000 triples under 15 predicates take 8 us, 585
// with that, and 1M under 300 take 12, 840 with it.  A search of the whole table
// in each wave, through vector registers, took 18 us more at 50M.
constexpr int DIST_IPT = 32;
constexpr uint32_t DIST_THREADS = 1024;
constexpr uint32_t DIST_ROWS = DIST_THREADS * DIST_IPT;
constexpr uint32_t DIST_FEW = 16;    // predicates of a wave's rows that are counted under masks
constexpr uint32_t DIST_LDS = 1024;  // predicates of a block's rows that are counted in LDS

// last q of [lo, hi] with off[q] <= row (off[lo] is)
__device__ __forceinline__ uint32_t pred_at(const int64_t* __restrict__ off, uint32_t lo, uint32_t hi, int64_t row) {
    while (lo < hi) {
        const uint32_t m = (lo + hi + 1) / 2;
        if (off[m] <= row) lo = m;
        else hi = m - 1;
    }
    return lo;
}

__global__ __launch_bounds__(DIST_THREADS) void distinct_kernel(const int32_t* __restrict__ a,
                                                                const int32_t* __restrict__ b, int64_t n,
                                                                const int64_t* __restrict__ off, uint32_t np,
                                                                unsigned long long* __restrict__ cnt) {
    static_assert(DIST_IPT <= MQ_WAVE && DIST_LDS <= DIST_THREADS, "a lane per head word, a thread per count");
    __shared__ uint32_t sh[DIST_LDS];
    const int32_t* __restrict__ x = blockIdx.y ? b : a;
    unsigned long long* out = cnt + (blockIdx.y ? np : 0u);
    const int64_t r0 = (int64_t)blockIdx.x * DIST_ROWS;
    const int64_t r1 = min(r0 + (int64_t)DIST_ROWS, n);
    const uint32_t q0 = pred_at(off, 0, np - 1, r0), q1 = pred_at(off, 0, np - 1, r1 - 1);
    const bool lds = q1 - q0 < DIST_LDS;
    if (threadIdx.x < DIST_LDS) sh[threadIdx.x] = 0;
    __syncthreads();
    // in a scalar register, and so are the wave's predicates and their bounds
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MQ_WAVE);
    const int64_t w0 = r0 + (int64_t)wave * (DIST_IPT * MQ_WAVE);
    if (w0 < r1) {  // wave-uniform
        const uint32_t rows = (uint32_t)min((int64_t)(DIST_IPT * MQ_WAVE), r1 - w0);
        uint32_t before = w0 > 0 ? (uint32_t)x[w0 - 1] : ~(uint32_t)x[0];
        uint64_t word = 0;  // lane k: heads of rows [64 k, 64 k + 64) of the wave
        constexpr int PART = 16;
#pragma unroll
        for (int p = 0; p < DIST_IPT; p += PART) {
            uint32_t v[PART];
#pragma unroll
            for (int i = 0; i < PART; i++) v[i] = (uint32_t)x[w0 + min((p + i) * MQ_WAVE + lane(), rows - 1)];
#pragma unroll
            for (int i = 0; i < PART; i++) {
                const uint32_t prev = wave_prev(v[i], before);
                const uint64_t m = __ballot(prev != v[i] && (p + i) * MQ_WAVE + lane() < rows);
                before = last_lane(v[i]);
                if (lane() == (uint32_t)(p + i)) word = m;
            }
        }
        // a search among the block's predicates only: none where it holds one
        const uint32_t qa = pred_at(off, q0, q1, w0), qb = pred_at(off, q0, q1, w0 + rows - 1);
        if (qb - qa < DIST_FEW) {
            for (uint32_t q = qa; q <= qb; q++) {
                const int64_t lo = off[q] - w0, hi = off[q + 1] - w0;  // the predicate's rows, wave-relative
                const int64_t f = (int64_t)lane() * MQ_WAVE;  // the lane's first row
                uint64_t mask = ~0ull;
                if (lo > f) mask = lo - f >= MQ_WAVE ? 0ull : ~0ull << (lo - f);
                if (hi < f + MQ_WAVE) mask = hi <= f ? 0ull : mask & (~0ull >> (f + MQ_WAVE - hi));
                uint64_t heads = word;
                // a predicate's first row starts a run whatever came before it
                if (lo >= f && lo < f + MQ_WAVE) heads |= 1ull << (lo - f);
                const uint32_t c = last_lane(wave_incl_u32((uint32_t)__popcll(heads & mask)));
                if (lane() == 0 && c) {
                    if (lds) atomicAdd(&sh[q - q0], c);
                    else atomicAdd(out + q, (unsigned long long)c);
                }
            }
        } else {
            for (uint32_t k = 0; k < DIST_IPT; k++) {
                const uint64_t m = __shfl(word, (int)k);
                const uint32_t at = k * MQ_WAVE + lane();
                if (at >= rows) continue;
                const uint32_t q = pred_at(off, qa, qb, w0 + at);
                if (((m >> lane()) & 1ull) || w0 + at == off[q]) {
                    if (lds) atomicAdd(&sh[q - q0], 1u);
                    else atomicAdd(out + q, 1ull);
                }
            }
        }
    }
    __syncthreads();
    if (lds && threadIdx.x <= q1 - q0 && sh[threadIdx.x])
        atomicAdd(out + q0 + threadIdx.x, (unsigned long long)sh[threadIdx.x]);
}

hipError_t launch_distinct(const int32_t* pso_s, const int32_t* pos_o, int64_t n, const int64_t* off, uint32_t np,
                           unsigned long long* cnt, hipStream_t stream) {
    if (n == 0 || np == 0) return hipSuccess;
    const dim3 grid((uint32_t)((n - 1) / DIST_ROWS + 1), 2);
    distinct_kernel<<<grid, DIST_THREADS, 0, stream>>>(pso_s, pos_o, n, off, np, cnt);
    return hipGetLastError();
}

}  // namespace mq
