// Semi-join reduction ahead of the shuffle.  A record whose key does not
// occur on the other side of the join meets no partner in Reduce and gives
// no output row, so it need not be sorted at all.  When one side is much
// larger, the smaller side's keys go into a bitmap over the key range and
// the larger side is filtered against it in one pass that also writes the
// surviving records (relative key, record id) in input order, ready for the
// first radix pass.  Because the kept records keep their order and ids,
// the sorted sequence is the unfiltered one with only unmatched keys'
// records removed, and the join's rows come out unchanged, row for row.
#include "device_common.h"
#include "kernels.h"

#include <algorithm>

namespace mq {

// Keys outside [base, base + range) (a caller's key bound that does not hold)
// set nothing.  Repeated keys must not queue on their word, nor read it again
// and again: each block remembers the keys it set last in LDS, and where most
// of a wave's keys share a word with a neighbour (a side sorted on the key)
// the first lane of each such run sets the bits of all of them.  59M keys, 200
// distinct ones in no order: 115 us (770 with one look at the bitmap per
// key, one key per thread at a time); 10.5M ascending keys: 42 (332).
// Few, large blocks: every one of them asks for the hot words once.
constexpr uint32_t BS_THREADS = 1024, BS_BLOCKS = 512, BS_SEEN = 4096;

template <int UNROLL>
__global__ __launch_bounds__(BS_THREADS) void bitmap_set_kernel(const int32_t* __restrict__ keys, uint32_t n,
                                                              int32_t base, uint64_t range, uint32_t* __restrict__ bm) {
    __shared__ uint32_t seen[BS_SEEN];  // seen[k % BS_SEEN] == k: this block has set k
    for (uint32_t i = threadIdx.x; i < BS_SEEN; i += BS_THREADS) seen[i] = ~i;  // no key of that place
    __syncthreads();
    constexpr uint32_t TILE = BS_THREADS * UNROLL;
    const uint32_t ntiles = (n + TILE - 1) / TILE;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const uint32_t i0 = t * TILE + threadIdx.x / MQ_WAVE * (MQ_WAVE * UNROLL) + lane();
        uint32_t key[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; u++) key[u] = (uint32_t)keys[min(i0 + u * MQ_WAVE, n - 1)] - (uint32_t)base;
#pragma unroll
        for (int u = 0; u < UNROLL; u++) {
            const uint32_t k = key[u], word = k >> 5;
            uint32_t* mark = &seen[k % BS_SEEN];
            bool fresh = k < range && *mark != k;
            if (fresh) fresh = atomicExch(mark, k) != k;  // of several lanes with k, one
            if (__ballot(fresh) == 0ull) continue;
            uint32_t bits = fresh ? 1u << (k & 31u) : 0u;
            const bool follows = wave_prev(word, ~word) == word;
            if (__popcll(__ballot(follows)) >= MQ_WAVE / 2) {
                // neighbours with one word: the run's bits meet in its first lane
#pragma unroll
                for (int o = 1; o < MQ_WAVE; o <<= 1) {
                    const uint32_t w = __shfl_down(word, o, MQ_WAVE), b = __shfl_down(bits, o, MQ_WAVE);
                    if (lane() + o < MQ_WAVE && w == word) bits |= b;
                }
                if (follows) bits = 0;
            }
            if (bits && (__hip_atomic_load(&bm[word], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bits) != bits)
                atomicOr(&bm[word], bits);
        }
    }
}

// The filter in two launches over the same chunks, at most SEMI_BLOCKS of them:
// the first leaves one mask bit per record and a count per chunk, the second
// adds up the counts before its chunk and writes the kept records in input
// order.  No block waits for another: with one launch, tiles numbered by a
// counter (11 ns each) and a look-back over them took 42 us on 4M keys and 52
// on 10.5M; this takes 29 and 37.
constexpr uint32_t SEMI_THREADS = 1024, SEMI_IPT = 4, SEMI_BLOCKS = 2048;
constexpr uint32_t SEMI_TILE = SEMI_THREADS * SEMI_IPT;

__global__ __launch_bounds__(SEMI_THREADS) void semi_mask_kernel(SemiArgs a, uint32_t tiles_per) {
    __shared__ uint32_t s_wtot[SEMI_THREADS / MQ_WAVE];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    uint32_t run = 0;
    for (uint32_t t = 0; t < tiles_per; t++) {
        const uint64_t at = ((uint64_t)blockIdx.x * tiles_per + t) * SEMI_TILE + w * (SEMI_IPT * MQ_WAVE);
        if (at >= a.n) break;
        const uint32_t base = (uint32_t)at;
        uint32_t key[SEMI_IPT], word[SEMI_IPT];
#pragma unroll
        for (uint32_t i = 0; i < SEMI_IPT; i++)
            key[i] = (uint32_t)a.keys[min(base + i * MQ_WAVE + lane(), a.n - 1)] - (uint32_t)a.base;
#pragma unroll
        for (uint32_t i = 0; i < SEMI_IPT; i++) word[i] = a.bm[key[i] < a.range ? key[i] >> 5 : 0u];
#pragma unroll
        for (uint32_t i = 0; i < SEMI_IPT; i++) {
            const uint32_t first = base + i * MQ_WAVE;
            const uint64_t m =
                __ballot(first + lane() < a.n && key[i] < a.range && ((word[i] >> (key[i] & 31u)) & 1u));
            if (lane() == 0 && first < a.n) a.masks[first / MQ_WAVE] = m;
            run += (uint32_t)__popcll(m);
        }
    }
    if (lane() == 0) s_wtot[w] = run;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t i = 1; i < SEMI_THREADS / MQ_WAVE; i++) run += s_wtot[i];
        a.counts[blockIdx.x] = run;
    }
}

__global__ __launch_bounds__(SEMI_THREADS) void semi_write_kernel(SemiArgs a, uint32_t tiles_per, Mail mail) {
    constexpr uint32_t WAVES = SEMI_THREADS / MQ_WAVE;
    __shared__ uint32_t s_w[2][WAVES];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint64_t lt = lanemask_lt();
    uint32_t before = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += SEMI_THREADS) before += a.counts[i];
    before = (uint32_t)wave_sum((uint64_t)before);
    if (lane() == 0) s_w[0][w] = before;
    __syncthreads();
    uint32_t pos = 0;
    for (uint32_t i = 0; i < WAVES; i++) pos += s_w[0][i];
    const uint32_t mine = a.counts[blockIdx.x];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        *a.count = pos + mine;
        mail.data[0] = pos + mine;
        mail_post(mail);
    }
    if (mine == 0) return;
    for (uint32_t t = 0; t < tiles_per; t++) {
        const uint64_t tile0 = ((uint64_t)blockIdx.x * tiles_per + t) * SEMI_TILE;
        if (tile0 >= a.n) break;
        const uint64_t at0 = tile0 + w * (SEMI_IPT * MQ_WAVE);
        uint64_t km[SEMI_IPT];
        uint32_t run = 0;
#pragma unroll
        for (uint32_t i = 0; i < SEMI_IPT; i++) {
            km[i] = at0 + i * MQ_WAVE < a.n ? a.masks[at0 / MQ_WAVE + i] : 0ull;
            run += (uint32_t)__popcll(km[i]);
        }
        if (lane() == 0) s_w[(t + 1) & 1][w] = run;  // the other buffer: the last one is still read
        __syncthreads();
        uint32_t wex = 0, all = 0;
        for (uint32_t i = 0; i < WAVES; i++) {
            const uint32_t c = s_w[(t + 1) & 1][i];
            wex += i < w ? c : 0u;
            all += c;
        }
        uint32_t at = pos + wex;
        pos += all;
#pragma unroll
        for (uint32_t i = 0; i < SEMI_IPT; i++) {
            if ((km[i] >> lane()) & 1ull) {
                const uint32_t idx = (uint32_t)at0 + i * MQ_WAVE + lane();
                const uint32_t o = at + (uint32_t)__popcll(km[i] & lt);
                a.kout[o] = (uint32_t)a.keys[idx] - (uint32_t)a.base;
                a.vout[o] = a.id_base + idx;
            }
            at += (uint32_t)__popcll(km[i]);
        }
    }
}

// Every record of one side, written from position (*at_dev if given) + i.
__global__ __launch_bounds__(MQ_BLOCK) void side_records_kernel(const int32_t* __restrict__ keys, uint32_t n,
                                                                int32_t base, uint32_t mask, uint32_t id_base,
                                                                const uint32_t* __restrict__ at_dev,
                                                                uint32_t* __restrict__ kout,
                                                                uint32_t* __restrict__ vout) {
    const uint32_t at = at_dev ? *at_dev : 0u;
    for (uint32_t i = blockIdx.x * MQ_BLOCK + threadIdx.x; i < n; i += gridDim.x * MQ_BLOCK) {
        kout[at + i] = ((uint32_t)keys[i] - (uint32_t)base) & mask;
        vout[at + i] = id_base + i;
    }
}

hipError_t launch_bitmap_set(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, uint32_t* bm,
                             hipStream_t stream) {
    if (n == 0) return hipSuccess;
    // a small side: one key per thread, all chains of loads and atomics side by side
    if (n <= BS_THREADS * BS_BLOCKS)
        bitmap_set_kernel<1><<<(n - 1) / BS_THREADS + 1, BS_THREADS, 0, stream>>>(keys, n, base, range, bm);
    else
        bitmap_set_kernel<16><<<BS_BLOCKS, BS_THREADS, 0, stream>>>(keys, n, base, range, bm);
    return hipGetLastError();
}

static uint32_t semi_tiles(uint32_t n) { return (n - 1) / SEMI_TILE + 1; }

hipError_t launch_semi_filter(const SemiArgs& args, void* scratch, Mail mail, hipStream_t stream) {
    if (args.n == 0) return hipSuccess;
    const uint32_t tiles = semi_tiles(args.n), per = (tiles - 1) / SEMI_BLOCKS + 1;
    const uint32_t blocks = (tiles - 1) / per + 1;
    SemiArgs a = args;
    a.masks = static_cast<uint64_t*>(scratch);
    a.counts = reinterpret_cast<uint32_t*>(a.masks + ((size_t)a.n - 1) / MQ_WAVE + 1);
    semi_mask_kernel<<<blocks, SEMI_THREADS, 0, stream>>>(a, per);
    semi_write_kernel<<<blocks, SEMI_THREADS, 0, stream>>>(a, per, mail);
    return hipGetLastError();
}

size_t semi_scratch_bytes(uint32_t n) {
    return n == 0 ? 0 : (((size_t)n - 1) / MQ_WAVE + 1) * 8 + (size_t)std::min(semi_tiles(n), SEMI_BLOCKS) * 4;
}

hipError_t launch_side_records(const int32_t* keys, uint32_t n, int32_t base, uint32_t mask, uint32_t id_base,
                               const uint32_t* at_dev, uint32_t* kout, uint32_t* vout, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t blocks = std::min<uint32_t>((n + MQ_BLOCK - 1) / MQ_BLOCK, 2048u);
    side_records_kernel<<<blocks, MQ_BLOCK, 0, stream>>>(keys, n, base, mask, id_base, at_dev, kout, vout);
    return hipGetLastError();
}

}  // namespace mq

namespace mq {

// Exact |RS| before any shuffle: the smaller side's keys are counted into a
// dense array over the key range, then every record of the larger side
// adds the count of its key (sum over keys of cL * cR, Algorithm 1's
// ReduceDuplicate without grouping).  Keys outside [base, base + range)
// count nothing.
// Each thread counts 16 consecutive keys, one atomic per run of equal keys;
// when the wave's 1024 keys are all one key (a hot key of a key-sorted
// side) one atomic counts them all, so hot keys do not serialise.
constexpr int KC_IPT = 16;

__global__ __launch_bounds__(MQ_BLOCK) void key_count_kernel(const int32_t* __restrict__ keys, uint32_t n, int32_t base,
                                                             uint64_t range, uint32_t* __restrict__ cnt) {
    constexpr uint32_t TILE = MQ_BLOCK * KC_IPT;
    for (uint64_t t0 = (uint64_t)blockIdx.x * TILE; t0 < n; t0 += (uint64_t)gridDim.x * TILE) {
        const uint64_t first = t0 + (uint64_t)threadIdx.x * KC_IPT;
        uint32_t k[KC_IPT];
#pragma unroll
        for (int i = 0; i < KC_IPT; i++)
            k[i] = first + i < n ? (uint32_t)keys[first + i] - (uint32_t)base : 0xffffffffu;
        const int cnt_here = first >= n ? 0 : (int)min((uint64_t)KC_IPT, n - first);
        const bool full = __ballot(cnt_here == KC_IPT) == ~0ull;
        const uint32_t k0 = __shfl(k[0], 0, MQ_WAVE), k1 = __shfl(k[KC_IPT - 1], MQ_WAVE - 1, MQ_WAVE);
        if (full && k0 == k1) {
            // sorted input, one key over the whole wave (unsorted input with
            // this property is one key too: the test is exact either way)
            bool same = true;
#pragma unroll
            for (int i = 0; i < KC_IPT; i++) same = same && k[i] == k0;
            if (__ballot(!same) == 0ull) {
                if (lane() == 0 && k0 < range) atomicAdd(&cnt[k0], (uint32_t)(MQ_WAVE * KC_IPT));
                continue;
            }
        }
        uint32_t cur = k[0], run = 0;
#pragma unroll
        for (int i = 0; i < KC_IPT; i++) {
            if (i < cnt_here) {
                if (k[i] != cur) {
                    if (cur < range) atomicAdd(&cnt[cur], run);
                    cur = k[i];
                    run = 0;
                }
                run++;
            }
        }
        if (run && cur < range) atomicAdd(&cnt[cur], run);
    }
}

__global__ __launch_bounds__(MQ_BLOCK) void key_dot_kernel(const int32_t* __restrict__ keys, uint32_t n, int32_t base,
                                                           uint64_t range, const uint32_t* __restrict__ cnt,
                                                           unsigned long long* __restrict__ total) {
    __shared__ uint64_t s_w[MQ_WAVES];
    uint64_t acc = 0;
    for (uint32_t i = blockIdx.x * MQ_BLOCK + threadIdx.x; i < n; i += gridDim.x * MQ_BLOCK) {
        const uint32_t k = (uint32_t)keys[i] - (uint32_t)base;
        if (k < range) acc += cnt[k];
    }
    acc = wave_sum(acc);
    if (lane() == 0) s_w[threadIdx.x / MQ_WAVE] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int w = 0; w < MQ_WAVES; w++) t += s_w[w];
        if (t) atomicAdd(total, (unsigned long long)t);
    }
}

// The same sum over one key of every aligned block of 64, chosen by a hash of
// the block: 64 times it estimates |RS|.  The counters are a 64th of the
// range (1 MB for 24-bit keys, so they stay in L2) and so are the atomics;
// what is left is one read of both key columns.
__device__ __forceinline__ bool sampled(uint32_t k) {
    return (((k >> 6) * 0x9E3779B1u) >> 26) == (k & 63u);
}
constexpr int KS_UNROLL = 8;
// few, large blocks: the two atomics that end each block of the sum queue on
// one address (16M keys: 41 us, against 78 with 2,048 blocks of 256 threads)
constexpr uint32_t KS_BLOCKS = 512, KS_THREADS = 1024;
// Each block counts the keys it meets in a table in LDS (a place per key, the
// first one there has it; the others count in memory) and adds its counts at
// the end: the atomics of a few keys, whose counters share a line, would queue
// on it (9M keys of 1,000 values: 1.59 ms, 15 us with the table; of 8M values 14.6
// and 14.5 us).
constexpr uint32_t KS_PLACES = 2048;

__global__ __launch_bounds__(KS_THREADS) void sample_count_kernel(const int32_t* __restrict__ keys, uint32_t n,
                                                                int32_t base, uint64_t range,
                                                                uint32_t* __restrict__ cnt) {
    __shared__ uint32_t s_key[KS_PLACES], s_cnt[KS_PLACES];
    for (uint32_t i = threadIdx.x; i < KS_PLACES; i += KS_THREADS) {
        s_key[i] = ~0u;  // no counter's number: those stay below 2^26
        s_cnt[i] = 0;
    }
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * KS_THREADS;
    for (uint64_t i0 = blockIdx.x * (uint64_t)KS_THREADS + threadIdx.x; i0 < n; i0 += stride * KS_UNROLL) {
        uint32_t k[KS_UNROLL];
#pragma unroll
        for (int u = 0; u < KS_UNROLL; u++) {
            const uint64_t i = i0 + u * stride;
            k[u] = i < n ? (uint32_t)keys[i] - (uint32_t)base : ~0u;
        }
#pragma unroll
        for (int u = 0; u < KS_UNROLL; u++) {
            if (i0 + u * stride < n && k[u] < range && sampled(k[u])) {  // about one lane in 64
                const uint32_t c = k[u] >> 6, at = c % KS_PLACES;
                const uint32_t has = atomicCAS(&s_key[at], ~0u, c);
                if (has == ~0u || has == c)
                    atomicAdd(&s_cnt[at], 1u);
                else
                    atomicAdd(&cnt[c], 1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < KS_PLACES; i += KS_THREADS)
        if (s_cnt[i]) atomicAdd(&cnt[s_key[i]], s_cnt[i]);
}

// acc: a 64-bit sum and a word of finished blocks, 0 before and after
__global__ __launch_bounds__(KS_THREADS) void sample_dot_kernel(const int32_t* __restrict__ keys, uint32_t n,
                                                              int32_t base, uint64_t range,
                                                              const uint32_t* __restrict__ cnt,
                                                              uint32_t* __restrict__ acc, Mail mail) {
    __shared__ uint64_t s_w[KS_THREADS / MQ_WAVE];
    const uint64_t stride = (uint64_t)gridDim.x * KS_THREADS;
    uint64_t sum = 0;
    for (uint64_t i0 = blockIdx.x * (uint64_t)KS_THREADS + threadIdx.x; i0 < n; i0 += stride * KS_UNROLL) {
        uint32_t k[KS_UNROLL];
#pragma unroll
        for (int u = 0; u < KS_UNROLL; u++) {
            const uint64_t i = i0 + u * stride;
            k[u] = i < n ? (uint32_t)keys[i] - (uint32_t)base : ~0u;
        }
#pragma unroll
        for (int u = 0; u < KS_UNROLL; u++)
            if (i0 + u * stride < n && k[u] < range && sampled(k[u])) sum += cnt[k[u] >> 6];
    }
    sum = wave_sum(sum);
    if (lane() == 0) s_w[threadIdx.x / MQ_WAVE] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < KS_THREADS / MQ_WAVE; w++) sum += s_w[w];
        unsigned long long* total = reinterpret_cast<unsigned long long*>(acc);
        atomicAdd(total, (unsigned long long)sum);
        __threadfence();
        if (atomicAdd(acc + 2, 1u) + 1 == gridDim.x) {
            __threadfence();
            const uint64_t t = atomicExch(total, 0ull);
            atomicExch(acc + 2, 0u);
            mail.data[0] = (uint32_t)t;
            mail.data[1] = (uint32_t)(t >> 32);
            mail_post(mail);
        }
    }
}

hipError_t launch_key_sample(const int32_t* a, uint32_t na, const int32_t* b, uint32_t nb, int32_t base,
                             uint64_t range, uint32_t* cnt, uint32_t* acc, Mail mail, hipStream_t stream) {
    auto blocks = [](uint32_t n) { return std::max(1u, std::min(n / (KS_THREADS * KS_UNROLL), KS_BLOCKS)); };
    hipError_t e = launch_fill_u32(cnt, key_sample_words(range), 0u, stream);
    if (e != hipSuccess) return e;
    sample_count_kernel<<<blocks(na), KS_THREADS, 0, stream>>>(a, na, base, range, cnt);
    sample_dot_kernel<<<blocks(nb), KS_THREADS, 0, stream>>>(b, nb, base, range, cnt, acc, mail);
    return hipGetLastError();
}

hipError_t launch_key_count(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, uint32_t* cnt,
                            hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t blocks = std::min<uint32_t>((n + MQ_BLOCK * KC_IPT - 1) / (MQ_BLOCK * KC_IPT), 4096u);
    key_count_kernel<<<blocks, MQ_BLOCK, 0, stream>>>(keys, n, base, range, cnt);
    return hipGetLastError();
}

hipError_t launch_key_dot(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, const uint32_t* cnt,
                          uint64_t* total, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t blocks = std::min<uint32_t>((n + MQ_BLOCK * 8 - 1) / (MQ_BLOCK * 8), 4096u);
    key_dot_kernel<<<blocks, MQ_BLOCK, 0, stream>>>(keys, n, base, range, cnt,
                                                    reinterpret_cast<unsigned long long*>(total));
    return hipGetLastError();
}

}  // namespace mq
