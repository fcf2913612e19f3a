// Sort and ReduceDuplicate of a small join in one block: up to SMALL_JOIN
// records are sorted in LDS and their segments, counts and offsets written
// out, so the whole join is this launch and the materialisation.  A small join
// is bound by its launches: 1,800 records took seven of them (histogram, its
// sum, two passes, three for the segments), 20 us of kernels and as much again
// between them; this one takes 11 us.
#include "device_common.h"
#include "kernels.h"
#include "tile_ops.h"

namespace mq {

constexpr int SJ_WAVES = 16, SJ_KPT = 4, SJ_BITS = 8;
constexpr uint32_t SJ_THREADS = SJ_WAVES * MQ_WAVE;
static_assert(SMALL_JOIN == SJ_THREADS * SJ_KPT, "one tile");

struct SmallSmem {
    uint32_t keys[SMALL_JOIN];
    uint32_t vals[SMALL_JOIN];
    uint32_t start[SMALL_JOIN];
    uint32_t split[SMALL_JOIN];
    uint16_t wcnt[SJ_WAVES][1 << SJ_BITS];  // per wave and digit: count, then first place
    uint32_t tmp[2][SJ_WAVES];
};

// exclusive prefix of v over the block's threads and their sum; `tmp` is free
// again after the next barrier
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* tmp, uint32_t& all) {
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t inc = wave_incl_u32(v);
    if (lane() == MQ_WAVE - 1) tmp[w] = inc;
    __syncthreads();
    uint32_t before = 0;
    all = 0;
#pragma unroll
    for (int i = 0; i < SJ_WAVES; i++) {
        before += (uint32_t)i < w ? tmp[i] : 0u;
        all += tmp[i];
    }
    return before + inc - v;
}

__global__ __launch_bounds__(SJ_THREADS) void small_join_kernel(SmallJoin a, Mail mail) {
    __shared__ SmallSmem sm;
    const uint32_t w = threadIdx.x / MQ_WAVE, t = threadIdx.x;
    const uint32_t n = a.n;
    const uint32_t o0 = w * SJ_KPT * MQ_WAVE + lane();
    uint32_t key[SJ_KPT], val[SJ_KPT];
    // records in input order, wave-striped; past the end padding keys of all
    // ones, which stay behind every record
#pragma unroll
    for (int i = 0; i < SJ_KPT; i++) {
        const uint32_t at = o0 + i * MQ_WAVE, idx = min(at, n - 1);
        if (a.kin) {
            key[i] = a.kin[idx];
            val[i] = a.vin[idx];
        } else {
            const bool right = idx >= a.src.n0;
            const uint32_t r = right ? idx - a.src.n0 : idx;
            const uint32_t rel = ((uint32_t)(right ? a.src.k1 : a.src.k0)[r] - (uint32_t)a.src.base) & a.src.mask;
            key[i] = a.src.carry ? rel << 1 | (right ? 1u : 0u) : rel;
            val[i] = a.src.carry ? (uint32_t)(right ? a.src.v1 : a.src.v0)[r] : idx;
        }
        if (at >= n) key[i] = 0xffffffffu;
    }

    // stable LSD passes over key bits [lo_bit, lo_bit + key_bits)
    uint16_t* cnt = sm.wcnt[w];
    const uint32_t end = (uint32_t)(a.lo_bit + a.key_bits);
    for (uint32_t shift = (uint32_t)a.lo_bit; shift < end; shift += (uint32_t)a.width) {
        const uint32_t nb = min((uint32_t)a.width, end - shift), mask = (1u << nb) - 1u;
        for (uint32_t d = lane(); d < (1u << SJ_BITS) / 2; d += MQ_WAVE) reinterpret_cast<uint32_t*>(cnt)[d] = 0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t rank[SJ_KPT];
#pragma unroll
        for (int i = 0; i < SJ_KPT; i++) {
            const uint32_t x = key[i] >> shift, dg = x & mask;
            uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
            for (int b = 0; b < SJ_BITS; b++) {
                if ((uint32_t)b < nb) {
                    const uint32_t spread = bit_spread(x, b);
                    const uint64_t m = __ballot(spread != 0);
                    lo = and_xnor(lo, (uint32_t)m, spread);
                    hi = and_xnor(hi, (uint32_t)(m >> 32), spread);
                }
            }
            const uint32_t old = cnt[dg];
            rank[i] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, old));
            __builtin_amdgcn_wave_barrier();
            if (rank[i] == old) cnt[dg] = (uint16_t)(old + __popc(lo) + __popc(hi));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // each digit's records: over the waves, then over the digits
        uint32_t run = 0, all;
        if (t < (1u << SJ_BITS)) {
#pragma unroll
            for (int i = 0; i < SJ_WAVES; i++) {
                const uint32_t c = sm.wcnt[i][t];
                sm.wcnt[i][t] = (uint16_t)run;
                run += c;
            }
        }
        const uint32_t ex = block_prefix(run, sm.tmp[0], all);
        if (t < (1u << SJ_BITS)) {
#pragma unroll
            for (int i = 0; i < SJ_WAVES; i++) sm.wcnt[i][t] = (uint16_t)(sm.wcnt[i][t] + ex);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SJ_KPT; i++) {
            const uint32_t place = cnt[(key[i] >> shift) & mask] + rank[i];
            sm.keys[place] = key[i];
            sm.vals[place] = val[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SJ_KPT; i++) {
            key[i] = sm.keys[o0 + i * MQ_WAVE];
            val[i] = sm.vals[o0 + i * MQ_WAVE];
        }
    }
    if (a.key_bits == 0) {  // one key: the input order is the sorted one
#pragma unroll
        for (int i = 0; i < SJ_KPT; i++) {
            sm.keys[o0 + i * MQ_WAVE] = key[i];
            sm.vals[o0 + i * MQ_WAVE] = val[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < SJ_KPT; i++) {
        const uint32_t at = o0 + i * MQ_WAVE;
        if (at < n) {
            a.kout[at] = key[i];
            a.vout[at] = val[i];
        }
    }

    // segments: a thread takes SJ_KPT consecutive records
    const uint32_t fs = a.side_bit ? 1u : 0u;
    auto right_of = [&](uint32_t i) { return fs ? (sm.keys[i] & 1u) != 0 : sm.vals[i] >= a.n_left; };
    uint32_t heads = 0, rights = 0, h = 0;  // bit j: record SJ_KPT * t + j
    const uint32_t i0 = t * SJ_KPT;
#pragma unroll
    for (int j = 0; j < SJ_KPT; j++) {
        const uint32_t i = i0 + j;
        if (i < n) {
            if (i == 0 || sm.keys[i - 1] >> fs != sm.keys[i] >> fs) {
                heads |= 1u << j;
                h++;
            }
            if (right_of(i)) rights |= 1u << j;
        }
    }
    uint32_t nseg;
    uint32_t sid = block_prefix(h, sm.tmp[1], nseg);  // heads before this thread's records
    bool prev_right = i0 > 0 && i0 < n && right_of(i0 - 1);
#pragma unroll
    for (int j = 0; j < SJ_KPT; j++) {
        const uint32_t i = i0 + j;
        if (i >= n) break;
        const bool head = (heads >> j) & 1u, right = (rights >> j) & 1u;
        if (head) sm.start[sid++] = i;
        const bool last = i + 1 == n || sm.keys[i + 1] >> fs != sm.keys[i] >> fs;
        // one record of each segment writes its split: the first RIGHT one, or
        // the last one of a segment without
        if (right ? head || !prev_right : last) sm.split[sid - 1] = right ? i : i + 1;
        prev_right = right;
    }
    __syncthreads();
    // at most 2,048 x 2,048 pairs in all: 32 bits
    uint32_t c[SJ_KPT], sum = 0, mx = 0;
#pragma unroll
    for (int j = 0; j < SJ_KPT; j++) {
        const uint32_t s = i0 + j;
        c[j] = 0;
        if (s < nseg) {
            const uint32_t st = sm.start[s], sp = sm.split[s], en = s + 1 < nseg ? sm.start[s + 1] : n;
            c[j] = (sp - st) * (en - sp);
        }
        sum += c[j];
        mx = max(mx, c[j]);
    }
    uint32_t total;
    uint32_t off = block_prefix(sum, sm.tmp[0], total);
#pragma unroll
    for (int j = 0; j < SJ_KPT; j++) {
        const uint32_t s = i0 + j;
        if (s < nseg) {
            a.seg_start[s] = sm.start[s];
            a.seg_split[s] = sm.split[s];
            a.seg_off[s] = off;
        }
        off += c[j];
    }
    mx = wave_max_u32(mx);
    __syncthreads();
    if (lane() == MQ_WAVE - 1) sm.tmp[1][w] = mx;
    __syncthreads();
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < SJ_WAVES; i++) mx = max(mx, sm.tmp[1][i]);
        *a.nseg = nseg;
        mail.data[0] = nseg;
        mail.data[2] = total;
        mail.data[3] = 0;
        mail.data[4] = mx;
        mail.data[5] = 0;
        mail_post(mail);
    }
}

hipError_t launch_small_join(SmallJoin a, Mail mail, hipStream_t stream) {
    if (a.n == 0 || a.n > SMALL_JOIN || a.lo_bit < 0 || a.key_bits < 0 || a.lo_bit + a.key_bits > 32)
        return hipErrorInvalidValue;
    a.width = small_join_width(a.key_bits);
    small_join_kernel<<<1, SJ_THREADS, 0, stream>>>(a, mail);
    return hipGetLastError();
}

}  // namespace mq
