// Reduce without a shuffle for two tables already in key order (a view of
// the PSO or POS index whose next sort column is the key, or the result of
// a join on the same key).  The stable sort of the two sides' records would
// be their merge, LEFT before RIGHT within a key, so the segments of
// Algorithm 1's ReduceDuplicate are the two sides' runs of each key: one
// pass over the smaller side finds, at the head of each run, the run's end
// (galloping) and the key's run in the larger side (binary search).  Keys on
// both sides become segments in ascending key order, with cL * cR output
// rows each; their count and offsets come from two decoupled look-backs, which
// two waves of a block do side by side (64,000 keys in 500K: 16 us, 18 in turn).
// Materialisation then reads both tables' columns in place.
#include "device_common.h"
#include "kernels.h"

#include <algorithm>

namespace mq {

// one smaller-side record per thread: the searches of a thread cannot
// overlap, those of different threads do
constexpr int MRG_IPT = 1;

// first index in [lo, hi) with a[i] >= v (a ascending)
__device__ __forceinline__ uint32_t lower_bound_i32(const int32_t* __restrict__ a, uint32_t lo, uint32_t hi,
                                                    int32_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// first index in [lo, hi) with a[i] > v (a ascending)
__device__ __forceinline__ uint32_t upper_bound_i32(const int32_t* __restrict__ a, uint32_t lo, uint32_t hi,
                                                    int32_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] <= v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// end of the run of v that starts at i (a[i] == v, a ascending, n < 2^31):
// gallop, then binary search; short runs cost a load or two
__device__ __forceinline__ uint32_t run_end(const int32_t* __restrict__ a, uint32_t i, uint32_t n, int32_t v) {
    uint32_t lo = i + 1, step = 1;  // a[lo - 1] == v
    for (;;) {
        const uint32_t probe = (uint32_t)min((uint64_t)n, (uint64_t)i + step);
        if (probe == n || a[probe] != v) return upper_bound_i32(a, lo, probe, v);
        lo = probe + 1;
        step <<= 1;
    }
}

// Both bounds of v in b[0, n) at once: lower (first b[i] >= v) and upper
// (first b[i] > v).  A table of MRG_SAMPLES evenly spaced keys in LDS gives
// each bound's bracket; the two global binary searches then run
// interleaved, so their loads overlap.
constexpr int MRG_SAMPLES = 2048;

__device__ __forceinline__ uint32_t sample_pos(uint32_t j, uint32_t n) {
    return (uint32_t)(((uint64_t)j * n) / MRG_SAMPLES);
}

__device__ __forceinline__ void bounds_i32(const int32_t* __restrict__ b, uint32_t n, const int32_t* samp, int32_t v,
                                           uint32_t& lower, uint32_t& upper) {
    // samples below v (jl) and at most v (ju), by binary search in LDS
    uint32_t jl = 0, jh = MRG_SAMPLES, ul = 0, uh = MRG_SAMPLES;
    while (jl < jh) {
        const uint32_t m = (jl + jh) >> 1;
        if (samp[m] < v) jl = m + 1;
        else jh = m;
    }
    while (ul < uh) {
        const uint32_t m = (ul + uh) >> 1;
        if (samp[m] <= v) ul = m + 1;
        else uh = m;
    }
    // the bound lies in (pos(j - 1), pos(j)], with pos(-1) = -1 and pos(S) = n
    uint32_t l0 = jl == 0 ? 0u : sample_pos(jl - 1, n) + 1, l1 = jl == MRG_SAMPLES ? n : sample_pos(jl, n);
    uint32_t u0 = ul == 0 ? 0u : sample_pos(ul - 1, n) + 1, u1 = ul == MRG_SAMPLES ? n : sample_pos(ul, n);
    while (l0 < l1 || u0 < u1) {
        const uint32_t lm = l0 + ((l1 - l0) >> 1), um = u0 + ((u1 - u0) >> 1);
        const bool lgo = l0 < l1, ugo = u0 < u1;
        const int32_t lv = lgo ? b[lm] : 0, uv = ugo ? b[um] : 0;
        if (lgo) {
            if (lv < v) l0 = lm + 1;
            else l1 = lm;
        }
        if (ugo) {
            if (uv <= v) u0 = um + 1;
            else u1 = um;
        }
    }
    lower = l0;
    upper = u0;
}

__global__ __launch_bounds__(MQ_BLOCK) void merge_segments_kernel(MergeArgs a, uint64_t* __restrict__ status,
                                                                  uint32_t* __restrict__ tile_ctr, uint32_t epoch,
                                                                  Mail mail) {
    constexpr uint32_t TILE = MQ_BLOCK * MRG_IPT;
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_wseg[MQ_WAVES];
    __shared__ uint64_t s_wrow[MQ_WAVES];
    __shared__ uint64_t s_ex[2];
    __shared__ int32_t s_samp[MRG_SAMPLES];
    const uint32_t ntiles = (a.ns + TILE - 1) / TILE;
    uint64_t* st_seg = status;           // segment counts
    uint64_t* st_row = status + ntiles;  // output rows
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint64_t lt = lanemask_lt();
    // nb >= 1: the caller returns early on an empty side
    for (uint32_t j = threadIdx.x; j < MRG_SAMPLES; j += MQ_BLOCK) s_samp[j] = a.bkey[sample_pos(j, a.nb)];
    __syncthreads();
    for (;;) {
        const uint32_t tile = next_tile(tile_ctr, &s_tile, ntiles + gridDim.x);
        if (tile >= ntiles) break;
        const uint32_t base = tile * TILE;
        uint32_t bl[MRG_IPT], bc[MRG_IPT], sc[MRG_IPT];
        uint64_t km[MRG_IPT];
        uint64_t rows[MRG_IPT];
        uint32_t wseg = 0;
        uint64_t wrow = 0;
#pragma unroll
        for (int k = 0; k < MRG_IPT; k++) {
            const uint32_t idx = base + (w * MRG_IPT + k) * MQ_WAVE + lane();
            bool keep = false;
            bl[k] = bc[k] = sc[k] = 0;
            if (idx < a.ns) {
                const int32_t key = a.skey[idx];
                if (idx == 0 || a.skey[idx - 1] != key) {
                    uint32_t lb, ub;
                    bounds_i32(a.bkey, a.nb, s_samp, key, lb, ub);
                    if (ub > lb) {
                        bl[k] = lb;
                        bc[k] = ub - lb;
                        sc[k] = run_end(a.skey, idx, a.ns, key) - idx;
                        keep = true;
                    }
                }
            }
            km[k] = __ballot(keep);
            rows[k] = keep ? (uint64_t)sc[k] * bc[k] : 0ull;
            wseg += (uint32_t)__popcll(km[k]);
            wrow += wave_sum(rows[k]);
        }
        if (lane() == 0) {
            s_wseg[w] = wseg;
            s_wrow[w] = wrow;
        }
        __syncthreads();
        uint32_t seg_before = 0, seg_tot = 0;
        uint64_t row_before = 0, row_tot = 0;
#pragma unroll
        for (int i = 0; i < MQ_WAVES; i++) {
            if ((uint32_t)i < w) {
                seg_before += s_wseg[i];
                row_before += s_wrow[i];
            }
            seg_tot += s_wseg[i];
            row_tot += s_wrow[i];
        }
        // two waves look back side by side, one for the segments, one for the rows
        if (w < 2) {
            const uint64_t ex = tile_prefix_wave0(w == 0 ? st_seg : st_row, tile, epoch, w == 0 ? seg_tot : row_tot);
            if (lane() == 0) s_ex[w] = ex;
        }
        __syncthreads();
        if (tile == ntiles - 1 && threadIdx.x == 0) {
            const uint32_t nseg = (uint32_t)s_ex[0] + seg_tot;
            const uint64_t total = sat_add(s_ex[1], row_tot > SAT40 ? SAT40 : row_tot);
            *a.nseg = nseg;
            mail.data[0] = nseg;
            mail.data[2] = (uint32_t)total;
            mail.data[3] = (uint32_t)(total >> 32);
            mail_post(mail);
        }
        uint32_t sp = (uint32_t)s_ex[0] + seg_before;
        uint64_t rp = sat_add(s_ex[1], row_before);
#pragma unroll
        for (int k = 0; k < MRG_IPT; k++) {
            const uint64_t rincl = wave_incl_scan(rows[k]);
            if ((km[k] >> lane()) & 1ull) {
                const uint32_t idx = base + (w * MRG_IPT + k) * MQ_WAVE + lane();
                const uint32_t at = sp + (uint32_t)__popcll(km[k] & lt);
                const uint32_t ls = a.small_is_left ? idx : bl[k], lc = a.small_is_left ? sc[k] : bc[k];
                const uint32_t rs = a.small_is_left ? bl[k] : idx, rc = a.small_is_left ? bc[k] : sc[k];
                a.seg_lstart[at] = ls;
                a.seg_lcount[at] = lc;
                a.seg_rstart[at] = rs;
                a.seg_rcount[at] = rc;
                a.seg_off[at] = sat_add(rp, rincl - rows[k]);
            }
            sp += (uint32_t)__popcll(km[k]);
            rp = sat_add(rp, __shfl(rincl, MQ_WAVE - 1, MQ_WAVE));
        }
    }
}

// The same for a small side of at most MRG_FEW rows, where the pass above is a
// chain: the samples' fetch, 22 steps in LDS, then a load per halving.  Here
// MRG_GROUP lanes search for one key together, so a level takes 1/16 of the
// bracket (500K keys: five loads one after the other), and the run's end on the
// small side is one more load beside them; two waves look back at once.  60,
// 1,000 and 8,000 keys in 500K: 5, 8 and 9.6 us (8, 10.5 and 12.7 above).  At
// 64,000 keys the 16 lanes a key are too many: 33 us against 16; 16,000 are even.
constexpr int MRG_GROUP = 16;
constexpr uint32_t MRG_FEW = 8192;
constexpr uint32_t FEW_THREADS = 1024, FEW_TILE = FEW_THREADS / MRG_GROUP;
static_assert(FEW_TILE == MQ_WAVE, "one wave takes the tile's keys");

__global__ __launch_bounds__(FEW_THREADS) void merge_few_kernel(MergeArgs a, uint64_t* __restrict__ status,
                                                                uint32_t* __restrict__ tile_ctr, uint32_t epoch,
                                                                Mail mail) {
    __shared__ uint32_t s_tile;
    __shared__ uint64_t s_ex[2];
    __shared__ uint32_t s_bl[FEW_TILE], s_bc[FEW_TILE], s_sc[FEW_TILE];
    const uint32_t ntiles = gridDim.x;
    const uint32_t tile = next_tile(tile_ctr, &s_tile, ntiles);
    const uint32_t slot = threadIdx.x / MRG_GROUP, gl = threadIdx.x % MRG_GROUP;
    const uint32_t idx = tile * FEW_TILE + slot;
    uint32_t bl = 0, bc = 0, sc = 0;
    if (idx < a.ns) {
        const int32_t key = a.skey[idx];
        const int32_t prev = a.skey[idx ? idx - 1 : 0u];
        const uint32_t ahead = idx + 1 + gl;
        const int32_t next = a.skey[min(ahead, a.ns - 1)];
        if (idx == 0 || prev != key) {
            const uint64_t same = __ballot(ahead < a.ns && next == key) >> (lane() - gl) & ((1ull << MRG_GROUP) - 1);
            uint32_t ub;
            group_bounds<MRG_GROUP, uint32_t>(a.bkey, 0u, a.nb, key, bl, ub);
            bc = ub - bl;
            sc = 1 + (uint32_t)__popcll(same);
            if (bc && sc == MRG_GROUP + 1) {  // a longer run: the rows of one key are a prefix of the rest
                uint32_t none, end;
                group_bounds<MRG_GROUP, uint32_t>(a.skey, idx + sc, a.ns, key, none, end);
                sc = end - idx;
            }
        }
    }
    if (gl == 0) {
        s_bl[slot] = bl;
        s_bc[slot] = bc;
        s_sc[slot] = sc;
    }
    __syncthreads();
    // two waves look back side by side, one for the segments, one for the rows
    const uint32_t w = threadIdx.x / MQ_WAVE;
    bl = s_bl[lane()];
    bc = s_bc[lane()];
    sc = s_sc[lane()];
    const uint64_t km = __ballot(bc != 0);
    const uint64_t rows = (uint64_t)sc * bc;
    const uint64_t rincl = wave_incl_scan(rows);
    const uint64_t seg_tot = (uint64_t)__popcll(km), row_tot = __shfl(rincl, MQ_WAVE - 1, MQ_WAVE);
    if (w < 2) {
        const uint64_t ex = tile_prefix_wave0(status + w * ntiles, tile, epoch, w == 0 ? seg_tot : row_tot);
        if (lane() == 0) s_ex[w] = ex;
    }
    __syncthreads();
    if (w > 0) return;
    const uint32_t es = (uint32_t)s_ex[0];
    const uint64_t er = s_ex[1];
    if (tile == ntiles - 1 && lane() == 0) {
        const uint64_t total = sat_add(er, row_tot > SAT40 ? SAT40 : row_tot);
        const uint32_t nseg = es + (uint32_t)seg_tot;
        *a.nseg = nseg;
        mail.data[0] = nseg;
        mail.data[2] = (uint32_t)total;
        mail.data[3] = (uint32_t)(total >> 32);
        mail_post(mail);
    }
    if (bc != 0) {
        const uint32_t at = es + (uint32_t)__popcll(km & lanemask_lt());
        const uint32_t i = tile * FEW_TILE + lane();
        a.seg_lstart[at] = a.small_is_left ? i : bl;
        a.seg_lcount[at] = a.small_is_left ? sc : bc;
        a.seg_rstart[at] = a.small_is_left ? bl : i;
        a.seg_rcount[at] = a.small_is_left ? bc : sc;
        a.seg_off[at] = sat_add(er, rincl - rows);
    }
}

uint32_t merge_tiles(uint32_t ns) {
    const uint32_t tile = ns <= MRG_FEW ? FEW_TILE : MQ_BLOCK * MRG_IPT;
    return (ns + tile - 1) / tile;
}

hipError_t launch_merge_segments(const MergeArgs& a, uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, Mail mail,
                                 hipStream_t stream) {
    if (a.ns == 0) return hipSuccess;
    if (a.ns <= MRG_FEW) {
        merge_few_kernel<<<merge_tiles(a.ns), FEW_THREADS, 0, stream>>>(a, status, tile_ctr, epoch, mail);
        return hipGetLastError();
    }
    const uint32_t blocks = std::min<uint32_t>(merge_tiles(a.ns), 256u * 8u);
    merge_segments_kernel<<<blocks, MQ_BLOCK, 0, stream>>>(a, status, tile_ctr, epoch, mail);
    return hipGetLastError();
}

}  // namespace mq
