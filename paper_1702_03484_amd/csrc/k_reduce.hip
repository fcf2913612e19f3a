// ReduceDuplicate of Algorithm 1 on gfx950: after the shuffle, records with
// equal keys are contiguous, LEFT records (payload < n_left) ahead of RIGHT
// records within each key.  Three phases:
//   segments     finds the first record of every distinct key, its LEFT/RIGHT
//                split, the pairs cL*cR and their exact output offsets,
//   materialize  writes the per-key cross products, with the output rows
//                split evenly over the grid (a key with a huge product is
//                spread over many blocks).
// Segments are read off bit maps (one bit per record: head, RIGHT) in two
// kernels with no ordering between blocks (no tile counter, no look-back): a
// sum pass in which block b owns a contiguous run of tiles and stores each
// tile's offset within the run and the run's total, one block that turns the
// run totals into prefix sums, then a pass with one tile per block whose offset
// is its run's prefix plus its in-run offset.  That last pass writes the
// segment arrays for the row-chunk kernel, or, where few rows meet per key,
// the output rows themselves.  Composite keys sorted word by word carry their
// segment starts as flags and go through the heads and count passes.
#include "device_common.h"
#include "kernels.h"
#include "tile_ops.h"

#include <algorithm>

namespace mq {

constexpr int HEADS_IPT = 16;
constexpr uint32_t HEADS_TILE = MQ_BLOCK * HEADS_IPT;
constexpr int COUNT_IPT = 8;
constexpr uint32_t COUNT_TILE = MQ_BLOCK * COUNT_IPT;
// blocks of a sum pass: one resident round of the sum kernels (up to 64
// VGPRs, 8 blocks per CU on 256 CUs), so each block sums only a few tiles
// (1,024 blocks: count phase of the 16M + 16M join 0.279 ms; 2,048: 0.247)
constexpr uint32_t RUN_BLOCKS = 2048;

struct RunGrid {
    uint32_t ntiles, chunk, blocks;
};

__host__ __device__ inline RunGrid run_grid(uint32_t ntiles) {
    RunGrid g;
    g.ntiles = ntiles;
    const uint32_t want = ntiles < RUN_BLOCKS ? ntiles : RUN_BLOCKS;
    g.chunk = want ? (ntiles + want - 1) / want : 0;
    g.blocks = g.chunk ? (ntiles + g.chunk - 1) / g.chunk : 0;
    return g;
}

// ---- segments straight from the sorted records -----------------------------
// A tile of sorted records is turned into two bit maps, segment heads and
// RIGHT records, one __ballot word per 64 records.  Everything about a
// segment whose head lies in the tile then comes from bit scans: its end is
// the next head, its split the first RIGHT record (within a key LEFT records
// come first), so one read of the keys gives the segments, their cL * cR
// pairs and the pairs' running sum together.  Each wave walks its words from
// the last to the first, carrying the next head and RIGHT record after the
// word in scalar registers, so a word costs some 25 vector instructions and
// no branch (looking the next bits up in LDS per head: 2,650 instructions a
// tile, and the sum pass of 32M records 87 us).  Only the tile's last segment
// can end past the tile; one wave looks for its end in the next 64 records
// and then by a 64-ary search.
//
//   seg_sum    segments and pairs per tile (each block sums a run of tiles),
//   seg_scan   one block: the run totals' prefixes, the totals to the host,
// then, once the host knows the totals, either
//   seg_write  segment starts, splits and offsets for the row-chunk
//              materialisation, or
//   mat_tile   the output rows themselves (small key products): the segments
//              never leave LDS.
// Tiles have 16 words per wave, or 4 for few records (below 2^18, where 4,096-
// record tiles would leave most of the chip idle).
constexpr int ST_IPT = 16, ST_IPT_FEW = 4;
constexpr uint32_t ST_FEW = 1u << 18;
constexpr uint32_t st_tile(int ipt) { return MQ_BLOCK * (uint32_t)ipt; }
static_assert(MQ_WAVES * ST_IPT <= 64, "one bit per ballot word");

struct SegIn {
    const uint32_t* keys;
    const uint32_t* vals;  // side of a record: payload >= n_left (fs = 0), or the key's low bit (fs = 1)
    uint32_t n, n_left;
};

struct SegTile {  // LDS
    uint64_t hm[MQ_WAVES * ST_IPT], rm[MQ_WAVES * ST_IPT];
    uint32_t hany[MQ_WAVES], rany[MQ_WAVES];  // per wave: one bit per ballot word that is not empty
};

// a wave's records of the tile at `base` (clamped to the last record), and the
// key before them
template <int IPT>
struct SegRecs {
    uint32_t k[IPT], v[IPT], kp;
};
template <int FS, int IPT>
__device__ __forceinline__ void seg_load(const SegIn& a, uint32_t base, SegRecs<IPT>& r) {
    const uint32_t first = base + threadIdx.x / MQ_WAVE * IPT * MQ_WAVE;  // of this wave
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const uint32_t idx = min(first + i * MQ_WAVE + lane(), a.n - 1);
        r.k[i] = a.keys[idx];
        r.v[i] = FS ? 0u : a.vals[idx];
    }
    r.kp = first > 0 ? a.keys[min(first, a.n) - 1] : 0u;
}

// The bit maps of the tile at `base` (this wave's words also in registers).
// Ends with a barrier.
template <int FS, int IPT>
__device__ __forceinline__ void seg_masks(SegTile& sm, const SegIn& a, uint32_t base, const SegRecs<IPT>& rec,
                                          uint64_t (&hm)[IPT], uint64_t (&rm)[IPT]) {
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t first = base + w * IPT * MQ_WAVE;  // of this wave
    const uint32_t(&k)[IPT] = rec.k;
    const uint32_t(&v)[IPT] = rec.v;
    uint32_t kp = rec.kp;
    uint32_t hany = 0, rany = 0;
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const uint32_t idx = first + i * MQ_WAVE + lane();
        const uint32_t p = wave_prev(k[i], kp);
        kp = last_lane(k[i]);
        hm[i] = __ballot(idx < a.n && (idx == 0 || (p >> FS) != (k[i] >> FS)));
        rm[i] = __ballot(idx < a.n && (FS ? (k[i] & 1u) != 0 : v[i] >= a.n_left));
        hany |= (hm[i] ? 1u : 0u) << i;
        rany |= (rm[i] ? 1u : 0u) << i;
    }
    if (lane() == 0) {
#pragma unroll
        for (int i = 0; i < IPT; i++) {
            sm.hm[w * IPT + i] = hm[i];
            sm.rm[w * IPT + i] = rm[i];
        }
        sm.hany[w] = hany;
        sm.rany[w] = rany;
    }
    __syncthreads();
}

template <int IPT>
__device__ __forceinline__ uint64_t any_words(const uint32_t (&any)[MQ_WAVES]) {
    uint64_t all = 0;
#pragma unroll
    for (int w = 0; w < MQ_WAVES; w++) all |= (uint64_t)any[w] << (w * IPT);
    return all;
}

// first set bit of the tile's map at or after position `from` (none: `none`)
__device__ __forceinline__ uint32_t next_bit(const uint64_t* words, uint64_t any, uint32_t from, uint32_t nwords,
                                             uint32_t none) {
    uint32_t r = from / MQ_WAVE;
    if (r >= nwords) return none;
    const uint64_t here = words[r] >> (from % MQ_WAVE);
    if (here) return from + (uint32_t)__builtin_ctzll(here);
    const uint64_t rows = r + 1 < 64 ? any >> (r + 1) : 0ull;
    if (!rows) return none;
    r += 1 + (uint32_t)__builtin_ctzll(rows);
    return r * MQ_WAVE + (uint32_t)__builtin_ctzll(words[r]);
}

// This lane's segments: for word i, LEFT and RIGHT counts of the segment
// headed by its record, up to the tile's last record (`lim` records), 0 and 0
// where it heads none, and RIGHT 0 for the tile's last segment when it may go
// on past the tile (`past`: seg_last has that one).
template <int IPT>
__device__ __forceinline__ void seg_counts(const SegTile& sm, const uint64_t (&hm)[IPT], const uint64_t (&rm)[IPT],
                                           uint32_t lim, bool past, uint32_t (&cl)[IPT], uint32_t (&cr)[IPT]) {
    constexpr uint32_t WORDS = MQ_WAVES * IPT;
    const uint32_t w = uni(threadIdx.x / MQ_WAVE);
    // the next head and RIGHT record after this wave's words
    uint32_t nh = uni(next_bit(sm.hm, any_words<IPT>(sm.hany), (w + 1) * IPT * MQ_WAVE, WORDS, lim));
    uint32_t nr = uni(next_bit(sm.rm, any_words<IPT>(sm.rany), (w + 1) * IPT * MQ_WAVE, WORDS, lim));
#pragma unroll
    for (int i = IPT - 1; i >= 0; i--) {
        const uint32_t word = (w * IPT + i) * MQ_WAVE, pos = word + lane();
        const uint64_t h = hm[i] >> 1 >> lane(), r = rm[i] >> lane();
        const uint32_t end = h ? pos + 1 + (uint32_t)__builtin_ctzll(h) : nh;
        const uint32_t sp = min(r ? pos + (uint32_t)__builtin_ctzll(r) : nr, end);
        const bool head = (hm[i] >> lane()) & 1ull;
        cl[i] = head ? sp - pos : 0u;
        cr[i] = head && !(past && end >= lim) ? end - sp : 0u;
        nh = hm[i] ? word + (uint32_t)__builtin_ctzll(hm[i]) : nh;
        nr = rm[i] ? word + (uint32_t)__builtin_ctzll(rm[i]) : nr;
    }
}

// first index in [lo, hi) where pred holds (false, then true), by 64 probes a
// level; every lane of the wave calls it
template <class Pred>
__device__ __forceinline__ uint32_t wave_first(uint32_t lo, uint32_t hi, Pred pred) {
    while (lo < hi) {
        const uint32_t step = (hi - lo + MQ_WAVE - 1) / MQ_WAVE;
        const uint64_t pos = (uint64_t)lo + (uint64_t)lane() * step;
        const uint32_t before = (uint32_t)__popcll(__ballot(pos < hi && !pred((uint32_t)pos)));
        if (before == 0) return lo;
        hi = (uint32_t)min((uint64_t)hi, (uint64_t)lo + (uint64_t)before * step);
        lo += (before - 1) * step + 1;
    }
    return lo;
}

// The tile's last segment when records follow the tile (`end` < n is the
// first of them): its head's position in the tile (false: the tile has no
// head) and its whole counts, by one wave.  ek, ev: keys and payloads of the
// 64 records from `end` on (clamped to the last record); key: the tile's last.
template <int FS, int IPT>
__device__ __forceinline__ bool seg_last(const SegTile& sm, const SegIn& a, uint32_t end, uint32_t key, uint32_t ek,
                                         uint32_t ev, uint32_t& pos, uint32_t& cl, uint32_t& cr) {
    constexpr uint32_t WORDS = MQ_WAVES * IPT, TILE = st_tile(IPT);
    const uint64_t hall = any_words<IPT>(sm.hany);
    if (!hall) return false;
    const uint32_t hw = 63u - (uint32_t)__builtin_clzll(hall);
    pos = hw * MQ_WAVE + 63u - (uint32_t)__builtin_clzll(sm.hm[hw]);
    uint32_t sp = next_bit(sm.rm, any_words<IPT>(sm.rany), pos, WORDS, TILE);
    const bool in = end + lane() < a.n;
    const uint64_t other = __ballot(!in || (ek >> FS) != (key >> FS));
    const uint32_t near = other ? (uint32_t)__builtin_ctzll(other) : (uint32_t)MQ_WAVE;  // records that follow, so far
    uint32_t stop = end + near;
    if (!other)
        stop = wave_first(end + MQ_WAVE, a.n, [&](uint32_t i) { return (a.keys[i] >> FS) != (key >> FS); });
    cl = sp - pos;
    cr = TILE - sp + (stop - end);
    if (sp == TILE) {  // no RIGHT record in the tile: find the first one
        const uint64_t right = __ballot(FS ? (ek & 1u) != 0 : ev >= a.n_left) & (other ? (1ull << near) - 1ull : ~0ull);
        sp = right ? end + (uint32_t)__builtin_ctzll(right) : stop;
        if (!right && !other)
            sp = wave_first(end + MQ_WAVE, stop,
                            [&](uint32_t i) { return FS ? (a.keys[i] & 1u) != 0 : a.vals[i] >= a.n_left; });
        cl += sp - end;
        cr = stop - sp;
    }
    return true;
}

__device__ __forceinline__ uint64_t seg_pairs_of(uint32_t cl, uint32_t cr) {
    const uint64_t c = (uint64_t)cl * cr;
    return c > SAT40 ? SAT40 : c;
}

// per tile: segments before it in its run (tseg) and pairs (trow); per run
// the totals and the largest single product.  One read of the keys (and of
// the payloads where they tell the side).
template <int FS, int IPT>
__global__ __launch_bounds__(MQ_BLOCK) void seg_sum_kernel(SegIn a, RunGrid g, uint32_t* __restrict__ tseg,
                                                           uint64_t* __restrict__ trow,
                                                           uint64_t* __restrict__ run_seg,
                                                           uint64_t* __restrict__ run_row,
                                                           uint64_t* __restrict__ run_max) {
    constexpr uint32_t TILE = st_tile(IPT);
    __shared__ SegTile sm;
    __shared__ uint32_t s_seg[MQ_WAVES], s_row[MQ_WAVES], s_max[MQ_WAVES];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    uint32_t segs = 0;
    uint64_t rows = 0, mx = 0;  // of the run so far (wave 0)
    const uint32_t t0 = blockIdx.x * g.chunk, t1 = min(t0 + g.chunk, g.ntiles);
    SegRecs<IPT> rec;  // the next tile's records are in flight while one is worked on
    seg_load<FS, IPT>(a, t0 * TILE, rec);
    for (uint32_t tile = t0; tile < t1; tile++) {
        const uint32_t base = tile * TILE, lim = min(TILE, a.n - base);
        const bool past = a.n - base > TILE;
        uint32_t ek = 0, ev = 0, lk = 0;
        if (w == 0 && past) {
            const uint32_t e = min(base + TILE + lane(), a.n - 1);
            ek = a.keys[e];
            if (!FS) ev = a.vals[e];
            lk = a.keys[base + TILE - 1];
        }
        uint32_t cl[IPT], cr[IPT];
        uint64_t hm[IPT], rm[IPT];
        seg_masks<FS, IPT>(sm, a, base, rec, hm, rm);
        if (tile + 1 < t1) seg_load<FS, IPT>(a, base + TILE, rec);
        seg_counts<IPT>(sm, hm, rm, lim, past, cl, cr);
        uint32_t sum = 0, m = 0, heads = 0;  // the products of a tile add up to at most 2^22
#pragma unroll
        for (int i = 0; i < IPT; i++) {
            const uint32_t c = __umul24(cl[i], cr[i]);
            heads += (uint32_t)__popcll(hm[i]);
            sum += c;
            m = max(m, c);
        }
        sum = last_lane(wave_incl_u32(sum));
        m = wave_max_u32(m);
        if (lane() == 0) {
            s_seg[w] = heads;
            s_row[w] = sum;
            s_max[w] = m;
        }
        __syncthreads();
        if (w == 0) {
            uint32_t ts = 0, tm = 0;
            uint64_t tr = 0;
#pragma unroll
            for (int i = 0; i < MQ_WAVES; i++) {
                ts += s_seg[i];
                tr += s_row[i];
                tm = max(tm, s_max[i]);
            }
            uint64_t oc = 0;
            uint32_t pos, ol, orr;
            if (past && seg_last<FS, IPT>(sm, a, base + TILE, lk, ek, ev, pos, ol, orr)) oc = seg_pairs_of(ol, orr);
            if (lane() == 0) {
                tseg[tile] = segs;
                trow[tile] = rows;
            }
            segs += ts;
            rows = sat_add(rows, tr + oc > SAT40 ? SAT40 : tr + oc);
            mx = max(mx, max((uint64_t)tm, oc));
        }
        __syncthreads();  // the maps are rewritten by the next tile
    }
    if (threadIdx.x == 0) {
        run_seg[blockIdx.x] = segs;
        run_row[blockIdx.x] = rows;
        run_max[blockIdx.x] = mx;
    }
}

// one block: both run totals become exclusive prefixes (pairs capped at
// 2^40 - 1); the sums and the largest product go to the host
constexpr uint32_t SEG_SCAN_PER = RUN_BLOCKS / MQ_BLOCK;
__global__ __launch_bounds__(MQ_BLOCK) void seg_scan_kernel(uint64_t* __restrict__ run_seg, uint64_t* __restrict__ run_row,
                                                            const uint64_t* __restrict__ run_max, uint32_t nruns,
                                                            uint32_t* __restrict__ nseg, Mail mail) {
    __shared__ uint64_t tmp[MQ_WAVES];
    __shared__ uint64_t s_mx[MQ_WAVES];
    uint64_t s[SEG_SCAN_PER], r[SEG_SCAN_PER], ss = 0, rs = 0, mx = 0;
#pragma unroll
    for (uint32_t j = 0; j < SEG_SCAN_PER; j++) {
        const uint32_t i = threadIdx.x * SEG_SCAN_PER + j;
        s[j] = i < nruns ? run_seg[i] : 0ull;
        r[j] = i < nruns ? run_row[i] : 0ull;
        if (i < nruns) mx = max(mx, run_max[i]);
        ss += s[j];
        rs += r[j];
    }
    uint64_t all_s, all_r;
    uint64_t es = block_excl_scan<uint64_t>(ss, tmp, &all_s), er = block_excl_scan<uint64_t>(rs, tmp, &all_r);
#pragma unroll
    for (uint32_t j = 0; j < SEG_SCAN_PER; j++) {
        const uint32_t i = threadIdx.x * SEG_SCAN_PER + j;
        if (i < nruns) {
            run_seg[i] = es;
            run_row[i] = er > SAT40 ? SAT40 : er;
        }
        es += s[j];
        er += r[j];
    }
#pragma unroll
    for (int o = MQ_WAVE / 2; o > 0; o >>= 1) mx = max(mx, (uint64_t)__shfl_xor(mx, o));
    if (lane() == 0) s_mx[threadIdx.x / MQ_WAVE] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < MQ_WAVES; i++) mx = max(mx, s_mx[i]);
        const uint64_t total = all_r > SAT40 ? SAT40 : all_r;
        *nseg = (uint32_t)all_s;
        mail.data[0] = (uint32_t)all_s;
        mail.data[2] = (uint32_t)total;
        mail.data[3] = (uint32_t)(total >> 32);
        mail.data[4] = (uint32_t)mx;
        mail.data[5] = (uint32_t)(mx >> 32);
        mail_post(mail);
    }
}

// This tile's segments and rows, per wave and lane: exclusive counts before
// each record's segment.  s_a, s_b: one word per wave of LDS.
struct TileBefore {
    uint32_t seg, row;
};
__device__ __forceinline__ TileBefore waves_before(uint32_t seg, uint32_t row, uint32_t* s_a, uint32_t* s_b) {
    const uint32_t w = threadIdx.x / MQ_WAVE;
    if (lane() == 0) {
        s_a[w] = seg;
        s_b[w] = row;
    }
    __syncthreads();
    TileBefore t{0, 0};
#pragma unroll
    for (int i = 0; i < MQ_WAVES; i++)
        if ((uint32_t)i < w) {
            t.seg += s_a[i];
            t.row += s_b[i];
        }
    return t;
}

// segment starts, splits and output offsets; one tile per block
template <int FS, int IPT>
__global__ __launch_bounds__(MQ_BLOCK) void seg_write_kernel(SegIn a, RunGrid g, const uint32_t* __restrict__ tseg,
                                                             const uint64_t* __restrict__ trow,
                                                             const uint64_t* __restrict__ run_seg,
                                                             const uint64_t* __restrict__ run_row,
                                                             uint32_t* __restrict__ seg_start,
                                                             uint32_t* __restrict__ seg_split,
                                                             uint64_t* __restrict__ seg_off) {
    constexpr uint32_t TILE = st_tile(IPT);
    __shared__ SegTile sm;
    __shared__ uint32_t s_a[MQ_WAVES], s_b[MQ_WAVES];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t tile = blockIdx.x, base = tile * TILE, lim = min(TILE, a.n - base);
    const bool past = a.n - base > TILE;
    SegRecs<IPT> rec;
    uint32_t cl[IPT], cr[IPT];
    uint64_t hm[IPT], rm[IPT];
    seg_load<FS, IPT>(a, base, rec);
    seg_masks<FS, IPT>(sm, a, base, rec, hm, rm);
    seg_counts<IPT>(sm, hm, rm, lim, past, cl, cr);
    uint32_t heads = 0, rows = 0;
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        heads += (uint32_t)__popcll(hm[i]);
        rows += __umul24(cl[i], cr[i]);  // the last segment's come after every other offset
    }
    const TileBefore t = waves_before(heads, last_lane(wave_incl_u32(rows)), s_a, s_b);
    const uint32_t seg0 = (uint32_t)run_seg[tile / g.chunk] + tseg[tile];
    uint32_t sid = seg0 + t.seg;
    uint64_t off = sat_add(sat_add(run_row[tile / g.chunk], trow[tile]), t.row);
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const uint32_t c = __umul24(cl[i], cr[i]), incl = wave_incl_u32(c);
        if ((hm[i] >> lane()) & 1ull) {
            const uint32_t at = sid + (uint32_t)__popcll(hm[i] & lt);
            const uint32_t idx = base + (w * IPT + i) * MQ_WAVE + lane();
            if (MQ_IN_BOUNDS(at, a.n)) {
                seg_start[at] = idx;
                if (!past || idx + cl[i] < base + TILE) seg_split[at] = idx + cl[i];  // else below
                seg_off[at] = sat_add(off, incl - c);
            }
        }
        sid += (uint32_t)__popcll(hm[i]);
        off = sat_add(off, last_lane(incl));
    }
    if (!past || w != MQ_WAVES - 1) return;
    // the tile's last segment when no RIGHT record of it lies in the tile
    const uint32_t end = base + TILE, e = min(end + lane(), a.n - 1);
    uint32_t pos, ol, orr;
    if (seg_last<FS, IPT>(sm, a, end, a.keys[end - 1], a.keys[e], FS ? 0u : a.vals[e], pos, ol, orr) &&
        pos + ol >= TILE && lane() == 0 && MQ_IN_BOUNDS(sid - 1, a.n))
        seg_split[sid - 1] = base + pos + ol;
}

// Scratch: run totals of segments and of pairs and run maxima (RUN_BLOCKS
// each), pairs before each tile, segments before each tile.
struct SegScratch {
    uint64_t *run_seg, *run_row, *run_max, *trow;
    uint32_t* tseg;
};
static bool seg_few(uint32_t n) { return n < ST_FEW; }
static RunGrid seg_grid(uint32_t n) {
    const uint32_t tile = st_tile(seg_few(n) ? ST_IPT_FEW : ST_IPT);
    return run_grid(n ? (n - 1) / tile + 1 : 0u);
}
static SegScratch seg_tiles(void* p, uint32_t n) {
    const RunGrid g = seg_grid(n);
    SegScratch s;
    s.run_seg = static_cast<uint64_t*>(p);
    s.run_row = s.run_seg + g.blocks;
    s.run_max = s.run_row + g.blocks;
    s.trow = s.run_max + g.blocks;
    s.tseg = reinterpret_cast<uint32_t*>(s.trow + g.ntiles);
    return s;
}

hipError_t launch_seg_sum(const uint32_t* keys, const uint32_t* vals, uint32_t n, uint32_t n_left, int side_bit,
                          uint32_t* nseg, void* scratch, Mail mail, hipStream_t stream) {
    if (n == 0) return hipErrorInvalidValue;
    const RunGrid g = seg_grid(n);
    const SegScratch s = seg_tiles(scratch, n);
    const SegIn a{keys, vals, n, n_left};
    auto* k = seg_few(n) ? (side_bit ? seg_sum_kernel<1, ST_IPT_FEW> : seg_sum_kernel<0, ST_IPT_FEW>)
                         : (side_bit ? seg_sum_kernel<1, ST_IPT> : seg_sum_kernel<0, ST_IPT>);
    k<<<g.blocks, MQ_BLOCK, 0, stream>>>(a, g, s.tseg, s.trow, s.run_seg, s.run_row, s.run_max);
    seg_scan_kernel<<<1, MQ_BLOCK, 0, stream>>>(s.run_seg, s.run_row, s.run_max, g.blocks, nseg, mail);
    return hipGetLastError();
}

hipError_t launch_seg_write(const uint32_t* keys, const uint32_t* vals, uint32_t n, uint32_t n_left, int side_bit,
                            uint32_t* seg_start, uint32_t* seg_split, uint64_t* seg_off, void* scratch,
                            hipStream_t stream) {
    if (n == 0) return hipErrorInvalidValue;
    const RunGrid g = seg_grid(n);
    const SegScratch s = seg_tiles(scratch, n);
    const SegIn a{keys, vals, n, n_left};
    auto* k = seg_few(n) ? (side_bit ? seg_write_kernel<1, ST_IPT_FEW> : seg_write_kernel<0, ST_IPT_FEW>)
                         : (side_bit ? seg_write_kernel<1, ST_IPT> : seg_write_kernel<0, ST_IPT>);
    k<<<g.ntiles, MQ_BLOCK, 0, stream>>>(a, g, s.tseg, s.trow, s.run_seg, s.run_row, seg_start, seg_split, seg_off);
    return hipGetLastError();
}

// ---- segments of a composite key sorted word by word -------------------------
// A record flagged in brk heads a segment too, which the keys alone do not
// show (and a segment's end cannot be searched for): segment heads and splits,
// then counts and offsets, in two passes each.

// Key and payload of record idx and of its neighbours, for every lane of a
// wave that covers 64 consecutive records (lanes past n see key ~0u).
struct RecView {
    uint32_t k, v, kprev, vprev, knext;
};

__device__ __forceinline__ RecView rec_view(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                            uint32_t n, uint32_t idx) {
    RecView r;
    const bool in = idx < n;
    r.k = in ? keys[idx] : ~0u;
    r.v = in ? vals[idx] : 0u;
    // neighbours from the adjacent lanes; the wave's edge lanes load them
    r.kprev = __shfl_up(r.k, 1, MQ_WAVE);
    r.vprev = __shfl_up(r.v, 1, MQ_WAVE);
    r.knext = __shfl_down(r.k, 1, MQ_WAVE);
    if (lane() == 0 && in && idx > 0) {
        r.kprev = keys[idx - 1];
        r.vprev = vals[idx - 1];
    }
    if (lane() == MQ_WAVE - 1 && idx + 1 < n) r.knext = keys[idx + 1];
    return r;
}

__device__ __forceinline__ bool rec_is_head(const RecView& r, uint32_t idx, uint32_t n) {
    return idx < n && (idx == 0 || r.kprev != r.k);
}

// sum pass: heads of every tile of the block's run
__global__ __launch_bounds__(MQ_BLOCK) void heads_sum_kernel(const uint32_t* __restrict__ keys,
                                                             const uint8_t* __restrict__ brk, uint32_t n,
                                                             uint64_t* __restrict__ run_tot,
                                                             uint32_t* __restrict__ tloc, RunGrid g) {
    __shared__ uint32_t s_wtot[MQ_WAVES];
    __shared__ uint32_t s_run;
    const uint32_t w = threadIdx.x / MQ_WAVE;
    if (threadIdx.x == 0) s_run = 0;
    const uint32_t t0 = blockIdx.x * g.chunk;
    const uint32_t t1 = min(t0 + g.chunk, g.ntiles);
    for (uint32_t tile = t0; tile < t1; tile++) {
        const uint32_t base = tile * HEADS_TILE;
        uint32_t k[HEADS_IPT];
        bool f[HEADS_IPT];
#pragma unroll
        for (int i = 0; i < HEADS_IPT; i++) {
            const uint32_t idx = base + (w * HEADS_IPT + i) * MQ_WAVE + lane();
            k[i] = idx < n ? keys[idx] : 0u;
            f[i] = idx < n && brk[idx] != 0;
        }
        uint32_t run = 0;
#pragma unroll
        for (int i = 0; i < HEADS_IPT; i++) {
            const uint32_t idx = base + (w * HEADS_IPT + i) * MQ_WAVE + lane();
            uint32_t kp = __shfl_up(k[i], 1, MQ_WAVE);
            if (lane() == 0 && idx > 0 && idx < n) kp = keys[idx - 1];
            const bool head = kp != k[i] || f[i];
            run += (uint32_t)__popcll(__ballot(idx < n && (idx == 0 || head)));
        }
        if (lane() == 0) s_wtot[w] = run;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
#pragma unroll
            for (int i = 0; i < MQ_WAVES; i++) tot += s_wtot[i];
            tloc[tile] = s_run;
            s_run += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) run_tot[blockIdx.x] = s_run;
}

// write pass: one tile per block
__global__ __launch_bounds__(MQ_BLOCK) void heads_write_kernel(const uint32_t* __restrict__ keys,
                                                               const uint8_t* __restrict__ brk,
                                                               const uint32_t* __restrict__ vals, uint32_t n,
                                                               uint32_t n_left,
                                                               const uint64_t* __restrict__ run_excl,
                                                               const uint32_t* __restrict__ tloc, RunGrid g,
                                                               uint32_t* __restrict__ seg_start,
                                                               uint32_t* __restrict__ seg_split) {
    __shared__ uint32_t s_wtot[MQ_WAVES];
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint64_t lt = lanemask_lt();
    const uint32_t tile = blockIdx.x;
    const uint32_t base = tile * HEADS_TILE;
    RecView r[HEADS_IPT];
    bool f[HEADS_IPT], fnext[HEADS_IPT];  // this record / the next one flagged in brk
#pragma unroll
    for (int i = 0; i < HEADS_IPT; i++) {
        const uint32_t idx = base + (w * HEADS_IPT + i) * MQ_WAVE + lane();
        r[i] = rec_view(keys, vals, n, idx);
        f[i] = idx < n && brk[idx] != 0;
        fnext[i] = idx + 1 < n && brk[idx + 1] != 0;
    }
    uint64_t hm[HEADS_IPT];
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < HEADS_IPT; i++) {
        const uint32_t idx = base + (w * HEADS_IPT + i) * MQ_WAVE + lane();
        hm[i] = __ballot(rec_is_head(r[i], idx, n) || f[i]);
        run += (uint32_t)__popcll(hm[i]);
    }
    if (lane() == 0) s_wtot[w] = run;
    __syncthreads();
    // heads before this tile: its run's prefix, then its offset within the run
    uint32_t pos = (uint32_t)run_excl[tile / g.chunk] + tloc[tile];
#pragma unroll
    for (int i = 0; i < MQ_WAVES; i++) pos += (uint32_t)i < w ? s_wtot[i] : 0u;
#pragma unroll
    for (int i = 0; i < HEADS_IPT; i++) {
        const uint32_t idx = base + (w * HEADS_IPT + i) * MQ_WAVE + lane();
        const bool h = (hm[i] >> lane()) & 1ull;
        const uint32_t bef = pos + (uint32_t)__popcll(hm[i] & lt);  // heads before this record
        if (idx < n) {
            const bool is_r = r[i].v >= n_left;
            const bool prev_r = r[i].vprev >= n_left;
            const bool last = idx + 1 == n || r[i].knext != r[i].k || fnext[i];
            const bool first_r = is_r && (h || !prev_r);
            if (h && MQ_IN_BOUNDS(bef, n)) seg_start[bef] = idx;
            if (first_r || (last && !is_r)) {
                const uint32_t sid = h ? bef : bef - 1u;  // record 0 is always a head
                if (MQ_IN_BOUNDS(sid, n)) seg_split[sid] = first_r ? idx : idx + 1;
            }
        }
        pos += (uint32_t)__popcll(hm[i]);
    }
}

// Scratch of the heads and count phases (u64 words first): heads run
// totals, count run totals, count run maxima, count per-tile offsets, then
// heads per-tile offsets (u32).
struct BrkScratch {
    uint64_t *h_run, *c_run, *c_max, *c_tloc;
    uint32_t* h_tloc;
};

static RunGrid heads_grid(uint32_t n) { return run_grid(n ? (n - 1) / HEADS_TILE + 1 : 0u); }
static RunGrid count_grid(uint32_t max_seg) { return run_grid(max_seg ? (max_seg - 1) / COUNT_TILE + 1 : 1u); }

static BrkScratch brk_scratch(void* p, uint32_t n) {
    const RunGrid gh = heads_grid(n), gc = count_grid(n);
    BrkScratch s;
    s.h_run = static_cast<uint64_t*>(p);
    s.c_run = s.h_run + gh.blocks;
    s.c_max = s.c_run + gc.blocks;
    s.c_tloc = s.c_max + gc.blocks;
    s.h_tloc = reinterpret_cast<uint32_t*>(s.c_tloc + gc.ntiles);
    return s;
}

size_t seg_scratch_bytes(uint32_t n, bool brk) {
    if (!brk) {
        const RunGrid g = seg_grid(n);
        return 8ull * (3ull * g.blocks + g.ntiles) + 4ull * g.ntiles;
    }
    const RunGrid gh = heads_grid(n), gc = count_grid(n);
    return 8ull * (gh.blocks + 2ull * gc.blocks + gc.ntiles) + 4ull * gh.ntiles;
}

hipError_t launch_seg_heads(const uint32_t* keys, const uint32_t* vals, const uint8_t* brk, uint32_t n,
                            uint32_t n_left, uint32_t* seg_start, uint32_t* seg_split, uint32_t* nseg, void* scratch,
                            hipStream_t stream) {
    if (n == 0) return hipErrorInvalidValue;
    const RunGrid g = heads_grid(n);
    const BrkScratch ss = brk_scratch(scratch, n);
    heads_sum_kernel<<<g.blocks, MQ_BLOCK, 0, stream>>>(keys, brk, n, ss.h_run, ss.h_tloc, g);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_scan_runs(ss.h_run, g.blocks, nullptr, nseg, nullptr, nullptr, nullptr, stream);
    if (e != hipSuccess) return e;
    heads_write_kernel<<<g.ntiles, MQ_BLOCK, 0, stream>>>(keys, brk, vals, n, n_left, ss.h_run, ss.h_tloc, g,
                                                         seg_start, seg_split);
    return hipGetLastError();
}

__device__ __forceinline__ uint64_t block_reduce_sum(uint64_t v, uint64_t* tmp) {
#pragma unroll
    for (int o = MQ_WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane() == 0) tmp[threadIdx.x / MQ_WAVE] = v;
    __syncthreads();
    uint64_t t = 0;
#pragma unroll
    for (int i = 0; i < MQ_WAVES; i++) t += tmp[i];
    __syncthreads();
    return t;
}

// pairs of segment s: (split - start) * (end - split), capped at 2^40 - 1
__device__ __forceinline__ uint64_t seg_pairs(const uint32_t* __restrict__ seg_start,
                                              const uint32_t* __restrict__ seg_split, uint32_t n, uint32_t ns,
                                              uint32_t s) {
    if (s >= ns) return 0;
    const uint32_t st = seg_start[s];
    const uint32_t en = s + 1 < ns ? seg_start[s + 1] : n;
    const uint32_t sp = seg_split[s];
    const uint64_t c = (uint64_t)(sp - st) * (uint64_t)(en - sp);
    return c > SAT40 ? SAT40 : c;
}

// The segment count lives on the device; both count kernels are sized for
// max_seg segments and treat tiles past the real count as empty.
__global__ __launch_bounds__(MQ_BLOCK) void count_sum_kernel(uint32_t n, const uint32_t* __restrict__ seg_start,
                                                             const uint32_t* __restrict__ nseg_p,
                                                             const uint32_t* __restrict__ seg_split,
                                                             uint64_t* __restrict__ run_tot,
                                                             uint64_t* __restrict__ run_max,
                                                             uint64_t* __restrict__ tloc, RunGrid g) {
    __shared__ uint64_t s_tmp[MQ_WAVES];
    __shared__ uint64_t s_run;
    uint64_t mx = 0;  // this thread's largest count
    const uint32_t ns = n == 0 ? 0u : *nseg_p;
    if (threadIdx.x == 0) s_run = 0;
    const uint32_t t0 = blockIdx.x * g.chunk;
    const uint32_t t1 = min(t0 + g.chunk, g.ntiles);
    for (uint32_t tile = t0; tile < t1; tile++) {
        // any order within the tile: coalesced, segment base + i * 256 + thread
        const uint32_t base = tile * COUNT_TILE;
        uint64_t sum = 0;
        if (base < ns) {
#pragma unroll
            for (int i = 0; i < COUNT_IPT; i++) {
                const uint64_t c = seg_pairs(seg_start, seg_split, n, ns, base + i * MQ_BLOCK + threadIdx.x);
                sum += c;
                mx = c > mx ? c : mx;
            }
        }
        const uint64_t tot = block_reduce_sum(sum, s_tmp);
        if (threadIdx.x == 0) {
            tloc[tile] = s_run;
            s_run = sat_add(s_run, tot > SAT40 ? SAT40 : tot);
        }
        __syncthreads();
    }
#pragma unroll
    for (int o = MQ_WAVE / 2; o > 0; o >>= 1) {
        const uint64_t y = __shfl_xor(mx, o);
        mx = y > mx ? y : mx;
    }
    if (lane() == 0) s_tmp[threadIdx.x / MQ_WAVE] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        run_tot[blockIdx.x] = s_run;
        for (int i = 0; i < MQ_WAVES; i++) mx = s_tmp[i] > mx ? s_tmp[i] : mx;
        run_max[blockIdx.x] = mx;
    }
}

__global__ __launch_bounds__(MQ_BLOCK) void count_write_kernel(uint32_t n, const uint32_t* __restrict__ seg_start,
                                                               const uint32_t* __restrict__ nseg_p,
                                                               const uint32_t* __restrict__ seg_split,
                                                               const uint64_t* __restrict__ run_excl,
                                                               const uint64_t* __restrict__ tloc, RunGrid g,
                                                               uint64_t* __restrict__ seg_off) {
    __shared__ uint64_t s_tmp[MQ_WAVES];
    const uint32_t ns = n == 0 ? 0u : *nseg_p;
    const uint32_t tile = blockIdx.x;
    const uint32_t ntiles = ns ? (ns - 1) / COUNT_TILE + 1 : 0u;
    if (tile >= ntiles) return;
    // wave-striped: slot i of wave w holds segments base + (w * IPT + i) * 64 + lane
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t base = tile * COUNT_TILE + w * COUNT_IPT * MQ_WAVE;
    uint32_t st[COUNT_IPT], sp[COUNT_IPT];
#pragma unroll
    for (int i = 0; i < COUNT_IPT; i++) {
        const uint32_t s = base + i * MQ_WAVE + lane();
        st[i] = s < ns ? seg_start[s] : n;
        sp[i] = s < ns ? seg_split[s] : n;
    }
    uint64_t cnt[COUNT_IPT];
    uint64_t wsum = 0;  // this wave's pairs before slot i
    uint64_t excl[COUNT_IPT];
#pragma unroll
    for (int i = 0; i < COUNT_IPT; i++) {
        const uint32_t s = base + i * MQ_WAVE + lane();
        uint32_t en = __shfl_down(st[i], 1, MQ_WAVE);
        if (lane() == MQ_WAVE - 1) en = s + 1 < ns ? seg_start[s + 1] : n;
        if (s + 1 >= ns) en = n;
        const uint64_t c = s < ns ? (uint64_t)(sp[i] - st[i]) * (uint64_t)(en - sp[i]) : 0ull;
        cnt[i] = c > SAT40 ? SAT40 : c;
        const uint64_t inc = wave_incl_scan<uint64_t>(cnt[i]);
        excl[i] = wsum + inc - cnt[i];
        wsum += (uint64_t)__shfl(inc, MQ_WAVE - 1, MQ_WAVE);
    }
    if (lane() == 0) s_tmp[w] = wsum;
    __syncthreads();
    // pairs before this tile: its run's prefix (capped), then its offset within the run
    uint64_t off = sat_add(run_excl[tile / g.chunk], tloc[tile]), wex = 0;
#pragma unroll
    for (int i = 0; i < MQ_WAVES; i++) wex += (uint32_t)i < w ? s_tmp[i] : 0ull;
    off = sat_add(off, wex > SAT40 ? SAT40 : wex);
#pragma unroll
    for (int i = 0; i < COUNT_IPT; i++) {
        const uint32_t s = base + i * MQ_WAVE + lane();
        if (s < ns) seg_off[s] = sat_add(off, excl[i] > SAT40 ? SAT40 : excl[i]);
    }
}

hipError_t launch_seg_count(uint32_t n, const uint32_t* seg_start, const uint32_t* nseg, uint32_t max_seg,
                            const uint32_t* seg_split, uint64_t* seg_off, Mail mail, void* scratch,
                            hipStream_t stream) {
    if (max_seg > n) return hipErrorInvalidValue;  // the scratch is laid out for n
    const RunGrid g = count_grid(max_seg);
    const BrkScratch ss = brk_scratch(scratch, n);
    count_sum_kernel<<<g.blocks, MQ_BLOCK, 0, stream>>>(n, seg_start, nseg, seg_split, ss.c_run, ss.c_max, ss.c_tloc,
                                                       g);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_scan_runs(ss.c_run, g.blocks, nullptr, nullptr, ss.c_max, nseg, &mail, stream);
    if (e != hipSuccess) return e;
    count_write_kernel<<<g.ntiles, MQ_BLOCK, 0, stream>>>(n, seg_start, nseg, seg_split, ss.c_run, ss.c_tloc, g,
                                                         seg_off);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Materialisation: waves own chunks of 64*RPT consecutive output rows.
// ---------------------------------------------------------------------------
template <int NC>
struct MatShape {
    static constexpr int RPT = NC <= 4 ? 16 : (NC <= 8 ? 8 : 4);  // rows per lane
    static constexpr uint32_t WROWS = MQ_WAVE * RPT;               // rows per wave chunk
};

template <int NC, int NLC>
__device__ __forceinline__ MatJoin mat_join_of(const MatArgs& a) {
    MatJoin mj;
    mj.keys = a.keys;
    mj.vals = a.vals;
    mj.seg_start = a.seg_start;
    mj.seg_split = a.seg_split;
    mj.seg_off = a.seg_off;
    mj.ns = *a.nseg;
    mj.n = a.n;
    mj.n_left = a.n_left;
    mj.key_base = a.key_base;
    mj.key_shift = a.key_shift;
    mj.nl = NLC >= 0 ? NLC : a.nl;
    mj.nr = NLC >= 0 ? NC - 1 - NLC : a.nr;
    const bool merged = a.seg_cl != nullptr;
    mj.sorted_vals = merged || a.use_sval != 0;
    mj.seg_cl = a.seg_cl;
    mj.seg_cr = a.seg_cr;
#pragma unroll
    for (int c = 0; c < NC; c++) {
        mj.out[c] = a.out[c];
        if (c >= 1) {
            const bool left = c <= mj.nl;
            mj.src[c] = left ? a.lcol[c - 1] : a.rcol[c - 1 - mj.nl];
            // merge join: runs index the tables' own (key-sorted) columns
            mj.ssrc[c] = merged ? mj.src[c] : (left ? a.sval[c - 1] : a.sval[c - 1 - mj.nl]);
        }
    }
    return mj;
}

template <int NC, int NLC>
__global__ __launch_bounds__(MQ_BLOCK) void materialize_kernel(MatArgs a) {
    constexpr uint32_t WROWS = MatShape<NC>::WROWS;
    __shared__ uint64_t s_segs[MQ_WAVES][MAT_LDS_SEGS];
    const MatJoin mj = mat_join_of<NC, NLC>(a);
    // chunks strided over the waves (the rows being written at any moment
    // stay in one window of the output); a wave's previous segment is the
    // starting guess for its next chunk
    const int qn = a.sparse ? 1 : MatShape<NC>::RPT / 4;
    const uint32_t crows = a.sparse ? 4 * MQ_WAVE : WROWS;
    const uint64_t nchunks = (a.row_end - a.row_begin + crows - 1) / crows;
    const uint64_t gw = (uint64_t)blockIdx.x * MQ_WAVES + threadIdx.x / MQ_WAVE;
    const uint64_t nw = (uint64_t)gridDim.x * MQ_WAVES;
    uint32_t hint = 0;
    for (uint64_t c = gw; c < nchunks; c += nw) {
        const uint64_t j0 = a.row_begin + c * crows;
        mat_wave_chunk<NC, MatShape<NC>::RPT, NLC>(mj, j0, min(j0 + crows, a.row_end), hint,
                                                   s_segs[threadIdx.x / MQ_WAVE], qn);
    }
}

// Materialisation straight from the sorted records, for outputs whose key
// products are small (mat_seg_use: at most 64 pairs a key).  One tile of
// records per block: the segments with pairs (at least two records each) go
// to LDS as head position, cL and cR in one word, output key and row offset;
// the tile's rows then go out with consecutive threads on consecutive rows,
// each finding its segment by a binary search over the offsets in LDS.
template <int NC, int NLC, int FS, int IPT>
__global__ __launch_bounds__(MQ_BLOCK) void mat_tile_kernel(MatArgs a, RunGrid g, const uint64_t* __restrict__ trow,
                                                            const uint64_t* __restrict__ run_row) {
    constexpr uint32_t TILE = st_tile(IPT), MAXE = TILE / 2 + 1;  // the last segment may have one record here
    static_assert(MAT_SEG_MAX_PAIRS <= 127 && TILE <= 4096, "a segment in one word");
    __shared__ SegTile sm;
    __shared__ uint32_t s_a[MQ_WAVES], s_b[MQ_WAVES];
    __shared__ uint32_t s_ent[MAXE], s_off[MAXE], s_key[MAXE];
    const int nl = NLC >= 0 ? NLC : a.nl, nr = NLC >= 0 ? NC - 1 - NLC : a.nr;
    const int nc = 1 + nl + nr;
    const uint32_t w = threadIdx.x / MQ_WAVE;
    const uint32_t tile = blockIdx.x, base = tile * TILE, lim = min(TILE, a.n - base);
    const bool past = a.n - base > TILE;
    const SegIn in{a.keys, a.vals, a.n, a.n_left};
    uint32_t ek = 0, ev = 0, lk = 0;
    if (w == MQ_WAVES - 1 && past) {
        const uint32_t e = min(base + TILE + lane(), a.n - 1);
        ek = a.keys[e];
        if (!FS) ev = a.vals[e];
        lk = a.keys[base + TILE - 1];
    }
    SegRecs<IPT> rec;
    uint32_t cl[IPT], cr[IPT];
    uint64_t hm[IPT], rm[IPT];
    seg_load<FS, IPT>(in, base, rec);
    seg_masks<FS, IPT>(sm, in, base, rec, hm, rm);
    seg_counts<IPT>(sm, hm, rm, lim, past, cl, cr);
    uint32_t ents = 0, rows = 0;
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const uint32_t c = __umul24(cl[i], cr[i]);
        ents += (uint32_t)__popcll(__ballot(c != 0));
        rows += c;
    }
    const TileBefore t = waves_before(ents, last_lane(wave_incl_u32(rows)), s_a, s_b);
    uint32_t at = t.seg, off = t.row;
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const uint32_t c = __umul24(cl[i], cr[i]), incl = wave_incl_u32(c);
        const uint64_t m = __ballot(c != 0);
        if (c) {
            const uint32_t e = at + (uint32_t)__popcll(m & lt);
            s_ent[e] = ((w * IPT + i) * MQ_WAVE + lane()) | (cl[i] << 12) | (cr[i] << 19);
            s_off[e] = off + incl - c;
            s_key[e] = rec.k[i];
        }
        at += (uint32_t)__popcll(m);
        off += last_lane(incl);
    }
    __syncthreads();  // s_a and s_b have been read
    if (w == MQ_WAVES - 1) {
        // this wave's `at` and `off` count the whole tile; its last segment follows
        uint32_t pos = 0, ol = 0, orr = 0, oc = 0;
        if (past && seg_last<FS, IPT>(sm, in, base + TILE, lk, ek, ev, pos, ol, orr))
            oc = ol && orr ? ol * orr : 0u;  // at most MAT_SEG_MAX_PAIRS
        if (lane() == 0) {
            if (oc) {
                s_ent[at] = pos | (ol << 12) | (orr << 19);
                s_off[at] = off;
                s_key[at] = lk;
            }
            s_a[0] = at + (oc ? 1u : 0u);
            s_b[0] = off + oc;
        }
    }
    __syncthreads();
    const uint32_t ne = s_a[0], nrow = s_b[0];
    if (nrow == 0) return;
    const uint64_t row0 = run_row[tile / g.chunk] + trow[tile];
    const bool sorted_vals = a.use_sval != 0;
    const uint32_t top = 1u << (31 - __builtin_clz(ne));  // the search's first step
    // MR rows per thread at once: their searches and loads overlap
    constexpr int MR = NC <= 4 ? 4 : 2;
    for (uint32_t r0 = threadIdx.x; r0 < nrow; r0 += MR * MQ_BLOCK) {
        uint32_t r[MR], x[MR];
#pragma unroll
        for (int q = 0; q < MR; q++) {
            r[q] = min(r0 + q * MQ_BLOCK, nrow - 1);
            x[q] = 0;
        }
        for (uint32_t step = top; step; step >>= 1) {
#pragma unroll
            for (int q = 0; q < MR; q++) {
                const uint32_t y = x[q] + step;
                if (y < ne && s_off[y] <= r[q]) x[q] = y;
            }
        }
        uint32_t lpos[MR], rpos[MR];
        int32_t v[MR][NC];
#pragma unroll
        for (int q = 0; q < MR; q++) {
            const uint32_t ent = s_ent[x[q]], rr = r[q] - s_off[x[q]];
            const uint32_t st = base + (ent & 4095u), l = (ent >> 12) & 127u, rn = ent >> 19;
            const bool left_in = left_inner_of(l, rn, nl, nr);
            const uint32_t ci = left_in ? l : rn;
            const uint32_t outer = rr / ci, inner = rr - outer * ci;
            lpos[q] = st + (left_in ? inner : outer);
            rpos[q] = st + l + (left_in ? outer : inner);
            v[q][0] = (int32_t)((s_key[x[q]] >> a.key_shift) + (uint32_t)a.key_base);
        }
        if (!sorted_vals) {  // record ids to rows of the tables
#pragma unroll
            for (int q = 0; q < MR; q++) {
                lpos[q] = nl > 0 ? a.vals[lpos[q]] : 0u;
                rpos[q] = nr > 0 ? a.vals[rpos[q]] - a.n_left : 0u;
            }
        }
#pragma unroll
        for (int q = 0; q < MR; q++)
#pragma unroll
            for (int col = 1; col < NC; col++)
                if (col < nc) {
                    const int32_t* src = sorted_vals ? a.sval[col <= nl ? col - 1 : col - 1 - nl]
                                                     : (col <= nl ? a.lcol[col - 1] : a.rcol[col - 1 - nl]);
                    v[q][col] = src[col <= nl ? lpos[q] : rpos[q]];
                }
#pragma unroll
        for (int q = 0; q < MR; q++) {
            const uint64_t j = row0 + r0 + q * MQ_BLOCK;
            if (r0 + q * MQ_BLOCK >= nrow || !MQ_IN_BOUNDS(j, a.row_end)) continue;
#pragma unroll
            for (int col = 0; col < NC; col++)
                if (col < nc) a.out[col][j] = v[q][col];
        }
    }
}

// Segment-major materialisation (mat_seg_group): one wave per group of 64
// keys, for outputs whose key products are small.
template <int NC, int NLC>
__global__ __launch_bounds__(MQ_BLOCK) void mat_seg_kernel(MatArgs a) {
    __shared__ uint64_t s_grp[MQ_WAVES][MAT_SEG_LDS_WORDS];
    const MatJoin mj = mat_join_of<NC, NLC>(a);
    const uint32_t ngroups = (mj.ns + MQ_WAVE - 1) / MQ_WAVE;
    const uint32_t nw = gridDim.x * MQ_WAVES;
    for (uint32_t grp = blockIdx.x * MQ_WAVES + threadIdx.x / MQ_WAVE; grp < ngroups; grp += nw)
        mat_seg_group<NC, NLC>(mj, grp, a.row_end, s_grp[threadIdx.x / MQ_WAVE]);
}

// One pass over the sorted records: every record's value columns move into
// sorted order, so that materialisation reads contiguous ranges instead of
// gathering each output row's values through its record id.
constexpr int GV_UNROLL = 8;

__global__ __launch_bounds__(MQ_BLOCK) void gather_values_kernel(GatherArgs g) {
    const int nv = g.nl > g.nr ? g.nl : g.nr;
    const uint64_t i0 = (uint64_t)blockIdx.x * (MQ_BLOCK * GV_UNROLL) + threadIdx.x;
    uint32_t r[GV_UNROLL];
#pragma unroll
    for (int u = 0; u < GV_UNROLL; u++) r[u] = g.vals[min(i0 + u * MQ_BLOCK, (uint64_t)g.n - 1)];
    for (int c = 0; c < nv; c++) {
        // a side without this column reads one word for all its records
        const bool has_l = c < g.nl, has_r = c < g.nr;
        const int32_t* lc = has_l ? g.lcol[c] : g.rcol[0];
        const int32_t* rc = has_r ? g.rcol[c] : g.lcol[0];
        int32_t x[GV_UNROLL];
#pragma unroll
        for (int u = 0; u < GV_UNROLL; u++) {
            const bool left = r[u] < g.n_left;
            const uint32_t at = left ? (has_l ? r[u] : 0u) : (has_r ? r[u] - g.n_left : 0u);
            x[u] = (left ? lc : rc)[at];
        }
#pragma unroll
        for (int u = 0; u < GV_UNROLL; u++)
            if (i0 + u * MQ_BLOCK < g.n) g.out[c][i0 + u * MQ_BLOCK] = x[u];
    }
}

hipError_t launch_gather_values(const GatherArgs& g, hipStream_t stream) {
    if (g.n == 0 || (g.nl == 0 && g.nr == 0)) return hipSuccess;
    const uint32_t blocks = (g.n - 1) / (MQ_BLOCK * GV_UNROLL) + 1;
    gather_values_kernel<<<blocks, MQ_BLOCK, 0, stream>>>(g);
    return hipGetLastError();
}

hipError_t launch_mat_tiles(const MatArgs& a, int side_bit, void* scratch, hipStream_t stream) {
    const int nc = 1 + a.nl + a.nr;
    if (a.n == 0 || a.row_begin != 0 || a.seg_cl || nc > MAT_MAXNC) return hipErrorInvalidValue;
    if (side_bit && (a.nl > 1 || a.nr > 1)) return hipErrorInvalidValue;
    const RunGrid g = seg_grid(a.n);
    const SegScratch s = seg_tiles(scratch, a.n);
#define MQ_LAUNCH(C, L, F)                                                                              \
    if (seg_few(a.n))                                                                                   \
        mat_tile_kernel<C, L, F, ST_IPT_FEW><<<g.ntiles, MQ_BLOCK, 0, stream>>>(a, g, s.trow, s.run_row); \
    else                                                                                                \
        mat_tile_kernel<C, L, F, ST_IPT><<<g.ntiles, MQ_BLOCK, 0, stream>>>(a, g, s.trow, s.run_row)
#define MQ_CASE(C)                 \
    case C:                        \
        MQ_LAUNCH(C, -1, 0);       \
        break;
    if (side_bit) {  // carried values: at most one per side
        switch (nc * 2 + a.nl) {
            case 1 * 2 + 0: MQ_LAUNCH(1, 0, 1); break;
            case 2 * 2 + 0: MQ_LAUNCH(2, 0, 1); break;
            case 2 * 2 + 1: MQ_LAUNCH(2, 1, 1); break;
            default: MQ_LAUNCH(3, 1, 1); break;
        }
        return hipGetLastError();
    }
    switch (nc) {
        MQ_CASE(1) MQ_CASE(2) MQ_CASE(3) MQ_CASE(4) MQ_CASE(5) MQ_CASE(6) MQ_CASE(7) MQ_CASE(8)
        MQ_CASE(9) MQ_CASE(10) MQ_CASE(11) MQ_CASE(12) MQ_CASE(13) MQ_CASE(14) MQ_CASE(15) MQ_CASE(16)
        default: return hipErrorInvalidValue;
    }
#undef MQ_CASE
#undef MQ_LAUNCH
    return hipGetLastError();
}

hipError_t launch_materialize(const MatArgs& a, hipStream_t stream) {
    if (a.row_end <= a.row_begin) return hipSuccess;
    if (a.row_begin % 16) return hipErrorInvalidValue;
    if (a.seg_major && (a.row_begin != 0 || a.seg_cl != nullptr)) return hipErrorInvalidValue;
    const int nc = 1 + a.nl + a.nr;
    const uint64_t rows = a.row_end - a.row_begin;
    const uint64_t cap = a.max_blocks ? a.max_blocks : MAT_MAX_BLOCKS;
    // narrow joins get the value-column split fixed at compile time
#define MQ_LAUNCH(C, L)                                                                             \
    if (a.seg_major) {                                                                              \
        const uint64_t groups = (a.seg_count + MQ_WAVE - 1) / MQ_WAVE;                              \
        uint32_t blocks = (uint32_t)std::min<uint64_t>((groups + MQ_WAVES - 1) / MQ_WAVES, cap);       \
        mat_seg_kernel<C, L><<<std::max(blocks, 1u), MQ_BLOCK, 0, stream>>>(a);                     \
    } else {                                                                                        \
        const uint64_t crows = a.sparse ? 4 * MQ_WAVE : MatShape<C>::WROWS;                         \
        uint64_t chunks = (rows + crows - 1) / crows;                                               \
        uint32_t blocks = (uint32_t)std::min<uint64_t>((chunks + MQ_WAVES - 1) / MQ_WAVES, cap);       \
        materialize_kernel<C, L><<<blocks, MQ_BLOCK, 0, stream>>>(a);                               \
    }
    if (nc <= 4) {
        const int key = nc * 4 + a.nl;
        switch (key) {
            case 1 * 4 + 0: MQ_LAUNCH(1, 0) break;
            case 2 * 4 + 0: MQ_LAUNCH(2, 0) break;
            case 2 * 4 + 1: MQ_LAUNCH(2, 1) break;
            case 3 * 4 + 0: MQ_LAUNCH(3, 0) break;
            case 3 * 4 + 1: MQ_LAUNCH(3, 1) break;
            case 3 * 4 + 2: MQ_LAUNCH(3, 2) break;
            case 4 * 4 + 0: MQ_LAUNCH(4, 0) break;
            case 4 * 4 + 1: MQ_LAUNCH(4, 1) break;
            case 4 * 4 + 2: MQ_LAUNCH(4, 2) break;
            case 4 * 4 + 3: MQ_LAUNCH(4, 3) break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (nc) {
        case 5: MQ_LAUNCH(5, -1) break;
        case 6: MQ_LAUNCH(6, -1) break;
        case 7: MQ_LAUNCH(7, -1) break;
        case 8: MQ_LAUNCH(8, -1) break;
        case 9: MQ_LAUNCH(9, -1) break;
        case 10: MQ_LAUNCH(10, -1) break;
        case 11: MQ_LAUNCH(11, -1) break;
        case 12: MQ_LAUNCH(12, -1) break;
        case 13: MQ_LAUNCH(13, -1) break;
        case 14: MQ_LAUNCH(14, -1) break;
        case 15: MQ_LAUNCH(15, -1) break;
        case 16: MQ_LAUNCH(16, -1) break;
        default: return hipErrorInvalidValue;
    }
#undef MQ_LAUNCH
    return hipGetLastError();
}

}  // namespace mq
