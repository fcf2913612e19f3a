// Dictionary encoding of RDF terms on gfx950: byte-string terms <-> dense
// int32 identifiers, numbered in order of first appearance (the terms of
// Table 1 become the identifiers the join works on, and results decode back
// to terms).
//
// Encoding a batch of n terms (concatenated bytes + n + 1 offsets):
//   hash     of every term, eight bytes a step;
//   insert   open addressing with linear probing into a table of 64-bit
//            slots [hash >> 32 | ref]: ref is a dictionary identifier, or
//            (bit 31 set) the index of the batch's term that claimed the slot
//            with a 64-bit CAS.  A slot is never emptied while terms are
//            being inserted, so equal terms meet at the first slot their
//            probe sequence finds free or holding them;
//   first    per claimed slot, the lowest batch index of its term (atomicMin);
//   number   the first occurrences of new terms, scanned in batch order,
//            become identifiers dictionary_size + rank;
//   append   their bytes go to the dictionary's byte store (offsets from the
//            same scan) and the table's slots are re-pointed from batch
//            indices to identifiers.
// Decoding copies each identifier's bytes to offsets from a scan of lengths.
// Both copies are driven by the output: a block owns a range of output bytes.
#include "device_common.h"
#include "kernels.h"

#include <algorithm>

namespace mq {

constexpr uint32_t DICT_NEW = 1u << 31;      // ref names a batch index
constexpr uint32_t DICT_NONE = 0xFFFFFFFFu;  // term absent (lookups)
constexpr uint64_t DICT_EMPTY = ~0ull;

static uint32_t grid_of(uint64_t n, uint32_t per_block = 256 * 4, uint32_t cap = 16384) {
    const uint64_t g = (n + per_block - 1) / per_block;
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(g, cap));
}

// Bytes at any alignment (global loads need none).
__device__ __forceinline__ uint64_t load8(const uint8_t* p) {
    uint64_t v;
    __builtin_memcpy(&v, p, 8);
    return v;
}
__device__ __forceinline__ uint32_t load4(const uint8_t* p) {
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

// the last len % 8 bytes of a term (none: 0), from loads that stay inside it
__device__ __forceinline__ uint64_t tail8(const uint8_t* p, int64_t len) {
    const int m = (int)(len & 7);
    if (m == 0) return 0;
    if (len >= 8) return load8(p + len - 8) >> (64 - 8 * m);
    if (m >= 4) return (uint64_t)load4(p + m - 4) << (8 * (m - 4)) | load4(p);  // the overlap agrees
    uint64_t v = p[0];
    if (m > 1) v |= (uint64_t)p[1] << 8;
    if (m > 2) v |= (uint64_t)p[2] << 16;
    return v;
}

// Eight bytes a step, each folded in with a step of the 64-bit finaliser of
// MurmurHash3 (Appleby, public domain), the length first.  (A byte-wise
// FNV-1a, a serial multiply and a one-byte load per byte, made the insert of
// 3M terms of 33 bytes 0.58 ms; it is 0.30 ms, now bound by the chain of
// random reads: slot, the claiming term's offsets, its bytes.)
__device__ __forceinline__ uint64_t term_hash(const uint8_t* p, int64_t len) {
    uint64_t h = 0x9E3779B97F4A7C15ull ^ (uint64_t)len;
    auto fold = [&](uint64_t w) {
        h ^= w;
        h *= 0xFF51AFD7ED558CCDull;
        h ^= h >> 33;
    };
    int64_t k = 0;
    for (; k + 8 <= len; k += 8) fold(load8(p + k));
    if (len & 7) fold(tail8(p, len));
    h *= 0xC4CEB9FE1A85EC53ull;
    return h ^ (h >> 33);
}

__device__ __forceinline__ bool same_bytes(const uint8_t* a, const uint8_t* b, int64_t len) {
    int64_t k = 0;
    for (; k + 8 <= len; k += 8)
        if (load8(a + k) != load8(b + k)) return false;
    return (len & 7) == 0 || tail8(a, len) == tail8(b, len);
}

// offsets non-decreasing from 0: err |= 1 otherwise; *total = the last one
__global__ void dict_check_offsets_kernel(const int64_t* __restrict__ off, uint32_t n, uint32_t* err,
                                          int64_t* __restrict__ total) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += gridDim.x * blockDim.x) {
        const bool bad = i == 0 ? off[0] != 0 : off[i] < off[i - 1];
        if (bad) atomicOr(err, 1u);
        if (i == n) *total = off[n];
    }
}

__global__ void dict_insert_kernel(DictDev d, TermsDev t, int insert, uint32_t* __restrict__ rep,
                                   uint32_t* __restrict__ err) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < t.n; i += gridDim.x * blockDim.x) {
        const uint8_t* p = t.bytes + t.off[i];
        const int64_t len = t.off[i + 1] - t.off[i];
        const uint64_t h = term_hash(p, len);
        const uint64_t tag = h >> 32;
        const uint64_t mine = tag << 32 | (DICT_NEW | i);
        uint64_t slot = h & d.mask;
        uint32_t r = DICT_NONE;
        bool done = false;
        for (uint64_t probe = 0; probe <= d.mask && !done; probe++, slot = (slot + 1) & d.mask) {
            uint64_t cur = __hip_atomic_load(d.table + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cur == DICT_EMPTY) {
                if (!insert) {
                    done = true;  // r stays DICT_NONE
                    break;
                }
                const uint64_t prev = atomicCAS((unsigned long long*)(d.table + slot), DICT_EMPTY, mine);
                if (prev == DICT_EMPTY) {
                    r = DICT_NEW | i;
                    done = true;
                    break;
                }
                cur = prev;
            }
            if ((cur >> 32) != tag) continue;
            const uint32_t ref = (uint32_t)cur;
            const uint8_t* q;
            int64_t qlen;
            if (ref & DICT_NEW) {
                const uint32_t j = ref & ~DICT_NEW;
                q = t.bytes + t.off[j];
                qlen = t.off[j + 1] - t.off[j];
            } else {
                q = d.bytes + d.off[ref];
                qlen = d.off[ref + 1] - d.off[ref];
            }
            if (qlen == len && same_bytes(p, q, len)) {
                r = ref;
                done = true;
            }
        }
        if (!done) atomicOr(err, 2u);  // table full: cannot happen within the capacity checks
        rep[i] = r;
    }
}

// first[j] = lowest batch index whose term claimed slot-owner j (first[]
// pre-set to ~0), over the batch's terms [lo, hi).  A plain read skips the
// atomic once a lower index is in: a frequent term would otherwise send every
// occurrence's atomic to one address, and those serialise (about 11 ns each).
// The launcher takes the batch in growing ranges, so that what is in flight
// before a frequent term's index is in is a few thousand terms and not the
// half million that the chip holds: 3M Zipf terms, 1.10 ms as one range,
// 0.035 ms as three.
__global__ void dict_first_kernel(const uint32_t* __restrict__ rep, uint32_t lo, uint32_t hi,
                                  uint32_t* __restrict__ first) {
    for (uint32_t i = lo + blockIdx.x * blockDim.x + threadIdx.x; i < hi; i += gridDim.x * blockDim.x) {
        const uint32_t r = rep[i];
        if (r == DICT_NONE || !(r & DICT_NEW)) continue;
        uint32_t* f = first + (r & ~DICT_NEW);
        if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > i) atomicMin(f, i);
    }
}

// identifiers: a dictionary term keeps its own, a new term takes
// base + rank of its first occurrence, an absent one (lookup) -1
__global__ void dict_ids_kernel(const uint32_t* __restrict__ rep, const uint32_t* __restrict__ first,
                                const uint32_t* __restrict__ rank, uint32_t n, uint32_t base,
                                int32_t* __restrict__ ids) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t r = rep[i];
        ids[i] = r == DICT_NONE ? -1 : (r & DICT_NEW) ? (int32_t)(base + rank[first[r & ~DICT_NEW]]) : (int32_t)r;
    }
}

// slots claimed by batch terms now name their identifiers (commit) or are
// emptied again (rollback: the table is back to its state before the batch)
__global__ void dict_fix_kernel(DictDev d, const uint32_t* __restrict__ first, const uint32_t* __restrict__ rank,
                                uint32_t base, int commit) {
    for (uint64_t s = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; s <= d.mask;
         s += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t w = d.table[s];
        if (w == DICT_EMPTY || !((uint32_t)w & DICT_NEW)) continue;
        d.table[s] = commit ? (w & 0xFFFFFFFF00000000ull) | (uint64_t)(base + rank[first[(uint32_t)w & ~DICT_NEW]])
                            : DICT_EMPTY;
    }
}

// ---- numbering scans --------------------------------------------------------
// Items with a length each (a scan of counts and of bytes at once): the new
// terms of a batch in batch order, or the terms of identifiers to decode.  A
// reduce pass and one block over its partials give the totals; the write pass
// recomputes the items, and runs after the host has checked that they fit.
constexpr uint32_t SCAN_IPT = 8;
constexpr uint32_t SCAN_TILE = MQ_BLOCK * SCAN_IPT;

struct NewTerms {  // first occurrences of terms the dictionary lacked
    TermsDev t;
    const uint32_t* rep;
    const uint32_t* first;
    __device__ __forceinline__ bool at(uint32_t i, uint64_t* len, uint32_t*) const {
        const uint32_t r = rep[i];
        if (r == DICT_NONE || !(r & DICT_NEW) || first[r & ~DICT_NEW] != i) return false;
        *len = (uint64_t)(t.off[i + 1] - t.off[i]);
        return true;
    }
};

struct IdTerms {  // every identifier (err |= 1 for one outside [0, nterms), of no bytes)
    DictDev d;
    const int32_t* ids;
    __device__ __forceinline__ bool at(uint32_t i, uint64_t* len, uint32_t* err) const {
        const int32_t id = ids[i];
        if (id < 0 || (uint32_t)id >= d.nterms) {
            *err = 1u;
            *len = 0;
        } else {
            *len = (uint64_t)(d.off[id + 1] - d.off[id]);
        }
        return true;
    }
};

template <class Items>
__global__ __launch_bounds__(MQ_BLOCK) void scan_reduce_kernel(Items it, uint32_t n, uint64_t* __restrict__ pcnt,
                                                               uint64_t* __restrict__ plen, uint32_t* err) {
    __shared__ uint64_t tmp[2][MQ_WAVES];
    const uint32_t base = blockIdx.x * SCAN_TILE + threadIdx.x;
    uint64_t c = 0, s = 0;
    uint32_t bad = 0;
#pragma unroll
    for (uint32_t k = 0; k < SCAN_IPT; k++) {
        const uint32_t i = base + k * MQ_BLOCK;  // any order within the tile
        uint64_t len = 0;
        if (i < n && it.at(i, &len, &bad)) {
            c++;
            s += len;
        }
    }
    if (bad) atomicOr(err, 1u);
    c = wave_sum(c);
    s = wave_sum(s);
    if (lane() == 0) {
        tmp[0][threadIdx.x / MQ_WAVE] = c;
        tmp[1][threadIdx.x / MQ_WAVE] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < MQ_WAVES; w++) {
            c += tmp[0][w];
            s += tmp[1][w];
        }
        pcnt[blockIdx.x] = c;
        plen[blockIdx.x] = s;
    }
}

// one block: both partials -> exclusive prefixes, the sums to the totals
__global__ __launch_bounds__(MQ_BLOCK) void scan_parts_kernel(uint64_t* __restrict__ pcnt, uint64_t* __restrict__ plen,
                                                              uint32_t np, uint32_t* __restrict__ total_cnt,
                                                              uint64_t* __restrict__ total_len) {
    __shared__ uint64_t tmp[MQ_WAVES];
    const uint32_t per = (np + MQ_BLOCK - 1) / MQ_BLOCK;
    const uint32_t b0 = min(threadIdx.x * per, np), b1 = min(b0 + per, np);
    uint64_t c = 0, s = 0;
    for (uint32_t k = b0; k < b1; k++) {
        c += pcnt[k];
        s += plen[k];
    }
    uint64_t call, sall;
    uint64_t crun = block_excl_scan<uint64_t>(c, tmp, &call), srun = block_excl_scan<uint64_t>(s, tmp, &sall);
    for (uint32_t k = b0; k < b1; k++) {
        const uint64_t cv = pcnt[k], sv = plen[k];
        pcnt[k] = crun;
        plen[k] = srun;
        crun += cv;
        srun += sv;
    }
    if (threadIdx.x == 0) {
        *total_cnt = (uint32_t)call;
        *total_len = sall;
    }
}

// out(i, number of the item, its offset) for every item
template <class Items, class Out>
__global__ __launch_bounds__(MQ_BLOCK) void scan_write_kernel(Items it, uint32_t n, const uint64_t* __restrict__ pcnt,
                                                              const uint64_t* __restrict__ plen, Out out) {
    __shared__ uint64_t tmp[MQ_WAVES];
    const uint32_t base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_IPT;
    uint64_t len[SCAN_IPT], s = 0, c = 0;
    uint32_t has = 0, bad = 0;
#pragma unroll
    for (uint32_t k = 0; k < SCAN_IPT; k++) {
        len[k] = 0;
        if (base + k < n && it.at(base + k, &len[k], &bad)) {
            has |= 1u << k;
            c++;
            s += len[k];
        }
    }
    uint64_t all;
    uint64_t crun = pcnt[blockIdx.x] + block_excl_scan<uint64_t>(c, tmp, &all);
    uint64_t srun = plen[blockIdx.x] + block_excl_scan<uint64_t>(s, tmp, &all);
#pragma unroll
    for (uint32_t k = 0; k < SCAN_IPT; k++)
        if ((has >> k) & 1u) {
            out(base + k, (uint32_t)crun, srun);
            crun++;
            srun += len[k];
        }
}

struct NewOut {  // rank of the first occurrence, its index by rank, its offset in the byte store
    uint32_t* rank;
    uint32_t* index;
    int64_t* off;  // the offsets from the first new identifier on
    int64_t bbase;
    __device__ __forceinline__ void operator()(uint32_t i, uint32_t r, uint64_t at) const {
        rank[i] = r;
        index[r] = i;
        off[r] = bbase + (int64_t)at;
    }
};

struct IdOut {
    int64_t* pos;
    __device__ __forceinline__ void operator()(uint32_t i, uint32_t, uint64_t at) const { pos[i] = (int64_t)at; }
};

__global__ void dict_end_kernel(int64_t* p, int64_t v) { *p = v; }

static uint32_t scan_parts(uint32_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE; }
size_t scan_part_bytes(uint32_t n) { return 16ull * (scan_parts(n) + 1); }

template <class Items>
static hipError_t scan_totals(const Items& it, uint32_t n, void* part, uint32_t* total_cnt, uint64_t* total_len,
                              uint32_t* err, hipStream_t s) {
    if (n == 0 || n > DICT_SCAN_MAX) return hipErrorInvalidValue;  // callers skip empty batches
    const uint32_t np = scan_parts(n);
    uint64_t* pc = static_cast<uint64_t*>(part);
    scan_reduce_kernel<Items><<<np, MQ_BLOCK, 0, s>>>(it, n, pc, pc + np, err);
    scan_parts_kernel<<<1, MQ_BLOCK, 0, s>>>(pc, pc + np, np, total_cnt, total_len);
    return hipGetLastError();
}

template <class Items, class Out>
static hipError_t scan_write(const Items& it, uint32_t n, void* part, const Out& out, hipStream_t s) {
    if (n == 0 || n > DICT_SCAN_MAX) return hipErrorInvalidValue;
    const uint32_t np = scan_parts(n);
    uint64_t* pc = static_cast<uint64_t*>(part);
    scan_write_kernel<Items, Out><<<np, MQ_BLOCK, 0, s>>>(it, n, pc, pc + np, out);
    return hipGetLastError();
}

// ---- copying terms ----------------------------------------------------------
// Terms back to back in out[0 .. total): term i takes out[pos[i] - base ..
// pos[i + 1] - base) (the last one ends at total) from src.of(i).  HBM-bound
// on the written bytes and short on parallel work per term, so the output is
// what is split: a block owns up to COPY_BYTES consecutive bytes from a 16-byte
// boundary, finds its first term with a 64-ary search, stages offsets and
// sources of COPY_TERMS terms at a time in LDS, and each thread writes whole
// 16-byte pieces, looking its piece's term up in LDS and loading four bytes
// at a time where a term holds them.  A term of any length, and any run of
// empty terms, is spread the same way.  3M terms of 33 bytes: 0.44 ms with
// one wave per term and one byte per lane, 0.11 ms so.  A small output is
// split over COPY_BLOCKS blocks first, down to pieces of COPY_LEAST bytes: its
// terms are short, and a block takes 512 of them after another (decode of
// 10,000 terms of 3 bytes: 81 us in pieces of 8,192 bytes, 45 so; 400,000
// terms: 89 and 50).
constexpr uint32_t COPY_BYTES = 8192, COPY_LEAST = 512, COPY_BLOCKS = 1024;
constexpr uint32_t COPY_TERMS = 512;

struct BatchSrc {
    TermsDev t;
    const uint32_t* index;
    __device__ __forceinline__ const uint8_t* of(uint32_t r) const { return t.bytes + t.off[index[r]]; }
};
struct DictSrc {
    DictDev d;
    const int32_t* ids;
    __device__ __forceinline__ const uint8_t* of(uint32_t i) const { return d.bytes + d.off[ids[i]]; }
};

// last i in [lo, n) with pos[i] <= v (pos ascends, pos[lo] <= v); every lane of the wave calls it
__device__ __forceinline__ uint32_t term_at(const int64_t* __restrict__ pos, uint32_t lo, uint32_t n, int64_t v) {
    uint32_t hi = n - 1;
    while (hi > lo) {
        const uint32_t step = (hi - lo + MQ_WAVE) / MQ_WAVE;
        const uint64_t p = (uint64_t)lo + (uint64_t)lane() * step;
        const uint64_t m = __ballot(p <= hi && pos[p] <= v);  // a prefix of lanes, lane 0 always set
        const uint32_t top = 63u - (uint32_t)__clzll(m);
        lo += top * step;
        hi = min(hi, lo + step - 1);
    }
    return lo;
}

template <class Src>
__global__ __launch_bounds__(MQ_BLOCK) void copy_terms_kernel(Src src, const int64_t* __restrict__ pos, uint32_t n,
                                                              int64_t base, int64_t total, uint32_t per,
                                                              uint8_t* __restrict__ out) {
    __shared__ int32_t s_off[COPY_TERMS + 1];  // offsets from c0, clamped to the block's range
    __shared__ const uint8_t* s_src[COPY_TERMS];
    // this block's bytes [c0, c1) of the output; c0 is 16-byte aligned in memory but for the first block
    const int64_t skew = (int64_t)(reinterpret_cast<uintptr_t>(out) & 15u);
    const int64_t a0 = (int64_t)blockIdx.x * per - skew;  // aligned start (may lie before the output)
    const int64_t c0 = max(a0, (int64_t)0), c1 = min(a0 + (int64_t)per, total);
    int64_t cur = c0;
    uint32_t i = 0;
    while (cur < c1) {
        i = term_at(pos, i, n, base + cur);  // the term of byte cur (past any empty ones)
        const uint32_t m = min(n - i, COPY_TERMS);
        for (uint32_t k = threadIdx.x; k < m; k += MQ_BLOCK) {
            // the first may begin before the block; the last ones may lie past its end and go unread
            const int64_t p = pos[i + k] - base;
            s_off[k] = (int32_t)(min(max(p, c0), c1) - c0);
            s_src[k] = p < c1 ? src.of(i + k) + (p < c0 ? c0 - p : 0) : nullptr;
        }
        if (threadIdx.x == 0) s_off[m] = (int32_t)(min(i + m < n ? pos[i + m] - base : total, c1) - c0);
        __syncthreads();
        const int32_t lo = (int32_t)(cur - c0), hi = s_off[m];
        // 16-byte pieces of memory that meet [lo, hi)
        const int32_t lead = (int32_t)(c0 - a0);  // bytes of the first piece that lie before the output
        for (int32_t g = (lo + lead) / 16 + (int32_t)threadIdx.x; g * 16 - lead < hi; g += MQ_BLOCK) {
            const int32_t b0 = max(g * 16 - lead, lo), b1 = min(g * 16 - lead + 16, hi);
            uint32_t x = 0, y = m - 1;  // last term with s_off <= b0
            while (x < y) {
                const uint32_t mid = (x + y + 1) / 2;
                if (s_off[mid] <= b0) x = mid;
                else y = mid - 1;
            }
            if (b1 - b0 == 16) {
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int32_t at = b0 + 4 * q;
                    while (s_off[x + 1] <= at) x++;
                    if (s_off[x + 1] - at >= 4) {
                        w[q] = load4(s_src[x] + (at - s_off[x]));
                    } else {
                        uint32_t v = 0;
#pragma unroll
                        for (int b = 0; b < 4; b++) {
                            while (s_off[x + 1] <= at + b) x++;
                            v |= (uint32_t)s_src[x][at + b - s_off[x]] << (8 * b);
                        }
                        w[q] = v;
                    }
                }
                *reinterpret_cast<uint4*>(out + c0 + b0) = make_uint4(w[0], w[1], w[2], w[3]);
            } else {
                for (int32_t at = b0; at < b1; at++) {
                    while (s_off[x + 1] <= at) x++;
                    out[c0 + at] = s_src[x][at - s_off[x]];
                }
            }
        }
        cur = c0 + hi;
        __syncthreads();
    }
}

template <class Src>
static hipError_t copy_terms(const Src& src, const int64_t* pos, uint32_t n, int64_t base, int64_t total, uint8_t* out,
                             hipStream_t s) {
    if (n == 0 || total == 0) return hipSuccess;
    const uint64_t span = (uint64_t)total + (reinterpret_cast<uintptr_t>(out) & 15u);
    // a multiple of 16, so that every piece but the first starts on a 16-byte boundary
    const uint32_t per = (uint32_t)std::min<uint64_t>(
        COPY_BYTES, std::max<uint64_t>(COPY_LEAST, span / COPY_BLOCKS / 16 * 16));
    copy_terms_kernel<Src><<<(uint32_t)((span + per - 1) / per), MQ_BLOCK, 0, s>>>(src, pos, n, base, total, per, out);
    return hipGetLastError();
}

// ---- launchers ------------------------------------------------------------
hipError_t launch_dict_check_offsets(const int64_t* off, uint32_t n, uint32_t* err, int64_t* total, hipStream_t s) {
    dict_check_offsets_kernel<<<grid_of(uint64_t(n) + 1), 256, 0, s>>>(off, n, err, total);
    return hipGetLastError();
}

hipError_t launch_dict_encode_front(const DictDev& d, const TermsDev& t, int insert, DictScratch w, hipStream_t s) {
    if (t.n == 0) return hipSuccess;
    dict_insert_kernel<<<grid_of(t.n, 256, 65536), 256, 0, s>>>(d, t, insert, w.rep, w.err);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !insert) return e;
    for (uint32_t lo = 0, hi = 4096; lo < t.n; lo = hi, hi = hi > t.n / 32 ? t.n : hi * 32) {
        hi = std::min(hi, t.n);
        dict_first_kernel<<<grid_of(hi - lo), 256, 0, s>>>(w.rep, lo, hi, w.first);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return scan_totals(NewTerms{t, w.rep, w.first}, t.n, w.part, w.new_terms, w.new_bytes, w.err, s);
}

hipError_t launch_dict_ids(const TermsDev& t, DictScratch w, uint32_t base, int32_t* ids, hipStream_t s) {
    if (t.n == 0) return hipSuccess;
    dict_ids_kernel<<<grid_of(t.n), 256, 0, s>>>(w.rep, w.first, w.rank, t.n, base, ids);
    return hipGetLastError();
}

hipError_t launch_dict_append(const DictDev& d, const TermsDev& t, DictScratch w, uint32_t base, int64_t bbase,
                              uint32_t new_terms, int64_t new_bytes, hipStream_t s) {
    if (t.n == 0) return hipSuccess;
    hipError_t e = scan_write(NewTerms{t, w.rep, w.first}, t.n, w.part, NewOut{w.rank, w.index, d.off + base, bbase}, s);
    if (e != hipSuccess) return e;
    dict_end_kernel<<<1, 1, 0, s>>>(d.off + base + new_terms, bbase + new_bytes);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return copy_terms(BatchSrc{t, w.index}, d.off + base, new_terms, bbase, new_bytes, d.bytes + bbase, s);
}

hipError_t launch_dict_fix(const DictDev& d, DictScratch w, uint32_t base, int commit, hipStream_t s) {
    dict_fix_kernel<<<grid_of(d.mask + 1), 256, 0, s>>>(d, w.first, w.rank, base, commit);
    return hipGetLastError();
}

hipError_t launch_dict_decode_size(const DictDev& d, const int32_t* ids, uint32_t n, uint32_t* count, uint64_t* total,
                                   void* part, uint32_t* err, hipStream_t s) {
    return scan_totals(IdTerms{d, ids}, n, part, count, total, err, s);
}

hipError_t launch_dict_decode(const DictDev& d, const int32_t* ids, uint32_t n, int64_t total, void* part,
                              int64_t* pos, uint8_t* out, hipStream_t s) {
    hipError_t e = scan_write(IdTerms{d, ids}, n, part, IdOut{pos}, s);
    if (e != hipSuccess) return e;
    dict_end_kernel<<<1, 1, 0, s>>>(pos + n, total);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return copy_terms(DictSrc{d, ids}, pos, n, 0, total, out, s);
}

}  // namespace mq
