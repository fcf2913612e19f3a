// Host-side launchers of the gfx950 kernels (one translation unit per
// kernel family).  All launches are asynchronous on the given stream; a
// launcher returns the launch error, if any.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mail.h"

namespace mq {

constexpr uint32_t BLOCK_THREADS = 256;  // threads per block of every tiled kernel

// ---- shuffle: LSD radix sort (k_sort.hip) --------------------------------
// Keys of a first pass come from two int32 segments (k0[0..n0) then
// k1[0..n1)), minus `base`; the payload is the position in that
// concatenation.
// First-pass source of a join's shuffle: the LEFT key column k0 (n0 rows)
// then the RIGHT one k1 (n1 rows), keys relative to base.  carry = 0: the
// payload is the record's position in that concatenation (RIGHT records
// from n0 on).  carry = 1: the payload is the record's value cell (v0 or v1;
// a side without a value column points at any column of its rows and its
// payloads go unused) and the key is (relative key << 1) | side, so LEFT
// records still sort ahead of RIGHT ones within a key.
// Relative keys are cut to `mask`, the bits the sort orders: the segment
// kernels search for a run's end in sorted keys, and a caller's key bound that
// does not hold must leave them keys that are in order (such records then meet
// under the wrong keys).
struct SortSrc {
    const int32_t* k0;
    uint32_t n0;
    const int32_t* k1;
    uint32_t n1;
    int32_t base;
    const int32_t* v0;
    const int32_t* v1;
    int32_t carry;
    uint32_t mask = ~0u;
};

// Merge join of two tables already sorted on the key (k_merge.hip).  One
// pass over the smaller side: at the head of each key run, the run's end is
// found by galloping and the key's run in the larger side by binary search;
// keys present on both sides become segments (ascending key), each with its
// LEFT run, RIGHT run and output offset; *nseg gets their count.
struct MergeArgs {
    const int32_t* skey;   // smaller side's key column (sorted)
    uint32_t ns;
    const int32_t* bkey;   // larger side's key column (sorted)
    uint32_t nb;
    int32_t small_is_left;
    uint32_t* seg_lstart;
    uint32_t* seg_lcount;
    uint32_t* seg_rstart;
    uint32_t* seg_rcount;
    uint64_t* seg_off;
    uint32_t* nseg;
};
// mail: segments (1 word), a pad word, rows (2 words).  tile_ctr is 0 before
// and after the launch.
hipError_t launch_merge_segments(const MergeArgs& a, uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, Mail mail,
                                 hipStream_t stream);
uint32_t merge_tiles(uint32_t ns);

// Semi-join reduction (k_semi.hip).  Bits of keys - base are set in bm
// (range bits, cleared by the caller); the filter keeps the records of
// `keys` whose relative key is set, writing (relative key, id_base + index)
// in input order to kout/vout and the kept count to *count and the mail's
// first word.  scratch: semi_scratch_bytes(n), 8-byte aligned, at most 8 bytes
// per record of both sides; masks and counts are set from it.
struct SemiArgs {
    const int32_t* keys;
    uint32_t n;
    int32_t base;
    uint64_t range;  // bits in bm
    const uint32_t* bm;
    uint32_t id_base;
    uint32_t* kout;
    uint32_t* vout;
    uint32_t* count;
    uint64_t* masks;
    uint32_t* counts;
};
hipError_t launch_bitmap_set(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, uint32_t* bm,
                             hipStream_t stream);
hipError_t launch_semi_filter(const SemiArgs& a, void* scratch, Mail mail, hipStream_t stream);
size_t semi_scratch_bytes(uint32_t n);
// Exact join size: cnt[k - base] += 1 over one side's keys (cnt cleared by
// the caller, range entries), then *total += sum of cnt[k - base] over the
// other side's keys (*total cleared by the caller).
hipError_t launch_key_count(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, uint32_t* cnt,
                            hipStream_t stream);
hipError_t launch_key_dot(const int32_t* keys, uint32_t n, int32_t base, uint64_t range, const uint32_t* cnt,
                          uint64_t* total, hipStream_t stream);
// 1/64 of that sum, over a sample of the keys, in the mail (2 words).  cnt:
// key_sample_words(range) words of scratch; acc: three words (8-byte aligned),
// 0 before and after the launch.
inline uint64_t key_sample_words(uint64_t range) { return (range + 63) / 64; }
hipError_t launch_key_sample(const int32_t* a, uint32_t na, const int32_t* b, uint32_t nb, int32_t base,
                             uint64_t range, uint32_t* cnt, uint32_t* acc, Mail mail, hipStream_t stream);
// all n records of one side at kout/vout[(*at_dev or 0) + i], relative keys cut to mask
hipError_t launch_side_records(const int32_t* keys, uint32_t n, int32_t base, uint32_t mask, uint32_t id_base,
                               const uint32_t* at_dev, uint32_t* kout, uint32_t* vout, hipStream_t stream);

// Sort and segments of a small join in one launch (k_small.hip): the records
// of `src` (kin null) or at kin/vin, sorted on the key_bits bits from lo_bit on
// into kout/vout (may be kin/vin), segments and *nseg as launch_seg_write writes
// them, mail as launch_seg_sum's.
constexpr uint32_t SMALL_JOIN = 4096;
struct SmallJoin {
    SortSrc src;
    const uint32_t* kin;
    const uint32_t* vin;
    uint32_t n, n_left;
    int32_t lo_bit, key_bits, side_bit;
    int32_t width;  // digit width, set by the launch
    uint32_t* kout;
    uint32_t* vout;
    uint32_t* seg_start;
    uint32_t* seg_split;
    uint64_t* seg_off;
    uint32_t* nseg;
};
// digits of at most 8 bits, spread evenly
inline int small_join_width(int key_bits) {
    const int passes = key_bits > 8 ? (key_bits + 7) / 8 : 1;
    return key_bits > 0 ? (key_bits + passes - 1) / passes : 1;
}
hipError_t launch_small_join(SmallJoin a, Mail mail, hipStream_t stream);

// Counting shuffle of a join with few distinct keys (k_few.hip).  Every word
// of a bitmap of range bits becomes an entry (bits, bits set in the words
// before); the first FEW_KEYS set bits' positions go to keys (base added) and
// their number to the mail (2 words).  status: few_table_tiles look-back words.
constexpr uint32_t FEW_KEYS = 1023;  // a digit of 10 bits, its last value left for records without a partner
struct FewEntry {
    uint32_t bits, before;
};
hipError_t launch_few_table(const uint32_t* bm, uint64_t range, int32_t base, FewEntry* table, int32_t* keys,
                            uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, Mail mail, hipStream_t stream);
uint32_t few_table_tiles(uint64_t range);
// One side of that shuffle: rows whose key - base is in the table, grouped by
// the key's rank in it, in input order inside a group.  Row i's values are
// in[c][ids[i]] (ids null: in[c][i]) and go to out[c].
// The columns of a side are limited by the scratch, which stays below the 24
// bytes per record that the sort asks for: per LEFT row 6 of bitmap and table
// and 4 for the key and each column, per RIGHT row 8.1 of filtered records and 4
// for each column.
constexpr int FEW_COLS = 3;
struct FewSide {
    const int32_t* keys;
    const uint32_t* ids;
    uint32_t n;
    int32_t base;
    uint64_t range;
    const FewEntry* table;
    int32_t nv;
    const int32_t* in[FEW_COLS];
    int32_t* out[FEW_COLS];
};
// digit width for a table of nkeys <= FEW_KEYS keys
int few_bits(uint32_t nkeys);
// rows of each rank into hist[2^rb]; part: few_part_words(rb)
hipError_t launch_few_hist(const FewSide& s, int rb, uint32_t* part, uint32_t* hist, hipStream_t stream);
uint32_t few_part_words(int rb);
// Segments of nkeys keys from both sides' histograms; every key has rows on
// both sides.  Runs, output offsets and *nseg as launch_merge_segments writes
// them; lkey[first row of the LEFT run] = the key; mail: nkeys, a pad word,
// pairs (2 words, capped at 2^40 - 1), the LEFT rows that have a partner.
hipError_t launch_few_segments(const uint32_t* lhist, const uint32_t* rhist, const int32_t* keys, uint32_t nkeys,
                               uint32_t* seg_ls, uint32_t* seg_lc, uint32_t* seg_rs, uint32_t* seg_rc,
                               uint64_t* seg_off, uint32_t* nseg, int32_t* lkey, Mail mail, hipStream_t stream);
// the rows of s into their n_out places; s.nv >= 1; status: few_status_words
hipError_t launch_few_pass(const FewSide& s, int rb, const uint32_t* hist, uint32_t n_out, uint64_t* status,
                           uint32_t* tile_ctr, uint32_t epoch, hipStream_t stream);
size_t few_status_words(uint32_t n, int rb);

// Digit histograms of `passes` passes into hist[passes][2^rb] (overwritten);
// the first digit's lowest bit is bit `shift0` of the key.
// keys == nullptr: read the keys from `src`.  `part` is scratch of
// radix_hist_part_words(rb, passes) words.
hipError_t launch_radix_hist(const SortSrc& src, const uint32_t* keys, uint32_t n, int rb, int shift0, int passes,
                             uint32_t* part, uint32_t* hist, hipStream_t stream);
uint32_t radix_hist_part_words(int rb, int passes);
// hist[c] = the sum of part[r * width + c] over r < rows
hipError_t launch_hist_reduce(const uint32_t* part, uint32_t rows, uint32_t width, uint32_t* hist,
                              hipStream_t stream);
// One stable pass on the digit whose lowest bit is `shift`.  kin == nullptr: first-pass mode from
// `src` (vin ignored).  hist_pass = this pass's histogram; status holds
// radix_tiles(n,kpt,rb,true) * 2^rb words; tile_ctr is 0 before and after the
// launch.
hipError_t launch_radix_pass(int rb, int kpt, const SortSrc& src, const uint32_t* kin, const uint32_t* vin,
                             uint32_t* kout, uint32_t* vout, uint32_t n, int shift, const uint32_t* hist_pass,
                             uint64_t* status, uint32_t* tile_ctr, uint32_t epoch, hipStream_t stream);
// record tiles of a radix pass over n records (gen: the first pass, reading
// the input columns; its tiles are never larger than the other passes')
uint32_t radix_tiles(uint32_t n, int kpt, int rb, bool gen);

// ---- reduce (k_reduce.hip) -------------------------------------------------
// The segments of the sorted records (records of one key; LEFT ones first):
// *nseg and the mail get how many there are, the mail also their pairs (the
// sum of cL * cR, capped at 2^40 - 1) and the largest single product: words
// 0, 2-3 and 4-5.  The side of a record is the key's low bit (side_bit: a
// carried shuffle, segments then group keys >> 1) or payload >= n_left.
// scratch: seg_scratch_bytes(n, false) bytes, read again by launch_seg_write
// and launch_mat_tiles.
hipError_t launch_seg_sum(const uint32_t* keys, const uint32_t* vals, uint32_t n, uint32_t n_left, int side_bit,
                          uint32_t* nseg, void* scratch, Mail mail, hipStream_t stream);
// seg_start[s] = first position of the s-th distinct key, seg_split[s] =
// position of its first RIGHT record, or its end when it has none, seg_off[s]
// = pairs of the segments before it.
hipError_t launch_seg_write(const uint32_t* keys, const uint32_t* vals, uint32_t n, uint32_t n_left, int side_bit,
                            uint32_t* seg_start, uint32_t* seg_split, uint64_t* seg_off, void* scratch,
                            hipStream_t stream);
// The same for records with break flags (a composite key sorted word by word;
// launch_key_breaks: a flagged record starts a segment too): starts, splits
// and their count, then offsets and the mail as above.  max_seg bounds the
// device count *nseg (sizes the grids).  scratch: seg_scratch_bytes(n, true).
hipError_t launch_seg_heads(const uint32_t* keys, const uint32_t* vals, const uint8_t* brk, uint32_t n,
                            uint32_t n_left, uint32_t* seg_start, uint32_t* seg_split, uint32_t* nseg, void* scratch,
                            hipStream_t stream);
hipError_t launch_seg_count(uint32_t n, const uint32_t* seg_start, const uint32_t* nseg, uint32_t max_seg,
                            const uint32_t* seg_split, uint64_t* seg_off, Mail mail, void* scratch,
                            hipStream_t stream);
size_t seg_scratch_bytes(uint32_t n, bool brk);

// Value columns in sorted record order: for every record i, with
// r = vals[i], out[c][i] = lcol[c][r] (a LEFT record, r < n_left, c < nl) or
// rcol[c][r - n_left] (a RIGHT record, c < nr).
struct GatherArgs {
    const uint32_t* vals;
    uint32_t n, n_left;
    int32_t nl, nr;
    const int32_t* lcol[16];
    const int32_t* rcol[16];
    int32_t* out[16];
};
hipError_t launch_gather_values(const GatherArgs& g, hipStream_t stream);

struct MatArgs {
    const uint32_t* keys;      // sorted relative keys
    const uint32_t* vals;      // sorted payloads (record positions)
    const uint32_t* seg_start;
    const uint32_t* seg_split;
    const uint64_t* seg_off;
    const uint32_t* nseg;      // device count of segments
    uint32_t n;                // records
    uint32_t n_left;
    int32_t key_base;
    int32_t nl, nr;            // value columns of each side
    const int32_t* lcol[16];
    const int32_t* rcol[16];
    int32_t* out[16];          // 1 + nl + nr output columns
    uint64_t row_begin, row_end;  // materialise output rows [row_begin, row_end)
    const int32_t* sval[16];   // value columns in sorted record order (GatherArgs.out), if use_sval
    int32_t use_sval;
    // merge join (seg_cl != null): segment s pairs LEFT rows [seg_start[s],
    // + seg_cl[s]) of lcol with RIGHT rows [seg_split[s], + seg_cr[s]) of
    // rcol; keys is the LEFT key column (key_base 0); vals and sval unused
    const uint32_t* seg_cl;
    const uint32_t* seg_cr;
    // 1: one 256-row sub-chunk per wave (a sparse output: few rows per
    // segment, so the per-row searches want many waves); 0: the default
    int32_t sparse;
    // 1: keys carry the side in their low bit (output key = (key >> 1) + base)
    int32_t key_shift;
    // 1: segment-major writing (one wave per 64 keys; see mat_seg_use);
    // needs row_begin == 0, row_end == |RS| and seg_cl == null
    int32_t seg_major;
    uint32_t seg_count;  // host copy of *nseg (sizes the segment-major grid)
    uint32_t max_blocks; // grid cap of the launch (0: MAT_MAX_BLOCKS); waves stride over the work
};
constexpr uint32_t MAT_MAX_BLOCKS = 256 * 32;
// Segment-major materialisation pays for sparse outputs: fewer than
// MAT_SEG_ROWS_PER_SEG output rows per key on average and no key product
// above MAT_SEG_MAX_PAIRS, so a wave writes at most 4,096 rows.  With a few
// hundred rows per key, 64-key groups are too coarse a work item (a batch of
// such joins materialised 15% slower than with the row-chunk kernel).
constexpr uint64_t MAT_SEG_MAX_PAIRS = 64;
constexpr uint64_t MAT_SEG_ROWS_PER_SEG = 64;
__host__ __device__ inline bool mat_seg_use(uint64_t rows, uint64_t nseg, uint64_t max_pairs) {
    return rows < MAT_SEG_ROWS_PER_SEG * nseg && max_pairs <= MAT_SEG_MAX_PAIRS;
}
hipError_t launch_materialize(const MatArgs& a, hipStream_t stream);
// the rows straight from the sorted records (mat_seg_use outputs), after
// launch_seg_sum on the same records and scratch; a's segment arrays are not read
hipError_t launch_mat_tiles(const MatArgs& a, int side_bit, void* scratch, hipStream_t stream);

// ---- map and filters (k_map.hip) -----------------------------------------
// Stream compaction of the rows of up to 16 int32 columns that pass every
// equality term; copies the selected columns.  A term compares column a
// with column b (b >= 0) or with constant c (b < 0).
struct CompactArgs {
    const int32_t* in[16];
    int32_t nin;
    uint64_t n;
    int32_t nterm;
    int32_t term_a[6];
    int32_t term_b[6];
    int32_t term_c[6];
    int32_t nout;
    int32_t out_src[16];
    int32_t* out[16];
    uint64_t* count;           // device: rows kept
};
// u64 words of device scratch launch_compact needs for n rows (block
// counts, then one mask word per 64 rows of whole tiles)
size_t compact_scratch_words(uint64_t n);
// a.n >= 1.  status: compact_status_words() look-back words; run_ctr is 0
// before and after the launch; mail: the rows kept (2 words).
uint32_t compact_status_words();
hipError_t launch_compact(const CompactArgs& a, uint64_t* scratch, uint64_t* status, uint32_t* run_ctr, uint32_t epoch,
                          Mail mail, hipStream_t stream);

// Range location in sorted columns: for query q, lo/hi start as the given
// range; level 1 narrows it to rows whose col1 value equals v1, level 2
// (if col2) narrows further to col2 == v2.  out[2q], out[2q+1] = result.
struct LocateQuery {
    const int32_t* col1;
    const int32_t* col2;
    int64_t lo, hi;
    int32_t v1, v2;
};
// One query by value, its range in the mail (2 x 2 words); or nq queries and
// their ranges in host-visible memory, the mail posted when all are written
// (done_ctr is 0 before and after the launch).
hipError_t launch_locate_one(const LocateQuery& q, Mail mail, hipStream_t stream);
hipError_t launch_locate(const LocateQuery* q, int32_t nq, int64_t* out, uint32_t* done_ctr, Mail mail,
                         hipStream_t stream);
// the mail's data = src[0 .. words)
hipError_t launch_publish(const uint32_t* src, uint32_t words, Mail mail, hipStream_t stream);

// ---- batched joins (k_batch.hip) -----------------------------------------
// Every size and pointer of a batch lives in device memory (BatchHdr and
// its BatchJoin array), so one captured graph serves every batch that uses
// the same digit width, tile size and pass count.
constexpr int BATCH_MAXNC = 8;  // output columns per batched join

struct BatchJoin {
    const int32_t* lkey;
    const int32_t* rkey;
    const int32_t* lcol[BATCH_MAXNC];
    const int32_t* rcol[BATCH_MAXNC];
    int32_t* out[BATCH_MAXNC];  // set on the device by the placement kernel
    uint32_t nl, nr;            // rows of each side
    uint32_t rec_off;           // first record slot (a multiple of the record tile)
    uint32_t tile_off, ntiles;  // record tiles [tile_off, tile_off + ntiles)
    int32_t key_base;
    int32_t nvl, nvr;           // value columns of each side
    // results (written on the device)
    uint32_t nseg;
    uint32_t status;            // 0 ok, 1 did not fit the output region, 2 over 2^40 rows
    uint64_t total;             // exact |RS| (saturating at 2^40 - 1)
    uint64_t out_word;          // word offset of column 0 in the output region
    uint64_t col_words;         // words per column (a multiple of 64)
    uint64_t chunk_off;         // first materialisation work item
    uint64_t max_pairs;         // largest key product (zero before the launch)
    uint32_t seg_major;         // work items are groups of 64 keys, not row chunks
    // Semi-join reduction: a blocked Bloom filter (fmask + 1 words, a power
    // of two) of the keys of one side; records of the other side (RIGHT when
    // probe_right, else LEFT) whose key it does not hold are dropped before
    // the sort.  filt = nullptr: every record is kept.
    uint64_t* filt;
    uint32_t fmask;
    uint32_t probe_right;
    uint32_t nrec;              // records sorted: nl + nr, or (filtered) the kept count, written on the device
};

struct BatchHdr {
    BatchJoin* joins;
    const uint32_t* tile_join;  // record tile -> join
    uint32_t njoins;
    uint32_t total_tiles;
    uint32_t passes;
    uint32_t epoch0;            // kernels use epoch0 .. epoch0 + passes + 1
    uint32_t* keys[2];
    uint32_t* vals[2];
    uint64_t* seg_off;
    uint32_t* hist;             // [njoins][passes][2^rb]
    uint32_t* ctr;              // tile counters: passes + 4 words, zero before the launch
    uint64_t* status;
    int32_t* out_base;          // output region
    uint64_t out_cap_words;
    uint64_t out_used_words;    // result
    uint64_t total_chunks;      // result
    // value columns in sorted record order (record slots as keys/vals), used
    // by joins with at least as many output rows as records; nsval = 0: none
    int32_t* sval[BATCH_MAXNC - 1];
    uint32_t nsval;
    uint64_t* filt;             // every join's filter words (cleared by the launch)
    uint64_t filt_words;
};

// The whole batch in kernel launches (a graph capture records them).
hipError_t launch_batch(const BatchHdr* hdr_dev, int rb, int kpt, int passes, hipStream_t stream);
// Rows per materialisation chunk of the batched kernels.
uint32_t batch_chunk_rows();

// ---- dictionary encoding of terms (k_dict.hip) ------------------------------
// The dictionary on the device: a hash table of 64-bit slots (mask + 1 of
// them, a power of two; ~0 = empty), and the terms in identifier order as
// bytes with nterms + 1 offsets.
struct DictDev {
    uint64_t* table;
    uint64_t mask;
    int64_t* off;
    uint8_t* bytes;
    uint32_t nterms;
};
// A batch of n terms: bytes[off[i] .. off[i + 1]) is term i.
struct TermsDev {
    const uint8_t* bytes;
    const int64_t* off;
    uint32_t n;
};
// Per-batch device scratch: u32 arrays of n (rep, first; rank of each first
// occurrence of a new term, and its batch index by rank), scalars and the
// scan partials (scan_part_bytes(n)).  first must hold ~0 before the launch
// and err 0.
struct DictScratch {
    uint32_t *rep, *first, *rank, *index;
    uint32_t* new_terms;
    uint64_t* new_bytes;
    void* part;
    uint32_t* err;
};
constexpr uint32_t DICT_SCAN_MAX = 1u << 26;  // terms per batch
size_t scan_part_bytes(uint32_t n);
// err |= 1 unless off[0] == 0 and off is non-decreasing over n + 1 entries;
// *total = off[n]
hipError_t launch_dict_check_offsets(const int64_t* off, uint32_t n, uint32_t* err, int64_t* total, hipStream_t s);
// hash and insert (insert = 0: look up only), then count the new terms:
// *new_terms, *new_bytes and the scan partials
hipError_t launch_dict_encode_front(const DictDev& d, const TermsDev& t, int insert, DictScratch w, hipStream_t s);
// number the new terms (identifiers from base) and append them to the byte
// store from bbase on: rank, index, their offsets and bytes (after
// launch_dict_encode_front, with the totals it counted)
hipError_t launch_dict_append(const DictDev& d, const TermsDev& t, DictScratch w, uint32_t base, int64_t bbase,
                              uint32_t new_terms, int64_t new_bytes, hipStream_t s);
// ids[i]: the identifier of term i (new terms: base + rank; absent: -1)
hipError_t launch_dict_ids(const TermsDev& t, DictScratch w, uint32_t base, int32_t* ids, hipStream_t s);
// the slots the batch claimed: commit = 1 re-points them to identifiers,
// commit = 0 empties them, restoring the table
hipError_t launch_dict_fix(const DictDev& d, DictScratch w, uint32_t base, int commit, hipStream_t s);
// decoding: *total bytes of n identifiers and the scan partials (err |= 1
// for one outside the dictionary; *count is scratch); then their offsets
// pos[0 .. n] and bytes
hipError_t launch_dict_decode_size(const DictDev& d, const int32_t* ids, uint32_t n, uint32_t* count, uint64_t* total,
                                   void* part, uint32_t* err, hipStream_t s);
hipError_t launch_dict_decode(const DictDev& d, const int32_t* ids, uint32_t n, int64_t total, void* part,
                              int64_t* pos, uint8_t* out, hipStream_t s);

// ---- loading and indexing a store (k_index.hip) ---------------------------
// Bounds of s and o together and of p, and the IDs outside [0, 2^31 - 1).
struct IngestOut {
    int32_t so_min, so_max, p_min, p_max;
    uint32_t bad, pad;
};
// *out over n triples; unless ds == s the columns are copied to ds, dp, dq.
hipError_t launch_ingest(const int32_t* s, const int32_t* p, const int32_t* o, int32_t* ds, int32_t* dp, int32_t* dq,
                         uint64_t n, IngestOut* out, hipStream_t stream);
// w1 << 32 | w0 = (p - pmin) << 2 so | s << so | o (the caller makes sure it
// fits 64 bits; so in [0, 31]).
hipError_t launch_pack_triples(const int32_t* s, const int32_t* p, const int32_t* o, uint64_t n, int32_t pmin, int so,
                               uint32_t* w0, uint32_t* w1, hipStream_t stream);
// Sorted words back to columns; r0, r1 get the words with first and second
// exchanged, and (p - pmin, position) of every predicate's first row is appended to
// pred/pred_pos at atomicAdd(npred) (entries past cap are only counted).
hipError_t launch_unpack_pso(const uint32_t* w0, const uint32_t* w1, uint64_t n, int so, int32_t* first, int32_t* second,
                             uint32_t* r0, uint32_t* r1, int32_t* pred, int64_t* pred_pos,
                             uint32_t* npred, uint32_t cap, hipStream_t stream);
hipError_t launch_unpack_pos(const uint32_t* w0, const uint32_t* w1, uint64_t n, int so, int32_t* first,
                             int32_t* second, hipStream_t stream);
// Runs of equal values per predicate (rows [off[q], off[q + 1]), np + 1
// offsets) added to cnt[q] (pso_s) and cnt[np + q] (pos_o).
hipError_t launch_distinct(const int32_t* pso_s, const int32_t* pos_o, int64_t n, const int64_t* off, uint32_t np,
                           unsigned long long* cnt, hipStream_t stream);

// ---- utilities (k_util.hip) -----------------------------------------------
// Between the two passes of a two-pass scan: the run totals tot[0..nruns)
// (nruns <= 1024) become their exclusive prefix sums, in place, capped at
// 2^40 - 1; the sum goes to *total64 and/or *total32 (either may be null)
// mail (may be null): the sum, or, when run_max is given, *nseg, a pad word,
// the sum and the largest of run_max[0..nruns).
hipError_t launch_scan_runs(uint64_t* tot, uint32_t nruns, uint64_t* total64, uint32_t* total32,
                            const uint64_t* run_max, const uint32_t* nseg, const Mail* mail, hipStream_t stream);
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t stream);
hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t stream);
// out[i] = src[idx[i]] - base
hipError_t launch_gather(const int32_t* src, const uint32_t* idx, int32_t* out, uint64_t n, int32_t base,
                         hipStream_t stream);
// Composite keys of up to MAX_KEY_WORDS variables.  Packed: out[i] = OR
// over j of (col[j][i] - base[j]) << shift[j] as u32 (the caller makes sure
// the relative ranges fit side by side; shifts in [0, 31]).
constexpr int MAX_KEY_WORDS = 3;
struct PackArgs {
    const int32_t* col[MAX_KEY_WORDS];
    int32_t base[MAX_KEY_WORDS];
    int32_t shift[MAX_KEY_WORDS];
    int32_t ncols;
};
hipError_t launch_pack_keys(const PackArgs& a, uint64_t n, uint32_t* out, hipStream_t stream);
// Not packed: brk[i] = 1 when sorted record ids[i] differs from ids[i - 1]
// in any of the nw further key words (record r < n_left reads lcol[j][r],
// else rcol[j][r - n_left]); brk[0] = 0.
struct BreakArgs {
    const int32_t* lcol[MAX_KEY_WORDS];
    const int32_t* rcol[MAX_KEY_WORDS];
    uint32_t n_left;
    int32_t nw;
};
hipError_t launch_key_breaks(const BreakArgs& a, const uint32_t* ids, uint32_t n, uint8_t* brk, hipStream_t stream);
// out[i] = cell of record ids[i] minus base, the record being LEFT row
// ids[i] of lcol (ids[i] < n_left) or RIGHT row ids[i] - n_left of rcol.
hipError_t launch_side_gather(const int32_t* lcol, const int32_t* rcol, uint32_t n_left, const uint32_t* ids,
                              uint32_t n, int32_t base, uint32_t* out, hipStream_t stream);
// Min and max of the int32 values of two segments (at least one value) to the
// mail's first two words.  acc: three words, 0 before and after the launch.
hipError_t launch_minmax(const int32_t* a, uint64_t na, const int32_t* b, uint64_t nb, uint32_t* acc, Mail mail,
                         hipStream_t stream);
// Run boundaries of a sorted column: for every i with v[i] != v[i-1] (or
// i == 0) appends (v[i], i) to out_val/out_pos at atomicAdd(count).
hipError_t launch_run_bounds(const int32_t* v, uint64_t n, int32_t* out_val, int64_t* out_pos, uint32_t* count,
                             uint32_t cap, hipStream_t stream);
// Duplicate flags of the (p,s,o)-sorted store: keep[perm[i]] = 1 if triple
// i differs from triple i-1 (or i == 0), else 0.
hipError_t launch_dup_flags(const int32_t* p, const int32_t* s, const int32_t* o, const uint32_t* perm,
                            uint64_t n, int32_t* keep, hipStream_t stream);

}  // namespace mq
