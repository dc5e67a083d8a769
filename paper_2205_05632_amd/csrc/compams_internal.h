// Internal declarations shared by the kernel files and the C-ABI host code of libcompams.
// Nothing here is part of the public interface (include/compams.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "compams_tasks.h"

namespace compams {

// ---------------------------------------------------------------------------------------------
// Geometry shared by all kernels.
//
// A row (one worker's d coordinates) is cut into chunks of kChunk consecutive coordinates, a chunk into
// kRounds rounds of 256 coordinates; in a round lane l of a wavefront holds the four coordinates
// base + 256*round + 4*l + {0,1,2,3}, so that a wave's 128-bit accesses cover 1 KiB of contiguous memory and
// (round, lane, slot) order is ascending coordinate order.  The dense passes give a chunk to a workgroup
// (a quarter of its rounds to each wavefront), the sweeps over stored rows and lists a chunk to a wavefront.
// ---------------------------------------------------------------------------------------------
constexpr int kWG = 256;                 // threads per workgroup = 4 wavefronts
constexpr int kWaves = kWG / 64;
constexpr int kChunk = 4096;             // coordinates per chunk
constexpr int kRounds = kChunk / 256;    // rounds per chunk

// Which part of memory a die works on.  Consecutive workgroups run on the eight dies (XCDs) in turn, and the memory
// channels follow each other through every span of eight 4 KB pages.  Where the workgroups of a die always take the same
// page of a span, each channel is asked by one die only: a first pass's traffic (two arrays read, one written, 2.1 GB)
// streams at 6.75 TB/s so, at 6.2 with a workgroup per 16 KB in address order, at 6.05 with pages that change from group
// to group (pages of 1 and 2 KB do as well, 512 B 6.6, 256 B 5.9).  A page is a quarter of a chunk: one wavefront's part
// of the dense passes.
constexpr uint32_t kPageCoords = 1024;
constexpr uint32_t kDies = 8;
constexpr uint32_t kSpanCoords = kDies * kPageCoords;  // two chunks
constexpr uint32_t kSpansPerGroup = kWaves;            // spans that eight consecutive workgroups share, a wavefront each

// The quarter of a chunk that a wavefront of a dense pass takes, the workgroup being number `group` of the row's
// page_groups(): page (`group` + `turn`) % 8 of one of the four spans.
struct Quarter {
  uint32_t chunk, part;
};
__device__ __forceinline__ Quarter page_quarter(uint32_t group, uint32_t wave, uint32_t turn = 0) {
  const uint32_t page = (group + turn) % kDies, span = group / kDies * kSpansPerGroup + wave;
  return {span * (kSpanCoords / kChunk) + page / kWaves, page % kWaves};
}
// A dense pass asks for this much LDS that it has no use for: four or five workgroups per compute unit are enough to keep
// the memory busy, and with eight the channels change between more pages (the traffic above: 330 us with eight, 318 with
// five, 317 with four, 373 with three).  Block-sign's first pass does so in chunk order as well (a step, with / without:
// 8 x 12 M 269.5 / 271.9 us, 4 x 12 M 174.1 / 175.5; the same below 3 M).
constexpr size_t kStreamLds = 32768;
inline uint32_t page_groups(uint32_t num_chunks) { return (num_chunks + kDies - 1) / kDies * kDies; }
static_assert(kPageCoords * kWaves == kChunk, "a page is a wavefront's quarter of a chunk");
static_assert(kSpansPerGroup * kSpanCoords == kDies * kChunk, "eight workgroups take eight chunks");

// Radix levels over the 31-bit magnitude key (fp32 bit pattern without the sign):
// level 0 = bits 30..19 (the exponent and 4 mantissa bits), level 1 = bits 18..9, level 2 = bits 8..0.
constexpr int kL0Shift = 19;
constexpr int kNB0 = 1 << 12;
constexpr int kL1Shift = 9;
constexpr int kNB1 = 1 << 10;
constexpr int kNB2 = 1 << 9;
// The level-0 kernel keeps level-1 histograms of this many buckets, starting at the guessed one: the guess is one
// below the last threshold bucket, so a threshold that moved by one bucket either way still resolves there.
constexpr uint32_t kTracked = 3;
// Top-k inside every block: a block of at most this many coordinates (a bias, a norm weight) is one wavefront's
// work from reading g to writing its part of the list; it takes no part in histograms, sweeps or counting.
constexpr uint32_t kMicroCoords = 1024;
constexpr uint32_t kMicroFlag = 0x80000000u;  // WgSlot.seg of a first-pass workgroup that takes micro problems

// The band and the counting kernel split a row's chunks into at most kMaxCountBlocks contiguous blocks of count_cpw
// chunks (four wavefronts, eight chunks at a time: a multiple of 32).  d < 2^31 gives at most 2^19 chunks.  Rows of up
// to 1024 chunks have blocks of 8, two chunks to a wavefront, while there are fewer than kShortChunks chunks in all rows:
// blocks of 32 leave most of the chip idle then (4 rows of 300007: the counting kernel 18.1 -> 10.1 us; 16 rows of 1 M:
// the band kernel 14.6 -> 12.6 us).  In larger grids the row's histogram, which every block of the band kernel reads,
// outweighs that; where rows miss their window and have to be counted, the shorter blocks still gain.  Measured (us,
// blocks of 32 / of 8; band kernel, counting kernel of rows that miss): 16 x 640 chunks 15.6 / 15.6, 13.5 / 8.9; 64 x 245
// 15.2 / 17.7, 20.0 / 10.8; 64 x 512 17.4 / 26.9, 26.1 / 15.9; 64 x 1024 23.9 / 42.8, 22.3 / 16.1; long rows, 4 x 2048:
// 16.1 / 18.4, 14.8 / 9.2.
constexpr uint32_t kMaxCountBlocks = 256;
constexpr uint32_t kMaxCountCpw = 2048;
constexpr uint32_t kShortChunks = 32768;
inline uint32_t count_chunks_per_block(uint32_t num_chunks) {
  const uint32_t m = (num_chunks + 32 * kMaxCountBlocks - 1) / (32 * kMaxCountBlocks);
  return 32 * (m ? m : 1);
}
inline uint32_t count_chunks_per_row_block(uint32_t n, uint32_t num_chunks) {
  const bool few = static_cast<uint64_t>(n) * num_chunks < kShortChunks;
  return num_chunks <= 4 * kMaxCountBlocks && few ? 8 : count_chunks_per_block(num_chunks);
}
// Chunks that a wavefront takes at a time of a block of cpw: two or eight.
__host__ __device__ __forceinline__ uint32_t chunks_per_wave(uint32_t cpw) { return cpw < 32 ? cpw / 4 : 8; }

// The candidate list of a selection problem is kept as kSubLists runs, which the workgroups of its first pass append to in
// turn (in pages in another turn from one eight of them to the next), each run with a cursor in a 128-byte line of its own.
// Atomics to one address are performed one after the other (about 3 ns apart on MI355X); a chunk's allocation every 8 ns
// through a single cursor queued long enough to cost the first pass 9 of 352 us, and cursors that share a line were little
// better.
constexpr uint32_t kSubLists = 8;
constexpr uint32_t kCursorPitch = 32;  // words between the cursors of a problem
// A problem (row or block) of fewer chunks than this keeps its list as one run: its allocations are few, and
// with a handful of chunks the runs would be of very different lengths and an eighth of the capacity each
// would overflow for nothing.
constexpr uint32_t kSubListMinChunks = 64;
constexpr uint32_t kNoCursorSet = 0xffffffffu;
// So many chunks in all rows (one selection per row, rows of several runs) have their first pass in pages, with a segment of
// the lists for every quarter of a chunk.  First pass (us; k = d / 100, chunks in order / pages): 8 x 2730 chunks 170 /
// 172; 2 x 6240 99.7 / 99.7; 16 x 2730 339 / 339; 8 x 6240 406 / 385; 16 x 6240 818 / 755; k = d / 1000, 8 x 3907 245 /
// 237, 8 x 30381 1977 / 1837. The whole step, three contexts in turn: 64 x 733 465 / 467, 64 x 977 619 / 615, 32 x 1465
// 477 / 478, 24 x 1954 484 / 476, 16 x 2930 494 / 490, 3 x 17090 823 / 815.
constexpr uint32_t kPagedChunks = 45056;
static_assert(kPagedChunks >= kShortChunks, "rows in pages have blocks of 32 chunks and more: eight chunks to a wavefront");
// Block-sign, which keeps no lists, from so many on (first pass, chunks in order / pages): 16 x 733 chunks 96.7 / 99.2; 8
// x 2730 169 / 172; 2 x 12208 186.5 / 184; 8 x 3907 247 / 239; 8 x 5128 314 / 313; 16 x 2730 332 / 333; 64 x 733 368 /
// 355; 8 x 7325 466 / 443; 8 x 30381 1948 / 1844.
constexpr uint32_t kBsPagedChunks = 24576;
inline bool paged_first_pass(uint64_t n, uint32_t num_chunks) {
  return num_chunks >= kSubListMinChunks && n * num_chunks >= kPagedChunks;
}

constexpr uint32_t kCountersPerRow = 8;  // == COMPAMS_COUNTERS_PER_ROW of the public header

constexpr int kWireTile = 256;  // coordinate gaps per tile of a top-k message (one width per tile)

// Where a row's selection reads its elements from after level 0.
enum : uint32_t {
  kModeCand = 0,   // candidate list written by the first pass (threshold bucket was predicted)
  kModeNeedB = 1,  // candidate list written by a second dense pass that knows the exact level-0 bucket
  kModeDense = 2   // no candidate list (it would not fit): every later pass reads the whole row
};

// The band: a window of magnitude keys [band_lo, band_hi) in which the next step's threshold key is expected,
// set from the last two thresholds, cut into 2048 or 8192 buckets of equal width (band_bucket below).  The first pass
// counts, per chunk, the entries at or above band_hi, copies the entries inside the window to a short list of their own (a
// segment per chunk) and adds them to the row's bucket histogram.  If the threshold does fall inside (checked
// exactly), one launch finishes the selection from the short list alone (k_topk_band).
// A window holds up to about k entries, and a bucket may hold kBoundaryCap at most: 70 000 to 240 000 entries (k =
// 110 000 to 260 000, hundreds of steps into a run) fill 2048 buckets with 35 to 120 each, and one row in five went
// to the general kernels for that alone.  A window expected to hold no more than 16 entries to each of 2048 buckets
// keeps those: every workgroup of the band kernel reads the histogram (16 x 11.2 M coordinates, k = 111 816, windows of
// 14 000 entries: 15.7 us with 2048 buckets, 21.2 with 8192).
constexpr uint32_t kBandBucketsFew = 2048, kBandBucketsMany = 8192;
enum : uint32_t { kBandFew = 1, kBandMany = 2 };  // TopkRow::band_valid
// Room for so many is kept per problem.
__host__ __device__ __forceinline__ uint32_t band_buckets(uint32_t k) { return k < 16384 ? kBandBucketsFew : kBandBucketsMany; }
constexpr uint32_t kBandMaxEntries = 1u << 20;  // capacity of a band list at most
constexpr uint32_t kBoundaryCap = 64;      // entries in the bucket that holds the threshold key; more: general route
constexpr uint32_t kCursorAboveWord = 2;   // word of a run's cursor line that counts the run's entries above the band

// Which kernel found this step's threshold key.
enum : uint32_t {
  kFastNot = 0,   // the general ones
  kFastBand = 1,  // k_topk_band
  kFastPick = 2   // k_topk_pick: chunk records hold prefixes over the whole row, there are no further tables
};

// What is still to be set for the next step's first pass.
enum : uint32_t {
  kNextSet = 0,    // nothing: there is a guess and a window, or none
  kNextNone = 1,   // that there is no guess
  kNextGuess = 2   // guess and window
};

// Words of TopkWorkspace::flags: the queues of k_topk_general lie a cache line apart from one another and from what
// everybody reads.
constexpr uint32_t kQueuePitch = 32;
__host__ __device__ __forceinline__ uint32_t queue_word(uint32_t queue) { return (1 + queue) * kQueuePitch; }
constexpr size_t kFlagBytes = (1 + kQueues) * kQueuePitch * 4;
constexpr uint32_t kMissGaveUp = 7;  // COMPAMS_CNT_BAND_MISS of a problem that k_topk_general has given up waiting for

// Per-row control block of the top-k selection (device memory, written by single workgroups).
struct TopkRow {
  uint32_t cand_from;   // 0, or one more than the first key that the next first pass lists as a candidate
  uint32_t b_guess;     // a level-0 bucket at or below that key's
  uint32_t cursor;      // candidate entries allocated so far in this step (a list kept as one run) ...
  uint32_t cursor_band; // ... and band entries: the two are advanced together as one 64-bit word
  uint32_t band_valid;  // kBandFew / kBandMany: the next first pass may also fill the band list and the bucket histogram
  uint32_t band_lo, band_hi;  // keys; band_lo >= b_guess << kL0Shift, band_hi > band_lo
  uint32_t band_mul;    // bucket of a key inside the band: see band_bucket()
  // (read together by the last kernel, up to tie_last)
  uint32_t fast;        // kFast*, not 0: the threshold is known, the general kernels skip the problem
  uint32_t mode;        // kMode*
  uint32_t tau;         // the k-th largest key
  uint32_t r;           // how many keys equal to tau are selected
  uint32_t ties;        // how many keys equal tau
  uint32_t tie_last;    // fast: ties are taken up to and including this coordinate (of the problem)
  uint32_t n_src;       // entries in the candidate list (kModeCand / kModeNeedB)
  uint32_t bstar;       // level-0 bucket that holds the k-th largest key
  uint32_t need;        // keys still to be taken inside the current prefix
  uint32_t prefix1;     // bits 30..9 of the k-th largest key (after level 1)
  uint32_t level1_done;    // bits 30..9 of the threshold key are known (prefix1 / need are valid)
  uint32_t ticket[4];      // "last workgroup of the row" counters of kernels 1..4; zero between launches
  uint32_t n_lists;        // runs of the candidate list: kSubLists (run s from entry s * (capacity / kSubLists) on), or 1
  uint32_t n_sub[kSubLists];  // entries of each run (n_src in all)
  uint32_t tau_prev;       // the threshold key of the step before (0: none)
  uint32_t above;          // entries at or above band_hi (a list kept as one run; else in the runs' cursor lines)
  uint32_t bnd_n;          // entries of the threshold's bucket gathered so far (k_topk_band); zero between launches
  uint32_t ticket_band;    // "last workgroup" counter of k_topk_band; zero between launches
  float noise;             // not taken by k_topk_band: what its window's population says of the threshold's scatter (0:
                           // there was no window)
  uint32_t known_from;     // see set_next_band()
  uint32_t next;           // kNext*: what the last kernel is to make of the next step's window (selected in one launch), from ...
  uint32_t next_prev2;     // ... the threshold key two steps before, and the window's population and a key in it
  uint32_t next_population, next_ref;
  uint32_t phase;          // kPhase*: how far k_topk_general is with a problem left to it
  uint32_t pad[21];
};
static_assert(sizeof(TopkRow) == 256, "TopkRow layout");

// Entries from one problem's candidate list to the next one's: whole cache lines, where the general route may be one
// launch (blocks; rows of more chunks than k_topk_pick takes).
constexpr uint32_t kPickChunks = 16;
__host__ __device__ __forceinline__ uint64_t cand_pitch(uint32_t cap) { return (static_cast<uint64_t>(cap) + 15) / 16 * 16; }
__host__ __device__ __forceinline__ uint64_t row_cand_pitch(uint32_t cap, uint32_t num_chunks) {
  return num_chunks > kPickChunks ? cand_pitch(cap) : cap;
}

// Bucket of a key inside a band of `span` keys starting at lo: floor(rel * buckets / span) for rel = key - lo,
// computed as the high word of rel * mul with mul = floor(2^32 * buckets / span); a band of at most `buckets`
// keys (mul = 0) has a bucket per key.  Non-decreasing in the key and always below `buckets`.
__device__ __forceinline__ uint32_t band_multiplier_dev(uint32_t span, uint32_t buckets) {
  return span > buckets ? static_cast<uint32_t>((static_cast<uint64_t>(buckets) << 32) / span) : 0u;
}
__device__ __forceinline__ uint32_t band_bucket(uint32_t rel, uint32_t mul) { return mul ? __umulhi(rel, mul) : rel; }
// Where its count lies: of the many buckets a thread of the band kernel takes 32 consecutive ones, kept in four
// groups of 8 with a quarter of the table between them, so that its first 8 are found before it is known how many
// there are.  The few lie in one quarter, which differs from problem to problem: always the first, 32 KB apart, they
// would meet on a quarter of the memory channels (first pass of the ResNet-18 shape 350.6 us, in different quarters 339.2).
__device__ __forceinline__ uint32_t band_rotation(uint32_t k, uint32_t problem) {
  return band_buckets(k) == kBandBucketsMany ? problem & 3u : 0u;
}
__device__ __forceinline__ uint32_t band_slot(uint32_t bucket, bool many, uint32_t rotation) {
  return many ? ((((bucket >> 3) + rotation) & 3u) << 11) | ((bucket >> 5) << 3) | (bucket & 7u)
              : rotation * kBandBucketsFew + bucket;
}
static_assert(kBandBucketsFew == 256 * 8 && kBandBucketsMany == 4 * kBandBucketsFew, "slots above");

// One selection problem: a worker's whole row (top-k over the flattened gradient) or one block of a worker's
// row (top-k inside every block).  Index fields count entries of the respective workspace tables.
struct Seg {
  int64_t elem_off;      // first element, relative to the start of g and of e
  uint64_t chunk_base;   // first entry in the per-chunk tables (segment descriptors, count records)
  uint64_t seloff_base;  // first entry in sel_off (a segment has one entry more than it has quarters of chunks)
  uint64_t cand_base;    // first entry of the segment's candidate list
  uint64_t list_base;    // first entry of the segment's slice of the worker's (coordinate, value) list
  uint64_t band_base;    // first entry of the segment's band list
  uint64_t bhist_base;   // first bucket of the segment's band histogram
  uint32_t d, k;         // length, and how many coordinates are kept
  uint32_t num_chunks;
  uint32_t cap;          // capacity of the candidate list
  uint32_t band_cap;     // capacity of the band list
  uint32_t coord_base;   // coordinate of the first element within the worker's row
  uint32_t count_cpw;    // chunks per block of the counting kernel
  uint32_t groups_first, groups_sweep, count_blocks;  // workgroups the kernel classes give this segment (first pass:
                                                      // one per chunk)
  uint32_t micro;        // at most kMicroCoords coordinates: one wavefront of the first pass does the whole selection
  uint32_t groups_level0;
  uint32_t cursor_set;   // which set of kSubLists cursors the problem's list uses, or kNoCursorSet: one run, rowp->cursor
};
static_assert(sizeof(Seg) % 8 == 0, "Seg layout");

// Which segment, and which of its workgroups, a workgroup of a flat launch is.
struct WgSlot {
  uint32_t seg, group;
};

enum : uint32_t {
  kBandOff = 0,
  kBandLists = 1,   // the first pass lists and counts what the window holds (k_topk_band)
  kBandWindow = 2   // it only leaves out of the candidate list what lies below the window (k_topk_pick)
};

struct TopkOptions {
  uint32_t cap;            // candidate entries per row
  uint32_t predict;        // 1: carry the threshold bucket over to the next step's first pass
  uint32_t force_dense;    // 1: never build a candidate list (test / ablation)
  uint32_t band;           // kBand*: also carry a window for the threshold key itself over
  uint32_t band_cap;       // band entries per row
};

struct TopkWorkspace {
  TopkRow* rows;        // n
  uint32_t* counters;   // n * COMPAMS_COUNTERS_PER_ROW
  uint32_t* hist0;      // n * kNB0
  uint32_t* hist1;      // n * kNB1
  uint32_t* hist1x;     // n * kTracked * kNB1 : level-1 histograms of the tracked buckets
  uint32_t* hist2;      // n * kNB2
  uint32_t* xcur;       // sets of kSubLists cursors, kCursorPitch words apart: one set per row, or per segment of at
                        // least kSubListMinChunks chunks
  uint4* chunk_rec;     // n * num_chunks : keys above tau, keys equal to tau, and the exclusive prefixes of both
                        //                  within the chunk's count block
  uint2* blk;           // n * kMaxCountBlocks : the two totals of every count block
  uint2* blk_prefix;    // n * kMaxCountBlocks : for a problem selected by k_topk_band, the totals of the blocks
                        // before each block (the sums the last kernel would otherwise form per chunk), and how many
                        // of the kept entries of the threshold's bucket lie before each block
  uint32_t* sel_off;    // n * (4 num_chunks + 1) : where the slice of the worker's list starts that belongs to each
                        //                          quarter of a chunk
  uint32_t* count_gt;   // n : selected entries whose key lies strictly above the threshold key
  uint32_t* wire_total;    // n : words of the gap stream of the message being packed or unpacked
  uint32_t* wire_tile_off; // n * ceil(k / kWireTile) : where each tile of gaps starts in its stream
  uint32_t* wire_tile_sum; // n * ceil(k / kWireTile) : coordinates before each tile, while unpacking
  uint2* desc;          // n * num_chunks * desc_parts : (offset, count) of the segment in the candidate list
  uint2* desc2;         // n * num_chunks * desc_parts : offset of the segment in the band list; entries at or above the
                        //                               band | entries in the band << 13
  uint2* band;          // n * band_cap   : (coordinate, fp32 bits) of the entries inside the band
  uint32_t* bhist;      // band_buckets(k) per problem : how many band entries fall into each bucket; zero between steps
  uint2* bnd;           // n * kBoundaryCap : the entries of the bucket that holds the threshold key
  uint32_t* bnd_sel;    // n * kBoundaryCap : coordinates of the kept ones among them, ascending
  uint32_t* flags;      // [queue_word(q)]: shares drawn by k_topk_general.  [0]: some problem of this step was left to the
                        //      general kernels (set by k_topk_band, cleared by the step's last kernel): they return at once
                        //      otherwise
  uint2* cand;          // n * cap_alloc  : (coordinate, fp32 bits)
  int32_t* idx;         // n * k
  float* val;           // n * k
  uint32_t* tau;        // n
  // top-k inside every block only: the segments and, per kernel class, the workgroups of a flat launch
  const Seg* segs;
  const WgSlot* map_first;   // first pass: .group = chunk of the segment (or a workgroup of micro problems, see below)
  const WgSlot* map_level0;
  const WgSlot* map_sweep;
  const WgSlot* map_count;
  const uint32_t* micro_list;  // segments that are micro problems; a first-pass workgroup with kMicroFlag takes
                               // .group (<= 4) of them, from entry (.seg without the flag) on, one per wavefront
  const WgSlot* map_final;  // .seg = block (worker 0's segment of it), .group = chunk of the block
  uint32_t* sel_off_srv;    // n * (4 * chunks of a whole row + 1) : list offsets per quarter of a chunk, for the
                            //                                   server's lines run from lists
  uint32_t page_turn;   // first pass in pages: row i starts its dies' pages (i * page_turn) >> 16 further on
  uint32_t desc_parts;  // segments of a chunk: one, or (rows whose first pass goes in pages) one for every quarter
};

struct BlocksignWorkspace {
  uint32_t* offsets;    // M + 1 block offsets
  uint32_t* chunk_block; // num_chunks : index of the block that holds the chunk's first coordinate
  uint64_t* acc;        // n * M * acc_replicas * kLimbs : exact sums of |x| (32-bit digits carried in 64-bit words);
                        // the sum of a (row, block) is the sum of its replicas
  uint32_t acc_replicas;
  uint32_t* special;    // n * M : bit 0 = an infinity was seen, bit 1 = a NaN was seen
  uint32_t paged;       // the first pass takes the rows in pages (kBsPagedChunks)
  uint32_t* ticket;     // n : "last workgroup of the row" counters of the first pass; zero between launches
  float* scales;        // n * M
  uint32_t* bits;       // n * words
  uint32_t chunk_blocks;  // where every block lies inside one chunk: the most that a chunk has, else 0
};
constexpr int kLimbs = 10;  // 10 digits of 32 bits cover 2^-149 .. 2^171

struct AmsParams {
  float beta1, beta2, one_minus_beta1, one_minus_beta2, eps, lr, nf;
  int eps_out;  // 1: epsilon outside the square root
  int cached_arrays;  // how many of theta, m, v, vhat (in that order) are left in the memory-side cache for the next step, the
                      // others streamed past it (see step_cached_arrays)
};

// How many of the four state arrays the memory-side cache (256 MB) holds together, with room for what else passes through.
constexpr int64_t kCacheBudget = int64_t(212) << 20;
inline int cached_state_arrays(int64_t d) {
  const int64_t fit = kCacheBudget / (d * 4);
  return fit > 4 ? 4 : static_cast<int>(fit);
}

// How many a step keeps there.  The identity compressor, which reads the gradients in the same pass, writes through what
// fits (16 x 11.2 M, three contexts in turn / one context's steps one after the other: 172 / 167 us, streamed 173 / 175).
// Top-k and block-sign read and write all four with ordinary accesses or all with streaming ones.  Ordinary accesses are
// the faster ones where one context's steps follow each other with nothing in between, at every size that fits the cache
// at all (us, ordinary / streaming: top-k 8 x 8 M 189 / 199, 16 x 11.2 M 432 / 450; block-sign 8 x 8 M 165 / 173, 1 x 12
// M 87 / 98).  Where something else comes in between, as in a training program, they are so only while the state is
// small: the lines of a larger one are gone when the next step asks for them, and are written out in the way of what
// follows.  Three contexts in turn, ordinary / streaming, k = d / 100 (the line lies at (n + 32) d = 231 M, 7 M
// coordinates of one worker, 4.8 M of sixteen):
//   top-k       1 x 6 M 73.1 / 75.2, 1 x 8 M 96.7 / 93.8; 4 x 6 M 110.5 / 111.8, 4 x 7 M 130.7 / 125.4; 8 x 5.5 M 153.4 / 155.0,
//               8 x 7 M 192 / 186; 16 x 4.5 M 206 / 205, 16 x 5.5 M 255 / 251; 64 x 2 M 363 / 366, 64 x 3.5 M 575 / 568
//   block-sign  1 x 6.5 M 57.1 / 58.3, 1 x 8 M 71.7 / 67.6; 8 x 6 M 129.8 / 131.7, 8 x 7 M 155.2 / 153.3; 16 x 4.5 M 171.6 / 172.9,
//               16 x 5.5 M 207.1 / 206.7, 16 x 8 M 305 / 296; 64 x 2.5 M 343 / 342
//   per layer   2 x 6 M 93.9 / 98.5, 8 x 5.5 M 165.6 / 167.1, 16 x 5 M 244 / 240
// With 512 MB of other traffic before every step, which is not counted, neither is ahead by more than 5 % from 6 M on (16
// x 11 M: block-sign 412 / 404, top-k 475 / 474; 8 x 8 M: 178.9 / 177.9, 222 / 218).
constexpr int64_t kOrdinaryState = 231000000;
inline int step_cached_arrays(int64_t n, int64_t d, bool identity) {
  return identity ? cached_state_arrays(d) : (n + 32) * d <= kOrdinaryState ? 4 : 0;
}

// Moment and parameter lines of Algorithm 2 for one coordinate: every product, sum, square root and
// quotient is a separately rounded fp32 operation (the library is built without contraction).
__device__ __forceinline__ void ams_update(float gb, float& th, float& mm, float& vv, float& vh, const AmsParams& p) {
  const float mj = p.beta1 * mm + p.one_minus_beta1 * gb;
  const float vj = p.beta2 * vv + p.one_minus_beta2 * (gb * gb);
  const float vhj = (vh < vj) ? vj : vh;
  const float den = p.eps_out ? sqrtf(vhj) + p.eps : sqrtf(vhj + p.eps);
  mm = mj;
  vv = vj;
  vh = vhj;
  th = th - p.lr * (mj / den);
}

struct Geometry {
  uint32_t n;
  uint32_t d;
  int64_t ld;
  uint32_t num_chunks;
  uint32_t k;
  uint32_t num_blocks;
  uint32_t words;  // ceil(d / 32)
  uint32_t count_cpw;  // top-k: chunks per block of the counting kernel
};

// Kernel slots for optional timing.
enum KernelSlot {
  kSlotPassA = 0, kSlotBand, kSlotPick, kSlotGeneral, kSlotLevel0, kSlotLevel1, kSlotLevel2, kSlotCount,
  kSlotTopkFinal,
  kSlotBsPass1, kSlotBsFinal, kSlotBsPass2, kSlotBsAms,
  kSlotNoneAms, kSlotWireEncode, kSlotWireDecode, kNumSlots
};

struct Launcher;  // host-side helper that brackets launches with events (compams_api.hip)

// Host-side launch entry points, one per compressor (defined next to their kernels).
// whole: a step that stands for itself (fresh control blocks, no guess, nothing pending): the residual's zeros are
// written at once.
// It clears the tables from the control blocks up to the chunk records itself where rows have kSample coordinates or more.
constexpr uint32_t kSample = 4096;
hipError_t topk_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt, const AmsParams& ap,
                     const float* g, float* e, float* theta, float* m, float* v, float* vhat,
                     bool first_pass_may_predict, bool clear_pending, bool workers_only, bool whole, hipStream_t stream,
                     Launcher* L);
// Sizes of the flat launches of top-k inside every block.
struct TopkFlat {
  uint32_t wg_first, wg_level0, wg_sweep, wg_count, wg_final;
  // from worker i's segment of a block to worker i + 1's: segment index, chunk tables, list offsets, candidates
  uint32_t blocks, chunk_stride, seloff_stride;
  uint64_t cand_stride;
};
hipError_t topk_blocks_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt, const AmsParams& ap,
                            const TopkFlat& flat, const float* g, float* e, float* theta, float* m, float* v,
                            float* vhat, bool first_pass_may_predict, bool clear_pending, bool workers_only,
                            hipStream_t stream, Launcher* L);
hipError_t topk_server_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt, const AmsParams& ap,
                            float* theta, float* m, float* v, float* vhat, hipStream_t stream, Launcher* L);
hipError_t topk_apply_clear(const Geometry& geo, const TopkWorkspace& ws, float* e, hipStream_t stream);
hipError_t blocksign_step(const Geometry& geo, const BlocksignWorkspace& ws, const AmsParams& ap, const float* g,
                          float* e, float* theta, float* m, float* v, float* vhat, bool residual_pending,
                          bool workers_only, hipStream_t stream, Launcher* L);
hipError_t blocksign_server_step(const Geometry& geo, const BlocksignWorkspace& ws, const AmsParams& ap, float* theta,
                                 float* m, float* v, float* vhat, hipStream_t stream, Launcher* L);
hipError_t blocksign_apply_residual(const Geometry& geo, const BlocksignWorkspace& ws, float* e, hipStream_t stream);
hipError_t none_step(const Geometry& geo, const AmsParams& ap, const float* g, float* theta, float* m, float* v,
                     float* vhat, hipStream_t stream, Launcher* L);
hipError_t wire_encode_topk(const Geometry& geo, const TopkWorkspace& ws, uint32_t* messages, int64_t stride,
                            uint32_t* words_out, hipStream_t stream, Launcher* L);
hipError_t wire_decode_topk(const Geometry& geo, const TopkWorkspace& ws, const uint32_t* messages, int64_t stride,
                            const uint32_t* words, int32_t* idx_out, float* val_out, uint32_t* status,
                            bool quarter_offsets, hipStream_t stream, Launcher* L);
hipError_t wire_encode_blocksign(const Geometry& geo, const BlocksignWorkspace& ws, uint32_t* messages, int64_t stride,
                                 uint32_t* words_out, hipStream_t stream, Launcher* L);
hipError_t wire_decode_blocksign(const Geometry& geo, const uint32_t* messages, int64_t stride, const uint32_t* words,
                                 uint32_t* bits_out, float* scales_out, uint32_t* status, hipStream_t stream,
                                 Launcher* L);
hipError_t fill_u32(uint32_t* p, size_t count, uint32_t value, hipStream_t stream);
hipError_t fill_rows_f32(float* p, uint32_t n, int64_t ld, uint32_t d, float value, hipStream_t stream);
hipError_t stream_copy(void* dst, const void* src, size_t bytes, hipStream_t stream);
hipError_t inplace_probe(float* const* arrays, int n_arrays, size_t count, int cached_arrays, hipStream_t stream);

// Kernels of short steps take what their first loads need as leading plain arguments, which arrive in scalar registers;
// the structures that follow hold the same values.
// Launch with optional timing: when the slot is being timed, the launch is bracketed by a pair of events on
// the same stream.  (Events attached to the dispatch itself give the same durations but slow the step down
// by more than the bracketing does; measured on MI355X.)
void launcher_begin(Launcher* L, int slot, hipStream_t stream);
void launcher_end(Launcher* L, int slot, hipStream_t stream);

template <typename... KArgs, typename... Args>
inline void launch_lds(Launcher* L, int slot, void (*kernel)(KArgs...), const dim3& grid, const dim3& block, size_t lds,
                       hipStream_t stream, Args... args) {
  if (L) launcher_begin(L, slot, stream);
  hipLaunchKernelGGL(kernel, grid, block, lds, stream, static_cast<KArgs>(args)...);
  if (L) launcher_end(L, slot, stream);
}
template <typename... KArgs, typename... Args>
inline void launch(Launcher* L, int slot, void (*kernel)(KArgs...), const dim3& grid, const dim3& block,
                   hipStream_t stream, Args... args) {
  launch_lds(L, slot, kernel, grid, block, 0, stream, args...);
}

// A kernel template over the number of cached state arrays (0..4), picked at run time.
#define COMPAMS_LAUNCH_BY_CACHED(nc, L, slot, KERNEL, ...)                      \
  do {                                                                          \
    switch (nc) {                                                               \
      case 0: launch(L, slot, KERNEL(0), __VA_ARGS__); break;                   \
      case 1: launch(L, slot, KERNEL(1), __VA_ARGS__); break;                   \
      case 2: launch(L, slot, KERNEL(2), __VA_ARGS__); break;                   \
      case 3: launch(L, slot, KERNEL(3), __VA_ARGS__); break;                   \
      default: launch(L, slot, KERNEL(4), __VA_ARGS__); break;                  \
    }                                                                           \
  } while (0)

// How many workgroups per row the streaming kernels use: enough to keep 256 compute units busy
// with several workgroups each, whatever n is.
inline uint32_t groups_per_row(uint32_t n, uint32_t num_chunks) {
  const uint32_t target = 256 * 8;  // workgroups in flight over the whole grid
  uint32_t g = (target + n - 1) / n;
  const uint32_t max_g = (num_chunks + kWaves - 1) / kWaves;  // one chunk per wavefront at least
  if (g > max_g) g = max_g;
  if (g < 1) g = 1;
  return g;
}


}  // namespace compams
