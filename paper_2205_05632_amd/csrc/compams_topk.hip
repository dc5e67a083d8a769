// Top-k with error feedback (Definition 1 inside the worker lines of Algorithm 2) and the server
// lines for sparse messages, for gfx950.
//
// Per worker row:  x = e + g is stored in place of e, the k coordinates of largest magnitude key
// (fp32 pattern without the sign; ties to the lower coordinate) are written out as ascending
// (coordinate, value) lists, and the residual at those coordinates becomes zero.
//
// Kernels of a step.  In the steady state three of them do the work (first pass, band, final); the general
// ones in between return at once for every row whose threshold the band kernel has found:
//   first pass     x = e + g -> e as a grid of short workgroups, one chunk each.  When the previous step's
//                  threshold bucket is carried over as a guess, the same pass writes the candidate list: the
//                  entries at or above the guessed bucket, a segment per chunk.  When the last two thresholds
//                  also give a band of keys in which this step's threshold is expected, the candidates are the
//                  entries from a margin below the band upwards (at or above the guessed bucket), and the
//                  pass counts per chunk the entries above the band, lists the entries inside it (a segment per
//                  chunk again) and adds them to the row's histogram of 2048 or 8192 buckets across the band.
//   band           if the threshold key does lie in the band (decided exactly from the counts): per chunk the
//                  entries kept for certain, their prefixes inside blocks of chunks and the block totals; the
//                  few entries of the threshold's bucket are ranked by the last workgroup of the row, which
//                  gives tau, the ties to keep (by coordinate) and the next step's guess, and the next step's band or,
//                  up to 64 rows, what it follows from (final).
//   pick           rows of at most 16 chunks, in every step that may have a guess: the whole selection by one workgroup
//                  per row, in place of the band kernel and the general route.
//   The general route (12 + 10 + 9 key bits and a zero sign bit), for every other row, in four launches or in one:
//   level 0        histogram of the 12-bit threshold buckets, from the candidate list when the guess held (the
//                  list then holds at least k entries), else from the row itself; for a listed row also the
//                  level-1 histograms of the three buckets from the guess upwards, among which the threshold
//                  is expected.  The last workgroup of a row to finish finds the threshold bucket, checks the
//                  guess, resolves level 1 if it can, and sets the next step's guess.
//   level 1        only for rows that level 0 could not resolve: one more read of the row that writes the
//                  candidate list with the exact bucket and builds the level-1 histogram (10 bits), or a
//                  sweep of the list; rows that would not fit a list are histogrammed from the row itself.
//   level 2        histogram of the last 9 key bits over the matching candidates; yields the k-th largest
//                  key tau and how many keys equal to tau are taken; sets the next step's band.
//   count          per chunk: keys above tau and keys equal to tau, with prefixes inside contiguous blocks of
//                  chunks and the totals of every block.
//   final          per chunk of coordinates: the position of each worker's entries in its list follows from
//                  the block totals and prefixes; the selected entries are written there, then added in
//                  worker order into an LDS tile of the averaged gradient, then AMSGrad.  Up to 64 rows it also sets the
//                  next step's band of the rows that band or pick has selected.
// With top-k inside every block (one selection problem per worker and block) the same launches go over all
// problems at once through tables of workgroup slots; problems of at most 1024 coordinates are solved by one
// wavefront inside the first pass.
// A step without a state of its own (the step whose tables lie in a static array) has no guess to carry over: a kernel
// before the first pass takes one, and mostly a band, from a sample of every row.
// Zeroing the residual at the selected coordinates is not done by scattered stores: the next step's
// first pass treats the coordinates in the previous lists as zero while it forms x (and a small kernel
// applies the zeros when the caller asks for e).
//
// All routes give the same result; the guess only decides how many bytes move.  A candidate list is a
// set of per-chunk segments, each in ascending coordinate order, placed by integer atomic cursors (a row's
// list is kept as eight runs with a cursor each, chunk c appending to run c % 8): their physical order
// varies from run to run but nothing that is output depends on it.  No floating-point atomics are used
// anywhere.

#include <algorithm>
#include <type_traits>

#include "compams_device.h"
#include "compams_internal.h"

namespace compams {
namespace {

struct Quad {
  uint32_t key[4];
  bool ok[4];
};

template <bool FULL>
__device__ __forceinline__ void hist4(uint32_t* lh, const Quad& q, uint32_t& zeros) {
  if (FULL) {
    // common case: no zero key in the whole round -> four unconditional LDS adds
    const uint32_t kmin = min(min(q.key[0], q.key[1]), min(q.key[2], q.key[3]));
    if (ballot64(kmin == 0) == 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) atomicAdd(&lh[q.key[s] >> kL0Shift], 1u);
      return;
    }
  }
  // Zero keys (frequent in sparse gradients) would serialise on one LDS word: count them by ballot.
  uint32_t z = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const bool isz = q.ok[s] && q.key[s] == 0;
    const uint64_t bz = ballot64(isz);
    if (bz) z += popc64(bz);
    if (q.ok[s] && q.key[s] != 0) atomicAdd(&lh[q.key[s] >> kL0Shift], 1u);
  }
  zeros += z;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
  return v;
}

// Number of flagged entries of one round, and this lane's position among them in (lane, slot) order.
struct RoundRank {
  uint32_t total;
  uint32_t below;
};
__device__ __forceinline__ RoundRank rank_round(const bool flag[4]) {
  const uint64_t b0 = ballot64(flag[0]), b1 = ballot64(flag[1]), b2 = ballot64(flag[2]), b3 = ballot64(flag[3]);
  RoundRank rr;
  rr.total = popc64(b0) + popc64(b1) + popc64(b2) + popc64(b3);
  rr.below = rr.total ? count_below(b0) + count_below(b1) + count_below(b2) + count_below(b3) : 0;
  return rr;
}

// Stores that other workgroups of the same launch read (see last_group_of_row).
__device__ __forceinline__ void store_agent(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(uint2* p, uint2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the parts of the general route hand on: SAME: to the same launch, else to the next one.
template <bool SAME, typename T>
__device__ __forceinline__ void hand_on(T* p, T v) {
  if constexpr (SAME) store_agent(p, v);
  else *p = v;
}

// Candidate entries of the chunk a wavefront is walking are first staged in LDS (kStage entries per
// wavefront) so that the chunk's segment can be allocated with one atomic once its size is known and
// then written with coalesced stores.  A chunk with more candidates than that is re-read instead.
constexpr int kStage = 512;

__device__ __forceinline__ void stage_round(uint2* stage, uint32_t& n, uint32_t j, const uint32_t bits[4],
                                            const bool flag[4]) {
  const RoundRank rr = rank_round(flag);
  if (rr.total == 0) return;
  uint32_t pos = n + rr.below;
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (flag[s]) {
      if (pos < static_cast<uint32_t>(kStage)) stage[pos] = make_uint2(j + s, bits[s]);
      ++pos;
    }
  n += rr.total;
}

// Allocating a chunk's segment of the candidate list takes an atomic with return.  It is split in two so
// that a caller can put other work between the request and the first use of its result.
__device__ __forceinline__ uint32_t segment_request(TopkRow* rowp, uint32_t cnt) {
  uint32_t raw = 0;
  if (cnt && lane_id() == 0) raw = atomicAdd(&rowp->cursor, cnt);
  return raw;  // meaningful in lane 0 only; nobody has looked at it yet
}

// Write the chunk's segment: from the staging area if everything fitted there, else by reading the chunk's
// (already stored) corrected gradients again.
template <bool SAME>
__device__ __forceinline__ void segment_write(uint32_t raw, const uint2* stage, uint32_t cnt,
                                              const float* __restrict__ er, uint32_t d, uint32_t c,
                                              uint32_t thr_bucket, uint2* candr, uint32_t cap, uint2* descr,
                                              uint32_t parts) {
  const uint32_t lane = lane_id();
  uint32_t off = 0;
  if (cnt) {
    off = first_lane(raw);
    if (off + cnt <= cap) {  // otherwise the row's list has overflowed and will not be used
      if (cnt <= static_cast<uint32_t>(kStage)) {
        for (uint32_t q = lane; q < cnt; q += 64) hand_on<SAME>(candr + off + q, stage[q]);
      } else {
        uint32_t at = off;
        for (int r = 0; r < kRounds; ++r) {
          const uint32_t j = c * kChunk + r * 256 + lane * 4;
          float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
          if (j < d) x = *reinterpret_cast<const float4*>(er + j);
          const uint32_t bits[4] = {__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z),
                                    __float_as_uint(x.w)};
          bool flag[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) flag[s] = j + s < d && (key_of_bits(bits[s]) >> kL0Shift) >= thr_bucket;
          const RoundRank rr = rank_round(flag);
          uint32_t pos = at + rr.below;
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (flag[s]) {
              if (pos < off + cnt) hand_on<SAME>(candr + pos, make_uint2(j + s, bits[s]));
              ++pos;
            }
          at += rr.total;
        }
      }
    }
  }
  if (lane < parts) {  // (parts of it one behind the other, where a chunk has several segments)
    const uint32_t share = (cnt + parts - 1) / parts, at = share * lane < cnt ? share * lane : cnt;
    hand_on<SAME>(descr + c * parts + lane, make_uint2(off + at, cnt - at < share ? cnt - at : share));
  }
}

template <bool SAME>
__device__ __forceinline__ void flush_chunk(const uint2* stage, uint32_t cnt, const float* __restrict__ er, uint32_t d,
                                            uint32_t c, uint32_t thr_bucket, TopkRow* rowp, uint2* candr,
                                            uint32_t cap, uint2* descr, uint32_t parts) {
  const uint32_t raw = segment_request(rowp, cnt);
  segment_write<SAME>(raw, stage, cnt, er, d, c, thr_bucket, candr, cap, descr, parts);
}

// ---------------------------------------------------------------------------------------------
// "Last workgroup of the row": every workgroup of a row takes a ticket when it has finished; the one
// that draws the last ticket continues with the row-wide step.  No workgroup ever waits for another.
//
// Everything the last workgroup reads from the others travels through device-scope atomics (adds,
// stores) and is read back with device-scope atomic loads: those are performed at the level of the
// memory hierarchy that all compute units share, so no cache write-back or invalidation is needed
// (a full device-scope fence would write back and invalidate the whole L2 of the die at every call).
// Ordering: each wavefront waits until its own atomics have been acknowledged, the workgroup barrier
// collects all wavefronts, and only then is the ticket drawn.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ bool last_group_of_row(uint32_t* ticket, uint32_t groups, uint32_t* sh_flag) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // this wavefront's atomics have been performed
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = (t + 1 == groups);
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    *sh_flag = last ? 1u : 0u;
  }
  __syncthreads();
  return *sh_flag != 0;
}

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Many device-scope loads in flight at once.  The compiler waits for each atomic load before it issues the
// next, which turns a row-wide step of a few thousand words into a chain of memory round trips; buffer loads
// with the same cache policy (served by the level all compute units share) are ordinary loads to it and
// overlap.  A view covers `words` 32-bit words from p; reads beyond it return 0.
struct AgentView {
  __amdgpu_buffer_rsrc_t rsrc;
};
__device__ __forceinline__ AgentView agent_view(const uint32_t* p, uint32_t words) {
  AgentView v;
  v.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), 0, words * 4u, 0x00020000);
  return v;
}
__device__ __forceinline__ uint32_t load_agent(const AgentView& v, uint32_t word) {
  return __builtin_amdgcn_raw_buffer_load_b32(v.rsrc, word * 4u, 0, /*device-scope policy*/ 16);
}

__device__ __forceinline__ uint2 load_agent2(const AgentView& v, uint32_t pair) {
  return make_uint2(load_agent(v, 2 * pair), load_agent(v, 2 * pair + 1));
}

// ---------------------------------------------------------------------------------------------
// Finding the bucket in which a suffix count crosses `need`, by one workgroup of kWG threads.
// h: NB bucket counts in LDS.  Returns through out2 the largest s with sum_{b >= s} h[b] >= need and the
// count strictly above it.  Requires 1 <= need <= sum h.
// ---------------------------------------------------------------------------------------------
// WANTS of them at once (each returned in two words of out2).
template <int NB, int NT = kWG, int WANTS = 1>
__device__ void find_crossings(const uint32_t* h, const uint32_t (&needs)[WANTS], uint32_t* suf /* NT + 1 */, uint32_t* out2) {
  constexpr int PER = NB / NT;
  static_assert(NB % NT == 0 && NT % 64 == 0, "buckets per thread, whole wavefronts");
  const int t = threadIdx.x;
  const uint32_t lane = lane_id(), wave = t >> 6;
  uint32_t part = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) part += h[t * PER + i];
  // inclusive suffix sum over the threads: inside the wavefront by shuffles, across wavefronts through LDS
  uint32_t s = part;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_down(s, o, 64);
    if (lane + o < 64) s += up;
  }
  __syncthreads();  // everybody has read h and whatever suf / out2 held before
  if (lane == 0) suf[wave] = s;  // the wavefront's total
  if (t < 2 * WANTS) out2[t] = 0;
  __syncthreads();
  uint32_t higher = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w)
    if (static_cast<uint32_t>(w) > wave) higher += suf[w];
  s += higher;                       // entries in this thread's buckets and all buckets above them
  const uint32_t above_mine = s - part;  // entries in the buckets above this thread's
#pragma unroll
  for (int w = 0; w < WANTS; ++w) {
    const uint32_t need = needs[w];
    if (s >= need && above_mine < need) {  // exactly one thread when 1 <= need <= sum h
      uint32_t acc = above_mine;
      for (int i = PER - 1; i >= 0; --i) {
        const uint32_t hb = h[t * PER + i];
        if (acc + hb >= need) {
          out2[2 * w] = t * PER + i;
          out2[2 * w + 1] = acc;
          break;
        }
        acc += hb;
      }
    }
  }
  __syncthreads();
}
template <int NB, int NT = kWG>
__device__ __forceinline__ void find_crossing(const uint32_t* h, uint32_t need, uint32_t* suf, uint32_t* out2) {
  const uint32_t needs[1] = {need};
  find_crossings<NB, NT, 1>(h, needs, suf, out2);
}

// Copy a row's global histogram into LDS and clear it for the next step.
template <int NB, int NT = kWG>
__device__ __forceinline__ void take_hist(uint32_t* gh, uint32_t* h) {
  static_assert(NB % NT == 0, "buckets per thread");
  constexpr int PER = NB / NT;
  const AgentView view = agent_view(gh, NB);
  uint32_t x[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) x[i] = load_agent(view, i * NT + threadIdx.x);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    h[i * NT + threadIdx.x] = x[i];
    gh[i * NT + threadIdx.x] = 0;
  }
  __syncthreads();
}

// bstar and need are passed in (not re-read from the control block): the caller may have written them a
// moment ago, and a line of the control block read earlier by this compute unit may still sit in its L1.
template <bool SAME, int NT = kWG>
__device__ __forceinline__ void resolve_level1(TopkRow* rp, uint32_t bstar, uint32_t need, const uint32_t* h,
                                               uint32_t* suf, uint32_t* out2) {
  find_crossing<kNB1, NT>(h, need, suf, out2);
  if (threadIdx.x == 0) {
    hand_on<SAME>(&rp->prefix1, (bstar << (kL0Shift - kL1Shift)) | out2[0]);
    hand_on<SAME>(&rp->need, need - out2[1]);
    rp->level1_done = 1;
  }
}

__device__ __forceinline__ void emit_chunk(uint32_t mode, const float* __restrict__ er, uint32_t d, uint32_t c,
                                           const uint2* __restrict__ candr, uint2 ds,
                                           uint32_t cap, uint32_t tau, uint32_t r, bool all_ties, uint32_t eq_seen,
                                           uint32_t at, int32_t* __restrict__ idx, float* __restrict__ val, uint32_t k,
                                           uint32_t coord_base, bool by_coord = false, uint32_t tie_last = 0);

// A micro problem (top-k inside a block of at most kMicroCoords coordinates) from end to end by one wavefront:
// x = e + g with the pending zeros honoured, stored in place of e; the k-th largest key by a bit-by-bit search
// over the keys, which stay in registers (31 steps of ballots: the largest t with at least k keys >= t); the
// selected entries in coordinate order into the problem's part of the worker's list (ties as everywhere: in
// coordinate order until r are in), which the last kernel reads.
// bm: 32 words of LDS of this wavefront (PEND only).  No barrier: other wavefronts of the workgroup do other
// problems.
constexpr int kMicroRounds = static_cast<int>(kMicroCoords / 256);

template <bool PEND>
__device__ __forceinline__ void micro_problem(const float* __restrict__ g, float* __restrict__ e, const Seg& sg,
                                              uint32_t seg, const TopkWorkspace& ws, uint32_t* bm) {
  const uint32_t lane = lane_id();
  const float* gr = g + sg.elem_off;
  float* er = e + sg.elem_off;
  const uint32_t d = sg.d, k = sg.k;
  int32_t* idx = ws.idx + sg.list_base;
  float* val = ws.val + sg.list_base;
  if constexpr (PEND) {
    if (lane < kMicroCoords / 32) bm[lane] = 0;
    const uint32_t* so = ws.sel_off + sg.seloff_base;
    const uint32_t lo = so[0];
    const uint32_t hi = so[kWaves] < k ? so[kWaves] : k;  // (one chunk: its end)
    for (uint32_t q = lo + lane; q < hi; q += 64) {
      const uint32_t jl = static_cast<uint32_t>(idx[q]) - sg.coord_base;
      if (jl < kMicroCoords) atomicOr(&bm[jl >> 5], 1u << (jl & 31u));
    }
  }
  uint32_t key[kMicroRounds * 4];
  uint32_t okm = 0;  // bit 4r + s: this lane's slot s of round r is a coordinate of the problem
#pragma unroll
  for (int r = 0; r < kMicroRounds; ++r) {
    const uint32_t j = r * 256 + lane * 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) key[4 * r + s] = 0;
    if (j < d) {
      const float4 gv = *reinterpret_cast<const float4*>(gr + j);
      const float4 e_in = *reinterpret_cast<const float4*>(er + j);
      float4 ev = e_in;
      if constexpr (PEND) {
        const uint32_t nib = (bm[r * 8 + (lane >> 3)] >> ((lane & 7u) * 4u)) & 15u;
        if (nib & 1u) ev.x = 0.0f;
        if (nib & 2u) ev.y = 0.0f;
        if (nib & 4u) ev.z = 0.0f;
        if (nib & 8u) ev.w = 0.0f;
      }
      float4 x = make_float4(ev.x + gv.x, ev.y + gv.y, ev.z + gv.z, ev.w + gv.w);
      const bool ok1 = j + 1 < d, ok2 = j + 2 < d, ok3 = j + 3 < d;
      if (!ok1) x.y = e_in.y;  // columns >= d keep what they held
      if (!ok2) x.z = e_in.z;
      if (!ok3) x.w = e_in.w;
      *reinterpret_cast<float4*>(er + j) = x;
      key[4 * r + 0] = key_of_bits(__float_as_uint(x.x));
      key[4 * r + 1] = ok1 ? key_of_bits(__float_as_uint(x.y)) : 0u;
      key[4 * r + 2] = ok2 ? key_of_bits(__float_as_uint(x.z)) : 0u;
      key[4 * r + 3] = ok3 ? key_of_bits(__float_as_uint(x.w)) : 0u;
      okm |= (1u | (ok1 ? 2u : 0u) | (ok2 ? 4u : 0u) | (ok3 ? 8u : 0u)) << (4 * r);
    }
  }
  const int rounds = static_cast<int>((d + 255) / 256);  // wave-uniform; keys of later rounds are 0 and not looked at
  uint32_t tau = 0;
  for (int bit = 30; bit >= 0; --bit) {
    const uint32_t t = tau | (1u << bit);  // t >= 1: a slot outside the problem (key 0) never counts
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < kMicroRounds; ++r)
      if (r < rounds) {
#pragma unroll
        for (int s = 0; s < 4; ++s) cnt += popc64(ballot64(key[4 * r + s] >= t));
      }
    if (cnt >= k) tau = t;
  }
  uint32_t gt = 0, ties = 0;
#pragma unroll
  for (int r = 0; r < kMicroRounds; ++r)
    if (r < rounds) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool ok = (okm >> (4 * r + s)) & 1u;
        gt += popc64(ballot64(ok && key[4 * r + s] > tau));
        ties += popc64(ballot64(ok && key[4 * r + s] == tau));
      }
    }
  const uint32_t r_take = k - gt;  // 1 <= r_take <= ties
  if (lane == 0) {
    TopkRow* rowp = ws.rows + seg;
    rowp->mode = kModeDense;
    rowp->n_src = 0;
    rowp->cursor = 0;
    rowp->cursor_band = 0;
    rowp->cand_from = 0;
    rowp->band_valid = 0;
    rowp->fast = 0;
    rowp->b_guess = 0;
    rowp->level1_done = 1;
    rowp->tau = tau;
    rowp->r = r_take;
    rowp->ties = ties;
    ws.tau[seg] = tau;
    ws.count_gt[seg] = gt;
    uint32_t* cn = ws.counters + seg * kCountersPerRow;
    cn[0] = 0;
    cn[1] = 0;
    cn[2] = ties;
    cn[3] = r_take;
    cn[4] = 0;
    cn[5] = 1;
  }
  // the values come back from where this wavefront has just stored them
  emit_chunk(kModeDense, er, d, 0u, nullptr, make_uint2(0u, 0u), 0u, tau, r_take, r_take == ties, 0u, 0u, idx, val, k,
             sg.coord_base);
}

// ---------------------------------------------------------------------------------------------
// Which selection problem a workgroup works on.  UNI: one problem per worker row, all of one shape, grid
// (groups, rows): everything follows from the block indices.  Otherwise the launch is flat and tables say
// which segment (a block of a worker's row) and which of its workgroups this is; geo and opt are then
// narrowed to the segment's own shape.
// ---------------------------------------------------------------------------------------------
enum : int { kClassFirst = 0, kClassSweep = 1, kClassCount = 2, kClassLevel0 = 3 };

struct SegCtx {
  uint32_t seg;     // index into the per-problem tables (control blocks, histograms, thresholds)
  uint32_t group;   // this workgroup's index among the `groups` that share the problem
  uint32_t groups;
  int64_t elem_off;
  uint32_t coord_base;
  size_t chunk_base, seloff_base, cand_base, list_base, band_base;
  uint32_t cursor_set;  // see Seg
  size_t bhist_base;
};

// The context of workgroup `group` of segment `seg` in a flat launch.
__device__ __forceinline__ SegCtx seg_ctx_of(uint32_t seg, uint32_t group, uint32_t groups, const Seg& sg, Geometry& geo,
                                             TopkOptions& opt) {
  SegCtx c;
  c.seg = seg;
  c.group = group;
  c.groups = groups;
  c.elem_off = sg.elem_off;
  c.coord_base = sg.coord_base;
  c.chunk_base = sg.chunk_base;
  c.seloff_base = sg.seloff_base;
  c.cand_base = sg.cand_base;
  c.list_base = sg.list_base;
  c.band_base = sg.band_base;
  c.cursor_set = sg.cursor_set;
  c.bhist_base = sg.bhist_base;
  geo.d = sg.d;
  geo.k = sg.k;
  geo.num_chunks = sg.num_chunks;
  geo.count_cpw = sg.count_cpw;
  opt.cap = opt.cap < sg.cap ? opt.cap : sg.cap;
  opt.band_cap = opt.band_cap < sg.band_cap ? opt.band_cap : sg.band_cap;
  return c;
}

// The context of workgroup `group` of the row `seg`, `groups` of them.
__device__ __forceinline__ SegCtx row_ctx(uint32_t seg, uint32_t group, uint32_t groups, const Geometry& geo, const TopkOptions& opt) {
  SegCtx c;
  c.seg = seg;
  c.group = group;
  c.groups = groups;
  c.elem_off = static_cast<int64_t>(c.seg) * geo.ld;
  c.coord_base = 0;
  c.chunk_base = static_cast<size_t>(c.seg) * geo.num_chunks;
  c.seloff_base = static_cast<size_t>(c.seg) * (geo.num_chunks * kWaves + 1);
  c.cand_base = static_cast<size_t>(c.seg) * row_cand_pitch(opt.cap, geo.num_chunks);
  c.list_base = static_cast<size_t>(c.seg) * geo.k;
  c.band_base = static_cast<size_t>(c.seg) * opt.band_cap;
  c.bhist_base = static_cast<size_t>(c.seg) * band_buckets(geo.k);
  c.cursor_set = geo.num_chunks >= kSubListMinChunks ? c.seg : kNoCursorSet;  // short rows keep one run
  return c;
}

template <bool UNI, int CLASS>
__device__ __forceinline__ SegCtx seg_ctx(Geometry& geo, TopkOptions& opt, const TopkWorkspace& ws) {
  if (UNI) return row_ctx(blockIdx.y, blockIdx.x, gridDim.x, geo, opt);
  // (the records come through the vector path: through the scalar one the first pass was 1-2 % slower)
  const WgSlot slot = (CLASS == kClassFirst ? ws.map_first
                       : CLASS == kClassLevel0 ? ws.map_level0
                       : CLASS == kClassSweep ? ws.map_sweep : ws.map_count)[blockIdx.x];
  const Seg sg = ws.segs[slot.seg];
  return seg_ctx_of(slot.seg, slot.group,
                    CLASS == kClassFirst ? sg.groups_first
                    : CLASS == kClassLevel0 ? sg.groups_level0
                    : CLASS == kClassSweep ? sg.groups_sweep : sg.count_blocks,
                    sg, geo, opt);
}

constexpr uint32_t kRowWord(size_t offset) { return static_cast<uint32_t>(offset / 4); }

// How the parts of the general route hand things on: SAME: inside one launch, at device scope; else from launch to
// launch, with ordinary accesses (at device scope the four launches took 5 us more).
template <bool SAME>
struct Handed {  // words from p on, `words` of them
  const uint32_t* p;
  AgentView view;
  __device__ __forceinline__ Handed(const void* from, uint32_t words) : p(static_cast<const uint32_t*>(from)) {
    if constexpr (SAME) view = agent_view(p, words);
  }
  __device__ __forceinline__ uint32_t word(uint32_t at) const {
    if constexpr (SAME) return load_agent(view, at);
    else return p[at];
  }
  __device__ __forceinline__ uint2 pair(uint32_t at) const {
    if constexpr (SAME) return load_agent2(view, at);
    else return reinterpret_cast<const uint2*>(p)[at];
  }
};

template <bool SAME>
__device__ __forceinline__ Handed<SAME> handed_row(const TopkRow* rowp) {
  return Handed<SAME>(rowp, sizeof(TopkRow) / 4);
}

// The runs of a problem's candidate list (one, or kSubLists for a row of the one-selection-per-row form).
struct ListRuns {
  uint32_t lists, pitch;  // run s starts at entry s * pitch
  uint32_t n[kSubLists];
  uint32_t total;
  bool fits;              // no run has outgrown its share of the capacity
};

// As the first pass left them: from the cursors.
__device__ __forceinline__ ListRuns runs_from_cursors(const TopkWorkspace& ws, const TopkRow* rowp, uint32_t cursor_set,
                                                      uint32_t cap) {
  ListRuns L;
  L.total = 0;
  L.fits = true;
  if (cursor_set != kNoCursorSet) {  // uniform
    L.lists = kSubLists;
    L.pitch = cap / kSubLists;
    const uint32_t* cur = ws.xcur + static_cast<size_t>(cursor_set) * kSubLists * kCursorPitch;
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s) {
      L.n[s] = cur[s * kCursorPitch];
      L.total += L.n[s];
      L.fits = L.fits && L.n[s] <= L.pitch;
    }
  } else {
    L.lists = 1;
    L.pitch = 0;
    L.n[0] = rowp->cursor;
#pragma unroll
    for (uint32_t s = 1; s < kSubLists; ++s) L.n[s] = 0;
    L.total = L.n[0];
    L.fits = L.n[0] <= cap;
  }
  return L;
}

// As level 0 recorded them for the later sweeps.
template <bool SAME>
__device__ __forceinline__ ListRuns runs_of_row(const Handed<SAME>& row, uint32_t cap) {
  ListRuns L;
  L.lists = row.word(kRowWord(offsetof(TopkRow, n_lists)));
  L.pitch = cap / kSubLists;
  L.total = 0;
  L.fits = true;
#pragma unroll
  for (uint32_t s = 0; s < kSubLists; ++s) L.n[s] = row.word(kRowWord(offsetof(TopkRow, n_sub)) + s);
#pragma unroll
  for (uint32_t s = 0; s < kSubLists; ++s) {
    L.n[s] = s < L.lists ? L.n[s] : 0u;
    L.total += L.n[s];
  }
  return L;
}

// read(bits_of) with the entries of a problem's candidate list, as an earlier launch has left them.  A list that this
// launch has written (SAME; level 1, kModeNeedB) is read at device scope: segments lie behind one another, so that
// workgroups of several dies write parts of one line, and the line in the reader's own die may be from before.
template <bool SAME, typename F>
__device__ __forceinline__ void with_list(const uint2* __restrict__ candr, uint32_t cap, uint32_t mode, F&& read) {
  if (SAME && mode == kModeNeedB) {  // uniform
    const AgentView view = agent_view(reinterpret_cast<const uint32_t*>(candr), 2 * cap);
    read([=](uint32_t q) { return load_agent(view, 2 * q + 1); });
  } else {
    read([=](uint32_t q) { return candr[q].y; });
  }
}

// A sweep over a problem's candidate list by `threads` threads, of which the caller is number `first`: visit(bits)
// for the entries first, first + threads, ... of every run; bits_of(q) is the value of the list's entry q.  The loads of a
// trip are requested together -- four entries of a list kept as one run, one entry of each of the kSubLists runs
// otherwise -- because a thread's trips are a chain of round trips (run after run, the sweep of level 2 took 10.4 us
// instead of 7).
template <typename Bits, typename F>
__device__ __forceinline__ void sweep_list(Bits&& bits_of, const ListRuns& R, uint32_t first, uint32_t threads, F&& visit) {
  if (R.lists == 1) {  // uniform
    const uint32_t len = R.n[0];
    for (uint32_t q = first; q < len; q += 4 * threads) {
      uint32_t bits[4];
      bool ok[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        ok[w] = q + w * threads < len;
        bits[w] = ok[w] ? bits_of(q + w * threads) : 0u;
      }
#pragma unroll
      for (int w = 0; w < 4; ++w)
        if (ok[w]) visit(bits[w]);
    }
    return;
  }
  uint32_t longest = 0;
#pragma unroll
  for (uint32_t s = 0; s < kSubLists; ++s) longest = R.n[s] > longest ? R.n[s] : longest;
  for (uint32_t q = first; q < longest; q += threads) {
    uint32_t bits[kSubLists];
    bool ok[kSubLists];
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s) {
      ok[s] = q < R.n[s];
      bits[s] = ok[s] ? bits_of(s * R.pitch + q) : 0u;  // (below cap)
    }
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s)
      if (ok[s]) visit(bits[s]);
  }
}

// ---------------------------------------------------------------------------------------------
// One selection per row, first pass without histograms.  A workgroup takes ONE chunk and ends; wavefront w takes
// rounds 4w .. 4w+3 of it.  Measured on MI355X with plain streaming kernels of the same traffic (read g, read e,
// write e, 2.1 GB): a grid of such short workgroups, handed out in order, streams at 6.1-6.4 TB/s, while
// workgroups that each walk many chunks stay at 5.4-5.7 TB/s whatever their number, occupancy or prefetch depth.
// A short-lived workgroup cannot afford a 4096-bin histogram in LDS (to clear and to flush), so this pass has
// none: x = e + g (pending zeros honoured) is stored, and when the row carries a guess for the threshold bucket
// the entries at or above it are staged per wavefront in coordinate order, the chunk's segment of the candidate
// list is allocated with one atomic for the whole workgroup, and the four quarters are written behind one
// another.  The level-0 histogram is taken afterwards, from the candidate list (general_level0).
// In large problems (paged_first_pass) the workgroup takes the same page of four spans instead, a quarter of four different
// chunks (page_quarter): one allocation still, but a segment of the lists for every quarter.  Which page a die takes changes
// seven times over the rows: a crowded page (a matrix as wide as the span or a multiple, its large columns side by side)
// takes its die longer, and as one die's page in every row it held up the whole pass (8 x 25570000, k 5 %, 1024 large
// columns of 32768: 441 us in chunks, 598 with the pages as they are in every row, 407 so; 64 x 3002268, k 8 %: 412, 574,
// 413; without such columns 16 x 25570000 755 / 755, 64 x 3002268 356 / 363).  (Measured on the way: fewer instructions
// between the loads and the stores, and stores as soon as a round's loads have come, made it slower, 8 x 30381 chunks
// 1828 -> 1899 us; all stores behind a barrier 1866; four workgroups per compute unit instead of five 1820, eight 1843.)
// ---------------------------------------------------------------------------------------------
constexpr int kLeanRounds = kRounds / kWaves;  // rounds of a chunk per wavefront
constexpr int kStageQ = 512;                   // staged candidates per wavefront (of at most 1024 coordinates)
constexpr size_t kLeanLds = 14000;              // asked for on top of that: five workgroups per compute unit, see kStreamLds

// UNI: grid (chunks, rows).  Otherwise (top-k inside every block) the launch is flat over map_first: a workgroup
// per chunk of every segment in address order, and at the end the workgroups whose wavefronts take one micro
// problem each; coordinates below are the segment's own, the lists hold coordinates of the worker's row.
template <bool PEND, bool UNI, bool PAGED>
__global__ __launch_bounds__(kWG) void k_topk_lean(Geometry geo, const float* __restrict__ g, float* __restrict__ e,
                                                    TopkWorkspace ws, TopkOptions opt, uint32_t use_guess) {
  __shared__ uint2 stage_all[kWaves * kStageQ];
  __shared__ uint32_t bm_all[PEND ? kWaves * 32 : 1];
  __shared__ uint32_t sh_cnt[kWaves], sh_above[kWaves], sh_from[kWaves], sh_off, sh_boff;
  const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();
  if constexpr (!UNI) {
    const WgSlot slot = ws.map_first[blockIdx.x];
    if (slot.seg & kMicroFlag) {  // workgroup-uniform: up to four micro problems, one per wavefront
      if (wave < slot.group) {
        const uint32_t seg = ws.micro_list[(slot.seg & ~kMicroFlag) + wave];
        const Seg sg = ws.segs[seg];
        micro_problem<PEND>(g, e, sg, seg, ws, bm_all + (PEND ? wave * 32 : 0));
      }
      return;
    }
  }
  const SegCtx sc = seg_ctx<UNI, kClassFirst>(geo, opt, ws);
  const Quarter quarter = PAGED ? page_quarter(sc.group, wave, (sc.seg * ws.page_turn) >> 16) : Quarter{sc.group, wave};
  const uint32_t c = quarter.chunk, row = sc.seg;
  const float* gr = g + sc.elem_off;
  float* er = e + sc.elem_off;
  TopkRow* rowp = ws.rows + row;
  const uint32_t d = geo.d;
  const uint32_t q0 = c * kChunk + quarter.part * (kLeanRounds * 256);  // first coordinate of this wavefront's quarter
  const bool full = (c + 1) * static_cast<uint64_t>(kChunk) <= d;
  // The chunk's loads go out before anything else is asked for: nothing below decides their addresses.
  float4 gv[kLeanRounds], ev[kLeanRounds];
#pragma unroll
  for (int u = 0; u < kLeanRounds; ++u) {
    const uint32_t j = q0 + u * 256 + lane * 4;
    gv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    ev[u] = gv[u];
    if (full || j < d) {
      gv[u] = load_stream4(gr + j);
      ev[u] = load_stream4(er + j);
    }
  }
  // What this pass reads of the row's control block and of the previous step's list offsets was written by earlier
  // launches and is the same for the whole workgroup: it comes through the scalar path, whose answers do not
  // queue behind the chunk's loads (vector loads return in order) - the first eight words of the control block
  // with one load, the list offsets with it, and only then is any of it looked at (one round trip, not one per
  // condition).
  static_assert(offsetof(TopkRow, cand_from) == 0 && offsetof(TopkRow, b_guess) == 4 &&
                offsetof(TopkRow, band_valid) == 16 && offsetof(TopkRow, band_lo) == 20 &&
                offsetof(TopkRow, band_hi) == 24 && offsetof(TopkRow, band_mul) == 28 &&
                offsetof(TopkRow, cursor) == 8 && offsetof(TopkRow, cursor_band) == 12,
                "words read below; the two cursors form one 64-bit word");
  const U32x8 rw = table_u32x8(reinterpret_cast<const uint32_t*>(rowp));
  uint32_t prev_lo = 0, prev_hi = 0;
  if constexpr (PEND) {
    const uint32_t* prev_off = ws.sel_off + sc.seloff_base;
    if (!PAGED || q0 < d) {  // (eight workgroups take eight chunks, also where the row ends before)
      prev_lo = table_u32(prev_off, c * kWaves + quarter.part);
      prev_hi = table_u32(prev_off, c * kWaves + quarter.part + 1);
    }
  }
  const bool pred = use_guess && rw[0] != 0;  // workgroup-uniform
  // the band [blo, bhi) of keys: empty (no key is >= 0xffffffff) unless the row carries one
  const bool banded = pred && opt.band == kBandLists && rw[4] != 0;
  const uint32_t blo = banded ? rw[5] : 0xffffffffu;
  const uint32_t bhi = banded ? rw[6] : 0xffffffffu;
  const uint32_t bmul = banded ? rw[7] : 0u;
  const bool bmany = rw[4] == kBandMany;
  const uint32_t brot = band_rotation(geo.k, sc.seg);
  // Candidates: every key at or above cand_lo - the guessed bucket's first key, or, with a band, a key somewhat below
  // the band's first one: the threshold is expected inside the band, so that little below it is needed (a list of at
  // least k entries that holds every key from some key upwards holds the k largest, wherever that key lies inside a
  // bucket; a shorter one sends the row to the kernels that read it again).
  const uint32_t cand_lo = rw[0] - 1u;
  uint32_t* bh = ws.bhist + sc.bhist_base;
  uint32_t* bm = bm_all + (PEND ? wave * 32 : 0);
  if constexpr (PEND) {
    // the quarter's coordinates that were selected in the previous step: their residual counts as zero
    if (lane < 32) bm[lane] = 0;
    const int32_t* prev_idx = ws.idx + sc.list_base;
    const uint32_t lo = prev_lo;
    const uint32_t hi = prev_hi < geo.k ? prev_hi : geo.k;
    // 256 entries of the quarter's slice per trip, requested together (one round trip unless the quarter is crowded)
    for (uint32_t q = lo + lane; q < hi; q += 256) {
      uint32_t jv[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) jv[w] = q + 64 * w < hi ? static_cast<uint32_t>(prev_idx[q + 64 * w]) : 0xffffffffu;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t jl = jv[w] - sc.coord_base - q0;
        if (q + 64 * w < hi && jl < static_cast<uint32_t>(kLeanRounds * 256)) atomicOr(&bm[jl >> 5], 1u << (jl & 31u));
      }
    }
  }
  uint2* stage = stage_all + wave * kStageQ;
  uint32_t cnt = 0;
  uint32_t n_above = 0, n_from = 0;  // this lane's entries at or above the band's upper end / its lower end
#pragma unroll
  for (int u = 0; u < kLeanRounds; ++u) {
    const uint32_t j = q0 + u * 256 + lane * 4;
    const bool ok[4] = {full || j < d, full || j + 1 < d, full || j + 2 < d, full || j + 3 < d};
    float4 en = ev[u];
    if constexpr (PEND) {
      const uint32_t nib = (bm[u * 8 + (lane >> 3)] >> ((lane & 7u) * 4u)) & 15u;
      if (nib & 1u) en.x = 0.0f;
      if (nib & 2u) en.y = 0.0f;
      if (nib & 4u) en.z = 0.0f;
      if (nib & 8u) en.w = 0.0f;
    }
    float4 x = make_float4(en.x + gv[u].x, en.y + gv[u].y, en.z + gv[u].z, en.w + gv[u].w);
    if (!full) {  // columns >= d keep what they held
      if (!ok[1]) x.y = ev[u].y;
      if (!ok[2]) x.z = ev[u].z;
      if (!ok[3]) x.w = ev[u].w;
    }
    if (ok[0]) store_stream4(er + j, x);
    if (pred) {
      const uint32_t bits[4] = {__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z), __float_as_uint(x.w)};
      bool flag[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t key = key_of_bits(bits[s]);
        flag[s] = ok[s] && key >= cand_lo;
        n_above += (ok[s] && key >= bhi) ? 1u : 0u;
        n_from += (ok[s] && key >= blo) ? 1u : 0u;
      }
      const RoundRank rr = rank_round(flag);
      if (rr.total) {
        uint32_t pos = cnt + rr.below;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (flag[s]) {
            if (pos < static_cast<uint32_t>(kStageQ)) stage[pos] = make_uint2(j + s, bits[s]);
            ++pos;
          }
        cnt += rr.total;
      }
    }
  }
  if (!pred) return;  // workgroup-uniform
  // the chunk's segments of the candidate list and of the band list: one allocation for the four quarters
  const uint32_t above_w = banded ? wave_sum(n_above) : 0u;
  const uint32_t band_w = banded ? wave_sum(n_from) - above_w : 0u;  // this quarter's entries inside the band
  if (lane == 0) { sh_cnt[wave] = cnt; sh_above[wave] = above_w; sh_from[wave] = band_w; }
  __syncthreads();
  uint32_t before = 0, total = 0, bbefore = 0, btotal = 0, atotal = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t t = sh_cnt[w], tb = sh_from[w];
    before += static_cast<uint32_t>(w) < wave ? t : 0u;
    bbefore += static_cast<uint32_t>(w) < wave ? tb : 0u;
    total += t;
    btotal += tb;
    atotal += sh_above[w];
  }
  // the run this workgroup appends to, its share of the capacities and its cursors (candidates in the low half of a
  // 64-bit word, band entries in the high half: one atomic advances both)
  const bool runs = sc.cursor_set != kNoCursorSet;  // workgroup-uniform
  // In pages `group` % 8 alone is the page, so that a matrix whose rows are a multiple of 8192 long and whose large
  // columns lie side by side would fill one run of eight and be read again in every step (8 x 25570000, 1024 large
  // columns of 8192: 1108 us a step against 597 with the runs in turn).
  const uint32_t turn = PAGED ? sc.group / kDies + sc.group / (kDies * kDies) : 0u;
  const uint32_t run = runs ? (sc.group + turn) % kSubLists : 0u;
  const uint32_t run_cap = runs ? opt.cap / kSubLists : opt.cap;
  const uint32_t run_base = run * run_cap;
  const uint32_t brun_cap = runs ? opt.band_cap / kSubLists : opt.band_cap;
  const uint32_t brun_base = run * brun_cap;
  if (threadIdx.x == 0) {
    uint32_t* cur =
        runs ? ws.xcur + (static_cast<size_t>(sc.cursor_set) * kSubLists + run) * kCursorPitch : &rowp->cursor;
    const unsigned long long add = static_cast<unsigned long long>(total) | (static_cast<unsigned long long>(btotal) << 32);
    const unsigned long long old = add ? atomicAdd(reinterpret_cast<unsigned long long*>(cur), add) : 0ull;
    const uint32_t off = static_cast<uint32_t>(old), boff = static_cast<uint32_t>(old >> 32);
    sh_off = off;
    sh_boff = boff;
    if constexpr (!PAGED) {
      ws.desc[sc.chunk_base + c] = make_uint2(run_base + off, total);
      if (banded) ws.desc2[sc.chunk_base + c] = make_uint2(brun_base + boff, atotal | (btotal << 13));
    }
    if (atotal) atomicAdd(runs ? cur + kCursorAboveWord : &rowp->above, atotal);  // nobody waits for it
  }
  __syncthreads();
  const uint32_t off = sh_off, boff = sh_boff;
  if (PAGED && lane == 0 && c < geo.num_chunks) {  // a quarter has a segment of its own
    const size_t at = (sc.chunk_base + c) * kWaves + quarter.part;
    ws.desc[at] = make_uint2(run_base + off + before, cnt);
    if (banded) ws.desc2[at] = make_uint2(brun_base + boff + bbefore, above_w | (band_w << 13));
  }
  if (off + total > run_cap) return;  // the list has overflowed and will not be used (nor will the band)
  const bool band_fits = boff + btotal <= brun_cap;  // else the band has overflowed and will not be used
  uint2* dst = ws.cand + sc.cand_base + run_base + off + before;
  uint2* bdst = ws.band + sc.band_base + brun_base + boff + bbefore;
  uint32_t bat = 0;  // band entries of this quarter written so far
  if (cnt <= static_cast<uint32_t>(kStageQ)) {
    for (uint32_t q0s = 0; q0s < cnt; q0s += 64) {
      const uint32_t q = q0s + lane;
      uint2 en = make_uint2(0u, 0u);
      if (q < cnt) {
        en = stage[q];
        dst[q] = en;
      }
      if (band_w && band_fits) {  // wave-uniform
        const uint32_t key = key_of_bits(en.y);
        const bool inb = q < cnt && key >= blo && key < bhi;
        const uint64_t bb = ballot64(inb);
        if (inb) {
          bdst[bat + count_below(bb)] = en;
          atomicAdd(&bh[band_slot(band_bucket(key - blo, bmul), bmany, brot)], 1u);  // the row's bucket histogram; nobody waits for it
        }
        bat += popc64(bb);
      }
    }
  } else {
    // more candidates than the staging area holds: the quarter's (already stored) values are read again
    uint32_t at = 0;
    for (int u = 0; u < kLeanRounds; ++u) {
      const uint32_t j = q0 + u * 256 + lane * 4;
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (j < d) x = *reinterpret_cast<const float4*>(er + j);
      const uint32_t bits[4] = {__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z), __float_as_uint(x.w)};
      bool flag[4], inb[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t key = key_of_bits(bits[s]);
        flag[s] = j + s < d && key >= cand_lo;
        inb[s] = j + s < d && key >= blo && key < bhi;
      }
      const RoundRank rr = rank_round(flag);
      uint32_t pos = at + rr.below;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (flag[s]) {
          if (pos < cnt) dst[pos] = make_uint2(j + s, bits[s]);
          ++pos;
        }
      at += rr.total;
      if (band_w && band_fits) {  // wave-uniform
        const RoundRank br = rank_round(inb);
        uint32_t bpos = bat + br.below;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (inb[s]) {
            if (bpos < band_w) {
              bdst[bpos] = make_uint2(j + s, bits[s]);
              atomicAdd(&bh[band_slot(band_bucket(key_of_bits(bits[s]) - blo, bmul), bmany, brot)], 1u);
            }
            ++bpos;
          }
        bat += br.total;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The window of keys in which the next step's threshold is expected, from this step's threshold key `tau` and the
// one before (0: none).  The keys of positive floats order as the floats do, so the window is set in float
// arithmetic.  Training thresholds drift smoothly while the residuals build up (+34 %, +17 %, +10 %, +7.5 % ... over
// the first steps of the ResNet-18-shaped workload, +2 % at step ten): with d1 the last relative change and d0 the
// one before, a drift that is dying down (same sign, |d1| < |d0|) is taken to go on doing so, next = d1 * d1 / d0
// (not below d1 / 4), and to be off by at most half of what that took away from d1; changes of opposite signs are
// scatter about a level, next = 0, unsure by 0.7 of the larger one; a drift that grows is extrapolated flat, next = d1,
// unsure by 0.4 |d1| + |d1 - d0|.  The centre is tau (1 + next), the half-width
// 0.4 % + unsure + `noise`, an allowance for the scatter of the k-th largest of a sample from step to step.  With B
// entries found in a window of relative width w around the threshold, one entry more or fewer above a level moves the
// k-th largest key by w / B of its value and the count above a level scatters by about sqrt(k): k_topk_band passes 8 w
// sqrt(k) / B (the extrapolation more than doubles the scatter, and three times the result is allowed for); where no
// window has been looked at yet, 1.5 / sqrt(k) stands in (as if a fourteenth of the kept entries lay within one per cent
// of the threshold).  It only decides which route the next step takes, never a result.  guess_valid / guess: the bucket
// guess the next first pass will use; the window must lie at or above it so that every band entry is also a candidate.
// ---------------------------------------------------------------------------------------------
// A step's list held n entries, every key from list_from upwards; the guess for the next step may lie below that, where
// nothing is known, and is taken to add at most as many again.  Where even that would not leave room to spare, the key
// that a list without a window should start at: the present list's first (0: the guess's own).
__device__ __forceinline__ uint32_t known_from(uint32_t guess, uint32_t list_from, uint32_t n, uint32_t cap) {
  return (guess << kL0Shift) < list_from && n > cap / 4 ? list_from : 0u;
}

__device__ __forceinline__ float default_band_noise(uint32_t k) { return 1.5f / sqrtf(static_cast<float>(k)); }

__device__ __forceinline__ bool normal_key(uint32_t key) { return key >= 0x00800000u && key < 0x7f000000u; }

// Below the band's lower end lies a margin of half its half-width, at most 2 %: the candidate list starts there, so
// that a threshold just below the band (two steps in a hundred on the ResNet-18 and ResNet-50 shapes) is still in the
// list and costs the general kernels' sweeps (50 us), not two more reads of every row (470 us).  (Without the limit the
// wide windows of a run's first steps make lists so long that the next step is given no guess.)

// known_from: where no window follows, the next list starts there if that is above the guess's first key (see known_from()).
__device__ __forceinline__ void set_next_band(TopkRow* rowp, uint32_t tau, uint32_t tau_prev, uint32_t tau_prev2,
                                              uint32_t guess_valid, uint32_t guess, uint32_t known_from, float noise,
                                              uint32_t k, const TopkOptions& opt) {
  uint32_t valid = 0, lo = 0, hi = 0;
  uint32_t from = guess << kL0Shift;  // the first key that the next first pass lists
  float delta_set = 0.0f;
  if (guess_valid && opt.band && opt.band_cap && normal_key(tau)) {
    const float t1 = __uint_as_float(tau);
    float d1 = 0.0f;  // the last relative change of the threshold
    if (normal_key(tau_prev)) d1 = fminf(fmaxf(t1 / __uint_as_float(tau_prev), 0.5f), 2.0f) - 1.0f;
    float next = d1, unsure = 0.4f * fabsf(d1);  // the change expected next, and how far off that may be
    if (normal_key(tau_prev) && normal_key(tau_prev2)) {
      const float d0 = fminf(fmaxf(__uint_as_float(tau_prev) / __uint_as_float(tau_prev2), 0.5f), 2.0f) - 1.0f;
      if (d0 * d1 > 0.0f && fabsf(d1) < fabsf(d0)) {  // a drift that is dying down: let it go on doing so
        next = d1 * fmaxf(d1 / d0, 0.25f);
        unsure = 0.5f * fabsf(d1 - next);
      } else if (d0 * d1 <= 0.0f) {  // scatter about a level that stands still
        next = 0.0f;
        unsure = 0.7f * fmaxf(fabsf(d1), fabsf(d0));
      } else {
        unsure += fabsf(d1 - d0);
      }
    }
    const float delta = fminf(0.004f + unsure + fminf(fmaxf(noise, 0.0005f), 0.25f), 0.25f);
    delta_set = delta;
    const float centre = t1 * (1.0f + next);
    const float flo = centre * (1.0f - delta), fhi = centre * (1.0f + delta);
    lo = __float_as_uint(flo);
    hi = __float_as_uint(fhi);
    const uint32_t floor_key = guess << kL0Shift;
    if (lo < floor_key) lo = floor_key;
    valid = (hi < 0x7f800000u && hi > lo && lo >= 0x00800000u) ? 1u : 0u;
    const uint32_t margin = __float_as_uint(centre * (1.0f - delta - fminf(0.5f * delta, 0.02f)));
    if (valid && margin > from) from = margin;
  }
  if (!valid && known_from > from) from = known_from;
  rowp->cand_from = guess_valid ? from + 1u : 0u;
  // Buckets of the window's histogram: the population of the last window (noise is 8 w sqrt(k) / B) says how many
  // entries this one will hold; beyond 16 to a bucket of the few it gets the many.
  const bool many = band_buckets(k) == kBandBucketsMany &&
                    16.0f * delta_set * sqrtf(static_cast<float>(k)) > 16.0f * kBandBucketsFew * noise;
  rowp->band_valid = valid ? (many ? kBandMany : kBandFew) : 0u;
  rowp->band_lo = lo;
  rowp->band_hi = hi;
  rowp->band_mul = valid ? band_multiplier_dev(hi - lo, many ? kBandBucketsMany : kBandBucketsFew) : 0u;
}

// The kernels that select in one launch end in one workgroup's chain, of which the above (divisions and roots, one after
// the other) was 1 to 1.5 us: they leave what it needs in the control block, and a workgroup of the last kernel goes
// through it beside the others' work, one more than there are chunks (a step of 4 x 65536, k = 655: 24.3 us, with that
// and the ranking of k_topk_pick 23.2; 16 x 1 M 70.4, now 69.6).  Top-k inside blocks: a wavefront of every problem's
// first chunk; in whole rows that kept the first chunk 0.4 us longer, in every step (4 x 65536 23.26 us a step, now
// 23.13).
// Only where there is a lane of a wavefront for every row: more of them keep its compute unit busy, 1.4 us for every 64,
// while in the selecting kernel every row has a workgroup of its own (us, all rows in the selecting kernel / in the last
// one: a step of 32 x 600000 75.4 / 74.6, 24 x 300000 49.5 / 48.9, 64 x 100000 59.7 / 59.1, 64 x 4096 43.4 / 43.7, 300 x
// 4096 134.7 / 140.8, 4000 x 4096 1547 / 1640; the workers' half 300 x 4096 27.2 / 33.8, 4000 x 4096 120 / 218).
// population: entries of the window lo .. hi that was looked at (0: none), ref: a key in it.
__host__ __device__ __forceinline__ bool window_later(uint32_t n) { return n <= 64; }
__device__ __forceinline__ float population_noise(uint32_t population, uint32_t lo, uint32_t hi, uint32_t ref, uint32_t k) {
  return population ? 8.0f * ((__uint_as_float(hi) - __uint_as_float(lo)) / __uint_as_float(ref)) * sqrtf(static_cast<float>(k)) /
                          static_cast<float>(population)
                    : default_band_noise(k);
}
__device__ __forceinline__ void leave_next(TopkRow* rowp, uint32_t n, uint32_t k, const TopkOptions& opt, uint32_t valid, uint32_t guess,
                                           uint32_t known, uint32_t tau, uint32_t tau_prev, uint32_t tau_prev2, uint32_t population,
                                           uint32_t lo, uint32_t hi, uint32_t ref) {
  rowp->b_guess = guess;
  if (!window_later(n)) {
    set_next_band(rowp, tau, tau_prev, tau_prev2, valid, guess, known, population_noise(population, lo, hi, ref, k), k, opt);
    return;
  }
  rowp->next = valid ? kNextGuess : kNextNone;
  rowp->known_from = known;
  rowp->next_prev2 = tau_prev2;
  rowp->next_population = population;
  rowp->next_ref = ref;
}
__device__ __forceinline__ void set_next(TopkRow* rowp, uint32_t k, const TopkOptions& opt) {
  const uint32_t next = rowp->next, lo = rowp->band_lo, hi = rowp->band_hi, population = rowp->next_population;
  if (next == kNextSet) return;
  rowp->next = kNextSet;
  set_next_band(rowp, rowp->tau, rowp->tau_prev, rowp->next_prev2, next == kNextGuess ? 1u : 0u, rowp->b_guess, rowp->known_from,
                population_noise(population, lo, hi, rowp->next_ref, k), k, opt);
}

// The runs of a problem's band list, from the high halves of the cursors the first pass advanced.
__device__ __forceinline__ ListRuns band_runs_from_cursors(const TopkWorkspace& ws, const TopkRow* rowp,
                                                           uint32_t cursor_set, uint32_t cap) {
  ListRuns L;
  L.total = 0;
  L.fits = true;
  if (cursor_set != kNoCursorSet) {  // uniform
    L.lists = kSubLists;
    L.pitch = cap / kSubLists;
    const uint32_t* cur = ws.xcur + static_cast<size_t>(cursor_set) * kSubLists * kCursorPitch;
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s) {
      L.n[s] = cur[s * kCursorPitch + 1];
      L.total += L.n[s];
      L.fits = L.fits && L.n[s] <= L.pitch;
    }
  } else {
    L.lists = 1;
    L.pitch = 0;
    L.n[0] = rowp->cursor_band;
#pragma unroll
    for (uint32_t s = 1; s < kSubLists; ++s) L.n[s] = 0;
    L.total = L.n[0];
    L.fits = L.n[0] <= cap;
  }
  return L;
}

// How a wavefront that takes up to `chunks` (1 .. 8) chunks at a time shares its lanes out among their segments, `parts`
// (one or four) to a chunk: every segment has the same number of lanes, which take its entries in turn, so that the
// segments of all the chunks are requested together however short they are.
struct SegmentLanes {
  uint32_t lanes;    // lanes per segment
  uint32_t segment;  // the lane's, counted from the group's first
  uint32_t chunk;    // ... and its chunk
  uint32_t sub;      // the lane's number among those of the segment
  uint32_t share;    // lanes per chunk
  bool first;        // it is the first lane of its chunk
};
__device__ __forceinline__ SegmentLanes segment_lanes(uint32_t chunks, uint32_t parts) {
  // (powers of two: shifts, as what follows waits for the result before it can ask for anything)
  const uint32_t lane = lane_id(), chunk_shift = chunks > 1u ? __builtin_clz(chunks - 1u) - 26u : 6u;
  const uint32_t shift = parts > 1u ? chunk_shift - 2u : chunk_shift;
  SegmentLanes s;
  s.lanes = 1u << shift;
  s.segment = lane >> shift;
  s.chunk = lane >> chunk_shift;
  s.sub = lane & (s.lanes - 1u);
  s.share = 1u << chunk_shift;
  s.first = (lane & (s.share - 1u)) == 0;
  return s;
}
// Sum over the lanes of a chunk.
__device__ __forceinline__ uint32_t chunk_sum(uint32_t v, const SegmentLanes& s) {
  for (uint32_t o = 1; o < s.share; o <<= 1) v += __shfl_xor(v, o, 64);  // uniform
  return v;
}

// ---------------------------------------------------------------------------------------------
// The selection in one launch, for problems whose threshold key falls inside the band the first pass was given.
// Same geometry as the counting kernel: a workgroup owns a contiguous block of geo.count_cpw chunks.
//   1. Every workgroup of a problem reads the problem's bucket histogram of band entries (2048 or 8192 counts,
//      added up by the first pass) and the count A of entries at or above the band, and finds by itself the
//      bucket that holds the k-th largest key: it exists iff A < k <= A + (entries in the band); both lists must
//      have fitted and the bucket must hold at most kBoundaryCap entries.  Otherwise the problem is left to the
//      general kernels that follow.  All workgroups of a problem read the same data and decide alike.
//   2. Per chunk: kept for certain = entries at or above the band + band entries in a bucket above the threshold's;
//      the workgroup leaves these counts with their prefixes inside the block, and the block's total, in the
//      tables the last kernel reads (the "equal to tau" columns stay 0).  Band entries in the threshold's bucket
//      are gathered in a small array of the problem.
//   3. The last workgroup of the problem to finish ranks the gathered entries by (key descending, coordinate
//      ascending): the first k - (entries above the bucket) of them are kept, the last of those holds tau;
//      an entry anywhere is kept iff key > tau, or key == tau and coordinate <= tie_last.  The coordinates of
//      the kept ones, ascending, let the last kernel add them to the positions of the chunks after them.
//      It also leaves what the next step's guess and band follow from (leave_next) and clears the histogram.
// ---------------------------------------------------------------------------------------------
template <bool UNI, bool QUARTERS>
__global__ __launch_bounds__(kWG) void k_topk_band(Geometry geo, TopkWorkspace ws, TopkOptions opt, uint32_t use_guess) {
  __shared__ uint32_t suf[kWG / 64];
  __shared__ uint32_t out3[3];
  __shared__ uint32_t l_gt[kMaxCountCpw];
  __shared__ uint32_t scratch[kWG / 64 + 1];
  __shared__ uint32_t sh_flag;
  __shared__ uint2 b_en[kBoundaryCap];
  __shared__ uint32_t b_rank[kBoundaryCap];
  const SegCtx sc = seg_ctx<UNI, kClassCount>(geo, opt, ws);
  const uint32_t row = sc.seg, t = threadIdx.x;
  const uint32_t cpw = geo.count_cpw, nc = geo.num_chunks, k = geo.k;
  const uint32_t start = sc.group * cpw;
  if (start >= nc) return;  // uniform; the grid has exactly the blocks that exist
  const uint32_t end = start + cpw < nc ? start + cpw : nc;
  TopkRow* rowp = ws.rows + row;
  uint32_t* bh = ws.bhist + sc.bhist_base;
  const uint32_t wave = uniform_u32(t >> 6), lane = lane_id();
  // A wavefront takes up to eight chunks at a time: all its lanes the entries of one after the other, or, where a chunk
  // has a segment for every quarter, the lanes shared out among the segments (SegmentLanes).  (Shared out also where
  // there is one segment to a chunk, this kernel took, us: blocks of 12 x 60000 13.8 -> 15.5, 16 x 733 chunks 13.8 ->
  // 15.9.) Everything that can be asked for before anything is known goes out together (a workgroup's work is a chain of
  // round trips otherwise): the control block and the cursors, the bucket histogram, the counts above the band, the first
  // descriptors.
  constexpr int kGroup = 8;  // chunks a wavefront takes at a time, at most
  constexpr uint32_t kParts = QUARTERS ? kWaves : 1;
  const uint2* d2 = ws.desc2 + sc.chunk_base * kParts;
  const uint32_t group = chunks_per_wave(cpw);
  const uint32_t c_first = start + wave * group;
  const SegmentLanes sl = segment_lanes(kGroup, kParts);  // (quarters: group is eight)
  auto descriptor = [&](uint32_t c0) {
    const bool mine = QUARTERS ? c0 + sl.chunk < end : lane < group && c0 + lane < end;
    return mine ? d2[c0 * kParts + (QUARTERS ? sl.segment : lane)] : make_uint2(0, 0);
  };
  uint2 ds = make_uint2(0, 0);
  if (opt.band) ds = descriptor(c_first);  // (no such table without a band)
  // (thread t's buckets are consecutive: 8 of the few, 32 of the many, of which the first 8 lie where the few do and the
  // others are asked for below, with the band entries)
  constexpr uint32_t kQuadsFew = kBandBucketsFew / kWG / 4, kQuadsMany = kBandBucketsMany / kWG / 4;
  uint4 x[kQuadsMany];
  const uint32_t rot = band_rotation(k, row);
  const uint4* bh4 = reinterpret_cast<const uint4*>(bh) + t * kQuadsFew;
#pragma unroll
  for (uint32_t i = 0; i < kQuadsMany; ++i)
    x[i] = i < kQuadsFew ? bh4[rot * (kBandBucketsFew / 4) + i] : make_uint4(0, 0, 0, 0);
  uint32_t total_above = rowp->above;
  if (sc.cursor_set != kNoCursorSet) {
    total_above = 0;
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s)
      total_above += ws.xcur[(static_cast<size_t>(sc.cursor_set) * kSubLists + s) * kCursorPitch + kCursorAboveWord];
  }
  const uint32_t blo = rowp->band_lo, bhi = rowp->band_hi, bmul = rowp->band_mul, bg = rowp->b_guess;
  const uint32_t list_from = rowp->cand_from - 1u;  // (with a candidate list)
  const uint32_t tau_before = rowp->tau, tau_before2 = rowp->tau_prev;  // the last two threshold keys (asked for
                                                                       // here: the last workgroup needs them)
  const ListRuns cand = runs_from_cursors(ws, rowp, sc.cursor_set, opt.cap);
  const ListRuns band = band_runs_from_cursors(ws, rowp, sc.cursor_set, opt.band_cap);
  // all of it was written by earlier launches: the same for every workgroup of the problem
  const bool banded = use_guess && opt.band && !opt.force_dense && rowp->cand_from != 0 && rowp->band_valid != 0;
  const bool many = rowp->band_valid == kBandMany;
  const uint32_t buckets = many ? kBandBucketsMany : kBandBucketsFew;
  uint32_t* bh_used = many ? bh : bh + rot * kBandBucketsFew;
  const uint32_t per_quads = many ? kQuadsMany : kQuadsFew;  // uniform
  // What the window's population says of the threshold's scatter, also where this route is not taken.
  auto noise = [&] {
    return banded && bhi > blo && band.total ? 8.0f * ((__uint_as_float(bhi) - __uint_as_float(blo)) / __uint_as_float(blo)) *
                                                   sqrtf(static_cast<float>(k)) / static_cast<float>(band.total)
                                             : 0.0f;
  };
  if (!(banded && cand.fits && band.fits && bhi > blo)) {
    // Not this route.  The first pass may still have counted (lists that did not fit): one workgroup clears the
    // problem's histogram and counters; nobody of this launch makes use of them.
    if (sc.group == 0) {
      if (banded)
        for (uint32_t b = t; b < buckets; b += kWG) bh_used[b] = 0;
      if (t == 0) {
        rowp->fast = kFastNot;
        rowp->noise = noise();
        rowp->above = 0;
        if (sc.cursor_set != kNoCursorSet)
          for (uint32_t s = 0; s < kSubLists; ++s)
            ws.xcur[(static_cast<size_t>(sc.cursor_set) * kSubLists + s) * kCursorPitch + kCursorAboveWord] = 0;
        uint32_t* cn = ws.counters + row * kCountersPerRow;
        cn[4] = 0;
        cn[5] = !banded ? 1u : (!cand.fits ? 2u : 3u);  // no band was set; the candidate list / the band list overflowed
        rowp->phase = kPhaseLevel0;
        ws.flags[0] = 1;  // work for the general kernel
      }
    }
    return;
  }
  // the band entries of this wavefront's first chunks: requested before the histogram is looked at
  const uint2* bandr = ws.band + sc.band_base;
  uint2 a[kGroup];   // the first 64 entries of every chunk's segment, or (quarters) a lane's first entries of its segment
  uint32_t cnt = 0;  // entries of the lane's segment
  uint32_t chunk_off[kGroup], chunk_cnt[kGroup];  // one segment to a chunk: wave-uniform
  auto request = [&](uint32_t q0) {
    if constexpr (QUARTERS) {
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const uint32_t q = q0 + u * sl.lanes + sl.sub;
        a[u] = q < cnt ? bandr[ds.x + q] : make_uint2(0, 0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        chunk_off[u] = __builtin_amdgcn_readlane(ds.x, u);
        chunk_cnt[u] = __builtin_amdgcn_readlane(cnt, u);
        a[u] = lane < chunk_cnt[u] ? bandr[chunk_off[u] + lane] : make_uint2(0, 0);
      }
    }
  };
  auto take = [&] {
    cnt = (ds.y >> 13) & 0x1fffu;
    if (ds.x > opt.band_cap) cnt = 0;  // segments always lie inside the list; never read outside it
    else if (cnt > opt.band_cap - ds.x) cnt = opt.band_cap - ds.x;
    request(0);
  };
  if (many) {  // uniform
#pragma unroll
    for (uint32_t i = kQuadsFew; i < kQuadsMany; ++i) x[i] = bh4[((i / kQuadsFew + rot) & 3u) * (kBandBucketsFew / 4) + i % kQuadsFew];
  }
  take();
  // ---- 1. the bucket of the threshold key: the thread whose buckets the count from the top crosses finds it ----
  bool inside = total_above < k && k - total_above <= band.total;  // uniform
  const uint32_t miss = total_above >= k ? 4u : (inside ? 6u : 5u);  // the threshold lies above / below the band; or (6) ...
  uint32_t bstar = 0, need = 0, n_boundary = 0;
  if (inside) {
    const uint32_t want = k - total_above;
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t i = 0; i < kQuadsMany; ++i) mine += x[i].x + x[i].y + x[i].z + x[i].w;
    uint32_t from_here = mine;  // entries in this thread's buckets and those of the threads above it
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_down(from_here, o, 64);
      if (lane + o < 64) from_here += up;
    }
    if (lane == 0) suf[wave] = from_here;
    if (t < 3) out3[t] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w)
      if (w > wave) from_here += suf[w];
    uint32_t above = from_here - mine;
    if (from_here >= want && above < want) {  // exactly one thread
      bool found = false;
      auto look = [&](uint32_t count, uint32_t bucket) {
        if (found) return;
        if (above + count >= want) {
          found = true;
          out3[0] = bucket;
          out3[1] = above;
          out3[2] = count;
        } else {
          above += count;
        }
      };
#pragma unroll
      for (int i = static_cast<int>(kQuadsMany) - 1; i >= 0; --i) {
        if (i >= static_cast<int>(kQuadsFew) && !many) continue;  // uniform
        const uint32_t first = (t * per_quads + i) * 4;
        look(x[i].w, first + 3);
        look(x[i].z, first + 2);
        look(x[i].y, first + 1);
        look(x[i].x, first);
      }
    }
    __syncthreads();
    bstar = out3[0];
    need = want - out3[1];       // how many entries of bucket bstar are kept: 1 <= need <= out3[2]
    n_boundary = out3[2];
    inside = n_boundary <= kBoundaryCap;
  }
  // ---- 2. per chunk: entries kept for certain; the threshold bucket's entries are gathered ----
  if (inside) {
    uint2* bnd = ws.bnd + static_cast<size_t>(row) * kBoundaryCap;
    for (uint32_t c0 = c_first; c0 < end; c0 += kWaves * group) {
      if (c0 != c_first) {  // wave-uniform
        ds = descriptor(c0);
        take();
      }
      auto gather = [&](bool at, const uint2& en) {
        if (!at) return;
        const uint32_t slot = atomicAdd(&rowp->bnd_n, 1u);
        if (slot < kBoundaryCap) {  // always: the histogram counted these entries
          __hip_atomic_store(&bnd[slot].x, en.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&bnd[slot].y, en.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      };
      if constexpr (QUARTERS) {
        uint32_t gt = sl.sub == 0 ? ds.y & 0x1fffu : 0u;  // this lane's part of the chunk's count
        for (uint32_t q0 = 0; ballot64(q0 < cnt) != 0; q0 += kGroup * sl.lanes) {
          if (q0) request(q0);
#pragma unroll
          for (int u = 0; u < kGroup; ++u) {
            const bool ok = q0 + u * sl.lanes + sl.sub < cnt;
            const uint32_t bucket = band_bucket(key_of_bits(a[u].y) - blo, bmul);
            gt += ok && bucket > bstar ? 1u : 0u;
            gather(ok && bucket == bstar, a[u]);
          }
        }
        gt = chunk_sum(gt, sl);
        if (sl.first && c0 + sl.chunk < end) l_gt[c0 - start + sl.chunk] = gt;
      } else {
        uint32_t mine = 0;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
          uint32_t gt = 0;  // wave-uniform
          for (uint32_t q = 0; q < chunk_cnt[u]; q += 64) {  // one trip unless the chunk holds more than 64 band entries
            const bool ok = q + lane < chunk_cnt[u];
            const uint2 en = q == 0 ? a[u] : (ok ? bandr[chunk_off[u] + q + lane] : make_uint2(0, 0));
            const uint32_t bucket = band_bucket(key_of_bits(en.y) - blo, bmul);
            gt += popc64(ballot64(ok && bucket > bstar));
            gather(ok && bucket == bstar, en);
          }
          if (lane == static_cast<uint32_t>(u)) mine = gt;
        }
        if (lane < group && c0 + lane < end) l_gt[c0 - start + lane] = (ds.y & 0x1fffu) + mine;
      }
    }
    __syncthreads();
    // exclusive prefixes within the block: thread t takes `per` consecutive chunks
    const uint32_t len = end - start;
    const uint32_t per = (cpw + kWG - 1) / kWG;  // <= kMaxCountCpw / kWG
    const uint32_t first = t * per;
    uint32_t sum_gt = 0;
    for (uint32_t i = 0; i < per; ++i)
      if (first + i < len) sum_gt += l_gt[first + i];
    uint32_t tot_gt;
    uint32_t pre_gt = block_excl_scan<kWG>(sum_gt, scratch, &tot_gt);
    uint4* rec = ws.chunk_rec + sc.chunk_base + start;
    for (uint32_t i = 0; i < per; ++i)
      if (first + i < len) {
        const uint32_t g = l_gt[first + i];
        rec[first + i] = make_uint4(g, 0u, pre_gt, 0u);
        pre_gt += g;
      }
    if (t == 0) {  // (device-scope stores: the problem's last workgroup adds the blocks' totals up)
      uint2* tot = ws.blk + static_cast<size_t>(row) * kMaxCountBlocks + sc.group;
      __hip_atomic_store(&tot->x, tot_gt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&tot->y, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // ---- 3. the problem-wide part, by whichever of its workgroups finishes last ----
  if (!last_group_of_row(&rowp->ticket_band, sc.groups, &sh_flag)) return;
  for (uint32_t b = t; b < buckets; b += kWG) bh_used[b] = 0;  // every workgroup has read it
  if (inside) {
    // the gathered entries (written by other workgroups with device-scope stores: read at that scope)
    const uint2* bnd = ws.bnd + static_cast<size_t>(row) * kBoundaryCap;
    const AgentView view = agent_view(reinterpret_cast<const uint32_t*>(bnd), 2 * kBoundaryCap);
    // ... and with the same round trip the blocks' totals, for their prefix sums: the last kernel then needs one
    // number per worker and chunk instead of a sum over all the blocks before the chunk's
    static_assert(kMaxCountBlocks <= kWG, "a thread per count block");
    const AgentView totals = agent_view(reinterpret_cast<const uint32_t*>(ws.blk + static_cast<size_t>(row) * kMaxCountBlocks),
                                        2 * kMaxCountBlocks);
    const uint32_t my_total = t < sc.groups ? load_agent(totals, 2 * t) : 0u;
    if (t < kBoundaryCap) {
      uint2 en = make_uint2(0xffffffffu, 0u);
      if (t < n_boundary) en = make_uint2(load_agent(view, 2 * t), load_agent(view, 2 * t + 1));
      b_en[t] = en;
    }
    uint32_t all_totals;
    const uint32_t blocks_before = block_excl_scan<kWG>(my_total, scratch, &all_totals);  // (barriers of its own)
    // rank by (key descending, coordinate ascending): coordinates are distinct, so ranks are
    bool kept = false;
    uint32_t my_key = 0, my_coord = 0xffffffffu;
    if (t < n_boundary) {
      my_key = key_of_bits(b_en[t].y);
      my_coord = b_en[t].x;
      uint32_t rank = 0;
      for (uint32_t q = 0; q < n_boundary; ++q) {
        const uint32_t kq = key_of_bits(b_en[q].y), cq = b_en[q].x;
        rank += (kq > my_key || (kq == my_key && cq < my_coord)) ? 1u : 0u;
      }
      kept = rank < need;
      if (rank == need - 1) { out3[0] = my_key; out3[1] = my_coord; }  // the last kept one: tau and the last tie taken
    }
    __syncthreads();
    const uint32_t tau = out3[0], last_coord = out3[1];
    // ties, and the kept entries' coordinates in ascending order
    if (t < kBoundaryCap) b_rank[t] = 0xffffffffu;
    __syncthreads();
    uint32_t is_tie = 0;
    if (t < n_boundary) {
      is_tie = my_key == tau ? 1u : 0u;
      if (kept) {
        uint32_t pos = 0;
        for (uint32_t q = 0; q < n_boundary; ++q) {
          const uint32_t kq = key_of_bits(b_en[q].y), cq = b_en[q].x;
          const bool kept_q = kq > tau || (kq == tau && cq <= last_coord);
          pos += (kept_q && cq < my_coord) ? 1u : 0u;
        }
        b_rank[pos] = my_coord;
      }
    }
    __syncthreads();
    static_assert(kBoundaryCap <= 64, "the first wavefront holds all of it");
    if (wave == 0) {
      const uint32_t ties = popc64(ballot64(is_tie != 0));
      const uint32_t ties_in = popc64(ballot64(is_tie != 0 && my_coord <= last_coord));
      if (lane == 0) { suf[0] = ties; suf[1] = ties_in; }
    }
    __syncthreads();
    const uint32_t n_ties = suf[0];
    uint32_t* sel = ws.bnd_sel + static_cast<size_t>(row) * kBoundaryCap;
    if (t < kBoundaryCap) sel[t] = b_rank[t];
    if (t < sc.groups) {
      const uint32_t block_lo = t * cpw * kChunk;  // (below d: 32 bits hold it)
      uint32_t kept_before = 0;
      for (uint32_t q = 0; q < need; ++q) kept_before += b_rank[q] < block_lo ? 1u : 0u;
      ws.blk_prefix[static_cast<size_t>(row) * kMaxCountBlocks + t] = make_uint2(blocks_before, kept_before);
    }
    if (t == 0) {
      // ties kept: those at coordinates <= last_coord; all of them if the last tie is kept
      const uint32_t ties_kept = suf[1], ties_after = n_ties - ties_kept;
      const uint32_t tau_prev = tau_before;
      rowp->fast = kFastBand;
      rowp->level1_done = 1;
      rowp->mode = kModeCand;
      rowp->n_src = cand.total;
      rowp->tau_prev = tau_prev;
      rowp->tau = tau;
      rowp->r = ties_kept;
      rowp->ties = n_ties;
      rowp->tie_last = ties_after ? last_coord : 0xffffffffu;
      ws.tau[row] = tau;
      ws.count_gt[row] = k - ties_kept;
      uint32_t* cn = ws.counters + row * kCountersPerRow;
      cn[0] = 0;
      cn[1] = cand.total;
      cn[2] = n_ties;
      cn[3] = ties_kept;
      cn[4] = band.total;
      cn[5] = 0;
      // Guess for the next step, as the general route sets it but from what is known here: the candidate list held
      // cand.total entries, every key from a key of bucket bg or above upwards.  Below that nothing is known: the bucket
      // below bg is taken to hold at most as many again, what bg itself holds below the list is left to known_from().
      const uint32_t b0 = tau >> kL0Shift;  // >= bg
      uint32_t valid = 0, guess = 0;
      if (opt.predict) {
        const uint32_t bound = b0 > bg ? cand.total : 2u * cand.total;  // entries from bucket b0 - 1 upwards
        if (b0 && bound <= opt.cap / 2) { valid = 1; guess = b0 - 1; }
        else if (cand.total <= opt.cap / 2) { valid = 1; guess = b0; }
      }
      leave_next(rowp, geo.n, k, opt, valid, guess, known_from(guess, list_from, cand.total, opt.cap), tau, tau_prev, tau_before2,
                 band.total, blo, bhi, blo);
    }
  } else if (t == 0) {
    rowp->fast = kFastNot;
    rowp->noise = noise();
    uint32_t* cn = ws.counters + row * kCountersPerRow;
    cn[4] = 0;
    cn[5] = miss;  // (6): ... its bucket holds more entries than are ranked here
    rowp->phase = kPhaseLevel0;
    ws.flags[0] = 1;  // work for the general kernel
  }
  if (t == 0) {
    rowp->above = 0;
    rowp->bnd_n = 0;
    if (inside) {  // the cursors go back to zero for the next step (else the general kernels still read them)
      rowp->cursor = 0;
      rowp->cursor_band = 0;
    }
    if (sc.cursor_set != kNoCursorSet) {
      for (uint32_t s = 0; s < kSubLists; ++s) {
        uint32_t* cur = ws.xcur + (static_cast<size_t>(sc.cursor_set) * kSubLists + s) * kCursorPitch;
        if (inside) { cur[0] = 0; cur[1] = 0; }
        cur[kCursorAboveWord] = 0;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The whole selection of a short row (at most kPickChunks chunks) by one workgroup: it takes the place of the band
// kernel and of the general route's four, whose launches and row-wide steps cost a short row more than its bytes (4 rows
// of 65536 coordinates: band 11.0 us and four launches of 1.3 to 2.6 us that return at once -> 9.9 us; the whole pass
// 31.0 -> 24.2).
//   1. Elements: the candidate list if the guess held, else the row's stored values, chunk after chunk.  The first trip of
//      four per thread stays in registers; what goes beyond is read again in every sweep, four trips requested together.
//   2. The bucket that holds the k-th largest key, by histograms of kPickBins buckets in LDS, each over the bucket the
//      one before found: from a list, buckets of a thousandth of an octave from the list's lower end upwards, so that
//      the first one usually leaves a handful of entries (key bits from the top, as for a row, would put a list's keys
//      into a few buckets, on which the LDS atomics queue).
//   3. At most kPickRank entries left: they are ranked by (key descending, coordinate ascending), up to 64 of them by every
//      wavefront for itself, without a barrier in between (4 rows of 65536: 2.7 us of the kernel's 9.7, now 1.8).  More can
//      only be equal keys: the last tie to take is found by the same histograms over the coordinates.
//   4. Per chunk the entries kept, and their prefix over the row, for the last kernel; what the next step's guess and window
//      follow from (leave_next).
// Where the line lies (whole step in us, 4 rows, the general kernels / this one): k = d / 100 16 chunks 30.6 / 24.6, 32
// chunks 30.8 / 28.6, 48 chunks 31.1 / 33.7; k = d / 10 16 chunks 39.5 / 39.1, 20 chunks 40.1 / 42.9.  What bounds it is
// one compute unit's instructions, about 20 us for a sweep over 65536 coordinates.  A row whose list did not hold (a
// selection of half the row, magnitudes that are few and equal) still takes it: 4 x 65536, k = 32768 164 / 101, k = 19660
// of three magnitudes 198 / 170.  A step of which it is known beforehand that no row has a guess (the first of a context,
// prediction off) goes to the general kernels: 4 x 65536, k = 655 56 / 95.
// A row's window only narrows what the first pass lists (opt.band = kBandWindow); whether the threshold lay inside is
// counted as on the band route.
// ---------------------------------------------------------------------------------------------
constexpr int kPickThreads = 1024;
constexpr int kPickBins = 2048;
constexpr uint32_t kPickQuad = 4;    // elements of a thread per trip
constexpr uint32_t kPickRank = 256;  // (ranked by comparing all with all: a thousand of them take 27 us, one more sweep less)
constexpr uint32_t kPickCrowd = 16;

struct PickShared {
  uint32_t lh[kPickBins];
  uint32_t suf[kPickThreads + 1];
  uint32_t out2[2];
  uint2 rank_en[kPickRank];
  uint32_t chunk_cnt[kPickChunks];
  uint32_t count, ties, ties_in, tau, last, from0, from1, window, bucket;
};

// What the selection reads of a row's control block, all of it requested together.
struct PickRow {
  uint32_t n_cand, cand_from, b_guess, band_valid, band_lo, band_hi, band_mul, tau, tau_prev;
};

// LISTED: the row's elements are the entries of its candidate list, else the coordinates of the row.
template <bool LISTED>
__device__ __forceinline__ void pick_row(PickShared& sh, const float* __restrict__ e, const Geometry& geo,
                                         const TopkWorkspace& ws, const TopkOptions& opt, const SegCtx& sc,
                                         const PickRow& in_row, bool pred, const uint2 (&first)[kPickQuad]) {
  const uint32_t row = sc.seg, t = threadIdx.x, lane = lane_id();
  const uint32_t k = geo.k;
  TopkRow* rowp = ws.rows + row;
  const float* er = e + sc.elem_off;
  const uint2* candr = ws.cand + sc.cand_base;
  const uint32_t n_cand = in_row.n_cand, bg = in_row.b_guess;
  const uint32_t blo = in_row.band_lo, bhi = in_row.band_hi, bmul = in_row.band_mul, cand_lo = in_row.cand_from - 1u;
  const uint32_t tau_before = in_row.tau, tau_before2 = in_row.tau_prev;
  const bool windowed = pred && opt.band && in_row.band_valid != 0;
  const uint32_t count = LISTED ? n_cand : geo.d;
  // A trip takes kPickQuad elements of every thread: entries of the list 1024 apart, or (from the second trip on) a quad
  // of the row's coordinates; over the row it is a chunk.
  struct Trip { uint2 en[kPickQuad]; };
  constexpr uint32_t kTripElements = kPickQuad * kPickThreads;
  static_assert(kTripElements == kChunk, "a trip over the row is a chunk");
  auto number = [&](uint32_t q0, uint32_t u) { return LISTED ? q0 + u * kPickThreads + t : q0 + kPickQuad * t + u; };
  auto load = [&](uint32_t q0, Trip& to) {
    if constexpr (LISTED) {
#pragma unroll
      for (uint32_t u = 0; u < kPickQuad; ++u) to.en[u] = number(q0, u) < count ? candr[number(q0, u)] : make_uint2(0u, 0u);
    } else {
      const uint32_t j = number(q0, 0);
      const float4 x = j < count ? *reinterpret_cast<const float4*>(er + j) : make_float4(0.f, 0.f, 0.f, 0.f);
      to.en[0] = make_uint2(j, __float_as_uint(x.x));
      to.en[1] = make_uint2(j + 1, __float_as_uint(x.y));
      to.en[2] = make_uint2(j + 2, __float_as_uint(x.z));
      to.en[3] = make_uint2(j + 3, __float_as_uint(x.w));
    }
  };
  // The first trip stays in registers, elements 1024 apart also of the row: a row of a few hundred coordinates is then one
  // element of a thread (8 x 5 coordinates: 17.5 us a step as quads, 16.5 so; 8 x 100 20.8 / 19.4).
  Trip held;
#pragma unroll
  for (uint32_t u = 0; u < kPickQuad; ++u) {
    const uint32_t q = u * kPickThreads + t;
    held.en[u] = LISTED ? first[u] : q < count ? make_uint2(q, __float_as_uint(er[q])) : make_uint2(0u, 0u);
  }
  // visit(element, whether it exists, first element of the trip) for every element, whole wavefronts at a time
  auto sweep = [&](auto&& visit) {
    constexpr uint32_t kAhead = 4;  // trips requested together
#pragma unroll
    for (uint32_t u = 0; u < kPickQuad; ++u)
      if (u * kPickThreads < count) visit(held.en[u], u * kPickThreads + t < count, 0u);  // uniform
#pragma unroll 1
    for (uint32_t q0 = kTripElements; q0 < count; q0 += kAhead * kTripElements) {
      Trip trip[kAhead];
#pragma unroll
      for (uint32_t w = 0; w < kAhead; ++w)
        if (q0 + w * kTripElements < count) load(q0 + w * kTripElements, trip[w]);  // uniform
#pragma unroll
      for (uint32_t w = 0; w < kAhead; ++w)
        if (q0 + w * kTripElements < count) {
#pragma unroll
          for (uint32_t u = 0; u < kPickQuad; ++u)
            visit(trip[w].en[u], number(q0 + w * kTripElements, u) < count, q0 + w * kTripElements);
        }
    }
  };
  // One more in lh[b] for every lane with `in`.  Additions to one word are performed one after the other: a word that
  // kPickCrowd lanes or more share (equal magnitudes, zeros) is counted by a ballot.
  auto count_in = [&](bool in, uint32_t b) {
    uint64_t left = ballot64(in);
    while (left) {
      const uint32_t b0 = __builtin_amdgcn_readlane(b, __builtin_ctzll(left));
      const uint64_t same = ballot64(in && b == b0);
      if (popc64(same) < kPickCrowd) {
        if (in) atomicAdd(&sh.lh[b], 1u);
        break;
      }
      if (lane == 0) atomicAdd(&sh.lh[b0], popc64(same));
      in = in && b != b0;
      left &= ~same;
    }
  };
  if (t < kPickChunks) sh.chunk_cnt[t] = 0;
  if (t == 0) sh.count = sh.ties = sh.ties_in = sh.from0 = sh.from1 = sh.window = sh.bucket = 0;
  // ---- 2. [lo, hi]: keys among which the k-th largest is the need-th largest ----
  uint32_t lo = LISTED ? cand_lo : 0u, hi = 0xffffffffu;
  uint32_t shift = LISTED ? 13u : 20u;  // (20: the buckets reach from 0 to 2^31)
  uint32_t need = k, inside = 0;
#pragma unroll 1
  for (;;) {
    for (int b = t; b < kPickBins; b += kPickThreads) sh.lh[b] = 0;
    __syncthreads();
    sweep([&](const uint2& en, bool ok, uint32_t) {
      const uint32_t key = key_of_bits(en.y), b = (key - lo) >> shift;
      const bool in = ok && key >= lo && key <= hi;
      if constexpr (LISTED) {  // (a list's keys spread over the buckets; counting the crowded ones apart costs 0.3 us)
        if (in && b + 1 < kPickBins) atomicAdd(&sh.lh[b], 1u);
        const uint64_t above = ballot64(in && b + 1 >= kPickBins);  // the last bucket holds everything above it
        if (above && lane == 0) atomicAdd(&sh.lh[kPickBins - 1], popc64(above));
      } else {
        count_in(in, b < kPickBins - 1 ? b : kPickBins - 1);
      }
    });
    __syncthreads();
    find_crossing<kPickBins, kPickThreads>(sh.lh, need, sh.suf, sh.out2);
    const uint32_t b = sh.out2[0];
    need -= sh.out2[1];
    inside = sh.lh[b];
    lo += b << shift;
    if (b + 1 < kPickBins) {
      const uint32_t top = lo + ((1u << shift) - 1u);
      hi = top < hi ? top : hi;
    }
    __syncthreads();  // everybody has read the histogram and the crossing
    if (inside <= kPickRank || lo == hi) break;
    // the next buckets: a 2048th of this one, or (the open last bucket) up to the largest key
    shift = hi == 0xffffffffu ? 20u : (shift > 11u ? shift - 11u : 0u);
  }
  // ---- 3. tau and the last tie to take ----
  uint32_t tau, tie_last, ties, ties_kept;
  if (inside <= kPickRank) {
    sweep([&](const uint2& en, bool ok, uint32_t) {
      const uint32_t key = key_of_bits(en.y);
      if (ok && key >= lo && key <= hi) sh.rank_en[atomicAdd(&sh.count, 1u)] = make_uint2(en.x, key);
    });
    __syncthreads();
    uint32_t last;
    if (inside <= 64) {  // every wavefront ranks them for itself: no more barriers (they took a third of the ranking)
      const bool have = lane < inside;
      const uint2 mine = have ? sh.rank_en[lane] : make_uint2(0u, 0u);
      uint32_t rank = have ? 0u : 64u;
      for (uint32_t q = 0; q < inside; ++q) {  // uniform
        const uint32_t coord = __builtin_amdgcn_readlane(mine.x, q), key = __builtin_amdgcn_readlane(mine.y, q);
        rank += (key > mine.y || (key == mine.y && coord < mine.x)) ? 1u : 0u;
      }
      const uint32_t at = __builtin_ctzll(ballot64(rank == need - 1));  // the last kept one
      tau = __builtin_amdgcn_readlane(mine.y, at);
      last = __builtin_amdgcn_readlane(mine.x, at);
      const bool tie = have && mine.y == tau;
      ties = popc64(ballot64(tie));
      ties_kept = popc64(ballot64(tie && mine.x <= last));
    } else {
      uint32_t my_key = 0, my_coord = 0, rank = 0;
      if (t < inside) {
        my_coord = sh.rank_en[t].x;
        my_key = sh.rank_en[t].y;
        for (uint32_t q = 0; q < inside; ++q) {
          const uint2 o = sh.rank_en[q];
          rank += (o.y > my_key || (o.y == my_key && o.x < my_coord)) ? 1u : 0u;
        }
        if (rank == need - 1) { sh.tau = my_key; sh.last = my_coord; }  // the last kept one
      }
      __syncthreads();
      tau = sh.tau;
      last = sh.last;
      if (t < inside && my_key == tau) {
        atomicAdd(&sh.ties, 1u);
        if (my_coord <= last) atomicAdd(&sh.ties_in, 1u);
      }
      __syncthreads();
      ties = sh.ties;
      ties_kept = sh.ties_in;
    }
    tie_last = ties_kept < ties ? last : 0xffffffffu;
  } else {
    tau = lo;
    ties = inside;
    ties_kept = need;
    tie_last = 0xffffffffu;
    if (need < inside) {  // the need-th smallest coordinate among the entries equal to tau
      uint32_t c_lo = 0, left = need;
      constexpr uint32_t kCoordShift = 5;
      static_assert((kPickChunks * kChunk) >> kCoordShift <= kPickBins && (1u << kCoordShift) <= kPickBins, "two levels");
#pragma unroll 1
      for (uint32_t c_shift = kCoordShift;; c_shift = 0) {
        for (int b = t; b < kPickBins; b += kPickThreads) sh.lh[b] = 0;
        __syncthreads();
        sweep([&](const uint2& en, bool ok, uint32_t) {
          const uint32_t rel = (en.x - c_lo) >> c_shift;  // mirrored below: the smallest coordinates on top
          count_in(ok && key_of_bits(en.y) == tau && en.x >= c_lo && rel < kPickBins, kPickBins - 1 - rel);
        });
        __syncthreads();
        find_crossing<kPickBins, kPickThreads>(sh.lh, left, sh.suf, sh.out2);
        c_lo += (kPickBins - 1 - sh.out2[0]) << c_shift;
        left -= sh.out2[1];
        __syncthreads();
        if (c_shift == 0) break;
      }
      tie_last = c_lo;
    }
  }
  // ---- 4. kept entries per chunk; what the counters and the next step's guess need ----
  const uint32_t b0 = tau >> kL0Shift;
  const uint32_t tau_bucket = windowed && tau >= blo && tau < bhi ? band_bucket(tau - blo, bmul) : 0xffffffffu;
  uint32_t n_from0 = 0, n_from1 = 0, n_window = 0, n_same = 0;  // this wavefront's
  sweep([&](const uint2& en, bool ok, uint32_t q0) {
    const uint32_t key = key_of_bits(en.y), bucket = key >> kL0Shift;
    uint64_t kept = ballot64(ok && (key > tau || (key == tau && en.x <= tie_last)));
    if constexpr (!LISTED) {  // (a list holds them all)
      n_from0 += popc64(ballot64(ok && bucket >= b0));
      n_from1 += popc64(ballot64(ok && bucket + 1 >= b0));
    }
    if (windowed) {  // uniform
      const bool in_window = ok && key >= blo && key < bhi;
      n_window += popc64(ballot64(in_window));
      n_same += popc64(ballot64(in_window && band_bucket(key - blo, bmul) == tau_bucket));
    }
    if constexpr (LISTED) {
      const uint32_t c = en.x / kChunk;
      while (kept) {  // (a wavefront's 64 entries lie in a few chunks)
        const uint32_t c0 = __builtin_amdgcn_readlane(c, __builtin_ctzll(kept));
        const uint64_t here = ballot64(c == c0) & kept;
        if (lane == 0) atomicAdd(&sh.chunk_cnt[c0], popc64(here));
        kept &= ~here;
      }
    } else if (kept && lane == 0) {
      atomicAdd(&sh.chunk_cnt[q0 / kChunk], popc64(kept));
    }
  });
  if (lane == 0) {
    if (n_from0) atomicAdd(&sh.from0, n_from0);
    if (n_from1) atomicAdd(&sh.from1, n_from1);
    if (n_window) atomicAdd(&sh.window, n_window);
    if (n_same) atomicAdd(&sh.bucket, n_same);
  }
  __syncthreads();
  if (t < geo.num_chunks) {
    uint32_t before = 0;
    for (uint32_t u = 0; u < t; ++u) before += sh.chunk_cnt[u];
    ws.chunk_rec[sc.chunk_base + t] = make_uint4(sh.chunk_cnt[t], 0u, before, 0u);
  }
  if (t != 0) return;
  const uint32_t total = sh.from0;  // (from the row itself) entries from the threshold's bucket upwards
  const bool fits = total <= opt.cap && !opt.force_dense;
  rowp->fast = kFastPick;
  rowp->level1_done = 1;
  rowp->mode = LISTED ? kModeCand : kModeDense;
  rowp->n_src = LISTED ? n_cand : 0u;
  rowp->tau_prev = tau_before;
  rowp->tau = tau;
  rowp->r = ties_kept;
  rowp->ties = ties;
  rowp->tie_last = tie_last;
  rowp->cursor = 0;
  rowp->cursor_band = 0;
  ws.tau[row] = tau;
  ws.count_gt[row] = k - ties_kept;
  uint32_t* cn = ws.counters + row * kCountersPerRow;
  cn[0] = LISTED ? 0u : (fits ? 1u : 4u);
  cn[1] = LISTED ? n_cand : (fits ? total : 0u);
  cn[2] = ties;
  cn[3] = ties_kept;
  const uint32_t in_window = sh.window;
  uint32_t miss = 0;
  if (!windowed || opt.force_dense) miss = 1;
  else if (n_cand > opt.cap) miss = 2;
  else if (in_window > opt.band_cap) miss = 3;
  else if (tau >= bhi) miss = 4;
  else if (tau < blo) miss = 5;
  else if (sh.bucket > kBoundaryCap) miss = 6;
  cn[4] = miss ? 0u : in_window;
  cn[5] = miss;
  // Guess and window for the next step, as the other routes set them; from a list nothing is known below its lower
  // end: the bucket below the guess it was made with is taken to hold at most as many entries as all above it.
  uint32_t valid = 0, guess = 0;
  if (opt.predict && !opt.force_dense) {
    const uint32_t at_hand = LISTED ? n_cand : total;
    const uint32_t bound = LISTED ? (b0 > bg ? n_cand : 2u * n_cand) : sh.from1;
    if (b0 && bound <= opt.cap / 2) { valid = 1; guess = b0 - 1; }
    else if (at_hand <= opt.cap / 2) { valid = 1; guess = b0; }
  }
  leave_next(rowp, geo.n, k, opt, valid, guess, LISTED ? known_from(guess, cand_lo, n_cand, opt.cap) : 0u, tau, tau_before, tau_before2,
             miss == 0 && normal_key(tau) ? in_window : 0u, blo, bhi, tau);
}

__global__ __launch_bounds__(kPickThreads) void k_topk_pick(Geometry geo, const float* __restrict__ e, TopkWorkspace ws,
                                                             TopkOptions opt, uint32_t use_guess) {
  __shared__ PickShared sh;
  const SegCtx sc = seg_ctx<true, kClassFirst>(geo, opt, ws);  // grid (1, rows)
  const TopkRow* rp = ws.rows + sc.seg;
  const PickRow r{rp->cursor /* a short row's list is kept as one run */, rp->cand_from, rp->b_guess, rp->band_valid,
                  rp->band_lo, rp->band_hi, rp->band_mul, rp->tau, rp->tau_prev};
  // The list's first trip is requested with it (what the list does not hold is not looked at).  Every thread loads, the same
  // entry again where there is none: behind a condition the compiler masked the sign inside it, and the four loads waited
  // for each other (4 x 65536, k = 655: 24.8 us a step so, 24.3 as here).
  const uint2* candr = ws.cand + sc.cand_base;
  uint2 first[kPickQuad];
#pragma unroll
  for (uint32_t u = 0; u < kPickQuad; ++u) {
    const uint32_t q = u * kPickThreads + threadIdx.x;
    first[u] = candr[q < opt.cap ? q : 0u];
  }
  const bool pred = use_guess && r.cand_from != 0;
  const bool listed = pred && !opt.force_dense && r.n_cand >= geo.k && r.n_cand <= opt.cap;
  if (listed) pick_row<true>(sh, e, geo, ws, opt, sc, r, pred, first);  // uniform
  else pick_row<false>(sh, e, geo, ws, opt, sc, r, pred, first);
}

// ---------------------------------------------------------------------------------------------
// A guess for the first step of a row from a sample of its corrected gradients: kSample / 4 quads spread evenly over
// the row, one workgroup per row.  (What bounds it are the cache lines that one compute unit asks for: 8192 single
// coordinates take 37 us, in quads 12.7, 4096 in quads 7.7.)
// The guess is the bucket above which one and a half times the share k / d of the sample lies, plus three deviations of
// that count and three entries for small counts: the list then holds k entries or more but for one row in hundreds.  A row
// whose list would not fit by what the sample holds from that bucket upwards (few magnitudes; three of 4096 are more than
// 65536 entries from 90 M coordinates on) gets no guess: the list would be written and counted for nothing.  It decides only
// whether the row is read again.  (Eight entries instead of three, and no look at what fits: 34 M coordinates, k = 1000, 362
// us a call, now 338; 60 M, k = 100000, 580, now 523.)
// ---------------------------------------------------------------------------------------------
// The same sample gives the window of keys in which the threshold is expected, where the first pass is to keep band
// lists: from the bucket above which the expected count plus three deviations lies to the one above which the expected
// count less three deviations does, if the band list would hold what the sample says lies in it.  The band kernel then
// selects, as in a step that carries its window over, and the general route (30 us of the call for 4 x 300007, k = 3000,
// in four launches) returns at once. Fewer of the sample's entries above the threshold than sample_gives_window() asks
// for say too little: the window is two octaves wide and more, its entries' lists and counts cost the first pass what the
// selection gains, and half of the calls miss it.  (Two sets of 24 drawn shapes, times faster than without a window, in
// the mean: from 8 entries on 1.06 and 1.06, from 16 on 1.05 and 1.04, always 1.05; always: 4 x 1634958, k = 2524, 70.9
// -> 74.0 us; 4 x 297708, k = 1050 -- 14 entries -- 50.3 -> 45.4; 4 x 97241, k = 1445 49.8 -> 43.9.)  In long rows a wide
// window's entries meet on the histogram's crowded end: us a call without / with a window, unit normal and heavy-tailed
// values, 12 entries above the threshold: 4 x 1.8 M 71.8 / 67.9, 71.1 / 69.3; 4 x 2.6 M 80.2 / 77.4, 89.7 / 81.9; 4 x 2.9
// M 85.0 / 83.9, 84.1 / 91.8; 8 x 1.8 M 89.6 / 83.8, 88.1 / 84.5; 8 x 2.1 M 91.6 / 94.0, 95.9 / 96.8; 8 x 2.9 M 107.4 /
// 117.1, 107.6 / 130.9; 40 entries, where it is narrower: 4 x 2.9 M 87.0 / 78.9, 8 x 2.9 M 111.4 / 109.0.
// The launch also clears the tables that the call expects at zero, which took a launch of its own, 2 us: a workgroup its
// row's control block, further workgroups what follows the flags.
// (And where nearly all is kept, the sample does not say from where on.)
inline bool sample_gives_window(const Geometry& geo) {
  const uint64_t entries = geo.num_chunks <= 640 && static_cast<uint64_t>(geo.n) * geo.num_chunks <= 4096 ? 8 : 32;
  const uint64_t k = geo.k, d = geo.d;
  return k * kSample >= d * entries && 8 * k <= 5 * d;
}

__global__ __launch_bounds__(kPickThreads) void k_topk_sample(const float* __restrict__ g, const float* __restrict__ e,
                                                               int64_t ld, uint32_t d, uint32_t n, uint32_t k, uint32_t cap,
                                                               TopkRow* rows, Geometry geo, TopkWorkspace ws, TopkOptions opt) {
  geo.ld = ld; geo.d = d; geo.n = n; geo.k = k; opt.cap = cap; ws.rows = rows;
  __shared__ uint32_t lh[kNB0];
  __shared__ uint32_t suf[kPickThreads + 1];
  __shared__ uint32_t out2[6];
  const uint32_t row = blockIdx.x, t = threadIdx.x;
  if (row >= geo.n) {  // clears, 16 bytes a thread
    uint4* p = reinterpret_cast<uint4*>(ws.counters);
    const uint32_t quads = static_cast<uint32_t>(reinterpret_cast<uint4*>(ws.chunk_rec) - p);
    for (uint32_t q = (row - geo.n) * kPickThreads + t; q < quads; q += (gridDim.x - geo.n) * kPickThreads)
      p[q] = make_uint4(0, 0, 0, 0);
    return;
  }
  // the control block as the first pass reads it; nothing else in it but zeros
  uint32_t cand_from = 0, guess = 0, valid = 0, band_lo = 0, band_hi = 0, band_mul = 0;
  if (row == 0 && t < kQueues) ws.flags[queue_word(t)] = 0;
  if (row == 0 && t == 0) ws.flags[0] = opt.band == kBandLists ? 0u : 1u;  // without a band kernel the general ones are told here
  const float* gr = g + static_cast<int64_t>(row) * geo.ld;
  const float* er = e + static_cast<int64_t>(row) * geo.ld;
  constexpr uint32_t kQuads = kSample / 4;
  constexpr int kPer = kQuads / kPickThreads;
  static_assert(kQuads % kPickThreads == 0, "whole quads");
  const uint32_t whole_quads = geo.d / 4;  // at least kQuads: the host asks for no sample of a shorter row
  const float each = static_cast<float>(geo.d) / static_cast<float>(kSample);  // coordinates that a sampled one stands for
  const float share = static_cast<float>(geo.k) / each;
  const float want = 1.5f * share + 3.0f * sqrtf(share) + 3.0f;
  if (want < static_cast<float>(kSample) && want * each <= static_cast<float>(opt.cap)) {  // uniform
    float4 x[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t q = u * kPickThreads + t;
      const uint32_t j = 4u * static_cast<uint32_t>((static_cast<uint64_t>(q) * whole_quads) / kQuads);  // (a shift)
      const float4 ev = *reinterpret_cast<const float4*>(er + j), gv = *reinterpret_cast<const float4*>(gr + j);
      x[u] = make_float4(ev.x + gv.x, ev.y + gv.y, ev.z + gv.z, ev.w + gv.w);
    }
    for (int b = t; b < kNB0; b += kPickThreads) lh[b] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      atomicAdd(&lh[key_of_bits(__float_as_uint(x[u].x)) >> kL0Shift], 1u);
      atomicAdd(&lh[key_of_bits(__float_as_uint(x[u].y)) >> kL0Shift], 1u);
      atomicAdd(&lh[key_of_bits(__float_as_uint(x[u].z)) >> kL0Shift], 1u);
      atomicAdd(&lh[key_of_bits(__float_as_uint(x[u].w)) >> kL0Shift], 1u);
    }
    __syncthreads();
    // (three crossings; no band list: the first one)
    const float off = 3.0f * sqrtf(share) + 2.0f;
    const uint32_t needs[3] = {static_cast<uint32_t>(want), static_cast<uint32_t>(fminf(want, share + off)),
                               static_cast<uint32_t>(fmaxf(share - off, 1.0f))};
    find_crossings<kNB0, kPickThreads, 3>(lh, needs, suf, out2);
    if (static_cast<float>(out2[1] + lh[out2[0]]) * each <= static_cast<float>(opt.cap)) {  // uniform
      guess = out2[0];
      cand_from = (guess << kL0Shift) + 1u;
    }
    if (cand_from && opt.band == kBandLists) {  // uniform
      const uint32_t lo = out2[2], from_lo = out2[3] + lh[lo];
      const uint32_t hi = out2[4] + 1, above = out2[5];
      band_lo = lo << kL0Shift;
      band_hi = hi << kL0Shift;
      const float inside = static_cast<float>(from_lo - above) * each;
      const bool many = band_buckets(geo.k) == kBandBucketsMany && inside > 16.0f * kBandBucketsFew;
      if (lo > 15 && hi < 0xff0u && 1.25f * inside <= static_cast<float>(opt.band_cap)) valid = many ? kBandMany : kBandFew;
      band_mul = band_multiplier_dev(band_hi - band_lo, many ? kBandBucketsMany : kBandBucketsFew);
    }
  }
  static_assert(offsetof(TopkRow, cand_from) == 0 && offsetof(TopkRow, b_guess) == 4 && offsetof(TopkRow, band_valid) == 16 &&
                offsetof(TopkRow, band_lo) == 20 && offsetof(TopkRow, band_hi) == 24 && offsetof(TopkRow, band_mul) == 28,
                "words written below");
  if (t < sizeof(TopkRow) / 4)
    reinterpret_cast<uint32_t*>(ws.rows + row)[t] =
        t == 0 ? cand_from : t == 1 ? guess : t == 4 ? valid : t == 5 ? band_lo : t == 6 ? band_hi : t == 7 ? band_mul : 0u;
}

// ---------------------------------------------------------------------------------------------
// Level 0 after the lean first pass.  A row whose guess held (its candidate list holds at least k entries and
// did not overflow) gets the histogram of threshold buckets from the list -- every key at or above the guessed
// bucket is in it, so the k-th largest key of the list is the row's -- together with the level-1 histograms of
// the three buckets from the guess upwards.  Any other row (no guess yet, the guess was too high, the list
// overflowed) gets its histogram from the stored values themselves, one more read of the row.  The last
// workgroup of the row finds the threshold bucket, decides the route of the remaining kernels and leaves the
// guess for the next step.
// ---------------------------------------------------------------------------------------------
// What the four parts of the general route keep in LDS, besides what they share.
struct GeneralShared {
  uint32_t suf[kWG + 1];
  uint32_t scratch[kWG / 64 + 1];
  uint32_t out2[2];
  uint32_t flag, l1, bstar, need;
};
struct Level0Shared { uint32_t lh[kNB0], lh1[kTracked * kNB1]; };
struct Level1Shared { uint32_t lh[kNB1]; uint2 stage[kWaves * kStage]; };
struct Level2Shared { uint32_t lh[kNB2]; };
struct CountShared { uint32_t gt[kMaxCountCpw], eq[kMaxCountCpw]; };

// A part of a problem is done: the next one may begin.  By the thread that has written what the next one reads, with
// device-scope stores.
__device__ __forceinline__ void problem_at(TopkRow* rowp, uint32_t phase) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  store_agent(&rowp->phase, phase);
}

// (unrolled by hand: before it is in line, the compiler does not know how many threads there are, and in loops level 0
// took 1.6 us more)
template <uint32_t NB>
__device__ __forceinline__ void clear_bins(uint32_t* bins) {
  static_assert(NB % kWG == 0, "bins per thread");
#pragma unroll
  for (uint32_t i = 0; i < NB / kWG; ++i) bins[i * kWG + threadIdx.x] = 0;
}
template <uint32_t NB>
__device__ __forceinline__ void flush_bins(const uint32_t* bins, uint32_t* to) {
#pragma unroll
  for (uint32_t i = 0; i < NB / kWG; ++i) {
    const uint32_t h = bins[i * kWG + threadIdx.x];
    if (h) atomicAdd(&to[i * kWG + threadIdx.x], h);
  }
}

template <bool SAME>
__device__ __forceinline__ void general_level0(GeneralShared& sh, Level0Shared& lds, const float* __restrict__ e, const Geometry& geo,
                                               const TopkWorkspace& ws, const TopkOptions& opt, const SegCtx& sc, uint32_t use_guess) {
  uint32_t (&lh)[kNB0] = lds.lh;
  uint32_t (&lh1)[kTracked * kNB1] = lds.lh1;
  const uint32_t row = sc.seg;
  TopkRow* rowp = ws.rows + row;
  const uint32_t bg = rowp->b_guess;
  const ListRuns runs = runs_from_cursors(ws, rowp, sc.cursor_set, opt.cap);  // written by the previous launch
  const bool listed = use_guess && rowp->cand_from != 0 && runs.total >= geo.k && runs.fits && !opt.force_dense;
  clear_bins<kNB0>(lh);
  clear_bins<kTracked * kNB1>(lh1);
  __syncthreads();
  const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();
  if (listed) {
    const uint2* candr = ws.cand + sc.cand_base;
    sweep_list([=](uint32_t q) { return candr[q].y; }, runs, sc.group * kWG + threadIdx.x, sc.groups * kWG, [&](uint32_t bits) {
      const uint32_t key = key_of_bits(bits);
      const uint32_t bucket = key >> kL0Shift;
      atomicAdd(&lh[bucket], 1u);
      const uint32_t rel = bucket - bg;
      if (rel < kTracked) atomicAdd(&lh1[rel * kNB1 + ((key >> kL1Shift) & (kNB1 - 1))], 1u);
    });
  } else {
    const float* er = e + sc.elem_off;
    uint32_t zeros = 0;
    const uint32_t stride = sc.groups * kWaves;
    for (uint32_t c = sc.group * kWaves + wave; c < geo.num_chunks; c += stride) {
      const uint32_t base = c * kChunk + lane * 4;
#pragma unroll 4
      for (int r = 0; r < kRounds; ++r) {
        const uint32_t j = base + r * 256;
        if (c * kChunk + r * 256 >= geo.d) break;  // wave-uniform
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j < geo.d) x = *reinterpret_cast<const float4*>(er + j);
        Quad q;
        q.key[0] = key_of_bits(__float_as_uint(x.x)); q.key[1] = key_of_bits(__float_as_uint(x.y));
        q.key[2] = key_of_bits(__float_as_uint(x.z)); q.key[3] = key_of_bits(__float_as_uint(x.w));
#pragma unroll
        for (int s = 0; s < 4; ++s) q.ok[s] = j + s < geo.d;
        hist4<false>(lh, q, zeros);
      }
    }
    if (zeros && lane == 0) atomicAdd(&lh[0], zeros);
  }
  __syncthreads();
  uint32_t* gh = ws.hist0 + static_cast<size_t>(row) * kNB0;
  flush_bins<kNB0>(lh, gh);
  uint32_t* gh1 = ws.hist1x + static_cast<size_t>(row) * kTracked * kNB1;
  if (listed)
    flush_bins<kTracked * kNB1>(lh1, gh1);
  // ---- row-wide part, by whichever workgroup of the row finishes last ----
  if (!last_group_of_row(&rowp->ticket[0], sc.groups, &sh.flag)) return;
  take_hist<kNB0>(gh, lh);
  find_crossing<kNB0>(lh, geo.k, sh.suf, sh.out2);
  if (threadIdx.x == 0) {
    const uint32_t bstar = sh.out2[0], above = sh.out2[1];
    const uint32_t total = above + lh[bstar];  // entries with bucket >= bstar
    uint32_t mode, n_src, reads;
    if (listed) { mode = kModeCand; n_src = runs.total; reads = 0; }  // bstar >= bg: the list holds the k largest keys
    else if (total <= opt.cap && !opt.force_dense) { mode = kModeNeedB; n_src = total; reads = 1; }
    else { mode = kModeDense; n_src = 0; reads = 4; }
    hand_on<SAME>(&rowp->mode, mode);
    rowp->n_src = n_src;
    // the list's runs for the sweeps that follow: as the first pass left them, or the one run that the second
    // read of the row is about to write; the cursors go back to zero for that read and for the next step
    hand_on<SAME>(&rowp->n_lists, listed ? runs.lists : 1u);
#pragma unroll
    for (uint32_t s = 0; s < kSubLists; ++s) hand_on<SAME>(&rowp->n_sub[s], listed ? runs.n[s] : (s == 0 ? n_src : 0u));
    hand_on<SAME>(&rowp->cursor, 0u);
    rowp->cursor_band = 0;
    if (sc.cursor_set != kNoCursorSet) {
#pragma unroll
      for (uint32_t s = 0; s < kSubLists; ++s) {
        uint32_t* cur = ws.xcur + (static_cast<size_t>(sc.cursor_set) * kSubLists + s) * kCursorPitch;
        cur[0] = 0;
        cur[1] = 0;
      }
    }
    hand_on<SAME>(&rowp->bstar, bstar);
    hand_on<SAME>(&rowp->need, geo.k - above);
    rowp->level1_done = 0;
    // Guess for the next step: one bucket below this step's threshold bucket if the list that guess would
    // have produced now fits with room to spare, else the bucket itself, else no guess.  From a list, nothing
    // is known below its first key: the bucket below the guess it was made with is then taken to hold at most as many
    // entries as all the buckets above it together, what that guess's bucket holds below the list is left to known_from().
    uint32_t valid = 0, guess = 0;
    if (opt.predict && !opt.force_dense) {
      const uint32_t below = bstar ? ((listed && bstar == bg) ? total : lh[bstar - 1]) : 0;
      if (bstar && total + below <= opt.cap / 2) { valid = 1; guess = bstar - 1; }
      else if (total <= opt.cap / 2) { valid = 1; guess = bstar; }
    }
    hand_on<SAME>(&rowp->known_from, listed ? known_from(guess, rowp->cand_from - 1u, runs.total, opt.cap) : 0u);
    hand_on<SAME>(&rowp->cand_from, valid ? (guess << kL0Shift) + 1u : 0u);
    hand_on<SAME>(&rowp->b_guess, guess);
    uint32_t* cn = ws.counters + row * kCountersPerRow;
    cn[0] = reads;
    cn[1] = n_src;
    sh.l1 = (listed && bstar - bg < kTracked) ? 1u + (bstar - bg) : 0u;
    sh.bstar = bstar;
    sh.need = geo.k - above;
  }
  __syncthreads();
  if (listed) {
    const uint32_t which = sh.l1;  // 0: level 1 not available; 1 + t: histogram of bucket guess + t
    if (which) {
      const AgentView view = agent_view(gh1 + (which - 1) * kNB1, kNB1);
      uint32_t x[kNB1 / kWG];
#pragma unroll
      for (int i = 0; i < kNB1 / kWG; ++i) x[i] = load_agent(view, i * kWG + threadIdx.x);
#pragma unroll
      for (int i = 0; i < kNB1 / kWG; ++i) lh[i * kWG + threadIdx.x] = x[i];
    }
    clear_bins<kTracked * kNB1>(gh1);
    __syncthreads();
    if (which) resolve_level1<SAME>(rowp, sh.bstar, sh.need, lh, sh.suf, sh.out2);
  }
  if (SAME && threadIdx.x == 0) problem_at(rowp, phase_after_level0(sh.l1 != 0));
}

// ---------------------------------------------------------------------------------------------
// Level 1 for rows that could not resolve it in the first pass.
//   kModeNeedB: one more read of the row; writes the candidate list (bucket >= bstar) and the histogram.
//   kModeCand : the list exists (the threshold bucket was above the tracked ones): sweep it.
//   kModeDense: no list: histogram from the row itself.
// ---------------------------------------------------------------------------------------------
template <bool SAME>
__device__ __forceinline__ void general_level1(GeneralShared& sh, Level1Shared& lds, const float* __restrict__ e, const Geometry& geo,
                                               const TopkWorkspace& ws, const TopkOptions& opt, const SegCtx& sc) {
  uint32_t (&lh)[kNB1] = lds.lh;
  const uint32_t row = sc.seg;
  TopkRow* rowp = ws.rows + row;
  const Handed<SAME> view = handed_row<SAME>(rowp);
  const uint32_t mode = view.word(kRowWord(offsetof(TopkRow, mode)));
  const uint32_t bstar = view.word(kRowWord(offsetof(TopkRow, bstar))), need = view.word(kRowWord(offsetof(TopkRow, need)));
  clear_bins<kNB1>(lh);
  __syncthreads();
  const float* er = e + sc.elem_off;
  uint2* candr = ws.cand + sc.cand_base;
  auto visit = [&](uint32_t bits, bool ok) {
    const uint32_t key = key_of_bits(bits);
    if (ok && (key >> kL0Shift) == bstar) atomicAdd(&lh[(key >> kL1Shift) & (kNB1 - 1)], 1u);
  };
  if (mode == kModeNeedB) {
    uint2* descr = ws.desc + sc.chunk_base * ws.desc_parts;
    const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();
    uint2* stage = lds.stage + wave * kStage;
    const uint32_t stride = sc.groups * kWaves;
    for (uint32_t c = sc.group * kWaves + wave; c < geo.num_chunks; c += stride) {
      const uint32_t base = c * kChunk + lane * 4;
      uint32_t cnt = 0;
#pragma unroll 4
      for (int r = 0; r < kRounds; ++r) {
        const uint32_t j = base + r * 256;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j < geo.d) x = *reinterpret_cast<const float4*>(er + j);
        const uint32_t bits[4] = {__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z),
                                  __float_as_uint(x.w)};
        bool flag[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          flag[s] = j + s < geo.d && (key_of_bits(bits[s]) >> kL0Shift) >= bstar;
          visit(bits[s], j + s < geo.d);
        }
        stage_round(stage, cnt, j, bits, flag);
      }
      // fits by construction: the level-0 histogram counted exactly these entries
      flush_chunk<SAME>(stage, cnt, er, geo.d, c, bstar, rowp, candr, opt.cap, descr, ws.desc_parts);
    }
  } else if (mode == kModeCand) {
    const ListRuns runs = runs_of_row(view, opt.cap);
    const uint2* list = candr;
    sweep_list([=](uint32_t q) { return list[q].y; }, runs, sc.group * kWG + threadIdx.x, sc.groups * kWG,
               [&](uint32_t bits) { visit(bits, true); });
  } else {
    const uint32_t step = sc.groups * kWG * 4;
    for (uint32_t j = (sc.group * kWG + threadIdx.x) * 4; j < geo.d; j += step) {
      const float4 x = *reinterpret_cast<const float4*>(er + j);
      visit(__float_as_uint(x.x), true);
      visit(__float_as_uint(x.y), j + 1 < geo.d);
      visit(__float_as_uint(x.z), j + 2 < geo.d);
      visit(__float_as_uint(x.w), j + 3 < geo.d);
    }
  }
  __syncthreads();
  uint32_t* gh = ws.hist1 + static_cast<size_t>(row) * kNB1;
  flush_bins<kNB1>(lh, gh);
  if (!last_group_of_row(&rowp->ticket[1], sc.groups, &sh.flag)) return;
  take_hist<kNB1>(gh, lh);
  resolve_level1<SAME>(rowp, bstar, need, lh, sh.suf, sh.out2);
  if (SAME && threadIdx.x == 0) problem_at(rowp, kPhaseLevel2);
}

// ---------------------------------------------------------------------------------------------
// Level 2 (last 9 key bits) over the entries that match bits 30..9 of the threshold key.
// ---------------------------------------------------------------------------------------------
template <bool SAME>
__device__ __forceinline__ void general_level2(GeneralShared& sh, Level2Shared& lds, const float* __restrict__ e, const Geometry& geo,
                                               const TopkWorkspace& ws, const TopkOptions& opt, const SegCtx& sc) {
  uint32_t (&lh)[kNB2] = lds.lh;
  const uint32_t row = sc.seg;
  TopkRow* rowp = ws.rows + row;
  const Handed<SAME> view = handed_row<SAME>(rowp);
  const uint32_t mode = view.word(kRowWord(offsetof(TopkRow, mode)));
  const uint32_t want = view.word(kRowWord(offsetof(TopkRow, prefix1))), need = view.word(kRowWord(offsetof(TopkRow, need)));
  clear_bins<kNB2>(lh);
  __syncthreads();
  auto visit = [&](uint32_t bits, bool ok) {
    const uint32_t key = key_of_bits(bits);
    if (ok && (key >> kL1Shift) == want) atomicAdd(&lh[key & (kNB2 - 1)], 1u);
  };
  if (mode == kModeDense) {
    const float* er = e + sc.elem_off;
    const uint32_t step = sc.groups * kWG * 4;
    for (uint32_t j = (sc.group * kWG + threadIdx.x) * 4; j < geo.d; j += step) {
      const float4 x = *reinterpret_cast<const float4*>(er + j);
      visit(__float_as_uint(x.x), true);
      visit(__float_as_uint(x.y), j + 1 < geo.d);
      visit(__float_as_uint(x.z), j + 2 < geo.d);
      visit(__float_as_uint(x.w), j + 3 < geo.d);
    }
  } else {
    const ListRuns runs = runs_of_row(view, opt.cap);
    with_list<SAME>(ws.cand + sc.cand_base, opt.cap, mode, [&](auto bits_of) {
      sweep_list(bits_of, runs, sc.group * kWG + threadIdx.x, sc.groups * kWG, [&](uint32_t bits) { visit(bits, true); });
    });
  }
  __syncthreads();
  uint32_t* gh = ws.hist2 + static_cast<size_t>(row) * kNB2;
  flush_bins<kNB2>(lh, gh);
  if (!last_group_of_row(&rowp->ticket[2], sc.groups, &sh.flag)) return;
  take_hist<kNB2>(gh, lh);
  find_crossing<kNB2>(lh, need, sh.suf, sh.out2);
  if (threadIdx.x == 0) {
    const uint32_t s = sh.out2[0], above = sh.out2[1];
    const uint32_t tau = (want << kL1Shift) | s;
    const uint32_t r = need - above, ties = lh[s];
    const uint32_t tau_prev = rowp->tau, tau_prev2 = rowp->tau_prev;
    rowp->tau_prev = tau_prev;
    hand_on<SAME>(&rowp->tau, tau);
    rowp->r = r;
    rowp->ties = ties;
    ws.tau[row] = tau;
    ws.count_gt[row] = geo.k - r;
    uint32_t* cn = ws.counters + row * kCountersPerRow;
    cn[2] = ties;
    cn[3] = r;
    cn[4] = 0;
    if (SAME) problem_at(rowp, kPhaseCount);
    // the guess was set when the threshold bucket was found
    set_next_band(rowp, tau, tau_prev, tau_prev2, view.word(kRowWord(offsetof(TopkRow, cand_from))) != 0 ? 1u : 0u,
                  view.word(kRowWord(offsetof(TopkRow, b_guess))), view.word(kRowWord(offsetof(TopkRow, known_from))),
                  rowp->noise > 0.0f ? rowp->noise : default_band_noise(geo.k), geo.k, opt);
  }
}

// ---------------------------------------------------------------------------------------------
// Chunk-ordered sweeps.  A wavefront visits a chunk's entries round by round; within a round the
// order (lane, slot) is ascending coordinate order, in both sources.
// ---------------------------------------------------------------------------------------------
struct Entry4 {
  uint32_t j[4];
  uint32_t bits[4];
  bool ok[4];
};

// f(const Entry4&, int slots) is called wave-uniformly once per round.
template <typename F>
__device__ __forceinline__ void for_each_round(uint32_t mode, const float* __restrict__ er, uint32_t d, uint32_t c,
                                               const uint2* __restrict__ candr, uint2 ds, uint32_t cap, F&& f) {
  // ds: the chunk's segment of the candidate list (offset, count), the same in every lane; not looked at without a list
  const uint32_t lane = lane_id();
  if (mode == kModeDense) {
    const uint32_t base = c * kChunk + lane * 4;
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t j = base + r * 256;
      if (c * kChunk + r * 256 >= d) break;  // wave-uniform
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (j < d) x = *reinterpret_cast<const float4*>(er + j);
      Entry4 en;
      en.bits[0] = __float_as_uint(x.x); en.bits[1] = __float_as_uint(x.y);
      en.bits[2] = __float_as_uint(x.z); en.bits[3] = __float_as_uint(x.w);
#pragma unroll
      for (int s = 0; s < 4; ++s) { en.j[s] = j + s; en.ok[s] = j + s < d; }
      f(en, 4);
    }
  } else {
    const uint32_t off = first_lane(ds.x);
    uint32_t cnt = first_lane(ds.y);
    if (off > cap) cnt = 0;                      // segments always lie inside the list; never read outside it
    else if (cnt > cap - off) cnt = cap - off;
    constexpr int kAhead = 4;  // loads in flight per trip (long segments would otherwise be a chain of round trips)
    for (uint32_t t = 0; t < cnt; t += 64 * kAhead) {
      uint2 cv[kAhead];
#pragma unroll
      for (int w = 0; w < kAhead; ++w) {
        const uint32_t q = t + w * 64 + lane;
        cv[w] = q < cnt ? candr[off + q] : make_uint2(0, 0);
      }
#pragma unroll
      for (int w = 0; w < kAhead; ++w) {
        if (t + w * 64 >= cnt) break;  // wave-uniform
        Entry4 en;
        en.ok[0] = t + w * 64 + lane < cnt;
        en.j[0] = cv[w].x; en.bits[0] = cv[w].y;
#pragma unroll
        for (int s = 1; s < 4; ++s) { en.j[s] = 0; en.bits[s] = 0; en.ok[s] = false; }
        f(en, 1);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Counting: per chunk, how many keys lie above tau and how many equal it.  A workgroup owns a contiguous
// block of geo.count_cpw chunks; it leaves, per chunk, the two counts and their exclusive prefixes within
// the block, and per block the two totals.  The last kernel turns these into positions in the worker's
// list (a sum over at most kMaxCountBlocks block totals), so no workgroup waits for or follows another.
// ---------------------------------------------------------------------------------------------
template <bool QUARTERS, bool SAME>
__device__ __forceinline__ void general_count(GeneralShared& sh, CountShared& lds, const float* __restrict__ e, const Geometry& geo,
                                              const TopkWorkspace& ws, const TopkOptions& opt, const SegCtx& sc) {
  const uint32_t row = sc.seg;
  const uint32_t cpw = geo.count_cpw;
  const uint32_t start = sc.group * cpw;
  if (start >= geo.num_chunks) return;  // uniform; the grid has exactly the blocks that exist
  const uint32_t end = start + cpw < geo.num_chunks ? start + cpw : geo.num_chunks;
  const TopkRow* rowp = ws.rows + row;
  const Handed<SAME> view = handed_row<SAME>(rowp);
  const uint32_t mode = view.word(kRowWord(offsetof(TopkRow, mode))), tau = view.word(kRowWord(offsetof(TopkRow, tau)));
  const float* er = e + sc.elem_off;
  const uint2* candr = ws.cand + sc.cand_base;
  // (a chunk's descriptors may have been written in this launch)
  constexpr uint32_t kParts = QUARTERS ? kWaves : 1;
  const Handed<SAME> descr(ws.desc + sc.chunk_base * kParts, 2 * geo.num_chunks * kParts);
  const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();
  if (mode == kModeDense) {
    for (uint32_t c = start + wave; c < end; c += kWaves) {
      uint32_t gt = 0, eq = 0;
      for_each_round(mode, er, geo.d, c, candr, make_uint2(0u, 0u), opt.cap, [&](const Entry4& en, int slots) {
        for (int s = 0; s < slots; ++s) {
          const uint32_t key = key_of_bits(en.bits[s]);
          gt += popc64(ballot64(en.ok[s] && key > tau));
          eq += popc64(ballot64(en.ok[s] && key == tau));
        }
      });
      if (lane == 0) { lds.gt[c - start] = gt; lds.eq[c - start] = eq; }
    }
  } else if constexpr (QUARTERS) {
    // A wavefront takes eight consecutive chunks at a time, sixteen lanes for every quarter of a chunk: the first 32
    // entries of all quarters together, then, chunk by chunk, what any of its quarters holds beyond.  (Two lanes to a
    // quarter, all quarters at once, ask for every line of the list several times, and go through a crowded quarter in a
    // chain of 32 trips.  us, rows in chunks / in pages with two lanes / with sixteen: 8 x 25570000, k 1 % 18.3 / 24.3 /
    // 18.7, 10 % 65 / 102 / 48, 5 % in 1024 large columns of 32768 41 / 168 / 48; 8 x 124439808, 0.1 % 36.6 / 30.9 /
    // 27.0; 64 x 3002268, 1 % 12.5 / 22.4 / 16.8.)
    constexpr int kGroup = 8;
    constexpr uint32_t kLanes = 64 / kWaves, kFirst = 2 * kLanes, kAhead = 8;
    const uint32_t part = lane / kLanes, sub = lane % kLanes;
    for (uint32_t c0 = start + wave * kGroup; c0 < end; c0 += kWaves * kGroup) {
      uint2 all = make_uint2(0, 0);  // lane l: segment l % 32
      if (c0 + lane % 32 / kWaves < end) all = descr.pair(c0 * kWaves + lane % 32);
      if (all.x > opt.cap) all.y = 0;  // segments always lie inside the list; never read outside it
      else if (all.y > opt.cap - all.x) all.y = opt.cap - all.x;
      uint2 ds[kGroup];
      uint32_t first[kGroup], second[kGroup];
#pragma unroll
      for (int u = 0; u < kGroup; ++u) ds[u] = make_uint2(__shfl(all.x, u * kWaves + part, 64), __shfl(all.y, u * kWaves + part, 64));
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        first[u] = sub < ds[u].y ? candr[ds[u].x + sub].y : 0u;
        second[u] = sub + kLanes < ds[u].y ? candr[ds[u].x + sub + kLanes].y : 0u;
      }
#pragma unroll
      for (uint32_t u = 0; u < kGroup; ++u) {
        uint32_t gt = 0, eq = 0;  // wave-uniform
        auto add = [&](bool ok, uint32_t bits) {
          const uint32_t key = key_of_bits(bits);
          gt += popc64(ballot64(ok && key > tau));
          eq += popc64(ballot64(ok && key == tau));
        };
        add(sub < ds[u].y, first[u]);
        add(sub + kLanes < ds[u].y, second[u]);
        for (uint32_t q0 = kFirst; ballot64(q0 < ds[u].y) != 0; q0 += kAhead * kLanes) {
          uint32_t bits[kAhead];
#pragma unroll
          for (uint32_t w = 0; w < kAhead; ++w) {
            const uint32_t q = q0 + w * kLanes + sub;
            bits[w] = q < ds[u].y ? candr[ds[u].x + q].y : 0u;
          }
#pragma unroll
          for (uint32_t w = 0; w < kAhead; ++w) add(q0 + w * kLanes + sub < ds[u].y, bits[w]);
        }
        if (lane == 0 && c0 + u < end) { lds.gt[c0 + u - start] = gt; lds.eq[c0 + u - start] = eq; }
      }
    }
  } else {
    // A wavefront takes up to eight consecutive chunks at a time, the lanes shared out among their segments: the
    // descriptors come with one load, then kAhead entries of every lane together.  Where fewer chunks are there than it
    // could take, each has more lanes (blocks of 12 x 60000, one coordinate in 20: 9.1 us, eight lanes to a chunk in any
    // case 14.0).
    constexpr int kAhead = 16;
    const uint32_t group = chunks_per_wave(cpw);
    const SegmentLanes sl = segment_lanes(end - start < group ? end - start : group, 1u);
    with_list<SAME>(candr, opt.cap, mode, [&](auto bits_of) {
      for (uint32_t c0 = start + wave * group; c0 < end; c0 += kWaves * group) {
        uint2 ds = make_uint2(0, 0);
        if (c0 + sl.chunk < end) ds = descr.pair(c0 + sl.chunk);
        if (ds.x > opt.cap) ds.y = 0;  // segments always lie inside the list; never read outside it
        else if (ds.y > opt.cap - ds.x) ds.y = opt.cap - ds.x;
        uint32_t gt = 0, eq = 0;  // of this lane's entries
        for (uint32_t q0 = 0; ballot64(q0 < ds.y) != 0; q0 += kAhead * sl.lanes) {
          uint32_t bits[kAhead];
#pragma unroll
          for (int u = 0; u < kAhead; ++u) {
            const uint32_t q = q0 + u * sl.lanes + sl.sub;
            bits[u] = q < ds.y ? bits_of(ds.x + q) : 0u;
          }
#pragma unroll
          for (int u = 0; u < kAhead; ++u) {
            const bool ok = q0 + u * sl.lanes + sl.sub < ds.y;
            const uint32_t key = key_of_bits(bits[u]);
            gt += ok && key > tau ? 1u : 0u;
            eq += ok && key == tau ? 1u : 0u;
          }
        }
        gt = chunk_sum(gt, sl);
        eq = chunk_sum(eq, sl);
        if (sl.first && c0 + sl.chunk < end) { lds.gt[c0 - start + sl.chunk] = gt; lds.eq[c0 - start + sl.chunk] = eq; }
      }
    });
  }
  __syncthreads();
  // exclusive prefixes within the block: thread t takes `per` consecutive chunks
  const uint32_t len = end - start;
  const uint32_t per = (cpw + kWG - 1) / kWG;  // <= kMaxCountCpw / kWG
  const uint32_t first = threadIdx.x * per;
  uint32_t sum_gt = 0, sum_eq = 0;
  for (uint32_t i = 0; i < per; ++i)
    if (first + i < len) { sum_gt += lds.gt[first + i]; sum_eq += lds.eq[first + i]; }
  uint32_t tot_gt, tot_eq;
  uint32_t pre_gt = block_excl_scan<kWG>(sum_gt, sh.scratch, &tot_gt);
  uint32_t pre_eq = block_excl_scan<kWG>(sum_eq, sh.scratch, &tot_eq);
  uint4* rec = ws.chunk_rec + sc.chunk_base + start;
  for (uint32_t i = 0; i < per; ++i)
    if (first + i < len) {
      const uint32_t gt = lds.gt[first + i], eq = lds.eq[first + i];
      rec[first + i] = make_uint4(gt, eq, pre_gt, pre_eq);
      pre_gt += gt;
      pre_eq += eq;
    }
  if (threadIdx.x == 0) ws.blk[static_cast<size_t>(row) * kMaxCountBlocks + sc.group] = make_uint2(tot_gt, tot_eq);
}

// A part of the general route as a launch of its own.
template <bool UNI, bool QUARTERS, int PART>
__global__ __launch_bounds__(kWG) void k_topk_part(Geometry geo, const float* __restrict__ e, TopkWorkspace ws, TopkOptions opt,
                                                   uint32_t use_guess) {
  if (table_u32(ws.flags, 0) == 0) return;  // every problem of this step was selected by k_topk_band
  __shared__ GeneralShared sh;
  __shared__ std::conditional_t<PART == 0, Level0Shared, std::conditional_t<PART == 1, Level1Shared,
                                std::conditional_t<PART == 2, Level2Shared, CountShared>>> lds;
  const SegCtx sc = seg_ctx<UNI, PART == 0 ? kClassLevel0 : PART == 3 ? kClassCount : kClassSweep>(geo, opt, ws);
  const TopkRow* rowp = ws.rows + sc.seg;
  if (rowp->fast) return;                              // the same for the whole problem
  if (PART == 1 && rowp->level1_done) return;  // level 0 has resolved it
  if constexpr (PART == 0) general_level0<false>(sh, lds, e, geo, ws, opt, sc, use_guess);
  else if constexpr (PART == 1) general_level1<false>(sh, lds, e, geo, ws, opt, sc);
  else if constexpr (PART == 2) general_level2<false>(sh, lds, e, geo, ws, opt, sc);
  else general_count<QUARTERS, false>(sh, lds, e, geo, ws, opt, sc);
}

// ---------------------------------------------------------------------------------------------
// The general route in one launch, for the steps in which the band kernel usually leaves nothing to it: it returns at
// once then, where four launches return one after the other (1.7 us each: 16 x 1 M, k = 10000, 69.6 us a step, so 65.1).
// The four parts are cut into tasks and every part into as many shares as there are workgroups.  A workgroup draws a
// share (next_share), takes level 0's tasks of it, draws again if there are shares that nobody has taken, and goes
// through the tasks of its shares in the parts that follow.  A task waits until its problem's part before is done
// (wait_for_part; level 1's also where level 0 has resolved it and nothing is left to do: nobody has to know beforehand).
// The wait ends: a workgroup waits only when all shares belong to workgroups that are running, and only for parts before
// its task's; level 0 waits for nothing.  So it does not matter how many workgroups run at a time, or in what order they
// start.  Only a control block that somebody else writes meanwhile can keep a phase from coming; the wait is bounded for
// that.
// What bounds it is a chain for every part: the wait, the list or row, the histogram's atomics, the ticket, the last
// workgroup's crossing, about 6 us.  (Every share of every part drawn from one counter, and two tasks of level 1 and 2 to
// a workgroup: 16 x 1 M, all thresholds rising by 15 % a step, 113 us a step; so 96, four launches 92.)
// What one part leaves to the next goes through device-scope stores and loads (no fences: see last_group_of_row), the
// list that level 1 writes included (with_list).
// Where it is taken: see general_in_one().
// ---------------------------------------------------------------------------------------------
// Workgroups at most: two to a compute unit, so that there is room for 137 vector registers (128 of them: 12 bytes
// spilled, steps that miss 0.3 to 1 us longer).
constexpr uint32_t kGeneralMost = 512;

template <bool UNI>
__global__ __launch_bounds__(kWG, 3) void k_topk_general(const uint32_t* flags, const float* __restrict__ e, Geometry geo_all,
                                                      TopkWorkspace ws, TopkOptions opt_all, uint32_t use_guess, GeneralTasks tasks) {
  if (table_u32(flags, 0) == 0) return;  // every problem of this step was selected by k_topk_band
  __shared__ GeneralShared sh;
  __shared__ union {
    Level0Shared level0;
    Level1Shared level1;
    Level2Shared level2;
    CountShared count;
  } lds;
  __shared__ uint32_t sh_drawn, sh_phase;
  __shared__ uint16_t sh_share[kGeneralMost];  // the shares that this workgroup holds
  // (out of the arguments at once: looked up by a number, each look-up waited for memory)
  const uint32_t t0 = tasks.total[0], t1 = tasks.total[1], t2 = tasks.total[2], t3 = tasks.total[3];
  const uint32_t g0 = tasks.groups[0], g1 = tasks.groups[1], g2 = tasks.groups[2], g3 = tasks.groups[3];
  uint32_t held = 0;
  uint32_t seg = ~0u, fast = 0, at = 0;  // the problem looked at last: found by k_topk_band; its phase, as far as seen
  for (uint32_t part = 0; part < kGeneralParts; ++part) {
    const uint32_t total = part == 0 ? t0 : part == 1 ? t1 : part == 2 ? t2 : t3;
    const uint32_t groups = part == 0 ? g0 : part == 1 ? g1 : part == 2 ? g2 : g3;
    for (uint32_t i = 0; part == 0 || i < held; ++i) {
      uint32_t share;
      if (part == 0) {
        if (threadIdx.x < 64) {  // (a wavefront: a lane per queue)
          const uint32_t lane = lane_id();
          const uint32_t next = held == gridDim.x ? gridDim.x : next_share(
              blockIdx.x, i == 0, gridDim.x,
              [&] {
                const uint32_t q = lane % kQueues;
                return static_cast<uint32_t>(ballot64(lane < kQueues && load_agent(ws.flags + queue_word(q)) <
                                                                            queue_shares(q, gridDim.x)));
              },
              [&](uint32_t q) {
                uint32_t drawn = 0;
                if (lane == 0)
                  drawn = __hip_atomic_fetch_add(ws.flags + queue_word(q), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return first_lane(drawn);
              });
          if (lane == 0) sh_drawn = next;
        }
        __syncthreads();
        share = uniform_u32(sh_drawn);
        if (threadIdx.x == 0 && share < gridDim.x) sh_share[held] = static_cast<uint16_t>(share);
        __syncthreads();
        if (share >= gridDim.x) break;  // none is left
        ++held;
      } else {
        share = uniform_u32(sh_share[i]);
      }
      const TaskRange range = tasks_of(share, gridDim.x, total);
      for (uint32_t q = range.first; q < range.end; ++q) {
        Geometry geo = geo_all;
        TopkOptions opt = opt_all;
        SegCtx sc;
        if constexpr (UNI) {
          sc = row_ctx(q / groups, q % groups, groups, geo, opt);
        } else {
          const WgSlot slot = (part == 0 ? ws.map_level0 : part == 3 ? ws.map_count : ws.map_sweep)[q];
          const Seg sg = ws.segs[slot.seg];
          sc = seg_ctx_of(slot.seg, slot.group, part == 0 ? sg.groups_level0 : part == 3 ? sg.count_blocks : sg.groups_sweep, sg, geo,
                          opt);
        }
        TopkRow* rowp = ws.rows + sc.seg;
        if (sc.seg != seg) {
          seg = sc.seg;
          fast = rowp->fast;  // (written by an earlier launch: the same for the whole problem)
          at = 0;
        }
        if (fast) continue;
        if (at < part) {
          if (threadIdx.x == 0) {
            bool again = false;
            sh_phase = wait_for_part(part, kMostLooks, [&] {
              if (again) __builtin_amdgcn_s_sleep(2);
              again = true;
              return load_agent(&rowp->phase);
            });
          }
          __syncthreads();
          at = uniform_u32(sh_phase);
          __syncthreads();
        }
        const TaskTurn turn = turn_of(part, at);
        if (turn == kTurnStop) {
          if (threadIdx.x == 0) ws.counters[sc.seg * kCountersPerRow + 5] = kMissGaveUp;
          return;
        }
        if (turn == kTurnSkip) continue;
        if (part == 0) general_level0<true>(sh, lds.level0, e, geo, ws, opt, sc, use_guess);
        else if (part == 1) general_level1<true>(sh, lds.level1, e, geo, ws, opt, sc);
        else if (part == 2) general_level2<true>(sh, lds.level2, e, geo, ws, opt, sc);
        else general_count<false, true>(sh, lds.count, e, geo, ws, opt, sc);
        __syncthreads();  // the next task takes the same LDS
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// One wavefront writes the selected entries of chunk c of one selection problem to their places in the list:
// `at` is where the chunk's slice starts, eq_seen how many keys equal to tau lie in earlier chunks (ties are
// taken in coordinate order until r are in).  Coordinates are written relative to the worker's row
// (coord_base = the problem's first coordinate there).  by_coord: the ties to keep are given as "up to and
// including coordinate tie_last of the problem" (k_topk_band) instead of through r and eq_seen.
__device__ __forceinline__ void emit_chunk(uint32_t mode, const float* __restrict__ er, uint32_t d, uint32_t c,
                                           const uint2* __restrict__ candr, uint2 ds,
                                           uint32_t cap, uint32_t tau, uint32_t r, bool all_ties, uint32_t eq_seen,
                                           uint32_t at, int32_t* __restrict__ idx, float* __restrict__ val, uint32_t k,
                                           uint32_t coord_base, bool by_coord, uint32_t tie_last) {
  for_each_round(mode, er, d, c, candr, ds, cap, [&](const Entry4& en, int slots) {
    bool sel[4] = {false, false, false, false};
    if (by_coord) {
      for (int s = 0; s < slots; ++s) {
        const uint32_t key = key_of_bits(en.bits[s]);
        sel[s] = en.ok[s] && (key > tau || (key == tau && en.j[s] <= tie_last));
      }
    } else if (all_ties) {
      for (int s = 0; s < slots; ++s) sel[s] = en.ok[s] && key_of_bits(en.bits[s]) >= tau;
    } else {
      uint64_t be[4];
      uint32_t below = 0, total = 0;
      for (int s = 0; s < slots; ++s) {
        be[s] = ballot64(en.ok[s] && key_of_bits(en.bits[s]) == tau);
        below += count_below(be[s]);
        total += popc64(be[s]);
      }
      uint32_t rank = eq_seen + below;  // ties before this lane's first slot, in coordinate order
      for (int s = 0; s < slots; ++s) {
        const uint32_t key = key_of_bits(en.bits[s]);
        const bool is_eq = en.ok[s] && key == tau;
        sel[s] = en.ok[s] && (key > tau || (is_eq && rank < r));
        rank += is_eq;
      }
      eq_seen += total;
    }
    uint64_t bs[4];
    uint32_t below = 0, total = 0;
    for (int s = 0; s < slots; ++s) {
      bs[s] = ballot64(sel[s]);
      below += count_below(bs[s]);
      total += popc64(bs[s]);
    }
    uint32_t pos = at + below;
    for (int s = 0; s < slots; ++s)
      if (sel[s]) {
        if (pos < k) {  // always true when the counts are consistent
          idx[pos] = static_cast<int32_t>(coord_base + en.j[s]);
          val[pos] = __uint_as_float(en.bits[s]);
        }
        ++pos;
      }
    at += total;
  });
}

// ---------------------------------------------------------------------------------------------
// The last kernel: per chunk of coordinates.  Workers are taken in tiles of kTileWorkers; lane i of a wavefront holds
// what is to be known of worker i of the tile.
//   Selecting: the wavefronts share out the tile's workers.  Where a worker's entries of the chunk go in its
//              list follows from the tables (entries above the threshold in earlier chunks, plus the ties taken there:
//              in coordinate order until r are in); its candidates of the chunk are gone through 64 to a slot, kSlots
//              slots requested while the ones before are worked on.  The selected (coordinate, value) pairs are
//              written to the list and kept in LDS.  What a slot needs of its worker is taken out of the worker's lane when
//              the walk reaches it (64 x 520 chunks, k = d / 20, crowded: 582 -> 561 us a step).
//   Adding:    one barrier later the first wavefront (or, where some worker has many entries, every
//              wavefront for its own quarter of the chunk's coordinates) adds the workers' entries into an LDS tile of
//              the summed gradient, one worker after the other: the fp32 sum has exactly the order i = 0 .. n-1, and
//              one worker's coordinates are distinct and touched by one wavefront only, so there are no atomics and no
//              barrier per worker.  A worker with more selected entries than its share of the LDS is read back from its
//              list.
//   Update:    gbar = sum / n and the AMSGrad moment and parameter lines (server lines of Algorithm 2).
// The loops are kept as loops: a workgroup of a small problem spends more time fetching instructions than executing
// them.
// What bounds it: theta, m, v, vhat read and written in place (the pattern alone takes 75 of the 94 us on the
// ResNet-18 shape, 16 workers, state from HBM), then the slots' instructions and the lists' stores.  Measured against
// the same kernel with the lists read back from memory and a barrier per worker: ResNet-18 98 -> 94 us, GPT-2 shape
// 722 -> 685, 16 x 1 M 28 -> 18.5, 4 x 65536 10.7 -> 8.5, the server's half 87 -> 80.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kTileWorkers = 16;
constexpr uint32_t kSolo = 128;      // up to so many selected entries of every worker one wavefront adds them all
constexpr uint32_t kKept = 2048;     // selected entries of a tile kept in LDS, shared out evenly among its workers

// Wavefronts per chunk.  A chunk's time is the chain of its slots, which more wavefronts share; a grid that fills the chip
// anyway pays for the room they take.  How a row's selection is spread is not known beforehand: evenly, or crowded into the
// few chunks of the layers with large gradients.  Whole steps in us, with sixteen / eight / four, selections spread
// evenly; in a tenth of the row:
//   16 x 245 chunks, k = d / 100   70 / - / 72; 80 / - / 95
//   16 x 300, k = d / 100          88 / 82 / 83; 90 / 93 / 105     64 x 300, k = d / 20    323 / 291 / 306; 351 / 457 / 622
//   16 x 520, k = d / 100          133 / 121 / 122; 122 / 124 / 136
//   64 x 1024, k = d / 100         715 / 673 / 661; 703 / 693 / 740  64 x 1024, k = d / 20   909 / 838 / 818; 913 / 1003 / 1206
//   1 x 1024, k = d / 20           85 / 73 / 71; 83 / 80 / 83
// So a row has sixteen up to 512 chunks, where crowded selections gain more than even ones lose, eight up to 768, and
// beyond that four, or eight where every row keeps more than a hundred entries of a chunk.  Inside every block the
// selection is spread evenly by what it is (16 layers, 64 x 300, one entry in twenty: 380 / 332 / -; 64 x 768: - / 734 /
// 713).
constexpr int kFinalMany = 4, kFinalSome = 8, kFinalFew = 16;
inline int final_wavefronts(uint32_t workgroups, const Geometry& geo, bool uniform) {
  if (uniform) return workgroups <= 256 ? kFinalFew : workgroups <= 640 ? kFinalSome : kFinalMany;
  if (workgroups <= 512) return kFinalFew;
  const bool large = geo.n >= 4 && static_cast<uint64_t>(geo.k) * kChunk >= static_cast<uint64_t>(geo.d) * 100;
  return workgroups <= 768 || large ? kFinalSome : kFinalMany;
}

// ROLE: kWholeStep does all of it; kWorkerHalf writes the lists and stops (the workers' lines of Algorithm 2: the
// lists are the messages); kServerHalf adds up lists that were put into the workspace (the server's lines; where a
// quarter's slice of each list starts was found by the unpacking).
enum : int { kWholeStep = 0, kWorkerHalf = 1, kServerHalf = 2 };

// UNI: one selection problem per worker over its whole row, one workgroup per chunk of the row.  !UNI (not in
// the server's half): top-k inside every block; a workgroup takes one chunk of one block (flat launch over map_final) and
// goes through the workers' segments of that block, which lie a fixed stride apart in every table.
struct FinalCtx {
  uint32_t c;                     // chunk of the problem
  uint32_t base;                  // first coordinate of the chunk, in coordinates of the worker's row
  uint32_t coord_base, d_loc;     // the problem covers coordinates coord_base .. coord_base + d_loc of the row
  uint32_t k_loc, num_chunks, count_cpw, cap;
  bool micro;                     // the list entries are there already (written by the first pass)
  uint32_t row0, row_stride;      // control block of worker i: row0 + i * row_stride
  size_t chunk0, chunk_stride, seloff0, seloff_stride, cand0, cand_stride, list0, list_stride;
};

template <bool UNI>
__device__ __forceinline__ FinalCtx final_ctx(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt,
                                              const TopkFlat& flat) {
  FinalCtx f;
  if (UNI) {
    f.c = blockIdx.x;
    f.base = f.c * kChunk;
    f.coord_base = 0; f.d_loc = geo.d; f.k_loc = geo.k; f.num_chunks = geo.num_chunks; f.count_cpw = geo.count_cpw;
    f.cap = opt.cap;
    f.micro = false;
    f.row0 = 0; f.row_stride = 1;
    f.chunk0 = 0; f.chunk_stride = geo.num_chunks;
    f.seloff0 = 0; f.seloff_stride = geo.num_chunks * kWaves + 1;
    f.cand0 = 0; f.cand_stride = row_cand_pitch(opt.cap, geo.num_chunks);
    f.list0 = 0; f.list_stride = geo.k;
  } else {
    const WgSlot slot = ws.map_final[blockIdx.x];
    const Seg sg = ws.segs[slot.seg];  // worker 0's segment of the block
    f.c = slot.group;
    f.coord_base = sg.coord_base;
    f.base = sg.coord_base + f.c * kChunk;
    f.d_loc = sg.d; f.k_loc = sg.k; f.num_chunks = sg.num_chunks; f.count_cpw = sg.count_cpw;
    f.cap = opt.cap < sg.cap ? opt.cap : sg.cap;
    f.micro = sg.micro != 0;
    f.row0 = slot.seg; f.row_stride = flat.blocks;
    f.chunk0 = sg.chunk_base; f.chunk_stride = flat.chunk_stride;
    f.seloff0 = sg.seloff_base; f.seloff_stride = flat.seloff_stride;
    f.cand0 = sg.cand_base; f.cand_stride = flat.cand_stride;
    f.list0 = sg.list_base; f.list_stride = geo.k;  // a worker's list holds the lists of all its blocks
  }
  return f;
}

// NC: how many of theta, m, v, vhat (in that order) are read and written with ordinary accesses, the others with
// streaming ones (a template parameter: as a run-time choice between otherwise identical branches the compiler
// merges them and drops the hint).
// CLEAR: the residual at the selected coordinates becomes zero at once (nothing is left to a next step).
// QUARTERS: a chunk has a segment of the candidate list for every quarter, else one.
template <int ROLE, bool UNI, int NC, int NW, bool CLEAR, bool QUARTERS>
__global__ __launch_bounds__(NW * 64, NW == kFinalSome ? 6 : 1) void k_topk_final(
    Geometry geo, float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v, float* __restrict__ vhat,
    const float* __restrict__ e, TopkWorkspace ws, TopkOptions opt, AmsParams p, TopkFlat flat) {
  static_assert(UNI || ROLE != kServerHalf, "the server's half works on whole rows");
  static_assert(NW == kWaves || ROLE != kServerHalf, "it knows the offsets of quarters");
  constexpr uint32_t kPart = kChunk / NW;  // coordinates of a wavefront's part of the chunk
  constexpr int kSlots = NW == kFinalFew ? 4 : 8;  // slots of 64 entries requested together (their code is fetched for each)
  static_assert(kTileWorkers % NW == 0 && NW % kWaves == 0 && NW <= 16, "workers and quarters are shared out evenly");
  __shared__ float4 gs4[ROLE == kWorkerHalf ? 1 : kChunk / 4];
  __shared__ float kept_val[ROLE == kWholeStep ? kKept : 1];
  __shared__ uint16_t kept_at[ROLE == kWholeStep ? kKept : 2];  // coordinates within the chunk
  __shared__ uint32_t sh_part[kTileWorkers][NW];  // a worker's selected entries in the chunk's parts
  __shared__ uint32_t sh_at[kTileWorkers];     // where its slice of the list starts
  float* gs = reinterpret_cast<float*>(gs4);
  const FinalCtx f = final_ctx<UNI>(geo, ws, opt, flat);
  const uint32_t c = f.c;
  const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();  // the wavefront's number: a scalar
  const uint32_t c_lo = c * kChunk;                                       // the chunk, in coordinates of the problem
  const uint32_t c_len = f.d_loc - c_lo < kChunk ? f.d_loc - c_lo : kChunk;
  const uint32_t q_lo = c_lo + wave * kPart;                              // this wavefront's part of it
  if (ROLE != kServerHalf && blockIdx.x == 0 && threadIdx.x < 1 + kQueues)  // the general kernel has run
    ws.flags[threadIdx.x < kQueues ? queue_word(threadIdx.x) : 0] = 0;
  // The workers' half has a workgroup per tile of workers, the others one that goes through all tiles.
  const uint32_t i_first = ROLE == kWorkerHalf ? blockIdx.y * kTileWorkers : 0u;
  if (UNI && !CLEAR && ROLE != kServerHalf && c == geo.num_chunks) {  // the workgroup beyond the chunks
    if (i_first == 0 && threadIdx.x < geo.n) set_next(ws.rows + threadIdx.x, f.k_loc, opt);
    return;
  }
  if (ROLE != kServerHalf && c == 0 && i_first == 0) {
    // the next step's first pass allocates its candidate lists from the start
    for (uint32_t i = threadIdx.x; i < geo.n; i += NW * 64) {
      ws.rows[f.row0 + i * f.row_stride].cursor = 0;
      ws.rows[f.row0 + i * f.row_stride].cursor_band = 0;
    }
    if (!UNI && !CLEAR && window_later(geo.n) && wave == NW - 1 && lane < geo.n)  // (it has workers of its own only from NW on)
      set_next(ws.rows + f.row0 + lane * f.row_stride, f.k_loc, opt);
  }
  if (ROLE != kWorkerHalf) {  // (before the tile's barrier: other wavefronts may add here)
#pragma unroll
    for (uint32_t r = 0; r < kPart / 256; ++r)
      gs4[wave * (kPart / 4) + r * 64 + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const uint32_t my_block = c / f.count_cpw;  // count blocks before this chunk's
  const uint32_t d_end = f.coord_base + f.d_loc;  // the chunk's coordinates end here at the latest
  const uint32_t j_lane = f.base + wave * kPart + lane * 4;  // the lane's first coordinate of the worker's row
  // Entries that are in the lists already: put there by the unpacking, or by the first pass for a micro problem.
  const bool listed = ROLE == kServerHalf || (!UNI && f.micro);
  const uint32_t share = kKept / (geo.n < kTileWorkers ? geo.n : kTileWorkers);  // of the LDS, per worker

  // Entries are gone through worker after worker, 64 to a slot.  `cnt` of lane i: the entries of worker i.
  struct Walk {
    uint32_t left;     // workers that follow the present one
    uint32_t i, t, n;  // the present one (kTileWorkers: none is left), its next entry, its entries
  };
  auto next_worker = [](Walk& w, uint32_t cnt) {
    w.i = kTileWorkers;
    w.t = w.n = 0;
    if (w.left) {
      w.i = static_cast<uint32_t>(__builtin_ctz(w.left));
      w.left &= w.left - 1u;
      w.n = __builtin_amdgcn_readlane(cnt, w.i);
    }
  };
  auto next_slot = [&](Walk& w, uint32_t cnt) {
    w.t += 64;
    if (w.t >= w.n) next_worker(w, cnt);
  };
  struct Slots { uint2 en[kSlots]; };

#pragma unroll 1
  for (uint32_t i0 = i_first; i0 < geo.n; i0 += kTileWorkers) {
    if (!listed) {  // uniform
      // ---- selecting: this wavefront's workers are those at lanes wave, wave + NW, ... ----
      const bool have = lane < kTileWorkers && (lane & (NW - 1)) == wave && i0 + lane < geo.n;
      const uint32_t i_lane = have ? i0 + lane : i0;  // (the other lanes read worker i0's tables and ignore them)
      const uint32_t rowi = f.row0 + i_lane * f.row_stride;
      static_assert(offsetof(TopkRow, fast) == 32 && offsetof(TopkRow, mode) == 36 && offsetof(TopkRow, tau) == 40 &&
                    offsetof(TopkRow, r) == 44 && offsetof(TopkRow, ties) == 48 && offsetof(TopkRow, tie_last) == 52,
                    "words read below");
      const uint4 ra = reinterpret_cast<const uint4*>(ws.rows + rowi)[2];
      const uint2 rb = reinterpret_cast<const uint2*>(ws.rows + rowi)[6];
      const size_t chunk_i = f.chunk0 + i_lane * f.chunk_stride + c;
      uint4 da, db = make_uint4(0, 0, 0, 0);  // the chunk's segments of the candidate list: one, or one for every quarter
      if constexpr (QUARTERS) {
        da = reinterpret_cast<const uint4*>(ws.desc)[2 * chunk_i];
        db = reinterpret_cast<const uint4*>(ws.desc)[2 * chunk_i + 1];
      } else {
        const uint2 ds = ws.desc[chunk_i];
        da = make_uint4(ds.x, ds.y, 0, 0);
      }
      const uint4 rec = ws.chunk_rec[f.chunk0 + i_lane * f.chunk_stride + c];
      uint2 pre = make_uint2(0, 0);
      if (my_block) pre = ws.blk_prefix[static_cast<size_t>(rowi) * kMaxCountBlocks + my_block];
      const bool fast = ra.x != 0;
      const bool dense = ra.x != kFastBand && ra.y == kModeDense;
      const bool partial = have && !fast && ra.w != rb.x;  // some of the row's ties are left out
      const uint32_t tau = ra.z, r = ra.w, tie = fast ? rb.y : 0xffffffffu;
      auto inside = [&](uint32_t off, uint32_t n) {  // segments always lie inside the list; never read outside it
        return off > f.cap ? 0u : n > f.cap - off ? f.cap - off : n;
      };
      // the segments as one list: entry q lies at q + shift, where the segment it is in says how far the list is shifted
      const uint32_t end0 = inside(da.x, da.y), end1 = end0 + inside(da.z, da.w), end2 = end1 + inside(db.x, db.y);
      const uint32_t shift0 = da.x, shift1 = da.z - end0, shift2 = db.x - end1, shift3 = db.z - end2;
      uint32_t cnt = end2 + inside(db.z, db.w);
      if (dense) cnt = c_len;    // no list: the chunk's coordinates themselves
      if (!have) cnt = 0;
      const uint32_t dense_mask = static_cast<uint32_t>(ballot64(dense));
      const uint32_t partial_mask = static_cast<uint32_t>(ballot64(partial));
      auto request = [&](Walk& w, Slots& to) {  // the next kSlots slots
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
          to.en[s] = make_uint2(0u, 0u);
          if (w.i < kTileWorkers) {  // wave-uniform
            const uint32_t q = w.t + lane, i = i0 + w.i;
            if (q < w.n) {
              if ((dense_mask >> w.i) & 1u)
                to.en[s] = make_uint2(c_lo + q, __float_as_uint((e + static_cast<int64_t>(i) * geo.ld + f.coord_base + c_lo)[q]));
              else {
                uint32_t at = __builtin_amdgcn_readlane(shift0, w.i);
                if constexpr (QUARTERS) {
                  at = q < static_cast<uint32_t>(__builtin_amdgcn_readlane(end0, w.i)) ? at : __builtin_amdgcn_readlane(shift1, w.i);
                  at = q < static_cast<uint32_t>(__builtin_amdgcn_readlane(end1, w.i)) ? at : __builtin_amdgcn_readlane(shift2, w.i);
                  at = q < static_cast<uint32_t>(__builtin_amdgcn_readlane(end2, w.i)) ? at : __builtin_amdgcn_readlane(shift3, w.i);
                }
                to.en[s] = (ws.cand + f.cand0 + i * f.cand_stride)[q + at];
              }
            }
            next_slot(w, cnt);
          }
        }
      };
      Walk now{static_cast<uint32_t>(ballot64(cnt != 0)), 0, 0, 0};
      next_worker(now, cnt);
      Walk ahead = now;
      Slots cur;
      request(ahead, cur);
      // positions
      uint32_t sums = static_cast<uint32_t>(ballot64(have && !fast && my_block != 0));
      while (sums) {  // the general kernels' problems: the totals of the count blocks before the chunk's are added up
        const uint32_t u = static_cast<uint32_t>(__builtin_ctz(sums));
        sums &= sums - 1u;
        const uint2* blk = ws.blk + static_cast<size_t>(f.row0 + (i0 + u) * f.row_stride) * kMaxCountBlocks;
        uint2 sum = make_uint2(0, 0);
        for (uint32_t b = lane; b < my_block; b += 64) {
          const uint2 t = blk[b];
          sum.x += t.x;
          sum.y += t.y;
        }
        const uint32_t sx = wave_sum(sum.x), sy = wave_sum(sum.y);
        if (lane == u) pre = make_uint2(sx, sy);
      }
      uint32_t at = pre.x + rec.z;  // where the worker's next entry goes
      uint32_t eq = 0;              // keys equal to tau so far (rows with ties to leave out)
      if (ra.x == kFastPick) {
        at = rec.z;                 // (the prefix over the whole row)
      } else if (fast) {
        // Selected by k_topk_band: the kept entries of the threshold's bucket are not in the tables; pre.y of them lie
        // before the chunk's count block, and those between the block's start and the chunk are counted here (their
        // coordinates are ascending, 0xffffffff beyond the last).
        const uint32_t* sel = ws.bnd_sel + static_cast<size_t>(rowi) * kBoundaryCap;
        uint32_t nb = pre.y;
        while (nb < kBoundaryCap && sel[nb] < c_lo) ++nb;
        at += nb;
      } else {
        eq = pre.y + rec.w;
        at += eq < r ? eq : r;  // ties go in coordinate order until r are in
      }
      const uint32_t at_first = at;
      if (lane < NW)
#pragma unroll
        for (uint32_t i = wave; i < kTileWorkers; i += NW) sh_part[i][lane] = 0;
      // What the slots of the present worker need, the same in every lane: taken out of its lane once.
      uint32_t tau_i = 0, tie_i = 0, at_i = 0, first_i = 0, eq_i = 0, r_i = 0, in_parts = 0;
      bool partial_i = false;
      auto enter = [&] {
        tau_i = __builtin_amdgcn_readlane(tau, now.i);
        tie_i = __builtin_amdgcn_readlane(tie, now.i);
        first_i = __builtin_amdgcn_readlane(at, now.i);
        at_i = first_i;
        partial_i = (partial_mask >> now.i) & 1u;
        if (partial_i) {
          eq_i = __builtin_amdgcn_readlane(eq, now.i);
          r_i = __builtin_amdgcn_readlane(r, now.i);
        }
        in_parts = 0;
      };
      if (now.i < kTileWorkers) enter();
#pragma unroll 1
      while (now.i < kTileWorkers) {
        Slots nxt;
        request(ahead, nxt);
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
          if (now.i < kTileWorkers) {  // wave-uniform
            const uint2 en = cur.en[s];
            const uint32_t key = key_of_bits(en.y);
            const bool ok = now.t + lane < now.n;
            bool is_tie = ok && key == tau_i && en.x <= tie_i;
            if (partial_i) {
              const uint64_t ties = ballot64(is_tie);
              is_tie = is_tie && eq_i + count_below(ties) < r_i;
              eq_i += popc64(ties);
            }
            const bool sel = is_tie || (ok && key > tau_i);
            const uint64_t taken = ballot64(sel);
            // lane u: how many of them lie in part u (the part's number is the coordinate's highest bits in the chunk)
            uint64_t in_part = taken;
#pragma unroll
            for (uint32_t bit = kPart; bit < static_cast<uint32_t>(kChunk); bit *= 2) {
              const uint64_t set = ballot64((en.x & bit) != 0);
              in_part &= (lane & (bit / kPart)) ? set : ~set;
            }
            in_parts += popc64(in_part);
            const uint32_t pos = at_i + count_below(taken);
            if (sel && pos < f.k_loc) {  // (always, when the counts are consistent)
              const size_t l = f.list0 + (i0 + now.i) * f.list_stride + pos;
              ws.idx[l] = static_cast<int32_t>(f.coord_base + en.x);
              ws.val[l] = __uint_as_float(en.y);
              // (nobody reads it again: a chunk of a row without a list is this wavefront's, slot after slot)
              if (CLEAR) const_cast<float*>(e)[static_cast<int64_t>(i0 + now.i) * geo.ld + f.coord_base + en.x] = 0.0f;
            }
            if (ROLE == kWholeStep) {
              const uint32_t kept = pos - first_i;
              if (sel && kept < share) {
                kept_val[now.i * share + kept] = __uint_as_float(en.y);
                kept_at[now.i * share + kept] = static_cast<uint16_t>(en.x - c_lo);
              }
            }
            at_i += popc64(taken);
            now.t += 64;
            if (now.t >= now.n) {  // the worker's last slot
              if (lane == now.i) at = at_i;
              if (lane < NW) sh_part[now.i][lane] = in_parts;
              next_worker(now, cnt);
              if (now.i < kTileWorkers) enter();
            }
          }
        cur = nxt;
      }
      if (have) {
        sh_at[lane] = at_first;
        // the next step's first pass finds the quarters' slices of the list here
        uint32_t* so = ws.sel_off + f.seloff0 + i_lane * f.seloff_stride + c * kWaves;
        uint32_t upto = at_first;
#pragma unroll
        for (uint32_t u = 0; u < NW; ++u) {
          if (u % (NW / kWaves) == 0) so[u / (NW / kWaves)] = upto;
          upto += sh_part[lane][u];
        }
        if (c + 1 == f.num_chunks) so[kWaves] = at;
      }
    } else if (ROLE != kServerHalf && threadIdx.x < kTileWorkers && i0 + threadIdx.x < geo.n) {
      uint32_t* so = ws.sel_off + f.seloff0 + (i0 + threadIdx.x) * f.seloff_stride;  // a micro problem: one chunk
      so[0] = 0;
#pragma unroll
      for (int w = 1; w <= kWaves; ++w) so[w] = f.k_loc;
    }
    if (ROLE == kWorkerHalf) return;
    if (!listed) __syncthreads();

    // ---- adding ----
    uint32_t all = 0, from = 0, part = 0;  // lane i: worker i's selected entries, those before the part, those in it
    if (ROLE == kWholeStep && !listed && lane < kTileWorkers && i0 + lane < geo.n) {
#pragma unroll
      for (uint32_t u = 0; u < NW; ++u) {
        const uint32_t x = sh_part[lane][u];
        all += x;
        from += u < wave ? x : 0u;
        part = u == wave ? x : part;
      }
    }
    if (ROLE == kWholeStep && !listed && ballot64(all > (share < kSolo ? share : kSolo)) == 0) {
      // No worker has more than two slots of selected entries in the chunk: the first wavefront adds them all (a
      // part each would be many more slots, hardly filled).
      if (wave == 0) {
        uint32_t left = static_cast<uint32_t>(ballot64(all != 0));
#pragma unroll 1
        while (left) {
          const uint32_t i = static_cast<uint32_t>(__builtin_ctz(left));
          left &= left - 1u;
          const uint32_t n = __builtin_amdgcn_readlane(all, i);
#pragma unroll
          for (uint32_t t = 0; t < kSolo; t += 64)
            if (t + lane < n) {
              float* g = gs + kept_at[i * share + t + lane];
              *g = *g + kept_val[i * share + t + lane];
            }
          __builtin_amdgcn_wave_barrier();  // the next worker's additions come after this one's
        }
      }
      __syncthreads();
    } else {
      // this wavefront's part of the coordinates
      const bool have = lane < kTileWorkers && i0 + lane < geo.n;
      const uint32_t i_lane = have ? i0 + lane : i0;
      uint32_t first = 0, cnt = 0;  // the worker's entries of the part: from entry `first` of its list on
      if (ROLE == kServerHalf) {
        const uint32_t* so = ws.sel_off_srv + static_cast<size_t>(i_lane) * (geo.num_chunks * kWaves + 1) + c * kWaves + wave;
        first = so[0];
        const uint32_t hi = so[1] < f.k_loc ? so[1] : f.k_loc;
        cnt = have && hi > first ? hi - first : 0u;
      } else if (listed) {
        cnt = have && wave < kMicroCoords / kPart ? f.k_loc : 0u;  // a micro problem: the whole list, of one chunk
      } else if (have) {
        cnt = part;
        first = sh_at[lane] + from;
        if (first > f.k_loc) cnt = 0;  // (never, when the counts are consistent)
        else if (cnt > f.k_loc - first) cnt = f.k_loc - first;
      }
      const uint32_t kept_mask = ROLE == kWholeStep && !listed ? static_cast<uint32_t>(ballot64(all <= share)) : 0u;
      auto request = [&](Walk& w, Slots& to) {
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
          to.en[s] = make_uint2(0u, 0u);
          if (w.i < kTileWorkers) {  // wave-uniform
            const uint32_t e_q = w.t + lane;
            if (e_q < w.n) {
              if ((kept_mask >> w.i) & 1u) {
                const uint32_t l = w.i * share + __builtin_amdgcn_readlane(from, w.i) + e_q;
                to.en[s] = make_uint2(c_lo + kept_at[l], __float_as_uint(kept_val[l]));
              } else {
                const size_t l = f.list0 + (i0 + w.i) * f.list_stride + __builtin_amdgcn_readlane(first, w.i) + e_q;
                to.en[s] = make_uint2(static_cast<uint32_t>(ws.idx[l]) - f.coord_base, __float_as_uint(ws.val[l]));
              }
            }
            next_slot(w, cnt);
          }
        }
      };
      Walk now{static_cast<uint32_t>(ballot64(cnt != 0)), 0, 0, 0};
      next_worker(now, cnt);
      Walk ahead = now;
      Slots cur;
      request(ahead, cur);
#pragma unroll 1
      while (now.i < kTileWorkers) {
        Slots nxt;
        request(ahead, nxt);
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
          if (now.i < kTileWorkers) {  // wave-uniform
            const uint32_t jl = cur.en[s].x - q_lo;
            if (now.t + lane < now.n && jl < kPart) {  // (others' coordinates; a malformed message's lie anywhere)
              float* g = gs + wave * kPart + jl;
              *g = *g + __uint_as_float(cur.en[s].y);
            }
            __builtin_amdgcn_wave_barrier();  // the next worker's additions come after this one's
            next_slot(now, cnt);
          }
        cur = nxt;
      }
    }
    if (!listed && i0 + kTileWorkers < geo.n) __syncthreads();  // the next tile's entries take this one's place in LDS
  }

  if (ROLE == kWorkerHalf) return;
#pragma unroll 1
  for (int r = 0; r < static_cast<int>(kPart / 256); ++r) {
    const uint32_t t = wave * (kPart / 4) + r * 64 + lane;
    const uint32_t j = j_lane + r * 256;
    if (j + 3 < d_end) {
      float4 th = load_state4<(NC > 0)>(theta, j), mm = load_state4<(NC > 1)>(m, j);
      float4 vv = load_state4<(NC > 2)>(v, j), vh = load_state4<(NC > 3)>(vhat, j);
      const float4 s = gs4[t];
      ams_update(s.x / p.nf, th.x, mm.x, vv.x, vh.x, p);
      ams_update(s.y / p.nf, th.y, mm.y, vv.y, vh.y, p);
      ams_update(s.z / p.nf, th.z, mm.z, vv.z, vh.z, p);
      ams_update(s.w / p.nf, th.w, mm.w, vv.w, vh.w, p);
      store_state4<(NC > 0)>(theta, j, th);
      store_state4<(NC > 1)>(m, j, mm);
      store_state4<(NC > 2)>(v, j, vv);
      store_state4<(NC > 3)>(vhat, j, vh);
    } else {
      for (uint32_t s = 0; s < 4 && j + s < d_end; ++s) {
        float th = theta[j + s], mm = m[j + s], vv = v[j + s], vh = vhat[j + s];
        ams_update(gs[4 * t + s] / p.nf, th, mm, vv, vh, p);
        theta[j + s] = th; m[j + s] = mm; v[j + s] = vv; vhat[j + s] = vh;
      }
    }
  }
}

// The residual at the coordinates selected in the last step becomes zero (the worker's error update of
// Algorithm 2 for the kept coordinates), applied on request.
__global__ __launch_bounds__(kWG) void k_topk_apply_clear(float* __restrict__ e, Geometry geo, TopkWorkspace ws) {
  const uint32_t row = blockIdx.y;
  float* er = e + static_cast<int64_t>(row) * geo.ld;
  const int32_t* idx = ws.idx + static_cast<size_t>(row) * geo.k;
  const uint32_t step = gridDim.x * kWG;
  for (uint32_t q = blockIdx.x * kWG + threadIdx.x; q < geo.k; q += step) {
    const uint32_t j = static_cast<uint32_t>(idx[q]);
    if (j < geo.d) er[j] = 0.0f;
  }
}

}  // namespace

#define COMPAMS_CHECK_LAUNCH()                    \
  do {                                            \
    hipError_t err__ = hipGetLastError();         \
    if (err__ != hipSuccess) return err__;        \
  } while (0)

namespace {

// The last kernel with NW wavefronts per chunk.
template <int ROLE, bool UNI, int NW, bool CLEAR, bool QUARTERS, typename... Args>
void launch_final_of(uint32_t n, int cached_arrays, Launcher* L, uint32_t workgroups, hipStream_t stream, Args... args) {
  const uint32_t more = UNI && !CLEAR && ROLE != kServerHalf && window_later(n) ? 1 : 0;  // for the next step's windows
  const dim3 grid(workgroups + more), wg(NW * 64);
  if constexpr (ROLE == kWorkerHalf) {
    // No state, and no order among the workers: a workgroup per tile of them.  With all tiles in one workgroup a few chunks
    // leave the chip idle (50000 coordinates in seven blocks: the half of 300 workers 128 us / 76 as here, of 64 52 / 45).
    const dim3 grid_tiles(workgroups + more, (n + kTileWorkers - 1) / kTileWorkers);
    launch(L, kSlotTopkFinal, k_topk_final<ROLE, UNI, 0, NW, CLEAR, QUARTERS>, grid_tiles, wg, stream, args...);
  } else if constexpr (CLEAR && NW == kFinalFew) {  // (so short that its whole state stays in the memory-side cache)
    launch(L, kSlotTopkFinal, k_topk_final<ROLE, UNI, 4, NW, CLEAR, QUARTERS>, grid, wg, stream, args...);
  } else if constexpr (CLEAR) {  // (a call that stands for itself has no option: four or none)
    if (cached_arrays) launch(L, kSlotTopkFinal, k_topk_final<ROLE, UNI, 4, NW, CLEAR, QUARTERS>, grid, wg, stream, args...);
    else launch(L, kSlotTopkFinal, k_topk_final<ROLE, UNI, 0, NW, CLEAR, QUARTERS>, grid, wg, stream, args...);
  } else {
#define COMPAMS_FINAL(NC) k_topk_final<ROLE, UNI, NC, NW, CLEAR, QUARTERS>
    COMPAMS_LAUNCH_BY_CACHED(cached_arrays, L, kSlotTopkFinal, COMPAMS_FINAL, grid, wg, stream, args...);
#undef COMPAMS_FINAL
  }
}

template <int ROLE, bool UNI, bool CLEAR, bool QUARTERS = false, typename... Args>
void launch_final(const Geometry& geo, int cached_arrays, Launcher* L, uint32_t workgroups, hipStream_t stream, Args... args) {
  switch (final_wavefronts(workgroups, geo, !UNI)) {
    case kFinalFew: launch_final_of<ROLE, UNI, kFinalFew, CLEAR, QUARTERS>(geo.n, cached_arrays, L, workgroups, stream, args...); break;
    case kFinalSome: launch_final_of<ROLE, UNI, kFinalSome, CLEAR, QUARTERS>(geo.n, cached_arrays, L, workgroups, stream, args...); break;
    default: launch_final_of<ROLE, UNI, kFinalMany, CLEAR, QUARTERS>(geo.n, cached_arrays, L, workgroups, stream, args...); break;
  }
}

}  // namespace

// Whether the general route is one launch: where a window gives the band kernel its chance, and the step is short enough
// for three launches to count.  us a step, four launches / one, two dozen steps into a run; windows mostly kept (a fifth
// to a third of the rows miss), thresholds that rise by 15 % a step, that jump tenfold, one magnitude only (the last
// three: most or all rows miss): 4 x 300007 40.9 / 37.3, 49.5 / 51.4, 46.9 / 46.3, 127.6 / 130.0; 8 x 1 M 58.4 / 55.2,
// 72.7 / 77.3, 73.3 / 74.4, 183.2 / 184.9; 16 x 1 M 74.5 / 71.6, 92.4 / 95.8, 95.0 / 95.0, 246.6 / 250.2; 64 x 250007
// 87.5 / 82.7, 104.6 / 105.2, 107.1 / 106.1, 344.6 / 347.2; 1 x 16 M 167.3 / 163.1, 197.0 / 189.0, 222.2 / 219.2, 707.3 /
// 709.4; 8 x 12 blocks of 60000 54.5 / 49.6, 64.5 / 60.5, 72.7 / 70.5, 148.7 / 151.6. Beyond the line the launches are
// less than three per cent of a step.
// Steps of a run that keep much: from two fifths of a row on a list seldom holds and the route is taken in every step (k
// = d / 2.7, d / 2.3, d / 1.5: 4 x 1 M 97.1 / 94.7, 112.8 / 111.6, 137.8 / 143.3; 1 x 4 M 120.5 / 118.7, 137.6 / 136.1,
// 163.1 / 168.6; 4 x 4 M 206.8 / 211.1, 236.2 / 248.2, 276.9 / 339.4; 16 x 1 M, d / 1.5, 231.4 / 302.4), and long lists
// are swept better by a full grid: a million entries of all rows (k = d / 8: 8 x 1 M 91.9 / 90.1, 16 x 1 M 125.1 / 128.1,
// 64 x 200000 153.8 / 157.5, 200 x 70000 288.4 / 303.6).
constexpr uint64_t kOneLaunchChunks = 4096;
// room: entries that a worker's lists hold (a list that the caller's option keeps short is left like a row of which much
// is kept: 16 x 1 M, k = 10000, a list of 20000 146.1 / 155.0).
static bool general_in_one(uint32_t use_guess, const TopkOptions& opt, const Geometry& geo, uint64_t chunks, uint64_t room,
                           bool whole) {
  const uint64_t k = geo.k, n = geo.n;
  return use_guess && opt.band && chunks <= kOneLaunchChunks && (whole || (5 * k <= 2 * room && n * k <= 1u << 20));
}
static_assert(kOneLaunchChunks < kPagedChunks, "k_topk_general counts chunks of one segment");
static_assert((kOneLaunchChunks + 1) * kGeneralMost < (1ull << 32), "tasks_of: a task has a chunk at least");
// (kGeneralMost = 256 / 512 / 1024: 16 x 1 M, rising thresholds 98 / 96 / 108 us a step, one magnitude 279 / 249 / 249; 1
// x 16 M 185 / 191 / 207, 723 / 709 / 720)
static uint32_t general_workgroups(const GeneralTasks& tasks) {
  return std::min(kGeneralMost, *std::max_element(tasks.total, tasks.total + 4));
}

constexpr size_t kClearBytes = 32768;  // a workgroup of the sampling launch clears

hipError_t topk_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& options, const AmsParams& ap,
                     const float* g, float* e, float* theta, float* m, float* v, float* vhat,
                     bool first_pass_may_predict, bool clear_pending, bool workers_only, bool whole, hipStream_t stream,
                     Launcher* L) {
  const int role = workers_only ? kWorkerHalf : kWholeStep;
  const uint32_t G = groups_per_row(geo.n, geo.num_chunks);
  const dim3 wg(kWG);
  const uint32_t use_guess = first_pass_may_predict || whole ? 1u : 0u;
  const bool paged = ws.desc_parts > 1;
  const dim3 grid_first(paged ? page_groups(geo.num_chunks) : geo.num_chunks, geo.n);
  const size_t lds_first = paged ? kLeanLds : 0;
  // Short rows are selected by a workgroup each (where the line lies: see there), unless no row of this step has a guess.
  const bool pick = geo.num_chunks <= kPickChunks && use_guess;
  TopkOptions opt = options;
  if (pick && opt.band) opt.band = kBandWindow;
  if (whole && !sample_gives_window(geo)) opt.band = kBandOff;
  // (4 rows of 300007, k = 3000: level 0 to count 49 us without a guess, with it 38 and 8 for the sample; 4 rows of 65536,
  // k = 655: the whole call 66 us by the general kernels without a guess, 34.4 with it and one workgroup per row)
  if (whole && geo.d >= kSample) {
    const size_t bytes = reinterpret_cast<const char*>(ws.chunk_rec) - reinterpret_cast<const char*>(ws.counters);
    const uint32_t clearing = static_cast<uint32_t>(std::min<size_t>((bytes + kClearBytes - 1) / kClearBytes, 256));
    launch(L, kSlotPick, k_topk_sample, dim3(geo.n + clearing), dim3(kPickThreads), stream, g, e, geo.ld, geo.d, geo.n, geo.k,
           opt.cap, ws.rows, geo, ws, opt);
    COMPAMS_CHECK_LAUNCH();
  }
  auto* first = clear_pending ? (paged ? k_topk_lean<true, true, true> : k_topk_lean<true, true, false>)
                              : (paged ? k_topk_lean<false, true, true> : k_topk_lean<false, true, false>);
  launch_lds(L, kSlotPassA, first, grid_first, wg, lds_first, stream, geo, g, e, ws, opt, use_guess);
  COMPAMS_CHECK_LAUNCH();
  if (pick) {
    launch(L, kSlotPick, k_topk_pick, dim3(1, geo.n), dim3(kPickThreads), stream, geo, e, ws, opt, use_guess);
    COMPAMS_CHECK_LAUNCH();
  } else {
    // the selection in one launch for the rows whose threshold lies in the band; it clears the rows' "fast" mark
    // otherwise, so it runs in every step (about a microsecond when it has nothing to do)
    const uint32_t count_blocks = (geo.num_chunks + geo.count_cpw - 1) / geo.count_cpw;  // <= kMaxCountBlocks
    if (!whole || opt.band) {
      launch(L, kSlotBand, paged ? k_topk_band<true, true> : k_topk_band<true, false>, dim3(count_blocks, geo.n), wg, stream, geo,
             ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
    }
    if (general_in_one(use_guess, opt, geo, static_cast<uint64_t>(geo.n) * geo.num_chunks, opt.cap, whole)) {
      // a task of every part to a workgroup: the second one's clearing, flushing and ticket would follow the first one's
      const uint32_t g1 = std::max(1u, std::min(kGeneralMost / geo.n, G));
      GeneralTasks tasks{{g1, g1, g1, count_blocks}, {}};
      for (uint32_t part = 0; part < kGeneralParts; ++part) tasks.total[part] = tasks.groups[part] * geo.n;
      launch(L, kSlotGeneral, k_topk_general<true>, dim3(general_workgroups(tasks)), wg, stream, ws.flags, e, geo, ws, opt,
             use_guess, tasks);
      COMPAMS_CHECK_LAUNCH();
    } else {
      // level 0 by about two workgroups per compute unit over all rows: each clears and flushes a whole histogram, and the
      // lists are short (measured on the headline workload: 37 us with 128 workgroups per row, 23 us with 32)
      const uint32_t g0 = std::min((512 + geo.n - 1) / geo.n, G);
      launch(L, kSlotLevel0, k_topk_part<true, false, 0>, dim3(g0, geo.n), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotLevel1, k_topk_part<true, false, 1>, dim3(G, geo.n), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotLevel2, k_topk_part<true, false, 2>, dim3(G, geo.n), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotCount, paged ? k_topk_part<true, true, 3> : k_topk_part<true, false, 3>, dim3(count_blocks, geo.n), wg, stream, geo, e,
             ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
    }
  }
  const TopkFlat none{};
  if (whole)
    launch_final<kWholeStep, true, true>(geo, ap.cached_arrays, L, geo.num_chunks, stream, geo, theta, m, v, vhat, e, ws, opt, ap,
                                         none);
  else if (role == kWorkerHalf && paged)
    launch_final<kWorkerHalf, true, false, true>(geo, 0, L, geo.num_chunks, stream, geo, theta, m, v, vhat, e, ws, opt, ap, none);
  else if (role == kWorkerHalf)
    launch_final<kWorkerHalf, true, false>(geo, 0, L, geo.num_chunks, stream, geo, theta, m, v, vhat, e, ws, opt, ap, none);
  else if (paged)
    launch_final<kWholeStep, true, false, true>(geo, ap.cached_arrays, L, geo.num_chunks, stream, geo, theta, m, v, vhat, e, ws, opt,
                                                ap, none);
  else
    launch_final<kWholeStep, true, false>(geo, ap.cached_arrays, L, geo.num_chunks, stream, geo, theta, m, v, vhat, e, ws, opt, ap,
                                          none);
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

// Top-k inside every block: the same kernels over segments (flat launches), then the lists are complete and
// the server's lines run from them.
hipError_t topk_blocks_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt, const AmsParams& ap,
                            const TopkFlat& flat, const float* g, float* e, float* theta, float* m, float* v,
                            float* vhat, bool first_pass_may_predict, bool clear_pending, bool workers_only,
                            hipStream_t stream, Launcher* L) {
  const dim3 wg(kWG);
  const uint32_t use_guess = first_pass_may_predict ? 1u : 0u;
  if (clear_pending)
    launch(L, kSlotPassA, k_topk_lean<true, false, false>, dim3(flat.wg_first), wg, stream, geo, g, e, ws, opt, use_guess);
  else
    launch(L, kSlotPassA, k_topk_lean<false, false, false>, dim3(flat.wg_first), wg, stream, geo, g, e, ws, opt, use_guess);
  COMPAMS_CHECK_LAUNCH();
  if (flat.wg_count) {
    launch(L, kSlotBand, k_topk_band<false, false>, dim3(flat.wg_count), wg, stream, geo, ws, opt, use_guess);
    COMPAMS_CHECK_LAUNCH();
  }
  if (flat.wg_sweep) {  // none if every block is a micro problem
    const GeneralTasks tasks{{}, {flat.wg_level0, flat.wg_sweep, flat.wg_sweep, flat.wg_count}};
    if (general_in_one(use_guess, opt, geo, static_cast<uint64_t>(geo.n) * flat.chunk_stride, geo.d, false)) {
      launch(L, kSlotGeneral, k_topk_general<false>, dim3(general_workgroups(tasks)), wg, stream, ws.flags, e, geo, ws, opt,
             use_guess, tasks);
      COMPAMS_CHECK_LAUNCH();
    } else {
      launch(L, kSlotLevel0, k_topk_part<false, false, 0>, dim3(flat.wg_level0), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotLevel1, k_topk_part<false, false, 1>, dim3(flat.wg_sweep), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotLevel2, k_topk_part<false, false, 2>, dim3(flat.wg_sweep), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
      launch(L, kSlotCount, k_topk_part<false, false, 3>, dim3(flat.wg_count), wg, stream, geo, e, ws, opt, use_guess);
      COMPAMS_CHECK_LAUNCH();
    }
  }
  const float* residuals = e;
  if (workers_only)
    launch_final<kWorkerHalf, false, false>(geo, 0, L, flat.wg_final, stream, geo, theta, m, v, vhat, residuals, ws, opt, ap, flat);
  else
    launch_final<kWholeStep, false, false>(geo, ap.cached_arrays, L, flat.wg_final, stream, geo, theta, m, v, vhat, residuals, ws,
                                           opt, ap, flat);
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

// The server's lines from lists that sit in the workspace (idx, val: n ascending lists of k entries), with the offsets
// of their quarters (sel_off_srv).
hipError_t topk_server_step(const Geometry& geo, const TopkWorkspace& ws, const TopkOptions& opt, const AmsParams& ap,
                            float* theta, float* m, float* v, float* vhat, hipStream_t stream, Launcher* L) {
  const float* no_e = nullptr;
  const TopkFlat none{};
  launch_final_of<kServerHalf, true, kFinalMany, false, false>(geo.n, ap.cached_arrays, L, geo.num_chunks, stream, geo, theta, m, v, vhat,
                                                               no_e, ws, opt, ap, none);
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t topk_apply_clear(const Geometry& geo, const TopkWorkspace& ws, float* e, hipStream_t stream) {
  uint32_t blocks = (geo.k + kWG - 1) / kWG;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_topk_apply_clear, dim3(blocks, geo.n), dim3(kWG), 0, stream, e, geo, ws);
  return hipGetLastError();
}

}  // namespace compams
