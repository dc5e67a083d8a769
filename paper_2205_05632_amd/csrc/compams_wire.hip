// The workers' messages as they would go on the wire (the send line among the worker lines of Algorithm 2),
// and back.  One message per worker, a sequence of 32-bit words:
//
//   top-k      [1, k, 256,  width words,  gap stream,  k value words]
//              gap_0 = idx_0, gap_q = idx_q - idx_{q-1} - 1.  The gaps are taken in tiles of 256 (the last one
//              may be shorter); tile t has its own width b_t = number of bits of its largest gap (at least 1),
//              kept as byte (t mod 4) of width word t div 4 (unused bytes 0).  In the stream the tiles follow
//              one another, each starting on a word boundary: gap i of a tile occupies the tile's bits
//              i*b_t .. i*b_t + b_t - 1, least significant bit first; bit u of a tile is bit (u mod 32) of its
//              word u div 32; unused bits of a tile's last word are 0.
//   block-sign [2, d, M,  ceil(d/32) sign words,  M scale words]
//
// A wavefront owns a tile.  Packing: the tile's gaps are staged in LDS and every stream word is written by one
// lane, which gathers the (at most 32) gaps that overlap it: no atomics touch the message.  Where a tile starts
// in the stream, and the coordinate before its first entry when unpacking, come from prefix sums over the
// tiles of a row: formed by every workgroup for itself where a row has few tiles, else by a launch of its own (one
// workgroup per row).  A message that is not well formed never makes a kernel read outside
// [message, message + stride): counts come from the configuration and widths are clamped to 1 .. 31.

#include "compams_device.h"
#include "compams_internal.h"

namespace compams {
namespace {

static_assert(kWireTile == 256, "a wavefront takes a tile as four gaps per lane");

__device__ __forceinline__ uint32_t gap_of(const int32_t* idx, uint32_t q) {
  const uint32_t cur = static_cast<uint32_t>(idx[q]);
  return q == 0 ? cur : cur - static_cast<uint32_t>(idx[q - 1]) - 1u;
}

__device__ __forceinline__ uint32_t width_of(uint32_t widest) {  // coordinates are below 2^31: at most 31
  return widest ? 32u - static_cast<uint32_t>(__clz(widest)) : 1u;
}

__device__ __forceinline__ uint32_t clamp_width(uint32_t b) { return b < 1u ? 1u : (b > 31u ? 31u : b); }

__device__ __forceinline__ uint32_t tile_count(uint32_t k, uint32_t t) {
  const uint32_t left = k - t * kWireTile;
  return left < kWireTile ? left : kWireTile;
}

__device__ __forceinline__ uint32_t tile_words(uint32_t cnt, uint32_t b) { return (cnt * b + 31u) >> 5; }

__device__ __forceinline__ uint32_t width_byte(const uint32_t* msg, uint32_t t) {
  return (msg[3 + (t >> 2)] >> (8u * (t & 3u))) & 0xffu;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    const uint32_t o = __shfl_xor(v, s, 64);
    v = o > v ? o : v;
  }
  return v;
}

// Widths of the tiles (into the message) and the words each tile will take (into tile_off, to be scanned).
__global__ __launch_bounds__(kWG) void k_wire_tile_width(const int32_t* __restrict__ idx_all, uint32_t k,
                                                          uint32_t tiles, uint32_t* __restrict__ messages,
                                                          int64_t stride, uint32_t* __restrict__ tile_off) {
  __shared__ uint32_t sb[kWaves];
  const uint32_t row = blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t t = blockIdx.x * kWaves + wave;
  const int32_t* idx = idx_all + static_cast<size_t>(row) * k;
  uint32_t b = 0;  // tiles beyond the last one leave a zero byte
  if (t < tiles) {
    const uint32_t cnt = tile_count(k, t);
    uint32_t mx = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t i = lane + 64u * s;
      if (i < cnt) {
        const uint32_t g = gap_of(idx, t * kWireTile + i);
        mx = g > mx ? g : mx;
      }
    }
    b = width_of(wave_max(mx));
    if (lane == 0) tile_off[static_cast<size_t>(row) * tiles + t] = tile_words(cnt, b);
  }
  if (lane == 0) sb[wave] = b;
  __syncthreads();
  if (threadIdx.x == 0)
    messages[static_cast<int64_t>(row) * stride + 3 + blockIdx.x] = sb[0] | (sb[1] << 8) | (sb[2] << 16) | (sb[3] << 24);
}

// Up to this many tiles per row (kDirectTiles * 256 entries of a list) every workgroup of the kernels that need the
// sums over the tiles before its own adds them up itself, four loads per thread at most; the launch between two short
// kernels that this replaces costs 4.7 us (437 tiles x 16 rows: packing 17.1 -> 13.7 us; unpacking, with the offsets of
// the quarters no longer found by a launch of their own, 34.3 -> 21.0 us).
// The work of a row grows with the square of its tiles: longer rows keep the launch.  (The line is one of registers, four
// loads per thread; the gain fades later.  With the launch / without, packing; unpacking, 16 rows: 437 tiles 15.1 / 12.5;
// 20.3 / 17.4 us, 1024 tiles 22.7 / 21.7; 30.2 / 27.6, 4000 tiles 70.5 / 70.8; 84.8 / 83.9.)
constexpr uint32_t kDirectTiles = 1024;

// What lies before tile t0 + (the wavefront's number) of a row's per-tile amounts, and the row's sum.
struct TileSums {
  uint32_t before, total;
};
__device__ __forceinline__ TileSums tile_sums_direct(const uint32_t* __restrict__ amounts, uint32_t tiles, uint32_t t0) {
  __shared__ uint32_t part[2][kWaves];
  const uint32_t wave = threadIdx.x >> 6;
  uint32_t before = 0, total = 0;
#pragma unroll
  for (uint32_t u = 0; u < kDirectTiles / kWG; ++u) {
    const uint32_t t = u * kWG + threadIdx.x;
    const uint32_t a = t < tiles ? amounts[t] : 0u;
    total += a;
    before += t < t0 ? a : 0u;
  }
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    before += __shfl_xor(before, s, 64);
    total += __shfl_xor(total, s, 64);
  }
  if (lane_id() == 0) {
    part[0][wave] = before;
    part[1][wave] = total;
  }
  __syncthreads();
  TileSums r{0, 0};
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    r.before += part[0][w];
    r.total += part[1][w];
    if (static_cast<uint32_t>(w) < wave && t0 + w < tiles) r.before += amounts[t0 + w];
  }
  return r;
}

// In place: per-tile amounts -> what lies before each tile; totals[row] (if given) gets the row's sum.
// One workgroup per row.
__global__ __launch_bounds__(kWG) void k_wire_tile_scan(uint32_t* __restrict__ tiles, uint32_t tiles_per_row,
                                                         uint32_t* __restrict__ totals) {
  __shared__ uint32_t scratch[kWG / 64 + 1];
  uint32_t* t = tiles + static_cast<size_t>(blockIdx.x) * tiles_per_row;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < tiles_per_row; base += kWG) {
    const uint32_t i = base + threadIdx.x;
    const uint32_t v = i < tiles_per_row ? t[i] : 0u;
    uint32_t total;
    const uint32_t before = block_excl_scan<kWG>(v, scratch, &total);
    if (i < tiles_per_row) t[i] = carry + before;
    carry += total;
  }
  if (totals && threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// DIRECT: tile_off holds the words of every tile, not yet summed (and totals nothing).
template <bool DIRECT>
__global__ __launch_bounds__(kWG) void k_wire_pack_topk(const int32_t* __restrict__ idx_all,
                                                         const float* __restrict__ val_all, uint32_t k,
                                                         uint32_t tiles, const uint32_t* __restrict__ tile_off,
                                                         const uint32_t* __restrict__ totals,
                                                         uint32_t* __restrict__ messages, int64_t stride,
                                                         uint32_t* __restrict__ words_out) {
  __shared__ uint32_t sg[kWaves][kWireTile];
  const uint32_t row = blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t t = blockIdx.x * kWaves + wave;
  const int32_t* idx = idx_all + static_cast<size_t>(row) * k;
  const float* val = val_all + static_cast<size_t>(row) * k;
  uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  const uint32_t width_words = (tiles + 3u) >> 2;
  const uint32_t* off_row = tile_off + static_cast<size_t>(row) * tiles;
  TileSums sums;
  if constexpr (DIRECT) sums = tile_sums_direct(off_row, tiles, blockIdx.x * kWaves);
  else sums = TileSums{t < tiles ? off_row[t] : 0u, totals[row]};
  const uint32_t stream_total = sums.total;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    msg[0] = 1u;
    msg[1] = k;
    msg[2] = kWireTile;
    words_out[row] = 3u + width_words + stream_total + k;
  }
  const bool live = t < tiles;
  const uint32_t cnt = live ? tile_count(k, t) : 0u;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t i = lane + 64u * s;
    sg[wave][i] = i < cnt ? gap_of(idx, t * kWireTile + i) : 0u;
  }
  __syncthreads();
  if (live) {
    const uint32_t b = width_byte(msg, t);  // written by the width kernel: 1 .. 31
    uint32_t* stream = msg + 3 + width_words + sums.before;
    const uint32_t nw = tile_words(cnt, b);
    for (uint32_t w = lane; w < nw; w += 64) {
      const uint32_t lo = w * 32u;
      const uint32_t q0 = lo / b;
      uint32_t q1 = (lo + 31u) / b;
      if (q1 > cnt - 1u) q1 = cnt - 1u;
      uint32_t word = 0;
      for (uint32_t q = q0; q <= q1; ++q) {
        const uint32_t g = sg[wave][q];
        const int32_t sh = static_cast<int32_t>(q * b) - static_cast<int32_t>(lo);
        word |= sh >= 0 ? (g << sh) : (g >> (-sh));  // |sh| <= 31
      }
      stream[w] = word;
    }
  }
  uint32_t* values = msg + 3 + width_words + stream_total;
  const uint32_t step = gridDim.x * kWG;
  for (uint32_t q = blockIdx.x * kWG + threadIdx.x; q < k; q += step) values[q] = __float_as_uint(val[q]);
}

// Gap i of a tile whose stream starts at `tile` and has nw words (i < cnt, so the field lies inside them).
__device__ __forceinline__ uint32_t field_of(const uint32_t* __restrict__ tile, uint32_t nw, uint32_t i, uint32_t b) {
  const uint32_t pos = i * b;
  const uint32_t w = pos >> 5, sh = pos & 31u;
  uint64_t two = tile[w];
  if (w + 1 < nw) two |= static_cast<uint64_t>(tile[w + 1]) << 32;
  return static_cast<uint32_t>(two >> sh) & ((1u << b) - 1u);
}

// status[row]: 0 well formed; bit 0: not a message of this kind and size, or a width outside 1 .. 31; bit 1 (set
// while unpacking): length differs; bit 2 (set while unpacking): a coordinate at or beyond d.
// Also leaves in tile_off where each tile starts in its stream (from the clamped widths), and the stream's length in
// totals[row].  One workgroup per row.
__global__ __launch_bounds__(kWG) void k_wire_check_topk(const uint32_t* __restrict__ messages, int64_t stride,
                                                          uint32_t k, uint32_t tiles,
                                                          uint32_t* __restrict__ tile_off,
                                                          uint32_t* __restrict__ totals,
                                                          uint32_t* __restrict__ status) {
  __shared__ uint32_t st;
  __shared__ uint32_t scratch[kWG / 64 + 1];
  const uint32_t row = blockIdx.x;
  const uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  if (threadIdx.x == 0) st = (msg[0] != 1u || msg[1] != k || msg[2] != kWireTile) ? 1u : 0u;
  __syncthreads();
  bool bad = false;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < tiles; base += kWG) {
    const uint32_t t = base + threadIdx.x;
    uint32_t words = 0;
    if (t < tiles) {
      const uint32_t b = width_byte(msg, t);
      bad |= b < 1u || b > 31u;
      words = tile_words(tile_count(k, t), clamp_width(b));
    }
    uint32_t total;
    const uint32_t before = block_excl_scan<kWG>(words, scratch, &total);
    if (t < tiles) tile_off[static_cast<size_t>(row) * tiles + t] = carry + before;
    carry += total;
  }
  if (bad) atomicOr(&st, 1u);
  __syncthreads();
  if (threadIdx.x == 0) {
    status[row] = st;
    totals[row] = carry;
  }
}

// The gaps of a lane's four consecutive entries of tile t (zero beyond the tile) and their number.
struct LaneGaps {
  uint32_t gap[4];
  uint32_t n;
};
// start: where the tile starts in the stream.
__device__ __forceinline__ LaneGaps lane_gaps(const uint32_t* __restrict__ msg, uint32_t k, uint32_t tiles, uint32_t t,
                                              uint32_t start) {
  const uint32_t lane = lane_id();
  const uint32_t cnt = tile_count(k, t);
  const uint32_t b = clamp_width(width_byte(msg, t));
  const uint32_t* tile = msg + 3 + ((tiles + 3u) >> 2) + start;
  const uint32_t nw = tile_words(cnt, b);
  LaneGaps g;
  g.n = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t i = lane * 4u + s;
    g.gap[s] = 0;
    if (i < cnt) {
      g.gap[s] = field_of(tile, nw, i, b);
      g.n = s + 1;
    }
  }
  return g;
}

__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
  return v;
}

// Coordinates covered by each tile (sum of gap + 1), to be scanned into the coordinate before each tile.
__global__ __launch_bounds__(kWG) void k_wire_tile_sums(const uint32_t* __restrict__ messages, int64_t stride,
                                                         uint32_t k, uint32_t tiles,
                                                         const uint32_t* __restrict__ tile_off,
                                                         uint32_t* __restrict__ tile_sum) {
  const uint32_t row = blockIdx.y, wave = threadIdx.x >> 6;
  const uint32_t t = blockIdx.x * kWaves + wave;
  if (t >= tiles) return;  // wave-uniform; no barrier below
  const uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  const LaneGaps g = lane_gaps(msg, k, tiles, t, tile_off[static_cast<size_t>(row) * tiles + t]);
  uint32_t sum = g.n;
#pragma unroll
  for (int s = 0; s < 4; ++s) sum += g.gap[s];
  sum = wave_total(sum);
  if (lane_id() == 0) tile_sum[static_cast<size_t>(row) * tiles + t] = sum;
}

// Both at once for rows of up to kDirectTiles tiles: every workgroup goes through the row's widths itself, four of them
// (a word) to a thread, for what lies before its own four tiles; the first one leaves status and total.  What it saves is
// a launch of one workgroup per row (a step in two halves, us, with that launch / so: 16 x 1 M, k = 10000 89.4 / 88.0; 16
// x 11181642, k = 111816 485.6 / 483.5; 64 x 1 M 208.8 / 207.6; 8 x 25 M, k = 262144, 1024 tiles, 620.4 / 617.6).
__global__ __launch_bounds__(kWG) void k_wire_measure_topk(const uint32_t* __restrict__ messages, int64_t stride, uint32_t k,
                                                            uint32_t tiles, uint32_t* __restrict__ tile_off,
                                                            uint32_t* __restrict__ totals, uint32_t* __restrict__ status,
                                                            uint32_t* __restrict__ tile_sum) {
  static_assert(kDirectTiles <= 4 * kWG && kWaves == 4, "a word of widths to a thread, and to a workgroup's tiles");
  __shared__ uint32_t part[3][kWaves];
  const uint32_t row = blockIdx.y, wave = threadIdx.x >> 6, word = threadIdx.x;
  const uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  // words of a tile, and whether its width is one
  auto tile = [&](uint32_t widths, uint32_t t, bool& bad) {
    const uint32_t b = (widths >> (8u * (t & 3u))) & 0xffu;
    bad |= t < tiles && (b < 1u || b > 31u);
    return t < tiles ? tile_words(tile_count(k, t), clamp_width(b)) : 0u;
  };
  uint32_t total = 0;
  bool bad = false;
  if (4 * word < tiles) {
    const uint32_t widths = msg[3 + word];
#pragma unroll
    for (uint32_t s = 0; s < 4; ++s) total += tile(widths, 4 * word + s, bad);
  }
  uint32_t before = word < blockIdx.x ? total : 0u;
  before = wave_total(before);
  total = wave_total(total);
  const bool wave_bad = ballot64(bad) != 0;
  if (lane_id() == 0) {
    part[0][wave] = before;
    part[1][wave] = total;
    part[2][wave] = wave_bad ? 1u : 0u;
  }
  __syncthreads();
  before = total = 0;
  uint32_t any = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    before += part[0][w];
    total += part[1][w];
    any |= part[2][w];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    status[row] = any | (msg[0] != 1u || msg[1] != k || msg[2] != kWireTile ? 1u : 0u);
    totals[row] = total;
  }
  const uint32_t t = blockIdx.x * kWaves + wave;
  if (t >= tiles) return;  // wave-uniform; no barrier below
  const uint32_t widths = msg[3 + blockIdx.x];
  for (uint32_t s = 0; s < wave; ++s) before += tile(widths, blockIdx.x * kWaves + s, bad);
  const LaneGaps g = lane_gaps(msg, k, tiles, t, before);
  uint32_t sum = g.n;
#pragma unroll
  for (int s = 0; s < 4; ++s) sum += g.gap[s];
  sum = wave_total(sum);
  if (lane_id() == 0) {
    tile_off[static_cast<size_t>(row) * tiles + t] = before;
    tile_sum[static_cast<size_t>(row) * tiles + t] = sum;
  }
}

// DIRECT: tile_sum holds the coordinates each tile covers, not yet summed.  quarter_off (OFFSETS): where the slice of
// the list starts that belongs to each quarter (kChunk / kWaves coordinates) of a chunk, `quarters` + 1 words per row
// = number of listed coordinates below each quarter: entry q fills the quarters between its predecessor's (exclusive)
// and its own (inclusive), beyond the last entry follows one that fills the rest.  A short gap is filled by the entry's
// own lane, a long one by the whole wavefront (the kept coordinates crowd into a few layers: one lane that wrote all
// the quarters of a layer without any took 30 us).
template <bool DIRECT, bool OFFSETS>
__global__ __launch_bounds__(kWG) void k_wire_unpack_topk(const uint32_t* __restrict__ messages, int64_t stride,
                                                           const uint32_t* __restrict__ words, uint32_t k,
                                                           uint32_t d, uint32_t tiles,
                                                           const uint32_t* __restrict__ tile_off,
                                                           const uint32_t* __restrict__ totals,
                                                           const uint32_t* __restrict__ tile_sum,
                                                           int32_t* __restrict__ idx_out, float* __restrict__ val_out,
                                                           uint32_t* __restrict__ status, uint32_t quarters,
                                                           uint32_t* __restrict__ quarter_off) {
  const uint32_t row = blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t t = blockIdx.x * kWaves + wave;
  const uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  const uint32_t width_words = (tiles + 3u) >> 2;
  const uint32_t stream_total = totals[row];
  if (blockIdx.x == 0 && threadIdx.x == 0 && words && words[row] != 3u + width_words + stream_total + k)
    atomicOr(&status[row], 2u);
  uint32_t tile_before;
  if constexpr (DIRECT) tile_before = tile_sums_direct(tile_sum + static_cast<size_t>(row) * tiles, tiles, blockIdx.x * kWaves).before;
  else tile_before = t < tiles ? tile_sum[static_cast<size_t>(row) * tiles + t] : 0u;
  if (t < tiles) {  // wave-uniform
    const LaneGaps g = lane_gaps(msg, k, tiles, t, tile_off[static_cast<size_t>(row) * tiles + t]);
    uint32_t mine = g.n;
#pragma unroll
    for (int s = 0; s < 4; ++s) mine += g.gap[s];
    // coordinates before this lane's first entry: those before the tile + those of the lanes below
    uint32_t pos = tile_before + wave_incl_scan(mine) - mine;
    int32_t* idx = idx_out + static_cast<size_t>(row) * k + t * kWireTile + lane * 4u;
    bool beyond = false;
    constexpr uint32_t kQuarter = kChunk / kWaves, kShort = 4;
    uint32_t* so = OFFSETS ? quarter_off + static_cast<size_t>(row) * (quarters + 1) : nullptr;
    auto quarter_of = [&](uint32_t j) {  // (a coordinate beyond d is flagged below)
      const uint32_t u = j / kQuarter;
      return u < quarters ? u : quarters - 1;
    };
    auto fill = [&](uint32_t from, uint32_t to, uint32_t q) {  // quarters from .. to - 1 start at entry q of the list
      const uint32_t gap = to > from ? to - from : 0u;         // (a malformed message's coordinates may wrap)
      if (gap <= kShort)
        for (uint32_t u = 0; u < gap; ++u) so[from + u] = q;
      uint64_t big = ballot64(gap > kShort);
      while (big) {
        const int l = __builtin_ctzll(big);
        big &= big - 1;
        const uint32_t lo = __builtin_amdgcn_readlane(from, l), hi = __builtin_amdgcn_readlane(to, l);
        const uint32_t at = __builtin_amdgcn_readlane(q, l);
        for (uint32_t u = lo + lane; u < hi; u += 64) so[u] = at;
      }
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool there = static_cast<uint32_t>(s) < g.n;
      const uint32_t q = t * kWireTile + lane * 4u + s;
      uint32_t from = 0, to = 0;
      if (there) {
        const uint32_t j = pos + g.gap[s];
        beyond |= j >= d;
        idx[s] = static_cast<int32_t>(j);
        if (OFFSETS) {
          from = q ? quarter_of(pos - 1u) + 1u : 0u;  // (pos - 1: the entry before)
          to = quarter_of(j) + 1u;
        }
        pos = j + 1u;
      }
      if (OFFSETS) fill(from, to, q);
    }
    if (OFFSETS && t + 1 == tiles) {  // wave-uniform: the quarters after the last entry
      const bool last = g.n != 0 && t * kWireTile + lane * 4u + g.n == k;
      fill(last ? quarter_of(pos - 1u) + 1u : 0u, last ? quarters + 1u : 0u, k);
    }
    if (beyond) atomicOr(&status[row], 4u);
  }
  const uint32_t* values = msg + 3 + width_words + stream_total;
  float* val = val_out + static_cast<size_t>(row) * k;
  const uint32_t step = gridDim.x * kWG;
  for (uint32_t q = blockIdx.x * kWG + threadIdx.x; q < k; q += step) val[q] = __uint_as_float(values[q]);
}

__global__ __launch_bounds__(kWG) void k_wire_pack_blocksign(const uint32_t* __restrict__ bits_all,
                                                              const float* __restrict__ scales_all, uint32_t d,
                                                              uint32_t words, uint32_t M,
                                                              uint32_t* __restrict__ messages, int64_t stride,
                                                              uint32_t* __restrict__ words_out) {
  const uint32_t row = blockIdx.y;
  uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    msg[0] = 2u;
    msg[1] = d;
    msg[2] = M;
    words_out[row] = 3u + words + M;
  }
  const uint32_t* bits = bits_all + static_cast<size_t>(row) * words;
  const float* mu = scales_all + static_cast<size_t>(row) * M;
  const uint32_t step = gridDim.x * kWG;
  for (uint32_t w = blockIdx.x * kWG + threadIdx.x; w < words; w += step) msg[3 + w] = bits[w];
  for (uint32_t b = blockIdx.x * kWG + threadIdx.x; b < M; b += step) msg[3 + words + b] = __float_as_uint(mu[b]);
}

__global__ __launch_bounds__(kWG) void k_wire_unpack_blocksign(const uint32_t* __restrict__ messages, int64_t stride,
                                                                const uint32_t* __restrict__ words_in, uint32_t d,
                                                                uint32_t words, uint32_t M,
                                                                uint32_t* __restrict__ bits_out,
                                                                float* __restrict__ scales_out,
                                                                uint32_t* __restrict__ status) {
  const uint32_t row = blockIdx.y;
  const uint32_t* msg = messages + static_cast<int64_t>(row) * stride;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    uint32_t st = 0;
    if (msg[0] != 2u || msg[1] != d || msg[2] != M) st |= 1u;
    else if (words_in && words_in[row] != 3u + words + M) st |= 2u;
    status[row] = st;
  }
  uint32_t* bits = bits_out + static_cast<size_t>(row) * words;
  float* mu = scales_out + static_cast<size_t>(row) * M;
  const uint32_t step = gridDim.x * kWG;
  for (uint32_t w = blockIdx.x * kWG + threadIdx.x; w < words; w += step) bits[w] = msg[3 + w];
  for (uint32_t b = blockIdx.x * kWG + threadIdx.x; b < M; b += step) mu[b] = __uint_as_float(msg[3 + words + b]);
}

#define COMPAMS_CHECK_LAUNCH()                    \
  do {                                            \
    hipError_t err__ = hipGetLastError();         \
    if (err__ != hipSuccess) return err__;        \
  } while (0)

uint32_t copy_groups(uint32_t n, uint64_t items) {
  uint64_t g = (items + kWG * 8 - 1) / (kWG * 8);  // eight items per thread
  const uint64_t most = (256 * 8 + n - 1) / n;
  if (g > most) g = most;
  return g < 1 ? 1u : static_cast<uint32_t>(g);
}

}  // namespace

hipError_t wire_encode_topk(const Geometry& geo, const TopkWorkspace& ws, uint32_t* messages, int64_t stride,
                            uint32_t* words_out, hipStream_t stream, Launcher* L) {
  const uint32_t tiles = (geo.k + kWireTile - 1) / kWireTile;
  const dim3 grid((tiles + kWaves - 1) / kWaves, geo.n), wg(kWG);
  launch(L, kSlotWireEncode, k_wire_tile_width, grid, wg, stream, ws.idx, geo.k, tiles, messages, stride,
         ws.wire_tile_off);
  COMPAMS_CHECK_LAUNCH();
  if (tiles <= kDirectTiles) {
    launch(L, kSlotWireEncode, k_wire_pack_topk<true>, grid, wg, stream, ws.idx, ws.val, geo.k, tiles, ws.wire_tile_off,
           ws.wire_total, messages, stride, words_out);
  } else {
    launch(L, kSlotWireEncode, k_wire_tile_scan, dim3(geo.n), wg, stream, ws.wire_tile_off, tiles, ws.wire_total);
    COMPAMS_CHECK_LAUNCH();
    launch(L, kSlotWireEncode, k_wire_pack_topk<false>, grid, wg, stream, ws.idx, ws.val, geo.k, tiles, ws.wire_tile_off,
           ws.wire_total, messages, stride, words_out);
  }
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t wire_decode_topk(const Geometry& geo, const TopkWorkspace& ws, const uint32_t* messages, int64_t stride,
                            const uint32_t* words, int32_t* idx_out, float* val_out, uint32_t* status,
                            bool quarter_offsets, hipStream_t stream, Launcher* L) {
  const uint32_t tiles = (geo.k + kWireTile - 1) / kWireTile;
  const dim3 grid((tiles + kWaves - 1) / kWaves, geo.n), wg(kWG);
  uint32_t* none = nullptr;
  const bool direct = tiles <= kDirectTiles;
  if (direct) {
    launch(L, kSlotWireDecode, k_wire_measure_topk, grid, wg, stream, messages, stride, geo.k, tiles, ws.wire_tile_off, ws.wire_total,
           status, ws.wire_tile_sum);
    COMPAMS_CHECK_LAUNCH();
  } else {
    launch(L, kSlotWireDecode, k_wire_check_topk, dim3(geo.n), wg, stream, messages, stride, geo.k, tiles,
           ws.wire_tile_off, ws.wire_total, status);
    COMPAMS_CHECK_LAUNCH();
    launch(L, kSlotWireDecode, k_wire_tile_sums, grid, wg, stream, messages, stride, geo.k, tiles, ws.wire_tile_off,
           ws.wire_tile_sum);
    COMPAMS_CHECK_LAUNCH();
    launch(L, kSlotWireDecode, k_wire_tile_scan, dim3(geo.n), wg, stream, ws.wire_tile_sum, tiles, none);
    COMPAMS_CHECK_LAUNCH();
  }
  const uint32_t quarters = geo.num_chunks * kWaves;
#define COMPAMS_UNPACK(D, O)                                                                                         \
  launch(L, kSlotWireDecode, k_wire_unpack_topk<D, O>, grid, wg, stream, messages, stride, words, geo.k, geo.d, tiles, \
         ws.wire_tile_off, ws.wire_total, ws.wire_tile_sum, idx_out, val_out, status, quarters, ws.sel_off_srv)
  if (direct && quarter_offsets) COMPAMS_UNPACK(true, true);
  else if (direct) COMPAMS_UNPACK(true, false);
  else if (quarter_offsets) COMPAMS_UNPACK(false, true);
  else COMPAMS_UNPACK(false, false);
#undef COMPAMS_UNPACK
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t wire_encode_blocksign(const Geometry& geo, const BlocksignWorkspace& ws, uint32_t* messages, int64_t stride,
                                 uint32_t* words_out, hipStream_t stream, Launcher* L) {
  const dim3 grid(copy_groups(geo.n, geo.words), geo.n), wg(kWG);
  launch(L, kSlotWireEncode, k_wire_pack_blocksign, grid, wg, stream, ws.bits, ws.scales, geo.d, geo.words,
         geo.num_blocks, messages, stride, words_out);
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t wire_decode_blocksign(const Geometry& geo, const uint32_t* messages, int64_t stride, const uint32_t* words,
                                 uint32_t* bits_out, float* scales_out, uint32_t* status, hipStream_t stream,
                                 Launcher* L) {
  const dim3 grid(copy_groups(geo.n, geo.words), geo.n), wg(kWG);
  launch(L, kSlotWireDecode, k_wire_unpack_blocksign, grid, wg, stream, messages, stride, words, geo.d, geo.words,
         geo.num_blocks, bits_out, scales_out, status);
  COMPAMS_CHECK_LAUNCH();
  return hipSuccess;
}

}  // namespace compams
