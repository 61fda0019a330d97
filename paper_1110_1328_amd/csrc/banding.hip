// LSH banding candidate generation (Section 2): the hashes of an object are
// cut into n_bands bands of band_bits sign-random-projection bits each, and
// objects whose band key is equal in some band become a candidate pair.  A
// pair is emitted once, in the first band where its two keys are equal.
//
// On the device, for a group of bands at once (all of them unless the
// workspace is too small for that; n objects, N = bands n positions):
//   keys      every object's key of every band: the sort's (band, key) keys,
//             and a row of keys per object for the earlier-band test;
//   sort      (key, id) pairs by (band, key), stable (rocPRIM radix sort): the
//             bands one after another, each bucket listing its members by
//             increasing id;
//   buckets   the start of every position's bucket and every bucket's end;
//   row order (order_tile = 0), band by band: one wave per member row p counts
//             its partners q in (p, end) that share no earlier band; a scan of
//             the row counts (rocPRIM) gives the offsets; the same walk writes
//             (x, y) = (ids[p], ids[q]);
//   tiled order (order_tile = 16): a bucket's member pairs by 16 x 16 tiles.
//             A strip is one tile row of a bucket (16 members against the
//             bucket's members from there on); the strips are listed with
//             their first tile's number, one wave per strip runs the
//             earlier-band test (each tile's 256-bit mask) and a scan of the
//             strips' pair counts (rocPRIM) gives the candidate numbers.  Pairs
//             are then written from the masks; tile descriptors are written by
//             the test itself and get their first candidate's number after.
// The output order is band by band, bucket by increasing key, then the
// bucket's pairs in the order asked for, x < y.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "device_common.h"

namespace blsh {

constexpr int kBandBlock = 256;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Sort keys and ids of bands [j0, j0 + group): key[(j - j0) n + i] = (j - j0)
// << band_bits | bits [j b, j b + b) of object i's signature (LSB-first), with
// its id beside it.  With rows != null also the object's row of all n_bands
// keys: `stride` words apart, two keys of at most 16 bits to a word (PACK; the
// even band in the low half) or one.
template <bool PACK>
__global__ __launch_bounds__(kBandBlock) void k_band_keys(const uint32_t *sig, int64_t n_obj, int32_t row_words,
                                                          int32_t word_major, int32_t n_bands, int32_t band_bits,
                                                          int32_t j0, int32_t group, uint32_t *keys, uint32_t *ids,
                                                          uint32_t *rows, int32_t stride) {
  const int64_t i = int64_t(blockIdx.x) * kBandBlock + threadIdx.x;
  if (i >= n_obj) return;
  const uint32_t mask = band_bits == 32 ? 0xFFFFFFFFu : ((1u << band_bits) - 1u);
  auto word = [&](int w) -> uint32_t {
    return word_major ? sig[size_t(w) * n_obj + i] : sig[size_t(i) * row_words + w];
  };
  uint32_t low = 0;
  const int first = rows ? 0 : j0, last = rows ? n_bands : j0 + group;
  for (int j = first; j < last; ++j) {
    const int o = j * band_bits, w = o >> 5, sh = o & 31;
    uint32_t v = word(w) >> sh;
    if (sh + band_bits > 32) v |= word(w + 1) << (32 - sh);
    v &= mask;
    if (j >= j0 && j < j0 + group) {   // (a group of several bands: band_bits < 32)
      keys[size_t(j - j0) * n_obj + i] = group > 1 ? uint32_t(j - j0) << band_bits | v : v;
      ids[size_t(j - j0) * n_obj + i] = uint32_t(i);
    }
    if (rows) {
      if constexpr (PACK) {
        if (j & 1) rows[size_t(i) * stride + (j >> 1)] = low | v << 16;
        else if (j == n_bands - 1) rows[size_t(i) * stride + (j >> 1)] = v;
        low = v;
      } else {
        rows[size_t(i) * stride + j] = v;
      }
    }
  }
}

// Buckets of the sorted keys, kBoundChunk positions to a wave.  last[chunk] = the
// last position of the chunk where a bucket starts, 0 if none does (position 0,
// where one starts, reads the same): the chunk from its end until one is found.
constexpr int kBoundChunk = 256;
__device__ inline int64_t bound_chunk() {
  return int64_t(blockIdx.x) * (kBandBlock / kWave) + int64_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
}
__global__ __launch_bounds__(kBandBlock) void k_bucket_last(const uint32_t *skeys, int64_t n, uint32_t *last) {
  const int64_t chunk = bound_chunk(), p0 = chunk * kBoundChunk;
  if (p0 >= n) return;
  uint32_t found = 0;
  for (int64_t q = p0 + kBoundChunk - kWave; q >= p0 && found == 0; q -= kWave) {
    const int64_t p = q + lane_id();
    const uint64_t mask = __ballot(p < n && p > 0 && skeys[p] != skeys[p - 1]);
    if (mask != 0) found = uint32_t(q) + 63u - uint32_t(__clzll(mask));
  }
  if (lane_id() == 0) last[chunk] = found;
}

// bstart[p] = the start of p's bucket; bend[s] = the end of the bucket that
// starts at s (written at bucket starts only).  A chunk's first bucket is found
// from the chunks before it, 64 at a time.  (The call of 16 bands of 1M objects:
// 3.56 ms, 3.64 with a library's scan between two kernels.)
__global__ __launch_bounds__(kBandBlock) void k_bucket_bounds(const uint32_t *skeys, int64_t n, const uint32_t *last,
                                                              uint32_t *bstart, uint32_t *bend) {
  const int64_t chunk = bound_chunk(), p0 = chunk * kBoundChunk;
  if (p0 >= n) return;
  const int lane = lane_id();
  uint32_t start = 0;   // of the bucket that position q - 1 is in
  for (int64_t b = chunk; b > 0; b -= kWave) {
    const uint32_t v = b - 1 - lane >= 0 ? last[b - 1 - lane] : 0u;
    const uint64_t mask = __ballot(v != 0);
    if (mask != 0) {
      start = uint32_t(__builtin_amdgcn_readlane(int(v), __ffsll((unsigned long long)mask) - 1));
      break;
    }
  }
  const int64_t p1 = min<int64_t>(n, p0 + kBoundChunk);
  for (int64_t q = p0; q < p1; q += kWave) {
    const int64_t p = q + lane;
    const bool in = p < p1, first = in && p > 0 && skeys[p] != skeys[p - 1];
    const uint64_t mask = __ballot(first);
    auto start_at = [&](uint64_t m) { return m != 0 ? uint32_t(q) + 63u - uint32_t(__clzll(m)) : start; };
    const uint64_t below = mask & ((1ull << lane) - 1ull);
    const uint32_t before = start_at(below), mine = first ? uint32_t(p) : before;
    if (first) bend[before] = uint32_t(p);
    if (in) bstart[p] = mine;
    if (p + 1 == n) bend[mine] = uint32_t(n);
    start = start_at(mask);
  }
}

// Row order: bstart[p] becomes the end of p's partners, in place (a row then takes
// one read for its bounds, not a chain of two: 1 band of 1M objects, 65,536 buckets,
// 518 -> 452 us).
__global__ __launch_bounds__(kBandBlock) void k_bucket_row_ends(uint32_t *bstart, const uint32_t *bend, int64_t n,
                                                                int32_t max_bucket) {
  const int64_t p = int64_t(blockIdx.x) * kBandBlock + threadIdx.x;
  if (p >= n) return;
  const uint32_t s = bstart[p], e = bend[s];
  bstart[p] = max_bucket > 0 ? s + min(e - s, uint32_t(max_bucket)) : e;
}

struct BandArgs {
  const uint32_t *sids;      // sorted ids of the group
  const uint32_t *ends;      // of each position's partners
  const uint32_t *rows;      // [n_obj][stride]
  int32_t stride;
  int64_t n_obj;
  int64_t p0;                // first position of this band in the group
  int32_t band;
  int64_t *row_count;        // count pass
  const int64_t *row_off;    // emit pass
  const int64_t *base;       // emit pass: output offset of this band
  uint32_t *x_out, *y_out;
  int64_t capacity;
};

// Whether two key rows agree in one of the bands before `band`.
template <bool PACK>
__device__ inline bool earlier_band(const uint32_t *kx, const uint32_t *ky, int band) {
  const int nw = PACK ? (band + 1) >> 1 : band;
  for (int w = 0; w < nw; ++w) {
    const uint32_t v = kx[w] ^ ky[w];
    if constexpr (PACK) {
      if ((v & 0xFFFFu) == 0 || (2 * w + 1 < band && (v >> 16) == 0)) return true;
    } else {
      if (v == 0) return true;
    }
  }
  return false;
}

// One wave per member row p.  EMIT = false counts the kept pairs of the row;
// EMIT = true writes them in order.
template <bool EMIT, bool PACK>
__global__ __launch_bounds__(kBandBlock) void k_band_pairs(BandArgs a) {
  const int lane = lane_id();
  const int64_t waves = int64_t(gridDim.x) * (kBandBlock / kWave);
  const int64_t w0 = int64_t(blockIdx.x) * (kBandBlock / kWave) +
                     int64_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
  const int64_t out0 = EMIT ? *a.base : 0;
  for (int64_t r = w0; r < a.n_obj; r += waves) {
    const int64_t p = a.p0 + r;
    const int64_t e = a.ends[p];
    int64_t kept = 0;
    if (p + 1 < e) {
      const uint32_t x = a.sids[p];
      const uint32_t *kx = a.rows + size_t(x) * a.stride;
      const int64_t off = EMIT ? out0 + a.row_off[r] : 0;
      for (int64_t q0 = p + 1; q0 < e; q0 += kWave) {
        const int64_t q = q0 + lane;
        bool keep = false;
        uint32_t y = 0;
        if (q < e) {
          y = a.sids[q];
          keep = !earlier_band<PACK>(kx, a.rows + size_t(y) * a.stride, a.band);   // collided before: emitted there
        }
        const uint64_t mask = __ballot(keep);
        if (EMIT && keep) {
          const int64_t pos = off + kept + int64_t(lanes_below(mask));
          if (pos < a.capacity) {
            a.x_out[pos] = x;
            a.y_out[pos] = y;
          }
        }
        kept += __popcll(mask);
      }
    }
    if (!EMIT && lane == 0) a.row_count[r] = kept;
  }
}

// ---------------------------------------------------------------------------
// Tiled emission order: the upper triangle of a bucket's member positions cut
// into kTile x kTile tiles, listed by tile row, then tile column, each tile
// row-major -- a run of 256 candidates then touches about 2 kTile objects
// instead of one row's ~256, which the verification kernels' L1 reuses.
// ---------------------------------------------------------------------------
constexpr int kTileRec = 5;
constexpr int kTile = 16;        // 16 x 16 = 256 pair positions: one wave, 4 per lane
constexpr int kRowRegs = 8;      // key words of a row held in registers by the strip kernel
constexpr int kStripPer = 16;    // positions per thread of k_strips
constexpr int64_t kStripBlock = int64_t(kBandBlock) * kStripPer;

struct StripArgs {
  const uint32_t *sids, *bstart, *bend;
  const uint32_t *rows;      // [n_obj][stride], stride a multiple of 4
  int32_t stride;
  int64_t n_obj, n_pos;      // objects; positions of the group
  int32_t j0;                // the group's first band
  int32_t max_bucket;
  uint4 *strip;              // [strips] first position, bucket start, its members, band
  int64_t *stile;            // [strips] its first tile's number in the group
  int64_t *stot;             // [strips] its pairs
  const int64_t *soff;       // [strips] exclusive prefix of stot from the launch's first strip
  // pairs: [tiles of the launch][kTileRec]: the tile's mask (bit l of word i:
  // position 64 i + l), the pairs of its strip before the tile
  uint64_t *rec;
  // tiles: descriptors of the launch, and how many of them the caller's array holds
  blsh_tile *out;
  int64_t out_n;
  int64_t s_begin, s_end;    // strips of the launch
  int64_t tile0;             // the launch's first tile
  const int64_t *base;       // candidates before the launch
  uint32_t *x_out, *y_out;
  int64_t capacity;
};

// A strip as listed: its bucket's start b0 and member count (capped at
// max_bucket), its tile row ta, the bucket's tiles along a side and the band.
// (32-bit: a bucket whose padded size passes 2^32 has 2^55 tiles)
struct Strip {
  uint32_t b0, len, ta, nt;
  int band;
};
__device__ inline Strip listed_strip(const StripArgs &a, int64_t s) {
  const uint4 v = a.strip[s];
  return Strip{v.y, v.z, (v.x - v.y) / kTile, (v.z + kTile - 1) / kTile, int(v.w)};
}

// Tiles of the strip that starts at position p (bucket start b0), and the
// bucket's capped member count; 0 if none starts there (only a multiple of
// kTile positions into a bucket can; a bucket of one member has no tile).
__device__ inline int64_t strip_tiles(const StripArgs &a, int64_t p, int64_t b0, int64_t &len) {
  const int64_t off = p - b0;
  if (off % kTile) return 0;
  len = int64_t(a.bend[b0]) - b0;
  if (a.max_bucket > 0) len = min(len, int64_t(a.max_bucket));
  return len >= 2 && off < len ? (len + kTile - 1) / kTile - off / kTile : 0;
}

// Lists the strips of the group in position order: block b takes kStripBlock
// positions.  WRITE = false leaves the block's strips and tiles in part[2 b],
// part[2 b + 1]; WRITE = true (part then holds their exclusive prefixes)
// writes the list, and meta[2 j], meta[2 j + 1] = strips and tiles before band
// j of the group.
template <bool WRITE>
__global__ __launch_bounds__(kBandBlock) void k_strips(StripArgs a, int64_t *part, int64_t *meta) {
  __shared__ int64_t s_part[2][kBandBlock / kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int64_t p0 = int64_t(blockIdx.x) * kStripBlock + int64_t(threadIdx.x) * kStripPer;
  int64_t strips = 0, tiles = 0;
  int64_t len = 0;
  for (int i = 0; i < kStripPer; ++i) {
    if (p0 + i >= a.n_pos) break;
    const int64_t t = strip_tiles(a, p0 + i, a.bstart[p0 + i], len);
    strips += t > 0;
    tiles += t;
  }
  int64_t is = strips, it = tiles;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t us = __shfl_up(is, o), ut = __shfl_up(it, o);
    if (lane >= o) { is += us; it += ut; }
  }
  if (lane == kWave - 1) { s_part[0][wv] = is; s_part[1][wv] = it; }
  __syncthreads();
  int64_t bs = is - strips, bt = it - tiles;
  for (int w = 0; w < wv; ++w) { bs += s_part[0][w]; bt += s_part[1][w]; }
  if constexpr (!WRITE) {
    if (threadIdx.x == kBandBlock - 1) { part[2 * blockIdx.x] = bs + strips; part[2 * blockIdx.x + 1] = bt + tiles; }
  } else {
    bs += part[2 * blockIdx.x];
    bt += part[2 * blockIdx.x + 1];
    int64_t j = (p0 + a.n_obj - 1) / a.n_obj;   // the first band starting at p0 or later
    for (int i = 0; i < kStripPer; ++i) {
      const int64_t p = p0 + i;
      if (p >= a.n_pos) break;
      if (p == j * a.n_obj) { meta[2 * j] = bs; meta[2 * j + 1] = bt; ++j; }
      const int64_t b0 = a.bstart[p], t = strip_tiles(a, p, b0, len);
      if (t > 0) {
        a.strip[bs] = make_uint4(uint32_t(p), uint32_t(b0), uint32_t(len), uint32_t(a.j0 + j - 1));
        a.stile[bs] = bt;
        ++bs;
        bt += t;
      }
      if (p + 1 == a.n_pos) { meta[2 * j] = bs; meta[2 * j + 1] = bt; }
    }
  }
}

// Exclusive prefixes of the block sums of k_strips, in place.  One block.
__global__ __launch_bounds__(1024) void k_strip_scan(int64_t *part, int64_t nb) {
  __shared__ int64_t s_part[2][1024 / kWave], s_carry[2];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  if (threadIdx.x < 2) s_carry[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t b = b0 + threadIdx.x;
    int64_t v[2], x[2], before[2];
    for (int q = 0; q < 2; ++q) {
      x[q] = v[q] = b < nb ? part[2 * b + q] : 0;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int64_t u = __shfl_up(x[q], o);
        if (lane >= o) x[q] += u;
      }
      if (lane == kWave - 1) s_part[q][wv] = x[q];
    }
    __syncthreads();
    for (int q = 0; q < 2; ++q) {
      before[q] = s_carry[q];
      for (int w = 0; w < wv; ++w) before[q] += s_part[q][w];
      if (b < nb) part[2 * b + q] = before[q] + x[q] - v[q];
    }
    __syncthreads();
    if (threadIdx.x == 1023)
      for (int q = 0; q < 2; ++q) s_carry[q] = before[q] + x[q];
    __syncthreads();
  }
}

// The strips of a launch go round its waves so that an XCD's blocks take
// consecutive ones: the strips of a bucket then share their columns' key rows
// in one L2, and a block's four in one L1.
constexpr int64_t kStripBlocks = int64_t(1) << 22;   // most blocks of a launch (one wave per strip below that)
__device__ inline int64_t first_strip(const StripArgs &a) {
  return a.s_begin + xcd_tile(blockIdx.x, gridDim.x) * (kBandBlock / kWave) +
         int64_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
}
__device__ inline int64_t strip_step() { return int64_t(gridDim.x) * (kBandBlock / kWave); }

// The tiles of one strip, NW key words in registers (NW < 0: rows of more
// words than that, read again for every tile).  Lane l holds column l % 16 and
// rows 4 i + l / 16, i < 4, so that ballot i is word i of the tile's mask.  A
// column's keys are requested while the tile before is tested, its id one tile
// earlier still.  Two keys of a word are tested with one exclusive-or and one
// packed minimum (zero: equal).
template <bool PACK, int NW, bool DESC>
__device__ inline void strip_run(const StripArgs &a, const Strip &st, int64_t s) {
  constexpr bool WIDE = NW < 0;
  constexpr int NR = WIDE ? kRowRegs : NW;      // words tested at a time
  constexpr int NL = (NR + 3) / 4 * 4 + (NR == 0);   // words loaded
  const int lane = lane_id(), c = lane & 15, rs = lane >> 4;
  const int nw = PACK ? (st.band + 1) >> 1 : st.band;
  const uint32_t half = PACK && (st.band & 1) ? 0xFFFF0000u : 0u;   // the last word's upper key is not an earlier band's
  const uint32_t *ids = a.sids + st.b0;
  auto member = [&](uint32_t tb) { return ids[min(tb * kTile + c, st.len - 1)]; };
  auto load = [&](uint32_t id, int w0, uint32_t (&k)[NL]) {
    const uint4 *r = reinterpret_cast<const uint4 *>(a.rows + size_t(id) * uint32_t(a.stride) + w0);
#pragma unroll
    for (int q = 0; q < NL / 4; ++q)
      if (!WIDE || w0 + 4 * q < nw) {
        const uint4 v = r[q];
        k[4 * q] = v.x; k[4 * q + 1] = v.y; k[4 * q + 2] = v.z; k[4 * q + 3] = v.w;
      }
  };
  const uint32_t mine = member(st.ta);
  uint32_t nid = member(st.ta + 1);   // (past the bucket: its last member, unused)
  uint32_t rid[4], rk[4][NL], ck[NL], nk[NL];
  uint64_t row_ok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    rid[i] = uint32_t(__shfl(int(mine), 4 * i + rs));
    row_ok[i] = __ballot(st.ta * kTile + 4 * i + rs < st.len);
    if constexpr (!WIDE) load(rid[i], 0, rk[i]);
  }
  auto test = [&](int w0, uint32_t (&acc)[4]) {
#pragma unroll
    for (int w = 0; w < NR; ++w)
      if (!WIDE || w0 + w < nw) {
        const uint32_t over = (WIDE ? w0 + w == nw - 1 : w == NR - 1) ? half : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t v = (rk[i][w] ^ ck[w]) | over;
          if constexpr (PACK) {
            const u16x2 m = __builtin_elementwise_min(__builtin_bit_cast(u16x2, acc[i]), __builtin_bit_cast(u16x2, v));
            acc[i] = __builtin_bit_cast(uint32_t, m);
          } else {
            acc[i] = min(acc[i], v);
          }
        }
      }
  };
  // the part of a descriptor that the strip's tiles share: row count and ids
  uint32_t fixed = 0;
  if constexpr (DESC) {
    const uint32_t row = uint32_t(__shfl(int(mine), (lane - 12) & 15));
    if (lane >= 12 && lane < 28) fixed = st.ta * kTile + uint32_t(lane - 12) < st.len ? row : 0xFFFFFFFFu;
    if (lane == 2) fixed = min(uint32_t(kTile), st.len - st.ta * kTile);
  }
  int64_t run = 0, t = a.stile[s] - a.tile0;
  uint32_t nc = mine;   // id of this lane's column in the next tile
  if constexpr (!WIDE && NW > 0) load(mine, 0, nk);
  for (uint32_t tb = st.ta; tb < st.nt; ++tb, ++t) {
    uint32_t acc[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    const uint32_t cid = nc;
    nc = nid;
    if constexpr (WIDE) {
      nid = member(tb + 2);
      for (int w0 = 0; w0 < nw; w0 += NR) {
        load(cid, w0, ck);
#pragma unroll
        for (int i = 0; i < 4; ++i) load(rid[i], w0, rk[i]);
        test(w0, acc);
      }
    } else {
#pragma unroll
      for (int w = 0; w < NL; ++w) ck[w] = nk[w];
      if (tb + 1 < st.nt) {
        if constexpr (NW > 0) load(nc, 0, nk);
        nid = member(tb + 2);
      }
      test(0, acc);
    }
    uint64_t mask[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      mask[i] = row_ok[i] & __ballot(PACK ? min(acc[i] & 0xFFFFu, acc[i] >> 16) != 0 : acc[i] != 0);
    const uint64_t col_ok = __ballot(tb * kTile + c < st.len);
    if (tb == st.ta) {   // the upper triangle
#pragma unroll
      for (int i = 0; i < 4; ++i) mask[i] &= __ballot(4 * i + rs < c);
    }
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mask[i] &= col_ok;
      total += uint32_t(__popcll(mask[i]));
    }
    uint32_t v = fixed;
    auto put = [&](uint64_t x, auto at) {   // x in lanes at, at + 1
      v = write_lane<at.value>(uint32_t(x), v);
      v = write_lane<at.value + 1>(uint32_t(x >> 32), v);
    };
    using std::integral_constant;
    if constexpr (DESC) {
      // first (within the strip until k_strip_first), counts, mask, ids, zeros
      const uint32_t col = dpp<kDppRowRor12>(cid);   // lanes 28 .. 43: columns 0 .. 15
      if (lane >= 28 && lane < 44) v = tb * kTile + uint32_t(lane - 28) < st.len ? col : 0xFFFFFFFFu;
      put(uint64_t(run), integral_constant<int, 0>{});
      v = write_lane<3>(min(uint32_t(kTile), st.len - tb * kTile), v);
      put(mask[0], integral_constant<int, 4>{});
      put(mask[1], integral_constant<int, 6>{});
      put(mask[2], integral_constant<int, 8>{});
      put(mask[3], integral_constant<int, 10>{});
      if (t < a.out_n && lane < int(sizeof(blsh_tile) / 4)) reinterpret_cast<uint32_t *>(a.out + t)[lane] = v;
    } else {
      put(mask[0], integral_constant<int, 0>{});
      put(mask[1], integral_constant<int, 2>{});
      put(mask[2], integral_constant<int, 4>{});
      put(mask[3], integral_constant<int, 6>{});
      put(uint64_t(run), integral_constant<int, 8>{});
      if (lane < 2 * kTileRec) reinterpret_cast<uint32_t *>(a.rec + kTileRec * t)[lane] = v;
    }
    run += total;
  }
  if (lane == 0) a.stot[s] = run;
}

// The earlier-band test of the strips' tiles, one wave per strip: a mask and a
// running count per tile (pairs) or its descriptor (DESC), and the strip's count.
// Bound by instruction issue, vector and scalar about alike (2 vector
// instructions per key word and 64 positions, about 40 of each per tile
// beside): 2.45 ms for the 11.0M tiles of 1M objects, 16 bands of 12 bits,
// where one wave per tile, each searching for its bucket, gathering 16-byte key
// quarters per lane and writing masks for a second kernel to turn into
// descriptors, took 17.1 + 1.0 ms; the number of key words as a constant of
// the loop (the cases below) 2.45 against 3.25 ms as a variable.  The whole call: 3.65
// against 26.2 ms (it was 596 launches and 33 copies to the host, band by band;
// now 25 and 2).
template <bool PACK, bool DESC>
__global__ __launch_bounds__(kBandBlock) void k_strip_masks(StripArgs a) {
  static_assert(sizeof(blsh_tile) == 192 && kRowRegs == 8, "descriptor layout; the cases below");
  for (int64_t s = first_strip(a); s < a.s_end; s += strip_step()) {
    const Strip st = listed_strip(a, s);
    switch (PACK ? (st.band + 1) >> 1 : st.band) {   // wave-uniform
      case 0: strip_run<PACK, 0, DESC>(a, st, s); break;
      case 1: strip_run<PACK, 1, DESC>(a, st, s); break;
      case 2: strip_run<PACK, 2, DESC>(a, st, s); break;
      case 3: strip_run<PACK, 3, DESC>(a, st, s); break;
      case 4: strip_run<PACK, 4, DESC>(a, st, s); break;
      case 5: strip_run<PACK, 5, DESC>(a, st, s); break;
      case 6: strip_run<PACK, 6, DESC>(a, st, s); break;
      case 7: strip_run<PACK, 7, DESC>(a, st, s); break;
      case 8: strip_run<PACK, 8, DESC>(a, st, s); break;
      default: strip_run<PACK, -1, DESC>(a, st, s); break;
    }
  }
}

// The candidates of a strip's tiles as (x, y) pairs, one wave per strip; the
// loads of kOutTiles tiles are issued together (each tile alone is one round
// trip to memory).
constexpr int kOutTiles = 4;

__global__ __launch_bounds__(kBandBlock) void k_strip_pairs(StripArgs a) {
  const int lane = lane_id(), c = lane & 15, rs = lane >> 4;
  for (int64_t s = first_strip(a); s < a.s_end; s += strip_step()) {
    const Strip st = listed_strip(a, s);
    const uint32_t *ids = a.sids + st.b0;
    const uint32_t mine = ids[min(st.ta * kTile + c, st.len - 1)];
    uint32_t x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = uint32_t(__shfl(int(mine), 4 * i + rs));
    int64_t t = a.stile[s] - a.tile0;
    const int64_t out0 = *a.base + a.soff[s];
    for (uint32_t tb = st.ta; tb < st.nt; tb += kOutTiles, t += kOutTiles) {
      uint32_t y[kOutTiles];
      int64_t pos[kOutTiles];
      uint64_t mask[kOutTiles][4];
#pragma unroll
      for (int u = 0; u < kOutTiles; ++u) {
        const bool in = tb + u < st.nt;
        const uint64_t *rec = a.rec + kTileRec * (t + (in ? u : 0));
        y[u] = ids[min((tb + u) * kTile + c, st.len - 1)];
        pos[u] = out0 + int64_t(rec[4]);
#pragma unroll
        for (int i = 0; i < 4; ++i) mask[u][i] = in ? rec[i] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kOutTiles; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t at = pos[u] + int64_t(lanes_below(mask[u][i]));
          if (((mask[u][i] >> lane) & 1u) && at < a.capacity) {
            a.x_out[at] = x[i];
            a.y_out[at] = y[u];
          }
          pos[u] += __popcll(mask[u][i]);
        }
    }
  }
}

// Adds the candidates before its strip to the first candidate of every
// descriptor, one wave per strip, one tile per lane.
__global__ __launch_bounds__(kBandBlock) void k_strip_first(StripArgs a) {
  for (int64_t s = first_strip(a); s < a.s_end; s += strip_step()) {
    const uint4 v = a.strip[s];
    const int64_t t0 = a.stile[s] - a.tile0, before = *a.base + a.soff[s];
    const int64_t t1 = min(a.out_n, t0 + (v.z + kTile - 1) / kTile - (v.x - v.y) / kTile);
    for (int64_t t = t0 + lane_id(); t < t1; t += kWave) a.out[t].first += before;
  }
}

// base += (pairs counted last) = off[n-1] + count[n-1]
__global__ void k_band_advance(int64_t *base, const int64_t *off, const int64_t *count, int64_t n) {
  if (threadIdx.x == 0 && blockIdx.x == 0 && n > 0) *base += off[n - 1] + count[n - 1];
}

__global__ void k_band_zero(int64_t *base) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *base = 0;
}

static inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

static int ensure_tile_buf(blsh_ctx *ctx, size_t bytes) {
  if (ctx->tile_bytes >= bytes) return BLSH_OK;
  BLSH_HIP(hipDeviceSynchronize());
  if (ctx->tile_buf) (void)hipFree(ctx->tile_buf);
  ctx->tile_buf = nullptr;
  ctx->tile_bytes = 0;
  const size_t want = std::max(bytes, size_t(1) << 20);
  if (hipMalloc(&ctx->tile_buf, want) != hipSuccess) return fail(BLSH_ENOMEM, "banding: tile buffer of %zu bytes", want);
  ctx->tile_bytes = want;
  return BLSH_OK;
}

// Pairs: bands are taken together up to this many bytes of tile masks and
// counts (40 per tile); a single band always goes in one launch.
constexpr int64_t kTileBufBytes = int64_t(1) << 30;
// Bands are grouped while the workspace stays within this (or within what the
// context already holds; a fixed workspace is never exceeded): one group of
// 16 bands of 1M objects takes 0.6 GB.
constexpr size_t kGroupBytes = size_t(4) << 30;
constexpr int64_t kGroupPositions = int64_t(1) << 30;

struct BandLayout {
  size_t rows, keys, ids, skeys, sids, bstart, bend, count, off, strip, stile, stot, soff, part, meta, base, tmp, scan_at, total;
  size_t sort_tmp, scan_tmp;
};

// Workspace of a group of bands (row order: the row counts and offsets; tiled
// order: the strips -- at most one for every two positions).
static int band_layout(size_t n, int group, int key_bits, int stride, bool tiled, hipStream_t s,
                       BandLayout *l) {
  const size_t N = n * group, S = N / 2 + 1;
  l->sort_tmp = l->scan_tmp = 0;
  if (rocprim::radix_sort_pairs(nullptr, l->sort_tmp, (const uint32_t *)nullptr, (uint32_t *)nullptr,
                                (const uint32_t *)nullptr, (uint32_t *)nullptr, N, 0, unsigned(key_bits), s) !=
          hipSuccess ||
      rocprim::exclusive_scan(nullptr, l->scan_tmp, (const int64_t *)nullptr, (int64_t *)nullptr, int64_t(0),
                              tiled ? S : n, rocprim::plus<int64_t>(), s) != hipSuccess)
    return fail(BLSH_EDEVICE, "banding: temporary storage query failed");
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t o = at; at += align256(bytes); return o; };
  l->rows = take(n * stride * 4);
  l->sids = take(N * 4);
  l->bstart = take(N * 4);
  l->bend = take(N * 4);
  l->meta = take(size_t(2) * (group + 1) * 8);
  l->part = take(tiled ? (N + kStripBlock - 1) / kStripBlock * 16 : 0);
  l->base = take(8);
  // the sort's keys and ids are spent once the buckets are known; the tiled
  // order's strips, the row order's counts and the scans' storage take their place
  const size_t from = at;
  l->keys = take(N * 4);
  l->ids = take(N * 4);
  l->skeys = take(N * 4);
  l->tmp = take(std::max(l->sort_tmp, (N + kBoundChunk - 1) / kBoundChunk * 4));
  const size_t sorted = at;
  at = from;
  l->strip = take(tiled ? S * sizeof(uint4) : 0);
  l->stile = take(tiled ? S * 8 : 0);
  l->count = l->stot = take((tiled ? S : n) * 8);
  l->off = l->soff = take((tiled ? S : n) * 8);
  l->scan_at = take(l->scan_tmp);
  l->total = std::max(sorted, at);
  return BLSH_OK;
}

int band_candidates(blsh_ctx *ctx, const uint32_t *sig, int64_t n_obj, int32_t row_words, bool word_major,
                    int32_t n_bands, int32_t band_bits, int32_t max_bucket, int32_t tile, uint32_t *x_out,
                    uint32_t *y_out, int64_t capacity, int64_t *n_pairs, hipStream_t s, const BandTilesOut *to) {
  if (tile != 0 && tile != kTile) return fail(BLSH_EINVAL, "banding: order_tile must be 0 or %d", kTile);
  const size_t n = size_t(n_obj);
  // key rows: two keys to a word when they fit; the strip kernel reads them 16 bytes at a time
  const bool pack = band_bits <= 16, tiled = tile != 0;
  int stride = pack ? (n_bands + 1) / 2 : n_bands;
  if (tiled) stride = (stride + 3) & ~3;
  // as many bands to a group as the sort's 32-bit keys, the positions and the
  // workspace allow; one band always needs less than 8 (n_bands + 6) n bytes
  // beside the library's temporary storage
  auto key_bits_of = [&](int g) {
    int b = band_bits;
    for (int x = g - 1; x > 0; x >>= 1) ++b;
    return b;
  };
  const size_t most = ctx->ws_fixed ? ctx->ws_bytes : std::max(ctx->ws_bytes, kGroupBytes);
  BandLayout l{};
  int group = n_bands, rc = BLSH_OK;
  for (;; group = (group + 1) / 2) {
    const bool ok = key_bits_of(group) <= 32 && int64_t(group) * n_obj <= kGroupPositions;
    if (group > 1 && !ok) continue;
    if ((rc = band_layout(n, group, key_bits_of(group), stride, tiled, s, &l))) return rc;
    if (group > 1 && l.total > most) continue;
    rc = ensure_workspace(ctx, l.total);
    if (rc != BLSH_ENOMEM || group == 1) break;
    (void)hipGetLastError();   // not enough device memory for these bands together: fewer
  }
  if (rc) return rc;
  char *ws = static_cast<char *>(ctx->ws);
  auto u32 = [&](size_t o) { return reinterpret_cast<uint32_t *>(ws + o); };
  auto i64 = [&](size_t o) { return reinterpret_cast<int64_t *>(ws + o); };
  uint32_t *rows = u32(l.rows), *sids = u32(l.sids), *bstart = u32(l.bstart), *bend = u32(l.bend);
  int64_t *base = i64(l.base);
  int64_t tiles_total = 0;   // tiles output: descriptors written so far (all bands)

  LaunchScope ls(ctx, s, "band_candidates");
  const unsigned nb = unsigned((n + kBandBlock - 1) / kBandBlock);
  hipLaunchKernelGGL(k_band_zero, dim3(1), dim3(64), 0, s, base);
  for (int j0 = 0; j0 < n_bands; j0 += group) {
    const int g = std::min(group, n_bands - j0);
    const int64_t N = int64_t(g) * n_obj;
    hipLaunchKernelGGL(pack ? k_band_keys<true> : k_band_keys<false>, dim3(nb), dim3(kBandBlock), 0, s, sig, n_obj,
                       row_words, int(word_major), n_bands, band_bits, j0, g, u32(l.keys), u32(l.ids),
                       j0 == 0 ? rows : nullptr, stride);
    size_t t1 = l.sort_tmp;
    if (rocprim::radix_sort_pairs(ws + l.tmp, t1, u32(l.keys), u32(l.skeys), u32(l.ids), sids, size_t(N), 0,
                                  unsigned(key_bits_of(g)), s) != hipSuccess)
      return fail(BLSH_EDEVICE, "banding: radix sort failed");
    const unsigned cb = unsigned((N + kBoundChunk * 4 - 1) / (kBoundChunk * 4));
    uint32_t *last = u32(l.tmp);   // (the sort's storage is free again)
    hipLaunchKernelGGL(k_bucket_last, dim3(cb), dim3(kBandBlock), 0, s, u32(l.skeys), N, last);
    hipLaunchKernelGGL(k_bucket_bounds, dim3(cb), dim3(kBandBlock), 0, s, u32(l.skeys), N, last, bstart, bend);
    if (tiled) {
      StripArgs a{};
      a.sids = sids;
      a.bstart = bstart;
      a.bend = bend;
      a.rows = rows;
      a.stride = stride;
      a.n_obj = n_obj;
      a.n_pos = N;
      a.j0 = j0;
      a.max_bucket = max_bucket;
      a.strip = reinterpret_cast<uint4 *>(ws + l.strip);
      a.stile = i64(l.stile);
      a.stot = i64(l.stot);
      a.soff = i64(l.soff);
      a.base = base;
      a.x_out = x_out;
      a.y_out = y_out;
      a.capacity = capacity;
      int64_t *part = i64(l.part), *meta = i64(l.meta);
      const int64_t sb = (N + kStripBlock - 1) / kStripBlock;
      hipLaunchKernelGGL(k_strips<false>, dim3(unsigned(sb)), dim3(kBandBlock), 0, s, a, part, meta);
      hipLaunchKernelGGL(k_strip_scan, dim3(1), dim3(1024), 0, s, part, sb);
      hipLaunchKernelGGL(k_strips<true>, dim3(unsigned(sb)), dim3(kBandBlock), 0, s, a, part, meta);
      int64_t at[2 * (64 + 1)];   // strips and tiles before each band
      BLSH_HIP(hipMemcpyAsync(at, meta, size_t(2) * (g + 1) * 8, hipMemcpyDeviceToHost, s));
      BLSH_HIP(hipStreamSynchronize(s));
      int64_t buf_bytes = kTileBufBytes;
      for (int b0 = 0, b1; b0 < g; b0 = b1) {
        b1 = b0 + 1;
        while (b1 < g && (to || (at[2 * (b1 + 1) + 1] - at[2 * b0 + 1]) * kTileRec * 8 <= buf_bytes)) ++b1;
        const int64_t n_strips = at[2 * b1] - at[2 * b0], n_tiles = at[2 * b1 + 1] - at[2 * b0 + 1];
        if (n_tiles == 0) continue;
        a.s_begin = at[2 * b0];
        a.s_end = at[2 * b1];
        a.tile0 = at[2 * b0 + 1];
        if (to) {
          a.out = to->tiles + std::min(tiles_total, to->tile_cap);
          a.out_n = std::max<int64_t>(0, to->tile_cap - tiles_total);
        } else {
          rc = ensure_tile_buf(ctx, size_t(n_tiles) * kTileRec * 8);
          if (rc == BLSH_ENOMEM && b1 > b0 + 1) {   // one band at a time
            (void)hipGetLastError();
            buf_bytes = 0;
            b1 = b0;
            continue;
          }
          if (rc) return rc;
          a.rec = static_cast<uint64_t *>(ctx->tile_buf);
        }
        const dim3 sg(unsigned(std::min(kStripBlocks, (n_strips + kBandBlock / kWave - 1) / (kBandBlock / kWave))));
        hipLaunchKernelGGL(pack ? (to ? k_strip_masks<true, true> : k_strip_masks<true, false>)
                                : (to ? k_strip_masks<false, true> : k_strip_masks<false, false>),
                           sg, dim3(kBandBlock), 0, s, a);
        size_t t3 = l.scan_tmp;
        if (rocprim::exclusive_scan(ws + l.scan_at, t3, a.stot + a.s_begin, i64(l.soff) + a.s_begin, int64_t(0),
                                    size_t(n_strips), rocprim::plus<int64_t>(), s) != hipSuccess)
          return fail(BLSH_EDEVICE, "banding: scan failed");
        hipLaunchKernelGGL(to ? k_strip_first : k_strip_pairs, sg, dim3(kBandBlock), 0, s, a);
        tiles_total += n_tiles;
        hipLaunchKernelGGL(k_band_advance, dim3(1), dim3(64), 0, s, base, a.soff + a.s_begin, a.stot + a.s_begin,
                           n_strips);
      }
      continue;
    }
    hipLaunchKernelGGL(k_bucket_row_ends, dim3(unsigned((N + kBandBlock - 1) / kBandBlock)), dim3(kBandBlock), 0, s,
                       bstart, bend, N, max_bucket);
    const unsigned pair_blocks = unsigned(std::min<int64_t>(int64_t(ctx->n_cu) * 8, (n_obj + 3) / 4 + 1));
    for (int j = j0; j < j0 + g; ++j) {
      BandArgs a{};
      a.sids = sids;
      a.ends = bstart;
      a.rows = rows;
      a.stride = stride;
      a.n_obj = n_obj;
      a.p0 = int64_t(j - j0) * n_obj;
      a.band = j;
      a.row_count = i64(l.count);
      a.row_off = i64(l.off);
      a.base = base;
      a.x_out = x_out;
      a.y_out = y_out;
      a.capacity = capacity;
      hipLaunchKernelGGL((pack ? k_band_pairs<false, true> : k_band_pairs<false, false>), dim3(pair_blocks),
                         dim3(kBandBlock), 0, s, a);
      size_t t3 = l.scan_tmp;
      if (rocprim::exclusive_scan(ws + l.scan_at, t3, a.row_count, i64(l.off), int64_t(0), n,
                                  rocprim::plus<int64_t>(), s) != hipSuccess)
        return fail(BLSH_EDEVICE, "banding: scan failed");
      hipLaunchKernelGGL((pack ? k_band_pairs<true, true> : k_band_pairs<true, false>), dim3(pair_blocks),
                         dim3(kBandBlock), 0, s, a);
      hipLaunchKernelGGL(k_band_advance, dim3(1), dim3(64), 0, s, base, a.row_off, a.row_count, n_obj);
    }
  }
  BLSH_HIP(hipMemcpyAsync(n_pairs, base, 8, hipMemcpyDeviceToHost, s));
  BLSH_HIP(hipStreamSynchronize(s));
  if (hipGetLastError() != hipSuccess) return fail(BLSH_EDEVICE, "banding: launch failed");
  if (to) {
    *to->n_tiles = tiles_total;
    if (tiles_total > to->tile_cap)
      return fail(BLSH_ETRUNCATED, "banding: %lld tiles, capacity %lld", (long long)tiles_total,
                  (long long)to->tile_cap);
    return BLSH_OK;
  }
  return *n_pairs > capacity ? fail(BLSH_ETRUNCATED, "banding: %lld pairs, capacity %lld", (long long)*n_pairs,
                                    (long long)capacity)
                             : BLSH_OK;
}

}  // namespace blsh
