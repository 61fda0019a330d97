// Batched verification of many query lists of uneven lengths in one
// graph-launched pair of persistent kernels (Algorithm 1 per candidate).
//
// Phase 1 (k_batch_phase1, one launch per measure): the batch is cut into
//   wave tiles -- 128, 256 or 512 consecutive candidates of one SRP list (2, 4
//   or 8 per lane) or 64 or 128 of one minhash list (lane l owns candidates l
//   and 64 + l, a group of k/4 lanes compares each candidate's k hashes), the
//   shape per measure chosen by the autotuner -- and every wave of the fixed grid
//   runs an equal share of them (no work counter, no block barrier): a range,
//   but the tiles of a list that spans several waves go to them by turns; each XCD has
//   an eighth of every list (L2 locality of sorted ids).  The
//   query's hashes are wave-uniform.  Each list carries its own measure and
//   threshold, hence its own decision table, and each measure its own k.  A
//   candidate still undecided after `inreg_levels` levels (SRP object-major
//   rows: at least the 128 hashes one 16-byte load brings) is spilled to the
//   wave's own region of the measure's survivor queue (ballot compaction, no
//   atomics); when the region is full it simply continues in registers.
// Phase 2 (k_batch_offsets, k_batch_phase2): the survivor queues are cut into
//   equal shares for the waves of a second grid: one lane per SRP survivor, one
//   group of k/4 lanes per minhash survivor, running the remaining levels, up to
//   four levels' words loaded ahead.
//
// Accepted pairs are staged in slices (as in the single-call paths) and
// appended to the caller's list by k_batch_flush at the end of the batch.
//
// The kernels read all their arguments from one device-resident BatchBlock,
// so the graph that holds [phase 1 x 2, offsets, phase 2, flush] is captured
// once per (k pair, tile shapes, grid) and replayed for any batch: each call
// only refreshes the block and the tile prefix sums.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <set>
#include <utility>

#include "device_common.h"

namespace blsh {

constexpr int kMaxBatchTables = 64;
constexpr int kBBlock = 256;
// phase 1 wave tiles (the autotuner picks one shape per measure):
// SRP 128, 256 or 512 consecutive candidates (2, 4 or 8 per lane), minhash 64
// or 128 (1 or 2 per lane)
constexpr int kSrpTileDefault = 256;
constexpr int kMhTileDefault = 64;
// phase-1 blocks per CU: all resident at once (the SRP kernel's registers allow 7),
// so that the waves of a list keep pace.  512 lists of 56 M candidates (k = 16 / 64):
// 474 us with 4, 449 with 5, 437 with 6, 484 with 7, 499 with 8; 34 K candidates: 56 to 57.
constexpr int kBlocksDefault = 6;
constexpr int kExSrpTile = 1024;   // comparator: candidates per SRP block tile
constexpr int kExMhTile = 256;     // comparator: candidates per minhash block tile
constexpr int kXcds = 8;           // phase 1: list tiles split in kXcds position ranges, one per XCD
// survivor queue of a small batch: 170 entries a wave of the largest grid the
// autotuner takes (6 blocks a CU, 256 CUs).  A wave whose region is full runs its tile to the last level
// alone, which takes a batch of 34 K candidates 22 us longer.
constexpr int64_t kMinSpill = int64_t(1) << 20;
constexpr int64_t kBatchStage = 4096;   // accepted-pair staging entries per slice

struct BatchList {
  int64_t offset;
  int64_t length;
  uint32_t query;
  int32_t measure;
  int32_t table;
  int32_t pad;
};

struct SigView {
  const uint32_t *data;
  int64_t n_obj;
  int32_t row_words;
  int32_t word_major;
  const uint32_t *pfx;          // SRP: hashes 0..127 of object i at pfx + i * pfx_stride, or null
  int64_t pfx_stride;
};

struct BatchBlock {
  const BatchList *lists;
  // phase 1: [2 measures][kXcds][n_lists + 1], slice (me, x) counts the
  // tiles [x n_t / kXcds, (x+1) n_t / kXcds) of each list of measure me (n_t
  // tiles); comparator: [n_lists + 1]
  const int64_t *tile_prefix;
  int64_t n_lists, n_tiles;
  const uint32_t *cand;
  SigView sig[2];               // [BLSH_JACCARD], [BLSH_COSINE]
  const uint32_t *tables[kMaxBatchTables];
  int32_t n_levels[kMaxBatchTables];
  double alpha, beta;           // Jaccard prior
  uint8_t *code;
  uint64_t *acc_idx;
  float *acc_val;
  int64_t acc_cap;
  int64_t *n_acc;
  uint16_t *m_dbg;
  int32_t *status;
  // accepted-pair staging (as in the single-call paths): kSlices slices of
  // st_cap entries, counts at acc_cnt[s * kCntStride], appended to the list by
  // k_batch_flush; entries past a slice's capacity go to the list directly at
  // positions from the running count *acc_total.  Batches alternate between two
  // sets of these counts: the flush of one leaves those of the next (acc_next,
  // laid out as acc_cnt with the running count behind) zero.
  int64_t *acc_cnt, *acc_next;
  uint64_t *st_idx;
  float *st_val;
  int64_t st_cap;
  int64_t *acc_total;
  uint4 *spill[2];               // survivor queue per measure: spill_region entries per phase-1 wave
  uint32_t *spill_count[2];     // entries each phase-1 wave stored in its region
  // the regions that hold entries, in order (k_batch_offsets): x = entries of all
  // before, y = wave; at [spill_waves] the total and the number of such regions
  uint2 *spill_used[2];
  int64_t spill_region;
  int32_t spill_waves;          // waves of the phase-1 grid
  int32_t inreg_levels;
};

// Spill entry: x = candidate position (low), y = candidate position (high),
// z = list index, w = m | level << 16 (level = next level to run).
__device__ inline uint4 spill_entry(int64_t pos, uint32_t list, uint32_t m, uint32_t next_level) {
  return make_uint4(uint32_t(pos), uint32_t(uint64_t(pos) >> 32), list, m | (next_level << 16));
}

__device__ inline BatchList ld_list(const BatchList *p) {
  BatchList r;
  r.offset = ld_uniform(&p->offset);
  r.length = ld_uniform(&p->length);
  r.query = ld_uniform(&p->query);
  r.measure = ld_uniform(&p->measure);
  r.table = ld_uniform(&p->table);
  r.pad = 0;
  return r;
}

template <int G, int... S>
__device__ inline void group_bcast_all(uint32_t v, uint32_t *out, std::integer_sequence<int, S...>) {
  ((out[S] = group_bcast<G, S>(v)), ...);
}

// Wave-level compaction of accepted pairs into the wave's staging slice (the
// list itself past the slice's capacity); called by all lanes of the wave.
__device__ inline void emit_block(const BatchBlock &B, bool pred, int64_t idx, float val) {
  uint64_t mask = __ballot(pred);
  if (mask == 0) return;
  {
    const int sl = wave_slice();
    const int leader = __ffsll((unsigned long long)mask) - 1;
    unsigned long long base = 0;
    if (lane_id() == leader)
      base = atomicAdd((unsigned long long *)(B.acc_cnt + sl * kCntStride), (unsigned long long)__popcll(mask));
    base = __shfl(base, leader);
    const unsigned long long pos = base + lanes_below(mask);
    if (pred && int64_t(pos) < B.st_cap) {
      B.st_idx[size_t(sl) * B.st_cap + pos] = uint64_t(idx);
      B.st_val[size_t(sl) * B.st_cap + pos] = val;
      pred = false;
    }
    mask = __ballot(pred);
    if (mask == 0) return;
  }
  const int leader = __ffsll((unsigned long long)mask) - 1;
  unsigned long long base = 0;
  if (lane_id() == leader) base = atomicAdd((unsigned long long *)B.acc_total, (unsigned long long)__popcll(mask));
  base = __shfl(base, leader);
  if (pred) {
    const unsigned long long pos = base + lanes_below(mask);
    if (int64_t(pos) < B.acc_cap) {
      B.acc_idx[pos] = uint64_t(idx);
      B.acc_val[pos] = val;
    } else {
      raise_status(B.status, BLSH_ETRUNCATED);
    }
  }
}

// Survivor queue of a measure: phase-1 wave w owns the entries
// [w R, (w+1) R) (R = spill_region) and keeps its fill `n` in a register, so
// spilling takes a ballot and no atomic.  Bit p of `want`: the lane's
// candidate p; returns the bits whose entry was stored (the others found the
// region full and continue in registers).  Called by all lanes of the wave.
template <int P>
__device__ inline uint32_t spill_tile(const BatchBlock &B, int meas, int64_t wave, uint32_t &n, uint32_t want,
                                      const uint4 *e) {
  const int64_t R = B.spill_region;
  uint4 *region = B.spill[meas] + wave * R;
  uint32_t stored = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint64_t mask = __ballot((want >> p) & 1u);
    if ((want >> p) & 1u) {
      const int64_t pos = int64_t(n) + lanes_below(mask);
      if (pos < R) {
        region[pos] = e[p];
        stored |= 1u << p;
      }
    }
    n = uint32_t(min<int64_t>(R, int64_t(n) + __popcll(mask)));
  }
  return stored;
}

template <int K>
__device__ inline uint32_t srp_level_word_agree(const SigView &s, uint32_t q, uint32_t y, int j) {
  auto word = [&](uint32_t id, int w) -> uint32_t {
    return s.word_major ? s.data[size_t(w) * s.n_obj + id] : s.data[size_t(id) * s.row_words + w];
  };
  if constexpr (K == 32) return 32u - __popc(word(q, j) ^ word(y, j));
  else if constexpr (K == 64) return 64u - __popc(word(q, 2 * j) ^ word(y, 2 * j)) - __popc(word(q, 2 * j + 1) ^ word(y, 2 * j + 1));
  else return 16u - __popc(((word(q, j >> 1) ^ word(y, j >> 1)) >> ((j & 1) * 16)) & 0xFFFFu);
}

// ---------------------------------------------------------------------------
// phase 1: wave tiles
// ---------------------------------------------------------------------------
// agreement of level j from the XOR of two 128-bit prefixes
template <int K>
__device__ inline uint32_t prefix_agree(const uint32_t *d, int j) {
  if constexpr (K == 32) return 32u - __popc(d[j]);
  else if constexpr (K == 64) return 64u - __popc(d[2 * j]) - __popc(d[2 * j + 1]);
  else return 16u - __popc((d[j >> 1] >> ((j & 1) * 16)) & 0xFFFFu);
}

// What a wave keeps of a list from tile to tile (uniform).
struct ListState {
  int64_t end;              // one past the list's last candidate
  uint32_t query;
  int32_t id;
  const uint32_t *tab;
  int L, words;
  bool interval;            // the table's accept sets are intervals (thresholds at kTabAloOff)
};

__device__ inline ListState list_state(const BatchBlock &B, int64_t l, const BatchList &Ls) {
  ListState st;
  st.end = Ls.offset + Ls.length;
  st.query = Ls.query;
  st.id = int32_t(l);
  st.tab = ld_uniform(B.tables + Ls.table);
  st.L = ld_uniform(B.n_levels + Ls.table);
  st.words = int(ld_uniform(st.tab + 2));
  st.interval = (ld_uniform(st.tab + kTabFlagOff) & 1u) != 0;
  return st;
}

// Accept test of level j; alo: its interval's start.
__device__ inline bool accepted_at(const ListState &st, int j, int m, int alo) {
  return st.interval ? m >= alo : accept_bit(st.tab, st.words, j, m);
}

// Candidates base + 64 p + lane below end.
template <int P>
__device__ inline void load_ids(const BatchBlock &B, int64_t base, int64_t end, uint32_t (&y)[P]) {
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t c = base + p * kWave + lane_id();
    y[p] = c < end ? __builtin_nontemporal_load(B.cand + c) : 0u;
  }
}

// 64 P consecutive candidates of one SRP list: candidate base + 64 p + lane,
// its id in y[p].
template <int K, int P>
__device__ inline void srp_tile(const BatchBlock &B, const SigView &S, const ListState &st, int64_t base,
                                const uint32_t (&ids)[P], int64_t wave, uint32_t &n_spill) {
  constexpr int PL = 128 / K;          // levels held by a 128-bit prefix
  const int L = st.L;
  const int lane = lane_id();
  const uint32_t q = st.query;
  const bool q_ok = q < S.n_obj;
  // a prefix view (the caller's prefix array, or object-major rows that a
  // 16-byte load can start): one gather per side serves the first 128 hashes
  const bool pfx = S.pfx != nullptr;
  uint32_t y[P], alive = 0, bad = 0, in = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    y[p] = ids[p];
    if (base + p * kWave + lane < st.end) {
      in |= 1u << p;
      if (q_ok && y[p] < S.n_obj) alive |= 1u << p; else { bad |= 1u << p; y[p] = 0; }
    }
  }
  uint32_t m[P], emit = 0;
  uint8_t code[P];
#pragma unroll
  for (int p = 0; p < P; ++p) { m[p] = 0; code[p] = 0; }
  auto decide = [&](int p, int j) {
    if (int(m[p]) < int(ld_uniform(st.tab + kTabMinOff + j))) {
      code[p] = uint8_t((BLSH_PRUNED << 6) | j);
      alive &= ~(1u << p);
    } else if (accepted_at(st, j, int(m[p]), int(ld_uniform(st.tab + kTabAloOff + j)))) {
      code[p] = uint8_t((BLSH_ACCEPT_CONC << 6) | j);
      alive &= ~(1u << p);
      emit |= 1u << p;
    } else if (j == L - 1) {
      code[p] = uint8_t((BLSH_ACCEPT_NMAX << 6) | j);
      alive &= ~(1u << p);
      emit |= 1u << p;
    }
  };
  auto word_levels = [&](int j0, int j1) {
    for (int j = j0; j < j1 && __ballot(alive != 0); ++j) {
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (alive & (1u << p)) m[p] += srp_level_word_agree<K>(S, q, y[p], j);
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (alive & (1u << p)) decide(p, j);
    }
  };
  const int J = min(L, max(B.inreg_levels, pfx ? PL : 0));
  int j = 0;
  if (pfx && __ballot(alive != 0)) {
    // all gathers issued before any is consumed; a lane without a live
    // candidate reads the query's own row
    const u32x4 hq = ld_uniform(reinterpret_cast<const u32x4 *>(S.pfx + size_t(q) * S.pfx_stride));
    u32x4 hy[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
      hy[p] = *reinterpret_cast<const u32x4 *>(S.pfx + size_t((alive >> p) & 1u ? y[p] : q) * S.pfx_stride);
    uint32_t d[P][4];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      d[p][0] = hq.x ^ hy[p].x; d[p][1] = hq.y ^ hy[p].y;
      d[p][2] = hq.z ^ hy[p].z; d[p][3] = hq.w ^ hy[p].w;
    }
    const int JP = min(J, PL);
#pragma unroll
    for (int jj = 0; jj < PL; ++jj) {   // unrolled: d is indexed by constants
      if (jj < JP && __ballot(alive != 0)) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
          if (!(alive & (1u << p))) continue;
          m[p] += prefix_agree<K>(d[p], jj);
          decide(p, jj);
        }
      }
    }
    j = JP;
  }
  word_levels(j, J);
  // spill what is still undecided; what cannot be spilled continues here
  if (J < L) {
    uint4 e[P];
#pragma unroll
    for (int p = 0; p < P; ++p) e[p] = spill_entry(base + p * kWave + lane, uint32_t(st.id), m[p], uint32_t(J));
    alive &= ~spill_tile<P>(B, BLSH_COSINE, wave, n_spill, alive, e);
  }
  word_levels(J, L);
  if (bad) raise_status(B.status, BLSH_EBADID);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (!((in >> p) & 1u)) continue;
    const int64_t c = base + p * kWave + lane;
    B.code[c] = (bad >> p) & 1u ? uint8_t(0xFF) : code[p];
    if (B.m_dbg) B.m_dbg[c] = uint16_t(m[p]);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const bool e = (emit >> p) & 1u;
    const float v = e ? map_estimate(BLSH_COSINE, int(m[p]), ((code[p] & 63) + 1) * K, 1.0, 1.0) : 0.f;
    emit_block(B, e, base + p * kWave + lane, v);
  }
}

// 64 P consecutive candidates of one minhash list: lane l owns candidates
// base + 64 p + l; the group of G = k/4 lanes holding a candidate compares the
// k hashes of each of its G members in turn (lane r holds hashes 4r..4r+3 of
// the level), with the rows of a pass loaded for all P candidates before any
// comparison.
template <int K, int P>
__device__ inline void minhash_tile(const BatchBlock &B, const SigView &S, const ListState &st, int64_t base,
                                    const uint32_t (&ids)[P], int64_t wave, uint32_t &n_spill) {
  constexpr int G = K / 4;
  constexpr int CH = G < 8 ? G : 8;      // rows in flight per pass and candidate
  const int L = st.L;
  const int lane = lane_id(), r = lane & (G - 1);
  const uint32_t q = st.query;
  const bool q_ok = q < S.n_obj;
  uint32_t y[P], m[P], alive = 0, bad = 0, in = 0, emit = 0;
  uint8_t code[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    y[p] = ids[p];
    m[p] = 0;
    code[p] = 0;
    if (base + p * kWave + lane < st.end) {
      in |= 1u << p;
      if (q_ok && y[p] < S.n_obj) alive |= 1u << p; else bad |= 1u << p;
    }
  }
  auto level = [&](int j) {
    // a lane whose candidate is decided (or invalid) reads the query's row
    uint32_t ys[P][G];
#pragma unroll
    for (int p = 0; p < P; ++p)
      group_bcast_all<G>((alive >> p) & 1u ? y[p] : q, ys[p], std::make_integer_sequence<int, G>{});
    const size_t col = size_t(j) * K + 4 * r;
    const uint4 hq = *reinterpret_cast<const uint4 *>(S.data + size_t(q) * S.row_words + col);
    uint32_t own[P];
#pragma unroll
    for (int p = 0; p < P; ++p) own[p] = 0;
#pragma unroll
    for (int s0 = 0; s0 < G; s0 += CH) {
      uint4 hy[P][CH];
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int s = 0; s < CH; ++s)
          hy[p][s] = *reinterpret_cast<const uint4 *>(S.data + size_t(ys[p][s0 + s]) * S.row_words + col);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int s = 0; s < CH; ++s) {
          uint32_t cnt = uint32_t(hq.x == hy[p][s].x) + uint32_t(hq.y == hy[p][s].y) +
                         uint32_t(hq.z == hy[p][s].z) + uint32_t(hq.w == hy[p][s].w);
          cnt = group_sum<G>(cnt);
          if (r == s0 + s) own[p] = cnt;
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (!((alive >> p) & 1u)) continue;
      m[p] += own[p];
      const int mp = int(m[p]);
      if (mp < int(ld_uniform(st.tab + kTabMinOff + j))) {
        code[p] = uint8_t((BLSH_PRUNED << 6) | j);
        alive &= ~(1u << p);
      } else if (accepted_at(st, j, mp, int(ld_uniform(st.tab + kTabAloOff + j)))) {
        code[p] = uint8_t((BLSH_ACCEPT_CONC << 6) | j);
        alive &= ~(1u << p);
        emit |= 1u << p;
      } else if (j == L - 1) {
        code[p] = uint8_t((BLSH_ACCEPT_NMAX << 6) | j);
        alive &= ~(1u << p);
        emit |= 1u << p;
      }
    }
  };
  const int J = min(L, B.inreg_levels);
  for (int j = 0; j < J && __ballot(alive != 0); ++j) level(j);
  if (J < L) {
    uint4 e[P];
#pragma unroll
    for (int p = 0; p < P; ++p) e[p] = spill_entry(base + p * kWave + lane, uint32_t(st.id), m[p], uint32_t(J));
    alive &= ~spill_tile<P>(B, BLSH_JACCARD, wave, n_spill, alive, e);
  }
  for (int j = J; j < L && __ballot(alive != 0); ++j) level(j);
  if (bad) raise_status(B.status, BLSH_EBADID);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (!((in >> p) & 1u)) continue;
    const int64_t c = base + p * kWave + lane;
    B.code[c] = (bad >> p) & 1u ? uint8_t(0xFF) : code[p];
    if (B.m_dbg) B.m_dbg[c] = uint16_t(m[p]);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const bool e = (emit >> p) & 1u;
    const float v = e ? map_estimate(BLSH_JACCARD, int(m[p]), ((code[p] & 63) + 1) * K, B.alpha, B.beta) : 0.f;
    emit_block(B, e, base + p * kWave + lane, v);
  }
}

// Index of the list holding tile t (the last l with prefix[l] <= t).
__device__ inline int64_t list_of_tile(const int64_t *prefix, int64_t n_lists, int64_t t) {
  int64_t lo = 0, hi = n_lists - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (ld_uniform(prefix + mid) <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same by the whole wave, 64 lists a probe.
__device__ inline int64_t wave_list_of_tile(const int64_t *prefix, int64_t n_lists, int64_t t) {
  int64_t lo = 0, len = n_lists;
  while (len > 1) {
    const int64_t step = (len + kWave - 1) / kWave, at = lo + lane_id() * step;
    const uint64_t mask = __ballot(lane_id() * step < len && prefix[min(at, n_lists - 1)] <= t);   // a run from lane 0
    const int64_t hit = max(__popcll(mask), 1) - 1;
    lo += hit * step;
    len = min(step, len - hit * step);
  }
  return lo;
}

// The w-th of W equal parts of slice x's T tiles in order, list after list, belongs to wave w
// (lists of measure MEAS, 64 P candidates per tile).  Where a list spans several
// whole waves these share its tiles by turns, not by ranges, so that the waves
// of all long lists pass through their sorted ids together and read the same
// rows at about the same time.  (Parts of one size rounded up start at another
// place of every list where lists are of one length: 512 lists of 100,000, 1M rows of 1024
// bits, 711 us instead of 369.)  A list's query, thresholds and pointers are kept
// from tile to tile, and the next tile's ids requested before a tile is run.
template <int MEAS, int K, int P>
__device__ inline void phase1_range(const BatchBlock &B, int x, const int64_t *prefix, int64_t T, int64_t w, int64_t W,
                                    int64_t wave, uint32_t &n_spill) {
  constexpr int64_t tsz = int64_t(P) * kWave;
  const SigView S = B.sig[MEAS];
  const int64_t t0 = w * T / W, t1 = (w + 1) * T / W;
  if (t0 == t1) return;
  int64_t l = wave_list_of_tile(prefix, B.n_lists, t0);
  int64_t first = ld_uniform(prefix + l), next = ld_uniform(prefix + l + 1);
  for (int64_t t = t0; t < t1;) {
    while (t >= next) {   // lists with no tiles in this slice
      ++l;
      first = next;
      next = ld_uniform(prefix + l + 1);
    }
    const BatchList Ls = ld_list(B.lists + l);
    int64_t n = min(t1, next) - t;   // tiles of this list here, `stride` apart
    int64_t stride = 1, at = t - first;
    if (t == t0 && t1 <= next && T >= W) {   // the whole wave: one of those, [wa, wb), whose parts (none empty) lie within the list
      const int64_t wa = (first * W + T - 1) / T, wb = min(W, ((next + 1) * W + T - 1) / T - 1);
      stride = wb - wa;
      at = wa * T / W - first + (w - wa);
      n = (wb * T / W - first - at + stride - 1) / stride;
      t = t1;
    } else {
      t += n;
    }
    const int64_t tile = (int64_t(x) * ((Ls.length + tsz - 1) / tsz)) / kXcds + at;
    int64_t base = Ls.offset + tile * tsz;
    uint32_t y[P], yn[P];
    load_ids<P>(B, base, Ls.offset + Ls.length, y);
    const ListState st = list_state(B, l, Ls);
    for (; n > 0; --n, base += stride * tsz) {
      load_ids<P>(B, base + stride * tsz, n > 1 ? st.end : 0, yn);
      if constexpr (MEAS == BLSH_COSINE) srp_tile<K, P>(B, S, st, base, y, wave, n_spill);
      else minhash_tile<K, P>(B, S, st, base, y, wave, n_spill);
#pragma unroll
      for (int p = 0; p < P; ++p) y[p] = yn[p];
    }
  }
}

// Blocks are dealt round-robin over the XCDs (block b runs on XCD b mod 8),
// each with its own L2.  Phase 1 gives the blocks of XCD x the x-th eighth
// (by position) of every list's tiles: lists hold sorted candidate ids, so an
// XCD touches about an eighth of the signature rows and its L2 holds them.
// Within an XCD every wave takes an equal share of that XCD's tiles (phase1_range).  One
// launch runs the lists of one measure (MEAS), so the streaming minhash rows
// do not evict the SRP rows from L2.  Bound by a tile's chain -- ids from HBM, rows
// from L2, thresholds -- and for minhash by the lines that miss L2.  512 lists,
// 32 M SRP candidates (k = 64, a prefix array): 199 us reading each list's state
// and ids tile by tile, 159 with both ahead.
template <int MEAS, int K, int P>
__global__ __launch_bounds__(kBBlock) void k_batch_phase1(const BatchBlock *__restrict__ Bp) {
  const BatchBlock &B = *Bp;
  const int x = int(blockIdx.x) % kXcds;
  const int64_t nbx = (int64_t(gridDim.x) - x + kXcds - 1) / kXcds;      // blocks on this XCD (grid >= kXcds)
  const int64_t wx = int64_t(blockIdx.x / kXcds) * (kBBlock / kWave) +
                     int64_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
  const int64_t Wx = nbx * (kBBlock / kWave);
  const int64_t *prefix = B.tile_prefix + int64_t(MEAS * kXcds + x) * (B.n_lists + 1);
  const int64_t Tx = ld_uniform(prefix + B.n_lists);
  const int64_t wave = int64_t(blockIdx.x) * (kBBlock / kWave) +
                       int64_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
  uint32_t n_spill = 0;
  phase1_range<MEAS, K, P>(B, x, prefix, Tx, wx, Wx, wave, n_spill);
  if (lane_id() == 0)   // every wave of the grid reports its fill, 0 included
    B.spill_count[MEAS][wave] = n_spill;
}

// ---------------------------------------------------------------------------
// phase 2: spilled survivors
// ---------------------------------------------------------------------------
// The regions that hold entries, with the entries before each (one block per
// measure).  Empty ones are left out, so any 64 consecutive items of the queue
// lie in at most 64 consecutive regions of the list.
constexpr int kOffsetsBlock = 1024;
static_assert(kBBlock / kWave == 4, "four waves a block: the counts are whole 16-byte groups");
__global__ __launch_bounds__(kOffsetsBlock) void k_batch_offsets(const BatchBlock *__restrict__ Bp) {
  const BatchBlock &B = *Bp;
  __shared__ uint64_t s_sum[2][kOffsetsBlock / kWave];
  const uint4 *cnt = reinterpret_cast<const uint4 *>(B.spill_count[blockIdx.x]);
  uint2 *used = B.spill_used[blockIdx.x];
  const int W4 = B.spill_waves / 4, t = threadIdx.x;
  // regions in the high half, entries in the low
  uint64_t carry = 0;
  for (int w0 = 0, buf = 0; w0 < W4; w0 += kOffsetsBlock, buf ^= 1) {
    uint4 c = make_uint4(0, 0, 0, 0);
    if (w0 + t < W4) c = cnt[w0 + t];
    const uint32_t n[4] = {c.x, c.y, c.z, c.w};
    uint64_t own = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) own += (n[i] ? uint64_t(1) << 32 : 0) + n[i];
    uint64_t v = own;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t u = __shfl_up(v, o);
      if (lane_id() >= o) v += u;
    }
    if (lane_id() == kWave - 1) s_sum[buf][t / kWave] = v;
    __syncthreads();
    uint64_t before = carry + v - own;
#pragma unroll
    for (int w = 0; w < kOffsetsBlock / kWave; ++w) {
      const uint64_t u = s_sum[buf][w];
      if (w < t / kWave) before += u;
      carry += u;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (n[i]) {
        used[before >> 32] = make_uint2(uint32_t(before), uint32_t((w0 + t) * 4 + i));
        before += (uint64_t(1) << 32) + n[i];
      }
    }
  }
  if (t == 0) used[B.spill_waves] = make_uint2(uint32_t(carry), uint32_t(carry >> 32));
}

// Entries and regions of a measure's queue.
__device__ inline uint2 queue_end(const BatchBlock &B, int meas) {
  const uint32_t *p = reinterpret_cast<const uint32_t *>(B.spill_used[meas] + B.spill_waves);
  return make_uint2(ld_uniform(p), ld_uniform(p + 1));
}

// Entry i0 + k (k < 64, this lane's) of a measure's queue; `end` = (total, regions).
// Called by all lanes of the wave; lanes past the total take the last entry.
__device__ inline uint4 spilled_item(const BatchBlock &B, int meas, uint2 end, uint32_t i0, uint32_t k) {
  const uint2 *used = B.spill_used[meas];
  const uint32_t n = end.y, lane = lane_id();
  // last region starting at or before i0, 64 probes at a time
  uint32_t lo = 0, len = n;
  while (len > kWave) {
    const uint32_t step = (len + kWave - 1) / kWave, at = lo + lane * step;
    const uint64_t mask = __ballot(at < lo + len && used[min(at, n - 1)].x <= i0);   // lane 0's always is
    const uint32_t hit = uint32_t(__popcll(mask)) - 1;
    len = min(step, len - hit * step);
    lo += hit * step;
  }
  uint2 u = used[min(lo + lane, n - 1)];
  const uint32_t skip = uint32_t(__popcll(__ballot(lane < len && u.x <= i0))) - 1;
  if (skip != 0) {
    lo += skip;
    u = used[min(lo + lane, n - 1)];
  }
  // this lane's region among the 64 from there
  const uint32_t i = min(i0 + k, end.x - 1);
  int a = 0;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const uint32_t f = uint32_t(__shfl(int(u.x), a + o));
    if (lo + a + o < n && f <= i) a += o;
  }
  const uint32_t first = uint32_t(__shfl(int(u.x), a)), w = uint32_t(__shfl(int(u.y), a));
  return B.spill[meas][int64_t(w) * B.spill_region + (i - first)];
}

// A survivor's decisions: the thresholds of a level, and the accept test (a
// compare where the level's accept set is an interval, as its table says).
struct LevelRule {
  const uint32_t *tab;
  int words;
  bool interval;
  __device__ explicit LevelRule(const uint32_t *t) : tab(t), words(int(t[2])), interval((t[kTabFlagOff] & 1u) != 0) {}
  __device__ bool accepted(int j, int m, int alo) const { return interval ? m >= alo : accept_bit(tab, words, j, m); }
};

// SRP words of level j of q and y (k = 16: the word holding the level)
template <int K>
struct LevelWords {
  uint32_t q[K == 64 ? 2 : 1], y[K == 64 ? 2 : 1];
};
template <int K>
__device__ inline void load_level(const SigView &s, uint32_t q, uint32_t y, int j, LevelWords<K> &w) {
  auto word = [&](uint32_t id, int i) -> uint32_t {
    return s.word_major ? s.data[size_t(i) * s.n_obj + id] : s.data[size_t(id) * s.row_words + i];
  };
  if constexpr (K == 64) {
    w.q[0] = word(q, 2 * j);
    w.q[1] = word(q, 2 * j + 1);
    w.y[0] = word(y, 2 * j);
    w.y[1] = word(y, 2 * j + 1);
  } else {
    const int i = K == 32 ? j : j >> 1;
    w.q[0] = word(q, i);
    w.y[0] = word(y, i);
  }
}
template <int K>
__device__ inline uint32_t level_agree(const LevelWords<K> &w, int j) {
  if constexpr (K == 64) return 64u - __popc(w.q[0] ^ w.y[0]) - __popc(w.q[1] ^ w.y[1]);
  else if constexpr (K == 32) return 32u - __popc(w.q[0] ^ w.y[0]);
  else return 16u - __popc(((w.q[0] ^ w.y[0]) >> ((j & 1) * 16)) & 0xFFFFu);
}

// Levels of a survivor loaded together.  A survivor of the first levels is as
// often as not decided at its next one, so the first step of k = 64 (two words
// per side and level) and of minhash (a line per side) loads that alone; what is
// left by then tends to go deep, and four levels at a time shorten its chain of
// dependent reads.
template <int K>
constexpr int phase2_first() { return K == 64 ? 1 : 4; }
constexpr int kPhase2Ahead = 4;

// Every wave takes an equal share of each queue, by items of all phase-1 waves:
// related candidates have neighbouring ids, so single waves of phase 1 hold
// thousands of survivors where most hold none.  Bound by the chain of a survivor's
// dependent reads (entry, list, table, rows by steps).  512 lists of 56 M
// candidates, 0.6 M survivors (k = 16 / 64): 316 us with each block draining the
// regions of its own phase-1 waves one level at a time, 66 + 5 (the offsets) now;
// 64 lists of 6.9 M: the whole batch 187 -> 118 us.
template <int KJ, int KC>
__global__ __launch_bounds__(kBBlock) void k_batch_phase2(const BatchBlock *__restrict__ Bp) {
  constexpr int G = KJ / 4;
  const BatchBlock &B = *Bp;
  const int lane = lane_id();
  const uint32_t wave = blockIdx.x * (kBBlock / kWave) + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave));
  const uint32_t waves = gridDim.x * (kBBlock / kWave);
  // SRP survivors: one lane each
  {
    const SigView &S = B.sig[BLSH_COSINE];
    const uint2 end = queue_end(B, BLSH_COSINE);
    const uint32_t total = end.x;
    for (uint64_t i0 = uint64_t(wave) * kWave; i0 < total; i0 += uint64_t(waves) * kWave) {
      const bool act = i0 + lane < total;
      int64_t pos = 0;
      uint32_t m = 0;
      uint8_t code = 0;
      bool emit = false;
      const uint4 e = spilled_item(B, BLSH_COSINE, end, uint32_t(i0), lane);
      if (act) {
        pos = int64_t(uint64_t(e.x) | (uint64_t(e.y) << 32));
        const BatchList Ls = B.lists[e.z];
        const LevelRule T(B.tables[Ls.table]);
        const int L = B.n_levels[Ls.table];
        m = e.w & 0xFFFFu;
        const uint32_t q = Ls.query, yv = B.cand[pos];
        bool done = false;
        for (int j0 = int(e.w >> 16), n = phase2_first<KC>(); !done; j0 += n, n = kPhase2Ahead) {
          const int j1 = min(L, j0 + n);
          LevelWords<KC> lw[kPhase2Ahead];
          int lo[kPhase2Ahead], alo[kPhase2Ahead];
#pragma unroll
          for (int d = 0; d < kPhase2Ahead; ++d)
            if (j0 + d < j1) {
              load_level<KC>(S, q, yv, j0 + d, lw[d]);
              lo[d] = int(T.tab[kTabMinOff + j0 + d]);
              alo[d] = int(T.tab[kTabAloOff + j0 + d]);
            }
#pragma unroll
          for (int d = 0; d < kPhase2Ahead; ++d) {
            const int j = j0 + d;
            if (done || j >= j1) break;
            m += level_agree<KC>(lw[d], j);
            if (int(m) < lo[d]) { code = uint8_t((BLSH_PRUNED << 6) | j); done = true; }
            else if (T.accepted(j, int(m), alo[d])) { code = uint8_t((BLSH_ACCEPT_CONC << 6) | j); emit = true; done = true; }
            else if (j == L - 1) { code = uint8_t((BLSH_ACCEPT_NMAX << 6) | j); emit = true; done = true; }
          }
        }
        B.code[pos] = code;
        if (B.m_dbg) B.m_dbg[pos] = uint16_t(m);
      }
      const float v = emit ? map_estimate(BLSH_COSINE, int(m), ((code & 63) + 1) * KC, 1.0, 1.0) : 0.f;
      emit_block(B, emit, pos, v);
    }
  }
  // minhash survivors: one group of G lanes each
  {
    const SigView &S = B.sig[BLSH_JACCARD];
    const uint2 end = queue_end(B, BLSH_JACCARD);
    const uint32_t total = end.x;
    constexpr int PER_WAVE = kWave / G;
    const int g = lane / G, r = lane % G;
    for (uint64_t i0 = uint64_t(wave) * PER_WAVE; i0 < total; i0 += uint64_t(waves) * PER_WAVE) {
      const bool act = i0 + g < total;
      int64_t pos = 0;
      uint32_t m = 0;
      uint8_t code = 0;
      bool emit = false;
      const uint4 e = spilled_item(B, BLSH_JACCARD, end, uint32_t(i0), g);
      if (act) {   // (a group's lanes agree on everything below)
        pos = int64_t(uint64_t(e.x) | (uint64_t(e.y) << 32));
        const BatchList Ls = B.lists[e.z];
        const LevelRule T(B.tables[Ls.table]);
        const int L = B.n_levels[Ls.table];
        m = e.w & 0xFFFFu;
        const uint32_t *rq = S.data + size_t(Ls.query) * S.row_words + 4 * r;
        const uint32_t *ry = S.data + size_t(B.cand[pos]) * S.row_words + 4 * r;
        bool done = false;
        for (int j0 = int(e.w >> 16), n = 1; !done; j0 += n, n = kPhase2Ahead) {
          const int j1 = min(L, j0 + n);
          uint4 hq[kPhase2Ahead], hy[kPhase2Ahead];
          int lo[kPhase2Ahead], alo[kPhase2Ahead];
#pragma unroll
          for (int d = 0; d < kPhase2Ahead; ++d)
            if (j0 + d < j1) {
              hq[d] = *reinterpret_cast<const uint4 *>(rq + (j0 + d) * KJ);
              hy[d] = *reinterpret_cast<const uint4 *>(ry + (j0 + d) * KJ);
              lo[d] = int(T.tab[kTabMinOff + j0 + d]);
              alo[d] = int(T.tab[kTabAloOff + j0 + d]);
            }
#pragma unroll
          for (int d = 0; d < kPhase2Ahead; ++d) {
            const int j = j0 + d;
            if (done || j >= j1) break;
            m += group_sum<G>(uint32_t(hq[d].x == hy[d].x) + uint32_t(hq[d].y == hy[d].y) +
                              uint32_t(hq[d].z == hy[d].z) + uint32_t(hq[d].w == hy[d].w));
            if (int(m) < lo[d]) { code = uint8_t((BLSH_PRUNED << 6) | j); done = true; }
            else if (T.accepted(j, int(m), alo[d])) { code = uint8_t((BLSH_ACCEPT_CONC << 6) | j); emit = true; done = true; }
            else if (j == L - 1) { code = uint8_t((BLSH_ACCEPT_NMAX << 6) | j); emit = true; done = true; }
          }
        }
        if (r == 0) {
          B.code[pos] = code;
          if (B.m_dbg) B.m_dbg[pos] = uint16_t(m);
        }
      }
      emit = emit && r == 0;
      const float v = emit ? map_estimate(BLSH_JACCARD, int(m), ((code & 63) + 1) * KJ, B.alpha, B.beta) : 0.f;
      emit_block(B, emit, pos, v);
    }
  }
}

// ---------------------------------------------------------------------------
// exhaustive comparator over the same tiles: every candidate compares the
// full n_max hashes of its row with the query's, and the decision sequence of
// Algorithm 1 is replayed on the per-level counts (same output).
// ---------------------------------------------------------------------------
// first level in [j0, j1) at which the running count decides; updates m
__device__ inline int replay_level(const uint32_t *tab, int words, int L, int j, int m, uint8_t &code) {
  if (m < int(tab[kTabMinOff + j])) { code = uint8_t((BLSH_PRUNED << 6) | j); return 1; }
  if (accept_bit(tab, words, j, m)) { code = uint8_t((BLSH_ACCEPT_CONC << 6) | j); return 2; }
  if (j == L - 1) { code = uint8_t((BLSH_ACCEPT_NMAX << 6) | j); return 2; }
  return 0;
}

// SRP rows of W words: groups of G = W/4 lanes per candidate (one 16-byte load
// per lane), exclusive prefix of lane totals, first deciding lane by ballot.
template <int K, int G>
__device__ void srp_tile_exhaustive(const BatchBlock &B, const BatchList &Ls, int64_t tile_in_list,
                                    const uint32_t *tab, int L) {
  constexpr int LPL = 128 / K;                 // levels per lane
  constexpr int PER_BLOCK = kBBlock / G;
  const SigView &S = B.sig[BLSH_COSINE];
  const int words = int(tab[2]);
  const int lane = lane_id(), r = lane % G, g = threadIdx.x / G, gw = lane / G;
  const int64_t end = Ls.offset + Ls.length;
  const uint32_t q = Ls.query;
  const bool q_ok = q < S.n_obj;
  uint4 hq = make_uint4(0, 0, 0, 0);
  if (q_ok) hq = *reinterpret_cast<const uint4 *>(S.data + size_t(q) * S.row_words + 4 * r);
  const int64_t t0 = Ls.offset + tile_in_list * kExSrpTile;
  for (int64_t c0 = t0; c0 < min(end, t0 + kExSrpTile); c0 += PER_BLOCK) {
    const int64_t c = c0 + g;
    const bool in = c < end;
    uint32_t y = 0;
    bool ok = false;
    if (in) {
      y = B.cand[c];
      ok = q_ok && y < S.n_obj;
    }
    uint32_t cnt[LPL], tot = 0;
    if (ok) {
      const uint4 hy = *reinterpret_cast<const uint4 *>(S.data + size_t(y) * S.row_words + 4 * r);
      const uint32_t d[4] = {hq.x ^ hy.x, hq.y ^ hy.y, hq.z ^ hy.z, hq.w ^ hy.w};
#pragma unroll
      for (int qq = 0; qq < LPL; ++qq) {
        if constexpr (K == 16) cnt[qq] = 16u - __popc((d[qq >> 1] >> ((qq & 1) * 16)) & 0xFFFFu);
        else if constexpr (K == 32) cnt[qq] = 32u - __popc(d[qq]);
        else cnt[qq] = 64u - __popc(d[2 * qq]) - __popc(d[2 * qq + 1]);
        tot += cnt[qq];
      }
    } else {
#pragma unroll
      for (int qq = 0; qq < LPL; ++qq) cnt[qq] = 0;
    }
    uint32_t incl = tot;
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
      const uint32_t v = __shfl_up(incl, o, G);
      if (r >= o) incl += v;
    }
    uint32_t run = incl - tot;
    int dec = 0, dm = 0;
    uint8_t dcode = 0;
#pragma unroll
    for (int qq = 0; qq < LPL; ++qq) {
      run += cnt[qq];
      const int j = r * LPL + qq;
      uint8_t cd;
      if (!dec && ok && j < L) {
        const int rr = replay_level(tab, words, L, j, int(run), cd);
        if (rr) { dec = rr; dm = int(run); dcode = cd; }
      }
    }
    const uint64_t has = __ballot(dec != 0);
    const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1ull)) << (gw * G);
    const uint64_t mine = has & gmask;
    const int first = mine ? __ffsll((unsigned long long)mine) - 1 : gw * G;
    const int fdec = __shfl(dec, first), fm = __shfl(dm, first);
    const uint32_t fcode = __shfl(uint32_t(dcode), first);
    bool emit = false;
    if (in && r == 0) {
      B.code[c] = ok ? uint8_t(fcode) : uint8_t(0xFF);
      if (B.m_dbg) B.m_dbg[c] = uint16_t(fm);
      emit = ok && fdec == 2;
      if (!ok) raise_status(B.status, BLSH_EBADID);
    }
    const float v = emit ? map_estimate(BLSH_COSINE, fm, ((fcode & 63) + 1) * K, 1.0, 1.0) : 0.f;
    emit_block(B, emit, c, v);
  }
}

// Minhash rows: groups of 16 lanes per candidate, 64 hashes (256 B) per pass;
// per-level sums with DPP, then the levels replayed in order.
template <int K>
__device__ void minhash_tile_exhaustive(const BatchBlock &B, const BatchList &Ls, int64_t tile_in_list,
                                        const uint32_t *tab, int L, int H) {
  constexpr int G = 16;
  constexpr int LPC = 64 / K;                  // levels per 64-hash chunk
  constexpr int LL = K / 4;                    // lanes per level
  constexpr int PER_BLOCK = kBBlock / G;
  const SigView &S = B.sig[BLSH_JACCARD];
  const int words = int(tab[2]);
  const int lane = lane_id(), r = lane % G, g = threadIdx.x / G, gw = lane / G;
  const int64_t end = Ls.offset + Ls.length;
  const uint32_t q = Ls.query;
  const bool q_ok = q < S.n_obj;
  const int64_t t0 = Ls.offset + tile_in_list * kExMhTile;
  for (int64_t c0 = t0; c0 < min(end, t0 + kExMhTile); c0 += PER_BLOCK) {
    const int64_t c = c0 + g;
    const bool in = c < end;
    uint32_t y = 0;
    bool ok = false;
    if (in) {
      y = B.cand[c];
      ok = q_ok && y < S.n_obj;
    }
    int m = 0, dec = 0, dm = 0;
    uint8_t dcode = 0;
    for (int h0 = 0; h0 < H; h0 += 64) {
      uint32_t cnt = 0;
      if (ok) {
        const uint4 hq = *reinterpret_cast<const uint4 *>(S.data + size_t(q) * S.row_words + h0 + 4 * r);
        const uint4 hy = *reinterpret_cast<const uint4 *>(S.data + size_t(y) * S.row_words + h0 + 4 * r);
        cnt = uint32_t(hq.x == hy.x) + uint32_t(hq.y == hy.y) + uint32_t(hq.z == hy.z) + uint32_t(hq.w == hy.w);
      }
      cnt = group_sum<LL>(cnt);
#pragma unroll
      for (int sl = 0; sl < LPC; ++sl) {
        const uint32_t lev = __shfl(cnt, gw * G + sl * LL);
        m += int(lev);
        const int j = h0 / K + sl;
        uint8_t cd;
        if (!dec && ok && j < L) {
          const int rr = replay_level(tab, words, L, j, m, cd);
          if (rr) { dec = rr; dm = m; dcode = cd; }
        }
      }
    }
    bool emit = false;
    if (in && r == 0) {
      B.code[c] = ok ? dcode : uint8_t(0xFF);
      if (B.m_dbg) B.m_dbg[c] = uint16_t(dm);
      emit = ok && dec == 2;
      if (!ok) raise_status(B.status, BLSH_EBADID);
    }
    const float v = emit ? map_estimate(BLSH_JACCARD, dm, ((dcode & 63) + 1) * K, B.alpha, B.beta) : 0.f;
    emit_block(B, emit, c, v);
  }
}

// Block b of the fixed grid runs the block tiles [b T / NB, (b+1) T / NB).
template <int KJ, int KC>
__global__ __launch_bounds__(kBBlock) void k_batch_exhaustive(const BatchBlock *__restrict__ Bp) {
  const BatchBlock &B = *Bp;
  const int64_t T = B.n_tiles, NB = gridDim.x;
  const int64_t t0 = int64_t(blockIdx.x) * T / NB, t1 = (int64_t(blockIdx.x) + 1) * T / NB;
  if (t0 >= t1) return;
  int64_t l = list_of_tile(B.tile_prefix, B.n_lists, t0);
  int64_t first = ld_uniform(B.tile_prefix + l), next = ld_uniform(B.tile_prefix + l + 1);
  for (int64_t t = t0; t < t1; ++t) {
    while (t >= next) {
      ++l;
      first = next;
      next = ld_uniform(B.tile_prefix + l + 1);
    }
    const BatchList Ls = ld_list(B.lists + l);
    const uint32_t *tab = ld_uniform(B.tables + Ls.table);
    const int L = ld_uniform(B.n_levels + Ls.table);
    const int64_t tl = t - first;
    if (Ls.measure == BLSH_COSINE) {
      const int W = L * KC / 32;   // words compared: n_max bits
      if (W == 4) srp_tile_exhaustive<KC, 1>(B, Ls, tl, tab, L);
      else if (W == 8) srp_tile_exhaustive<KC, 2>(B, Ls, tl, tab, L);
      else if (W == 16) srp_tile_exhaustive<KC, 4>(B, Ls, tl, tab, L);
      else if (W == 32) srp_tile_exhaustive<KC, 8>(B, Ls, tl, tab, L);
      else srp_tile_exhaustive<KC, 16>(B, Ls, tl, tab, L);
    } else {
      minhash_tile_exhaustive<KJ>(B, Ls, tl, tab, L, L * KJ);
    }
  }
}

// Clears both sets of staging counts and running counts (one block of kSlices
// threads): before the first batch, and after one that was not launched whole.
__global__ void k_batch_reset(int64_t *cnt) {
  for (int set = 0; set < 2; ++set) {
    int64_t *c = cnt + set * (size_t(kSlices) + 1) * kCntStride;
    c[threadIdx.x * kCntStride] = 0;
    if (threadIdx.x == 0) c[size_t(kSlices) * kCntStride] = 0;
  }
}

// Appends the staging slices to the accepted list, one block per slice, no
// atomics: every block scans the kSlices counts, block s copies slice s after
// the slices before it and after the entries written directly; block 0
// stores the final count to *n_acc (which no block reads).  Leaves the next
// batch's counts zero.
__global__ __launch_bounds__(kBBlock) void k_batch_flush(const BatchBlock *__restrict__ Bp) {
  static_assert(kSlices == kBBlock, "one staging slice per thread of a block");
  const BatchBlock &B = *Bp;
  __shared__ int64_t s_cnt[kSlices];
  __shared__ int64_t s_base, s_total;
  const int t = threadIdx.x, sl = blockIdx.x;
  const int64_t c = min(B.acc_cnt[size_t(t) * kCntStride], B.st_cap);
  int64_t v = c;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t u = __shfl_up(v, o);
    if (lane_id() >= o) v += u;
  }
  s_cnt[t] = v;
  __syncthreads();
  int64_t before = 0;
  for (int w = 0; w < (t >> 6); ++w) before += s_cnt[w * kWave + kWave - 1];
  __syncthreads();
  s_cnt[t] = before + v - c;
  if (t == kSlices - 1) s_total = before + v;
  if (t == 0) s_base = *B.acc_total;
  __syncthreads();
  const int64_t n = min(B.acc_cnt[size_t(sl) * kCntStride], B.st_cap);
  const int64_t base = s_base + s_cnt[sl];
  const uint64_t *idx = B.st_idx + size_t(sl) * B.st_cap;
  const float *val = B.st_val + size_t(sl) * B.st_cap;
  bool trunc = false;
  for (int64_t i = t; i < n; i += kBBlock) {
    const int64_t pos = base + i;
    if (pos < B.acc_cap) {
      B.acc_idx[pos] = idx[i];
      B.acc_val[pos] = val[i];
    } else {
      trunc = true;
    }
  }
  if (trunc) raise_status(B.status, BLSH_ETRUNCATED);
  if (t == 0) B.acc_next[size_t(sl) * kCntStride] = 0;
  if (sl == 0 && t == 0) {
    B.acc_next[size_t(kSlices) * kCntStride] = 0;
    *B.n_acc = s_base + s_total;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct BatchState {
  BatchBlock *d_block = nullptr;
  BatchBlock *h_block = nullptr;        // pinned staging
  BatchList *d_lists = nullptr, *h_lists = nullptr;
  int64_t *d_prefix = nullptr, *h_prefix = nullptr;
  int64_t lists_cap = 0;
  // staging: two sets of kSlices counters (kCntStride apart) and the running
  // count, then kSlices x kBatchStage entries
  int64_t *d_stage_cnt = nullptr;
  int stage_set = 0;                    // set of the next batch; its counts are zero
  bool stage_dirty = true;              // unless this is set
  uint64_t *d_st_idx = nullptr;
  float *d_st_val = nullptr;
  uint4 *d_spill[2] = {nullptr, nullptr};
  int64_t spill_cap = 0;
  uint32_t *d_spill_count = nullptr;    // [2][spill_waves_cap]
  uint2 *d_spill_used = nullptr;        // [2][spill_waves_cap + 1]
  int64_t spill_waves_cap = 0;
  hipEvent_t staged{};
  bool staged_valid = false;
  hipStream_t cap_stream{};
  struct GraphKey {
    int mode, kj, kc, ts, tm, grid1, grid2;
    bool operator<(const GraphKey &o) const {
      return std::tie(mode, kj, kc, ts, tm, grid1, grid2) < std::tie(o.mode, o.kj, o.kc, o.ts, o.tm, o.grid1, o.grid2);
    }
  };
  std::map<GraphKey, hipGraphExec_t> graphs;
  // k per measure, SRP / minhash tile (candidates per wave tile), in-register
  // levels, blocks per CU
  struct Choice { int kj, kc, ts, tm, inreg, bpc; };
  std::map<std::vector<int64_t>, Choice> tuned;
  std::map<void (*)(const BatchBlock *), int> resident;   // blocks of a kernel that a CU holds at once
};

static void batch_free(BatchState *b) {
  if (!b) return;
  for (auto &g : b->graphs) (void)hipGraphExecDestroy(g.second);
  if (b->d_block) (void)hipFree(b->d_block);
  if (b->h_block) (void)hipHostFree(b->h_block);
  if (b->d_lists) (void)hipFree(b->d_lists);
  if (b->h_lists) (void)hipHostFree(b->h_lists);
  if (b->d_prefix) (void)hipFree(b->d_prefix);
  if (b->h_prefix) (void)hipHostFree(b->h_prefix);
  if (b->d_stage_cnt) (void)hipFree(b->d_stage_cnt);
  if (b->d_st_idx) (void)hipFree(b->d_st_idx);
  if (b->d_st_val) (void)hipFree(b->d_st_val);
  for (auto *p : b->d_spill) if (p) (void)hipFree(p);
  if (b->d_spill_count) (void)hipFree(b->d_spill_count);
  if (b->d_spill_used) (void)hipFree(b->d_spill_used);
  if (b->staged_valid) (void)hipEventDestroy(b->staged);
  if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
  delete b;
}

void batch_state_free(void *p) { batch_free(static_cast<BatchState *>(p)); }

static int batch_state(blsh_ctx *ctx, BatchState **out) {
  if (!ctx->batch) {
    auto *b = new (std::nothrow) BatchState();
    if (!b) return fail(BLSH_ENOMEM, "host allocation failed");
    if (hipMalloc(&b->d_block, sizeof(BatchBlock)) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void **>(&b->h_block), sizeof(BatchBlock), hipHostMallocDefault) != hipSuccess ||
        hipMalloc(&b->d_stage_cnt, 2 * (size_t(kSlices) + 1) * kCntStride * sizeof(int64_t)) != hipSuccess ||
        hipMalloc(&b->d_st_idx, size_t(kSlices) * kBatchStage * sizeof(uint64_t)) != hipSuccess ||
        hipMalloc(&b->d_st_val, size_t(kSlices) * kBatchStage * sizeof(float)) != hipSuccess ||
        hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->staged, hipEventDisableTiming) != hipSuccess) {
      batch_free(b);
      return fail(BLSH_ENOMEM, "batched state allocation failed");
    }
    b->staged_valid = true;
    ctx->batch = b;
    ctx->batch_free = batch_state_free;
  }
  *out = static_cast<BatchState *>(ctx->batch);
  return BLSH_OK;
}

static int grow_lists(BatchState *b, int64_t n_lists) {
  if (b->lists_cap >= n_lists) return BLSH_OK;
  BLSH_HIP(hipDeviceSynchronize());
  if (b->d_lists) (void)hipFree(b->d_lists);
  if (b->h_lists) (void)hipHostFree(b->h_lists);
  if (b->d_prefix) (void)hipFree(b->d_prefix);
  if (b->h_prefix) (void)hipHostFree(b->h_prefix);
  b->d_lists = b->h_lists = nullptr;
  b->d_prefix = b->h_prefix = nullptr;
  b->lists_cap = 0;
  const int64_t cap = std::max<int64_t>(n_lists, 1024);
  if (hipMalloc(&b->d_lists, cap * sizeof(BatchList)) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void **>(&b->h_lists), cap * sizeof(BatchList), hipHostMallocDefault) != hipSuccess ||
      hipMalloc(&b->d_prefix, 2 * kXcds * (cap + 1) * sizeof(int64_t)) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void **>(&b->h_prefix), 2 * kXcds * (cap + 1) * sizeof(int64_t),
                    hipHostMallocDefault) != hipSuccess)
    return fail(BLSH_ENOMEM, "list buffers");
  b->lists_cap = cap;
  return BLSH_OK;
}

static int grow_spill_counts(BatchState *b, int64_t waves) {
  if (b->spill_waves_cap >= waves) return BLSH_OK;
  BLSH_HIP(hipDeviceSynchronize());
  if (b->d_spill_count) (void)hipFree(b->d_spill_count);
  if (b->d_spill_used) (void)hipFree(b->d_spill_used);
  b->d_spill_count = nullptr;
  b->d_spill_used = nullptr;
  b->spill_waves_cap = 0;
  if (hipMalloc(&b->d_spill_count, size_t(2 * waves) * sizeof(uint32_t)) != hipSuccess ||
      hipMalloc(&b->d_spill_used, size_t(2 * (waves + 1)) * sizeof(uint2)) != hipSuccess)
    return fail(BLSH_ENOMEM, "spill counts");
  b->spill_waves_cap = waves;
  return BLSH_OK;
}

static int grow_spill(BatchState *b, int64_t cap) {
  if (b->spill_cap >= cap) return BLSH_OK;
  BLSH_HIP(hipDeviceSynchronize());
  for (auto *&p : b->d_spill) { if (p) (void)hipFree(p); p = nullptr; }
  b->spill_cap = 0;
  for (auto *&p : b->d_spill)
    if (hipMalloc(&p, size_t(cap) * sizeof(uint4)) != hipSuccess) return fail(BLSH_ENOMEM, "spill buffers");
  b->spill_cap = cap;
  return BLSH_OK;
}

typedef void (*BatchKernel)(const BatchBlock *);

template <int KC>
static BatchKernel phase1_srp(int ts) {
  return ts == 128 ? k_batch_phase1<BLSH_COSINE, KC, 2>
                   : ts == 512 ? k_batch_phase1<BLSH_COSINE, KC, 8> : k_batch_phase1<BLSH_COSINE, KC, 4>;
}

template <int KJ>
static BatchKernel phase1_mh(int tm) {
  return tm == 128 ? k_batch_phase1<BLSH_JACCARD, KJ, 2> : k_batch_phase1<BLSH_JACCARD, KJ, 1>;
}

template <int KJ, int KC>
static void launch_batch_kernels(BatchState *b, const BatchState::GraphKey &gk, hipStream_t s) {
  if (gk.mode == 1) {
    hipLaunchKernelGGL((k_batch_exhaustive<KJ, KC>), dim3(gk.grid1), dim3(kBBlock), 0, s, b->d_block);
  } else {
    hipLaunchKernelGGL(phase1_srp<KC>(gk.ts), dim3(gk.grid1), dim3(kBBlock), 0, s, b->d_block);
    hipLaunchKernelGGL(phase1_mh<KJ>(gk.tm), dim3(gk.grid1), dim3(kBBlock), 0, s, b->d_block);
    hipLaunchKernelGGL(k_batch_offsets, dim3(2), dim3(kOffsetsBlock), 0, s, b->d_block);
    hipLaunchKernelGGL((k_batch_phase2<KJ, KC>), dim3(gk.grid2), dim3(kBBlock), 0, s, b->d_block);
  }
  hipLaunchKernelGGL(k_batch_flush, dim3(kSlices), dim3(kBBlock), 0, s, b->d_block);
}

template <int KJ>
static void launch_batch_kernels_kc(BatchState *b, const BatchState::GraphKey &gk, hipStream_t s) {
  if (gk.kc == 16) launch_batch_kernels<KJ, 16>(b, gk, s);
  else if (gk.kc == 32) launch_batch_kernels<KJ, 32>(b, gk, s);
  else launch_batch_kernels<KJ, 64>(b, gk, s);
}

static int get_graph(BatchState *b, const BatchState::GraphKey &key, hipGraphExec_t *out) {
  auto it = b->graphs.find(key);
  if (it != b->graphs.end()) { *out = it->second; return BLSH_OK; }
  hipGraph_t g;
  BLSH_HIP(hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
  if (key.kj == 16) launch_batch_kernels_kc<16>(b, key, b->cap_stream);
  else if (key.kj == 32) launch_batch_kernels_kc<32>(b, key, b->cap_stream);
  else launch_batch_kernels_kc<64>(b, key, b->cap_stream);
  BLSH_HIP(hipStreamEndCapture(b->cap_stream, &g));
  hipGraphExec_t ex;
  hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return fail(BLSH_EDEVICE, "hipGraphInstantiate: %s", hipGetErrorString(e));
  b->graphs[key] = ex;
  *out = ex;
  return BLSH_OK;
}

// Blocks of the call's kernels that a CU holds at once: the comparator's, or the least
// of the used measures' phase 1.
static int resident_blocks(BatchState *b, const bool *need, int kj, int kc, int ts, int tm, int mode) {
  const int ij = kj == 16 ? 0 : kj == 32 ? 1 : 2, ic = kc == 16 ? 0 : kc == 32 ? 1 : 2;
  static const BatchKernel cmp[3][3] = {
      {k_batch_exhaustive<16, 16>, k_batch_exhaustive<16, 32>, k_batch_exhaustive<16, 64>},
      {k_batch_exhaustive<32, 16>, k_batch_exhaustive<32, 32>, k_batch_exhaustive<32, 64>},
      {k_batch_exhaustive<64, 16>, k_batch_exhaustive<64, 32>, k_batch_exhaustive<64, 64>}};
  const BatchKernel srp = ic == 0 ? phase1_srp<16>(ts) : ic == 1 ? phase1_srp<32>(ts) : phase1_srp<64>(ts);
  const BatchKernel mh = ij == 0 ? phase1_mh<16>(tm) : ij == 1 ? phase1_mh<32>(tm) : phase1_mh<64>(tm);
  int least = kBBlock;
  for (const BatchKernel k : {mode ? cmp[ij][ic] : nullptr, !mode && need[0] ? mh : nullptr, !mode && need[1] ? srp : nullptr}) {
    if (!k) continue;
    int &n = b->resident[k];
    if (n == 0 && (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kBBlock, 0) != hipSuccess || n < 1)) {
      (void)hipGetLastError();
      n = kBlocksDefault;
    }
    least = std::min(least, n);
  }
  return least;
}

// Blocks per CU of a call that neither fixes nor tunes them: as many as a CU holds at
// once, at most kBlocksDefault in phase 1, so that no wave starts when others have ended.
// The comparator (registers: 4 at k = 16 for cosine, 5 at 32, 6 at 64), 14 M candidates
// in 1000 lists of all lengths, sets: 4 a CU 2.80 ms, 6 3.56, 8 2.83 (k = 16); 5 1.39, 6 2.01,
// 8 1.65 (32); 6 1.81, 5 2.06, 8 2.47 (64).  Phase 1 of 216 M candidates, sets, k = 64 (5):
// 5 2.38 ms, 6 2.85, 8 2.48.
// Lists of one length that come several to a wave: a number that gives every wave whole
// lists, if one does, so that all waves start a list at the same time and read the same
// rows (1024 lists of 50,000, 1M rows of 1024 bits: 4 a CU 368 us, 8 422, 6 561; 4096 of
// 12,000: 494, 595, 749; rows read through a prefix array 340, 371, 325).  The comparator
// with 5 keeps in step over many candidates with 8 (512 lists of 50,000 sets 2.14 ms, 5 2.35).
// (Below 2^22 candidates the numbers are alike, and walking 20,000 short lists is not free.)
static int default_blocks(const blsh_ctx *ctx, const blsh_list_desc *lists, int64_t n_lists, int64_t n_cand, int mode,
                          int resident) {
  const int most = mode ? resident : std::min(resident, kBlocksDefault);
  if (mode ? resident != 5 || n_cand < int64_t(1) << 24 : n_cand < int64_t(1) << 22) return most;
  int64_t n[2] = {0, 0}, length[2] = {0, 0};
  for (int64_t i = 0; i < n_lists; ++i) {
    const int me = lists[i].measure == BLSH_COSINE;
    if (n[me]++ == 0) length[me] = lists[i].length;
    else if (length[me] != lists[i].length) return most;
  }
  if (mode) return 8;
  for (const int bpc : {most, 4, 5, 8}) {
    const int64_t waves = int64_t(ctx->n_cu) * bpc / kXcds * (kBBlock / kWave);   // of an XCD
    if (n[0] % waves == 0 && n[1] % waves == 0) return bpc;
  }
  return most;
}

int verify_batched(blsh_ctx *ctx, const blsh_list_desc *lists, int64_t n_lists, const uint32_t *cand, int64_t n_cand,
                   const blsh_sigs *jac, const blsh_sigs *cos, double eps, double delta, double gamma,
                   blsh_prior prior, int32_t kj, int32_t kc, blsh_result *res, int32_t *k_used, hipStream_t s,
                   int (*check_sigs_fn)(const blsh_sigs *, int, int *, int *), int mode) {
  BatchState *b = nullptr;
  int rc = batch_state(ctx, &b);
  if (rc) return rc;
  // --- tables per (measure, t); each measure has its own k ---
  const int k_given[2] = {kj, kc};
  int n_max[2] = {0, 0}, row_words[2] = {0, 0};
  const blsh_sigs *sv[2] = {jac, cos};
  bool need[2] = {false, false};
  for (int64_t i = 0; i < n_lists; ++i) need[lists[i].measure == BLSH_COSINE] = true;
  for (int me = 0; me < 2; ++me) {
    if (!need[me]) continue;
    if (!sv[me]) return fail(BLSH_EINVAL, "a list needs %s signatures", me ? "cosine" : "Jaccard");
    if (sv[me]->measure != me) return fail(BLSH_EINVAL, "signature set has the wrong measure");
    const std::vector<int> ks = k_given[me] ? std::vector<int>{k_given[me]} : std::vector<int>{16, 32, 64};
    for (int kk : ks)
      if ((rc = check_sigs_fn(sv[me], kk, &n_max[me], &row_words[me]))) return rc;
  }
  std::vector<double> ts;
  for (int64_t i = 0; i < n_lists; ++i) ts.push_back(lists[i].t);
  std::sort(ts.begin(), ts.end());
  ts.erase(std::unique(ts.begin(), ts.end()), ts.end());
  if (2 * ts.size() > size_t(kMaxBatchTables)) return fail(BLSH_EINVAL, "at most %d distinct thresholds per batch", kMaxBatchTables / 2);
  // --- work decomposition (does not depend on k) ---
  if ((rc = grow_lists(b, n_lists))) return rc;
  if (b->staged_valid) BLSH_HIP(hipEventSynchronize(b->staged));   // previous call's staging copies are done
  // list descriptors; the tile prefix sums depend on the tile shapes and are
  // built by prepare()
  const int n_slices = mode ? 1 : 2 * kXcds;
  for (int64_t i = 0; i < n_lists; ++i) {
    const blsh_list_desc &d = lists[i];
    BatchList &bl = b->h_lists[i];
    bl.offset = d.offset;
    bl.length = d.length;
    bl.query = d.query;
    bl.measure = d.measure;
    bl.table = int32_t(std::lower_bound(ts.begin(), ts.end(), d.t) - ts.begin()) * 2 + (d.measure == BLSH_COSINE);
    bl.pad = 0;
  }
  // tile prefix sums for SRP / minhash tiles of srp_tile / mh_tile candidates:
  // one array (comparator) or one per (measure, XCD slice)
  int64_t tiles = 0;
  auto build_prefix = [&](int64_t srp_tile, int64_t mh_tile) {
    tiles = 0;
    for (int x = 0; x < n_slices; ++x) b->h_prefix[int64_t(x) * (n_lists + 1)] = 0;
    for (int64_t i = 0; i < n_lists; ++i) {
      const blsh_list_desc &d = lists[i];
      const int64_t tsz = d.measure == BLSH_COSINE ? srp_tile : mh_tile;
      const int64_t nt = (d.length + tsz - 1) / tsz;
      tiles += nt;
      for (int x = 0; x < n_slices; ++x) {
        int64_t *px = b->h_prefix + int64_t(x) * (n_lists + 1);
        if (mode) {
          px[i + 1] = px[i] + nt;
        } else {
          const int me = x / kXcds, xs = x % kXcds;
          px[i + 1] = px[i] + (me == d.measure ? (int64_t(xs + 1) * nt) / kXcds - (int64_t(xs) * nt) / kXcds : 0);
        }
      }
    }
  };
  int64_t prefix_shape[2] = {-1, -1};   // tile shapes of the prefix sums last uploaded in this call
  const int64_t spill_cap = ctx->tuning.batch_spill_cap > 0
                                ? int64_t(ctx->tuning.batch_spill_cap)
                                : std::max<int64_t>(kMinSpill, std::min<int64_t>(n_cand, int64_t(1) << 24));
  if ((rc = grow_spill(b, spill_cap))) return rc;

  auto prepare = [&](int kkj, int kkc, int64_t srp_tile, int64_t mh_tile, int inreg, int grid1) -> int {
    const int kk[2] = {kkj, kkc};
    // the pinned staging (block, prefix sums) is read by the copies enqueued by
    // the previous prepare (the autotuner enqueues several per call): wait for
    // those copies before rewriting it
    BLSH_HIP(hipEventSynchronize(b->staged));
    if (prefix_shape[0] != srp_tile || prefix_shape[1] != mh_tile) {
      build_prefix(srp_tile, mh_tile);
      BLSH_HIP(hipMemcpyAsync(b->d_prefix, b->h_prefix, n_slices * (n_lists + 1) * sizeof(int64_t),
                              hipMemcpyHostToDevice, s));
      prefix_shape[0] = srp_tile;
      prefix_shape[1] = mh_tile;
    }
    BatchBlock &B = *b->h_block;
    std::memset(&B, 0, sizeof(B));
    B.lists = b->d_lists;
    B.tile_prefix = b->d_prefix;
    B.n_lists = n_lists;
    B.n_tiles = tiles;
    B.cand = cand;
    for (int me = 0; me < 2; ++me) {
      if (!need[me]) continue;
      const blsh_sigs &g = *sv[me];
      const bool om_rows = g.layout == BLSH_OBJECT_MAJOR && row_words[me] % 4 == 0 && (uintptr_t(g.data) & 15) == 0;
      const uint32_t *pfx = me == BLSH_COSINE ? (g.prefix ? g.prefix : (om_rows ? g.data : nullptr)) : nullptr;
      B.sig[me] = SigView{g.data, g.n_obj, row_words[me], g.layout == BLSH_WORD_MAJOR ? 1 : 0, pfx,
                          g.prefix ? 4 : int64_t(row_words[me])};
    }
    for (size_t ti = 0; ti < ts.size(); ++ti)
      for (int me = 0; me < 2; ++me) {
        if (!need[me]) continue;
        const int L = n_max[me] / kk[me];
        TableKey key{me, ts[ti], eps, delta, gamma, me ? 1.0 : prior.alpha, me ? 1.0 : prior.beta, kk[me], L, 0};
        const uint32_t *dt = nullptr;
        int r2 = get_table(ctx, key, nullptr, &dt, s);
        if (r2) return r2;
        B.tables[ti * 2 + me] = dt;
        B.n_levels[ti * 2 + me] = L;
      }
    B.alpha = prior.alpha;
    B.beta = prior.beta;
    B.code = res->code;
    B.acc_idx = res->acc_idx;
    B.acc_val = res->acc_val;
    B.acc_cap = res->acc_capacity;
    B.n_acc = res->n_accepted;
    B.m_dbg = res->m_debug;
    B.status = ctx->d_status;
    const size_t set_words = (size_t(kSlices) + 1) * kCntStride;
    B.acc_cnt = b->d_stage_cnt + size_t(b->stage_set) * set_words;
    B.acc_next = b->d_stage_cnt + size_t(b->stage_set ^ 1) * set_words;
    B.acc_total = B.acc_cnt + size_t(kSlices) * kCntStride;
    B.st_idx = b->d_st_idx;
    B.st_val = b->d_st_val;
    B.st_cap = ctx->tuning.acc_stage_cap > 0
                   ? std::min<int64_t>(kBatchStage, std::max<int64_t>(1, ctx->tuning.acc_stage_cap / kSlices))
                   : kBatchStage;
    B.spill[0] = b->d_spill[0];
    B.spill[1] = b->d_spill[1];
    B.spill_waves = grid1 * (kBBlock / kWave);
    B.spill_region = spill_cap / B.spill_waves;
    B.spill_count[0] = b->d_spill_count;
    B.spill_count[1] = b->d_spill_count + B.spill_waves;
    B.spill_used[0] = b->d_spill_used;
    B.spill_used[1] = b->d_spill_used + B.spill_waves + 1;
    B.inreg_levels = inreg;
    BLSH_HIP(hipMemcpyAsync(b->d_block, b->h_block, sizeof(BatchBlock), hipMemcpyHostToDevice, s));
    // the pinned staging may be rewritten by the next call once these copies ran
    BLSH_HIP(hipEventRecord(b->staged, s));
    return BLSH_OK;
  };
  BLSH_HIP(hipMemcpyAsync(b->d_lists, b->h_lists, n_lists * sizeof(BatchList), hipMemcpyHostToDevice, s));

  auto run = [&](const BatchState::Choice &c) -> int {
    const int grid1 = std::max(kXcds, ctx->n_cu * c.bpc);   // phase 1 needs a block on every XCD slice
    int r2 = grow_spill_counts(b, int64_t(grid1) * (kBBlock / kWave));
    if (r2) return r2;
    const int ts = mode ? kExSrpTile : c.ts, tm = mode ? kExMhTile : c.tm;
    if ((r2 = prepare(c.kj, c.kc, ts, tm, c.inreg, grid1))) return r2;
    const int grid2 = std::max(1, ctx->n_cu * 6);
    hipGraphExec_t ex;
    if ((r2 = get_graph(b, BatchState::GraphKey{mode, c.kj, c.kc, ts, tm, grid1, grid2}, &ex))) return r2;
    if (b->stage_dirty) {
      hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(kSlices), 0, s, b->d_stage_cnt);
      BLSH_HIP(hipGetLastError());
    }
    b->stage_dirty = true;
    LaunchScope ls(ctx, s, mode ? "batched_exhaustive_graph" : "batched_graph");
    BLSH_HIP(hipGraphLaunch(ex, s));
    b->stage_dirty = false;
    b->stage_set ^= 1;
    return BLSH_OK;
  };

  // k of a measure no list uses is irrelevant: 32
  BatchState::Choice ch{kj ? kj : 32, kc ? kc : 32, kSrpTileDefault, kMhTileDefault, 2, 0};
  const int fixed_tile[2] = {ctx->tuning.batch_mh_tile, ctx->tuning.batch_srp_tile};
  if (fixed_tile[0] > 0) ch.tm = fixed_tile[0];
  if (fixed_tile[1] > 0) ch.ts = fixed_tile[1];
  ch.bpc = default_blocks(ctx, lists, n_lists, n_cand, mode, resident_blocks(b, need, ch.kj, ch.kc, ch.ts, ch.tm, mode));
  if ((kj == 0 || kc == 0) && mode == 0) {
    // autotune (cached per context and batch shape): each free k in turn with
    // the other fixed (the two measures' tiles share the grid but not their
    // work), then each used measure's tile shape at its k, then in-register
    // levels x blocks per CU at the chosen shapes
    std::vector<int64_t> key{n_lists, n_cand >> 16, int64_t(need[0]), int64_t(need[1]), n_max[0], n_max[1],
                             int64_t(ts.size()), kj, kc, fixed_tile[0], fixed_tile[1]};
    auto it = b->tuned.find(key);
    if (it != b->tuned.end()) {
      ch = it->second;
    } else {
      struct EventPair {
        hipEvent_t e[2] = {nullptr, nullptr};
        ~EventPair() {
          for (hipEvent_t x : e)
            if (x) (void)hipEventDestroy(x);
        }
      } ev;
      BLSH_HIP(hipEventCreate(&ev.e[0]));
      BLSH_HIP(hipEventCreate(&ev.e[1]));
      hipEvent_t e0 = ev.e[0], e1 = ev.e[1];
      auto time_of = [&](const BatchState::Choice &c, float *ms) -> int {
        int r2 = run(c);                                   // warm (tables, graph)
        if (r2) return r2;
        BLSH_HIP(hipEventRecord(e0, s));
        if ((r2 = run(c))) return r2;
        BLSH_HIP(hipEventRecord(e1, s));
        BLSH_HIP(hipEventSynchronize(e1));
        BLSH_HIP(hipEventElapsedTime(ms, e0, e1));
        return BLSH_OK;
      };
      for (int me = 0; me < 2; ++me) {
        if (k_given[me] || !need[me]) continue;
        float best = 1e30f;
        BatchState::Choice pick = ch;
        for (int kk : {16, 32, 64}) {
          BatchState::Choice c = ch;
          (me ? c.kc : c.kj) = kk;
          float ms = 0.f;
          if ((rc = time_of(c, &ms))) return rc;
          if (ms < best) { best = ms; pick = c; }
        }
        ch = pick;
      }
      for (int me = 0; me < 2; ++me) {
        if (!need[me] || fixed_tile[me] > 0) continue;
        static constexpr int kSrpShapes[] = {128, 256, 512}, kMhShapes[] = {64, 128};
        const int *shapes = me ? kSrpShapes : kMhShapes;
        const int n_shapes = me ? 3 : 2;
        float best = 1e30f;
        BatchState::Choice pick = ch;
        for (int i = 0; i < n_shapes; ++i) {
          BatchState::Choice c = ch;
          (me ? c.ts : c.tm) = shapes[i];
          float ms = 0.f;
          if ((rc = time_of(c, &ms))) return rc;
          if (ms < best) { best = ms; pick = c; }
        }
        ch = pick;
      }
      float best = 1e30f;
      BatchState::Choice pick = ch;
      for (int inreg : {1, 2, 4, kMaxLevels})   // kMaxLevels: every level in registers, no queue
        for (int bpc : {2, 4, kBlocksDefault}) {
          BatchState::Choice c = ch;
          c.inreg = inreg;
          c.bpc = bpc;
          float ms = 0.f;
          if ((rc = time_of(c, &ms))) return rc;
          if (ms < best) { best = ms; pick = c; }
        }
      ch = pick;
      b->tuned[key] = ch;
    }
  }
  if (ctx->tuning.batch_inreg > 0) ch.inreg = ctx->tuning.batch_inreg;
  if (ctx->tuning.batch_blocks_per_cu > 0) ch.bpc = ctx->tuning.batch_blocks_per_cu;
  if (fixed_tile[0] > 0) ch.tm = fixed_tile[0];
  if (fixed_tile[1] > 0) ch.ts = fixed_tile[1];
  if ((rc = run(ch))) return rc;
  if (k_used) { k_used[0] = ch.kj; k_used[1] = ch.kc; }
  ctx->tuning.last_batch_k_jaccard = ch.kj;
  ctx->tuning.last_batch_k_cosine = ch.kc;
  ctx->tuning.last_batch_inreg = ch.inreg;
  ctx->tuning.last_batch_blocks_per_cu = ch.bpc;
  ctx->tuning.last_batch_srp_tile = mode ? kExSrpTile : ch.ts;
  ctx->tuning.last_batch_mh_tile = mode ? kExMhTile : ch.tm;
  return BLSH_OK;
}

}  // namespace blsh
