// Signature generation kernels for gfx950 (Section 4 LSH families).
//
//   k_minhash          one wave per set, lanes over hash functions; each lane keeps
//                      the running minimum of (a_h e + b_h) mod (2^31 - 1) over the
//                      set's elements (Section 4.1).
//   k_srp_sparse, k_srp_settle  signs of sparse rows' projections (Section 4.2): most
//                      from approximate plane entries (Philox-4x32-10 + Box-Muller in
//                      fp32, a table of 2-byte codes where terms repeat) with an error
//                      bound, the others from FP64 sums of the entries themselves,
//                      optionally as stored in 2 bytes (Section 4.3).
//   k_srp_dense_mfma   dense rows times a Gaussian plane matrix on the matrix cores
//                      (v_mfma_f32_32x32x2f32); each wave keeps 32 rows of X in
//                      registers, the block stages a 32-plane slice of R in LDS, and
//                      the sign of every accumulator is packed with a wave ballot.
//   k_srp_dense_filter, k_srp_dense_settle  the same bits: bf16 products decide the signs
//                      that their error bound allows, the fp32 instructions the rest.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "srp_entries.h"

namespace blsh {

// ---------------------------------------------------------------------------
// Minhash
// ---------------------------------------------------------------------------
// x mod P of a 32-bit x
__device__ inline uint32_t mod_p(uint32_t x) {
  constexpr uint32_t P = 2147483647u;
  x = (x & P) + (x >> 31);
  return x >= P ? x - P : x;
}

// One hash of one element: with a, b, e < P the value v = a e + b is below
// P 2^31, so s = (v >> 31) + (v & P) < 2 P has v's residue, which is the smaller of
// s and s - P (as unsigned numbers).  On 2 v the shift is the product's high
// word: one 64-bit multiply-add, a shift, two additions and a three-way minimum.
__device__ inline uint32_t minhash_step(uint32_t best, uint32_t a2, uint64_t b2, uint32_t e) {
  constexpr uint32_t P = 2147483647u;
  const uint64_t v2 = uint64_t(a2) * e + b2;
  const uint32_t hi = uint32_t(v2 >> 32), lo = uint32_t(v2) >> 1, s = hi + lo;
  return min(min(best, s), s - P);
}

// A set at a time per wave (a wave takes several of a large collection, with the
// coefficients in registers and the next set's bounds requested: 1M sets of one
// element, 32 hashes, 161 -> 89 us); 64 elements are loaded at a time (reduced mod P
// once) and taken from their lanes one by one.  Bound by integer VALU: 8.2e7 elements x
// 256 hashes in 3.07 ms, 6.8e12 a second (two folds, a 64-bit compare and
// subtraction, an element at a time: 6.79 ms, 3.1e12).
template <int HPL>  // hashes per lane
__global__ __launch_bounds__(256) void k_minhash(const int64_t *offsets, const uint32_t *elems, int64_t n_sets,
                                                 const uint32_t *a, const uint32_t *b, int32_t n_hashes,
                                                 uint32_t *out, int32_t *status) {
  const int lane = lane_id();
  const int64_t waves = int64_t(gridDim.x) * 4;
  int64_t set = int64_t(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  if (set >= n_sets) return;
  int64_t s = ld_uniform(offsets + set), e = ld_uniform(offsets + set + 1);
  uint32_t a2[HPL];
  uint64_t b2[HPL];
#pragma unroll
  for (int i = 0; i < HPL; ++i) {
    const int h = lane + kWave * i;
    a2[i] = h < n_hashes ? 2u * mod_p(a[h]) : 0u;
    b2[i] = h < n_hashes ? 2u * mod_p(b[h]) : 0u;
  }
  for (;;) {
    // (a wave's last: its own again, not one line for all)
    const int64_t next = set + waves < n_sets ? set + waves : set;
    const int64_t s1 = ld_uniform(offsets + next), e1 = ld_uniform(offsets + next + 1);
    uint32_t best[HPL];
#pragma unroll
    for (int i = 0; i < HPL; ++i) best[i] = 0xFFFFFFFFu;
    if (e <= s) raise_status(status, BLSH_EINVAL);
    for (int64_t q = s; q < e; q += kWave) {
      const int n = int(min<int64_t>(kWave, e - q));
      const uint32_t el = lane < n ? mod_p(elems[q + lane]) : 0u;
      int j = 0;
      for (; j + 4 <= n; j += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t x = uint32_t(__builtin_amdgcn_readlane(int(el), j + u));
#pragma unroll
          for (int i = 0; i < HPL; ++i) best[i] = minhash_step(best[i], a2[i], b2[i], x);
        }
      }
      for (; j < n; ++j) {
        const uint32_t x = uint32_t(__builtin_amdgcn_readlane(int(el), j));
#pragma unroll
        for (int i = 0; i < HPL; ++i) best[i] = minhash_step(best[i], a2[i], b2[i], x);
      }
    }
#pragma unroll
    for (int i = 0; i < HPL; ++i) {
      const int h = lane + kWave * i;
      if (h < n_hashes) out[size_t(set) * n_hashes + h] = best[i];
    }
    set += waves;
    if (set >= n_sets) break;
    s = s1;
    e = e1;
  }
}

template <int G>
__device__ inline uint32_t group_or(uint32_t v) {
  if constexpr (G >= 2) v |= dpp<kDppQuadXor1>(v);
  if constexpr (G >= 4) v |= dpp<kDppQuadXor2>(v);
  if constexpr (G >= 8) v |= dpp<kDppHalfMirror>(v);
  return v;
}

// used[term] = 1 for every term < dim that some nonzero holds (used[] zeroed
// before).
__global__ __launch_bounds__(256) void k_srp_mark(const uint32_t *indices, int64_t nnz, int64_t dim,
                                                  uint8_t *used) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < nnz; i += int64_t(gridDim.x) * 256) {
    const uint32_t t = indices[i];
    if (int64_t(t) < dim) used[t] = 1;
  }
}

__global__ __launch_bounds__(256) void k_fill_u8(uint8_t *p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) p[i] = 0;
}

// ---------------------------------------------------------------------------
// Sparse projections: signs from approximate plane entries, open ones settled
// with the entries themselves.
//
// A bit is the sign of sum_t v_t g(term_t, h), summed in FP64 over the row's
// nonzeros in order (srp_settle below).  Its entries cost two FP64 Box-Muller
// pairs per four hashes, far more than the sum, so the sign is first looked for
// with entries g' that cost a fraction: the same Philox words through the
// hardware's fp32 logarithm, square root, sine and cosine, |g' - g| <= kFastErr,
// and, where terms repeat, a table of them as 16-bit multiples of 1 / kUnit.
// With S = sum v g' in fp32, the sum has S's sign wherever |S| exceeds
//   sum |v| (kFastErr + half a unit [table] + 2^-13 [2-byte entries])
//   + the fp32 additions' rounding;
// every other bit (about 1 in 1000 with the table and rows of 100 equal weights, 1 in
// 6,400 without) is marked open and settled: by the approximate entries themselves
// summed in FP64 where that is enough, else (1 in 30,000) by g.  So the bits are those of
// the FP64 sums, every one.
// ---------------------------------------------------------------------------
constexpr int kSumBlock = 32;            // nonzeros summed before they are added to the sum of a stretch
constexpr int kSumStretch = 1024;        // nonzeros of a stretch; a longer row's stretches are added in FP64

// Codes of the entries of the terms < dim that occur (used[term] != 0),
// table[term][n_bits]: a wave takes `per` (at most 64) terms, those that occur one by one (the
// term is wave-uniform, and with it Philox's first multiplications).  Used when each term
// occurs in several rows, so that an entry is drawn once instead of once per
// occurrence.  Bound by VALU (Philox's multiplications first): 1.37e9 entries of
// 668,880 terms in 1.27 ms, against 4.41 ms of FP64 logarithms, sines and cosines.
__global__ __launch_bounds__(256) void k_srp_table(int64_t dim, int32_t n_bits, uint32_t k0, uint32_t k1,
                                                   const uint8_t *used, int16_t *table, int32_t per) {
  const int Q = n_bits / 4, lane = lane_id();
  const int64_t n_groups = (dim + per - 1) / per;   // the terms' flags by one load
  for (int64_t gr = int64_t(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6); gr < n_groups;
       gr += int64_t(gridDim.x) * 4) {
    const int64_t t = gr * per + lane;
    for (uint64_t left = __ballot(lane < per && t < dim && used[t] != 0); left; left &= left - 1) {
      const uint32_t term = uint32_t(gr * per) + uint32_t(__ffsll((unsigned long long)left) - 1);   // wave-uniform
      for (int q = lane; q < Q; q += kWave) {
        float g[4];
        srp_fast4(term, uint32_t(q), k0, k1, g);
        int c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = int(__builtin_rintf(g[e] * kUnit));
        *reinterpret_cast<uint2 *>(table + size_t(term) * n_bits + 4 * q) =
            make_uint2(uint32_t(c[0] & 0xFFFF) | uint32_t(c[1]) << 16, uint32_t(c[2] & 0xFFFF) | uint32_t(c[3]) << 16);
      }
    }
  }
}

// S of rows [row0, row1) in units of 1 / kUnit and the bits it decides.  A wave
// takes one row and one slice of 64 QPL quads of its hashes (QPL consecutive
// quads per lane: 16-byte loads with two).  The whole grid goes slice by slice (4
// of 512 of 2048 hashes), so that every L2 holds one slice of the frequent terms'
// entries, not every slice of fewer terms, and the last-level cache more of the rest.
// Bound by table rows out of the caches: 1.0e7 nonzeros x 4 KB in 2.40 ms, 17 TB/s
// (slices of 256 hashes, 8-byte loads, a slice to an XCD: 3.25 ms; slices of 512
// over XCDs: 2.56 ms; 8 KB of fp32 entries, 1024 hashes per wave, FP64 sums: 6.6 ms).
// TABLE: entries of terms < dim are codes from the table, the rows of U
// nonzeros requested before any is used; others are drawn.
// err: the most an entry is off, in units.
template <bool TABLE, int QPL>
__global__ __launch_bounds__(256) void k_srp_sparse(const int64_t *offsets, const uint32_t *indices,
                                                    const float *values, int64_t n_rows, int64_t row0, int64_t row1,
                                                    int32_t n_bits, int32_t n_slices, uint32_t k0, uint32_t k1,
                                                    int32_t word_major, uint32_t *out, uint32_t *open,
                                                    const int16_t *table, int64_t dim, float err) {
  constexpr int U = TABLE ? 8 : 1;
  __shared__ double s_total[4 * QPL][256];   // sums of a long row's stretches (each thread its own)
  typedef uint32_t codes __attribute__((ext_vector_type(2 * QPL), aligned(8)));
  const int lane = lane_id();
  const int64_t row_blocks = int64_t(gridDim.x) / n_slices;
  const int slice = int(blockIdx.x / row_blocks);
  const int64_t row = row0 + (blockIdx.x % row_blocks) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  if (row >= row1) return;  // wave-uniform
  const int Q = n_bits / 4, W = n_bits / 32, q = (slice * kWave + lane) * QPL;   // (Q is a multiple of QPL)
  const int qc = min(q, Q - QPL);   // (lanes past the last quad repeat it)
  const int64_t s = ld_uniform(offsets + row), e = ld_uniform(offsets + row + 1);
  float acc[4 * QPL], sum[4 * QPL];
#pragma unroll
  for (int c = 0; c < 4 * QPL; ++c) acc[c] = sum[c] = 0.f;
  auto drawn = [&](uint32_t term, float v) {
#pragma unroll
    for (int i = 0; i < QPL; ++i) {
      float g[4];
      srp_fast4(term, uint32_t(qc + i), k0, k1, g);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[4 * i + c] = __builtin_fmaf(v * kUnit, g[c], acc[4 * i + c]);
    }
  };
  auto coded = [&](const codes &x, float v) {
#pragma unroll
    for (int i = 0; i < 2 * QPL; ++i) {
      acc[2 * i] = __builtin_fmaf(v, float(int16_t(x[i])), acc[2 * i]);
      acc[2 * i + 1] = __builtin_fmaf(v, float(int32_t(x[i]) >> 16), acc[2 * i + 1]);
    }
  };
  const uint32_t lane_off = uint32_t(qc) * 8u;
  auto entry = [&](uint32_t term) {
    return *reinterpret_cast<const codes *>(reinterpret_cast<const char *>(table + size_t(term) * uint32_t(n_bits)) + lane_off);
  };
  for (int64_t t0 = s; t0 < e; t0 += kSumBlock) {
    const int64_t t1 = min(e, t0 + kSumBlock);
    int64_t t = t0;
    if constexpr (TABLE) {
      for (; t + U <= t1; t += U) {
        uint32_t term[U];
        float v[U];
        bool in_table = true;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          term[u] = ld_uniform(indices + t + u);
          v[u] = ld_uniform(values + t + u);
          in_table = in_table && int64_t(term[u]) < dim;
        }
        if (!in_table) break;   // the rest of the block one nonzero at a time
        codes ent[U];
#pragma unroll
        for (int u = 0; u < U; ++u) ent[u] = entry(term[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) coded(ent[u], v[u]);
      }
    }
    for (; t < t1; ++t) {
      const uint32_t term = ld_uniform(indices + t);
      const float v = ld_uniform(values + t);
      if (TABLE && int64_t(term) < dim) coded(entry(term), v);
      else drawn(term, v);
    }
#pragma unroll
    for (int c = 0; c < 4 * QPL; ++c) { sum[c] += acc[c]; acc[c] = 0.f; }
    if ((t1 - s) % kSumStretch == 0 && t1 < e) {   // wave-uniform
      const bool first = t1 - s == kSumStretch;
#pragma unroll
      for (int c = 0; c < 4 * QPL; ++c) {
        s_total[c][threadIdx.x] = (first ? 0.0 : s_total[c][threadIdx.x]) + double(sum[c]);
        sum[c] = 0.f;
      }
    }
  }
  // the mass sum |v|
  float mass = 0.f;
  for (int64_t t = s + lane; t < e; t += kWave) mass += fabsf(values[t]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mass += __shfl_xor(mass, o);
  // roundings: one per nonzero of a block's sum (a drawn entry's product with
  // the unit: one more of its own term), one per block of a stretch, each 2^-24 of at most
  // 2^15 units of the mass; and those of the mass itself.  Near the bottom of the
  // float range a rounding is 2^-150 instead, at most 10 of them a nonzero: under
  // 2^-8 of the mass (two of the four roundings to spare) for any row of 2^32
  // nonzeros and a mass of 2^-100 or more.  A smaller mass decides nothing.
  const float n = float(e - s);
  const float T = mass < 0x1p-100f ? INFINITY : mass * (err + (kSumBlock + fminf(n, kSumStretch) / kSumBlock + 4.f) * 0x1p-9f) * (1.f + n * 0x1p-23f) * 1.001f;
  uint32_t nib = 0, unsure = 0;
#pragma unroll
  for (int c = 0; c < 4 * QPL; ++c) {
    // (the cast rounds by 2^-24 of the sum itself, which T has room for)
    const float S = e - s > kSumStretch ? float(s_total[c][threadIdx.x] + double(sum[c])) : sum[c];
    nib |= uint32_t(S >= 0.f) << c;
    unsure |= uint32_t(!(fabsf(S) > T && fabsf(S) < INFINITY)) << c;   // (an overflow decides nothing)
  }
  constexpr int G = 8 / QPL;   // lanes per word
  const int sh = 4 * QPL * (lane & (G - 1)), w = q >> 3;
  const uint32_t word = group_or<G>(q < Q ? nib << sh : 0u), mask = group_or<G>(q < Q ? unsure << sh : 0u);
  if ((lane & (G - 1)) == 0 && w < W) {
    if (word_major) out[size_t(w) * n_rows + row] = word;
    else out[size_t(row) * W + w] = word;
    open[size_t(row - row0) * W + w] = mask;
  }
}

// The open bits of rows [rows0, rows1) (open = null: every bit), worked out:
// the FP64 sum of v g over the row's nonzeros in order, g rounded to fp32 (Q16:
// the value of its 2-byte code).  Rows with more than half their bits open (weights
// outside the fp32 sums' range, or no workspace for masks) go four hashes to a
// thread, the entries of a quad drawn together.  Of the others a block lists the
// open bits of its `per` rows (at most kSettleRows) in LDS, 256 words at a time while they fit.  8 lanes take
// a bit, each every eighth nonzero, and sum the approximate entries themselves in
// FP64: that leaves only the entries' error, |v| kFastErr (Q16: a cell where an entry
// that much off might have another code, 3% of them), so that 1 bit in 30 of those
// the table left open remains.  What remains is
// drawn in FP64, a wave to a bit and 64 nonzeros at a time, the products (exact
// in FP64) added in order.  Rows of 100,000 equal weights leave 3% of their bits open:
// 64 of them take 45 ms in all (63 with FP64 entries for every bit; 6800 with every
// open bit drawn in FP64 by 8 lanes, the stretches added in fp32 and 14 to 34% of the bits open).
constexpr int kSettleList = 8192, kSettleRows = 32;
static_assert(kSettleList >= 256 * 32, "one round of words fits the list");
constexpr uint32_t kSettled = 0xFFFFFFFFu;

template <bool Q16>
__global__ __launch_bounds__(256) void k_srp_settle(const int64_t *offsets, const uint32_t *indices,
                                                    const float *values, int64_t n_rows, int64_t rows0, int64_t rows1,
                                                    int32_t per, int32_t n_bits, uint32_t k0, uint32_t k1,
                                                    int32_t word_major, uint32_t *out, const uint32_t *open) {
  __shared__ uint32_t s_bit[kSettleList];   // (row - row0) n_bits + hash (at most 32 x 2048), or kSettled
  __shared__ uint32_t s_wave[4];
  __shared__ uint32_t s_row[kSettleRows];   // open bits of a row, then whether it goes whole
  __shared__ int32_t s_whole[kSettleRows];
  const int W = n_bits / 32, Q = n_bits / 4, lane = lane_id(), wv = threadIdx.x >> 6, r = lane & 7;
  const int64_t row0 = rows0 + int64_t(blockIdx.x) * per;
  const int n_own = int(min<int64_t>(per, rows1 - row0)), words = n_own * W;
  if (threadIdx.x < kSettleRows) s_row[threadIdx.x] = 0;
  __syncthreads();
  if (open)
    for (int w = threadIdx.x; w < words; w += 256) {
      const uint32_t mask = open[size_t(row0 - rows0) * W + w];
      if (mask) atomicAdd(&s_row[w / W], uint32_t(__popc(mask)));
    }
  __syncthreads();
  const bool all = lane < n_own && (!open || 2 * s_row[lane % kSettleRows] > uint32_t(n_bits));
  const uint64_t whole = __ballot(all);   // (the same in every wave)
  __syncthreads();
  if (wv == 0 && lane < n_own) {
    s_row[lane] = all;
    if (all) s_whole[lanes_below(whole)] = lane;
  }
  __syncthreads();
  // (Q is a multiple of 8, so the lanes of a word are in the loop together)
  for (int it = threadIdx.x; it < __popcll(whole) * Q; it += 256) {
    const int64_t row = row0 + s_whole[it / Q];
    const int q = it % Q;
    const int64_t s = offsets[row], e = offsets[row + 1];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t t = s; t < e; ++t) {
      const double v = values[t];
      double g[4];
      srp_gauss4(indices[t], uint32_t(q), k0, k1, g);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = __builtin_fma(v, Q16 ? q16_value(q16_code(g[c])) : g[c], acc[c]);
    }
    uint32_t nib = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) nib |= uint32_t(acc[c] >= 0.0) << c;
    const uint32_t word = group_or<8>(nib << (4 * r));
    if (r == 0) out[word_major ? size_t(q >> 3) * n_rows + row : size_t(row) * W + (q >> 3)] = word;
  }
  if (!open) return;
  uint32_t count = 0;   // entries of the list (block-uniform)
  auto put = [&](int64_t row, uint32_t h, bool one) {
    uint32_t *word = word_major ? out + size_t(h >> 5) * n_rows + row : out + size_t(row) * W + (h >> 5);
    const uint32_t bit = 1u << (h & 31);
    if (one) atomicOr(word, bit);
    else atomicAnd(word, ~bit);
  };
  auto settle = [&]() {
    __syncthreads();
    for (uint32_t i0 = 0; i0 < count; i0 += 32) {   // block-uniform
      const uint32_t i = i0 + (threadIdx.x >> 3);
      const bool act = i < count;
      const uint32_t b = act ? s_bit[i] : 0u;
      const int64_t row = row0 + b / uint32_t(n_bits);
      const uint32_t h = b % uint32_t(n_bits);
      const int64_t s = offsets[row], e = act ? offsets[row + 1] : s;
      double sum = 0.0, mass = 0.0, slack = 0.0;
      for (int64_t t = s + r; t < e; t += 8) {
        const double v = values[t];
        double g = srp_fast1(indices[t], h, k0, k1), off = kFastErr;
        if constexpr (Q16) {   // the code's value, sure but near a cell's edge: there one cell off at most
          const double x = (g + 8.0) * 4096.0, c = floor(x);
          off = x - c < kFastErr * 4096.0 || x - c > 1.0 - kFastErr * 4096.0 ? 0x1p-12 : 0.0;
          g = (c + 0.5) * (1.0 / 4096.0) - 8.0;
        }
        sum = __builtin_fma(v, g, sum);
        slack += fabs(v) * off;
        mass += fabs(v);
      }
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {
        sum += __shfl_xor(sum, o);
        mass += __shfl_xor(mass, o);
        slack += __shfl_xor(slack, o);
      }
      // (the last term: the roundings of either FP64 sum, each 2^-53 of at most 7 times the mass)
      const double T = (slack + mass * double(e - s) * 0x1p-49) * 1.0001;
      if (act && r == 0 && fabs(sum) > T && fabs(sum) < INFINITY) {
        put(row, h, sum > 0.0);
        s_bit[i] = kSettled;
      }
    }
    __syncthreads();
    for (uint32_t i0 = wv * kWave; i0 < count; i0 += 4 * kWave) {   // wave-uniform
      const uint32_t mine = i0 + lane < count ? s_bit[i0 + lane] : kSettled;
      for (uint64_t left = __ballot(mine != kSettled); left; left &= left - 1) {
        const uint32_t b = uint32_t(__builtin_amdgcn_readlane(int(mine), __ffsll((unsigned long long)left) - 1));
        const int64_t row = row0 + b / uint32_t(n_bits);
        const uint32_t h = b % uint32_t(n_bits);
        const int64_t s = offsets[row], e = offsets[row + 1];
        double acc = 0.0;
        for (int64_t t = s; t < e; t += kWave) {
          double p = 0.0;
          if (t + lane < e) {
            double g = srp_gauss1(indices[t + lane], h, k0, k1);
            if constexpr (Q16) g = q16_value(q16_code(g));
            p = double(values[t + lane]) * g;
          }
          const int n = int(min<int64_t>(kWave, e - t));
          const uint64_t u = __builtin_bit_cast(uint64_t, p);
          for (int j = 0; j < n; ++j)
            acc += __builtin_bit_cast(double, uint64_t(uint32_t(__builtin_amdgcn_readlane(int(u), j))) |
                                                  uint64_t(uint32_t(__builtin_amdgcn_readlane(int(u >> 32), j))) << 32);
        }
        if (lane == 0) put(row, h, acc >= 0.0);
      }
    }
    __syncthreads();
    count = 0;
  };
  for (int w0 = 0; w0 < words; w0 += 256) {
    const int w = w0 + threadIdx.x;
    uint32_t mask = w >= words || s_row[w / W] ? 0u : open[size_t(row0 - rows0) * W + w];
    const uint32_t mine = uint32_t(__popc(mask));
    uint32_t before = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t u = __shfl_up(before, o);
      if (lane >= o) before += u;
    }
    __syncthreads();
    if (lane == kWave - 1) s_wave[wv] = before;
    __syncthreads();
    const uint32_t total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    before -= mine;
    for (int x = 0; x < wv; ++x) before += s_wave[x];
    if (count + total > uint32_t(kSettleList)) settle();
    uint32_t at = count + before;
    for (; mask; mask &= mask - 1) s_bit[at++] = uint32_t(w) * 32u + uint32_t(__ffs(int(mask)) - 1);
    count += total;
  }
  if (count) settle();
}

// ---------------------------------------------------------------------------
// Dense SRP on the matrix cores
// ---------------------------------------------------------------------------
typedef float floatx16 __attribute__((ext_vector_type(16)));

// The 32 x 32 product's ballots by row: row 8 (v / 4) + v % 4 of the low half
// of ballot v and the row 4 further of its high half go to their rows' lanes.
template <int... V>
__device__ inline void write_rows(uint32_t &word, const uint64_t (&b)[16], std::integer_sequence<int, V...>) {
  ((word = write_lane<8 * (V >> 2) + (V & 3)>(uint32_t(b[V]), word)), ...);
  ((word = write_lane<8 * (V >> 2) + (V & 3) + 4>(uint32_t(b[V] >> 32), word)), ...);
}

// The product of a block's rows (row0: this wave's first of 32) with the planes of
// tiles [t0, t1), 32 to a tile; a wave that is not `mine` only helps to stage them.
// AHEAD: the next slice of planes is read while one is multiplied (else after it:
// fewer registers, for a kernel that holds other things).
// X: [n_rows][D] fp32, R: [D][n_bits] fp32.  Block = 4 waves = 128 rows; the
// D dimension is split between the two half-waves: lanes 0..31 cover
// d in [0, D/2) and lanes 32..63 cover [D/2, D), so that each lane's A
// operands are one contiguous half-row of X.  The 32-plane slices of R are
// double-buffered in LDS: the next slice is read into registers before the
// current one's MFMA loop and written to the other buffer after it, so one
// barrier per slice remains and the reads overlap the matrix work.
template <int D, bool AHEAD>
__device__ inline void dense_chain(const float *X, int64_t n_rows, const float *R, int32_t n_bits, int32_t word_major,
                                   uint32_t *out, int64_t row0, int t0, int t1, bool mine, float (&sR)[2][D * 32]) {
  constexpr int HD = D / 2;
  constexpr int PER = D * 32 / 256;   // slice entries per thread; sR[b][d*32 + j] = R[d][col0 + j]
  const int lane = lane_id();
  const int h = lane >> 5, i = lane & 31;
  const int64_t my_row = row0 + i;
  float xa[HD];
  if (my_row < n_rows) {
    const float4 *src = reinterpret_cast<const float4 *>(X + size_t(my_row) * D + h * HD);
#pragma unroll
    for (int q = 0; q < HD / 4; ++q) {
      const float4 v = src[q];
      xa[4 * q] = v.x; xa[4 * q + 1] = v.y; xa[4 * q + 2] = v.z; xa[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int q = 0; q < HD; ++q) xa[q] = 0.f;
  }
  const int W = n_bits / 32;
  // row held in the result word by this lane (lanes 0..31): t = lane
  const int t = lane & 31;
  const int my_v = 4 * (t >> 3) + (t & 3), my_h = (t >> 2) & 1;
  constexpr int CH = AHEAD ? PER : 4;   // entries of a thread on their way to LDS
  float st[CH];
  // entry idx = threadIdx.x + 256 u of the slice: d = idx / 32, j = idx % 32.  Without AHEAD
  // d's part of u uniform, the thread's in 32 bits (fewer registers beside the filter);
  // with it an address a load (60,000 x 256 x 128: 42.5 us, 44.6 the other way).
  const uint32_t own = (threadIdx.x >> 5) * uint32_t(n_bits) + (threadIdx.x & 31);
  auto fetch = [&](int tile, int u0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int idx = int(threadIdx.x) + 256 * (u0 + u);
      if constexpr (AHEAD) st[u] = R[size_t(idx >> 5) * n_bits + tile * 32 + (idx & 31)];
      else st[u] = (R + size_t(8 * (u0 + u)) * uint32_t(n_bits) + tile * 32)[own];
    }
  };
  auto stash = [&](int b, int u0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) sR[b][int(threadIdx.x) + 256 * (u0 + u)] = st[u];
  };
  auto slice = [&](int tile, int b) {
#pragma unroll 1
    for (int u0 = 0; u0 < PER; u0 += CH) {
      fetch(tile, u0);
      stash(b, u0);
    }
  };
  if constexpr (AHEAD) {
    fetch(t0, 0);
    stash(0, 0);
  } else {
    slice(t0, 0);
  }
  __syncthreads();
  for (int tile = t0; tile < t1; ++tile) {
    const int b = (tile - t0) & 1;
    if (AHEAD && tile + 1 < t1) fetch(tile + 1, 0);
    if (mine) {
      floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  #pragma unroll
      for (int s = 0; s < HD; ++s) {
        const float bv = sR[b][(h * HD + s) * 32 + i];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[s], bv, acc, 0, 0, 0);
      }
      uint32_t word = 0;
  #pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint64_t mk = __ballot(acc[v] >= 0.f);
        if (my_v == v) word = my_h ? uint32_t(mk >> 32) : uint32_t(mk);
      }
      const int64_t r = row0 + t;
      if (lane < 32 && r < n_rows) {
        if (word_major) out[size_t(tile) * n_rows + r] = word;
        else out[size_t(r) * W + tile] = word;
      }
    }
    // buffer b ^ 1 was last read in the previous slice, before the barrier
    // that ended it; the barrier below orders these writes before its reads
    if (tile + 1 < t1) {
      if constexpr (AHEAD) stash(b ^ 1, 0);
      else slice(tile + 1, b ^ 1);
    }
    __syncthreads();
  }
}

template <int D>
__global__ __launch_bounds__(256, 2) void k_srp_dense_mfma(const float *X, int64_t n_rows, const float *R,
                                                        int32_t n_bits, int32_t word_major, uint32_t *out) {
  __shared__ float sR[2][D * 32];
  dense_chain<D, true>(X, n_rows, R, n_bits, word_major, out, int64_t(blockIdx.x) * 128 + (threadIdx.x >> 6) * 32, 0, n_bits / 32,
                 true, sR);
}

// ---------------------------------------------------------------------------
// Dense SRP, filtered: the same signs as k_srp_dense_mfma from bf16 matrix
// products, with every sign they leave open taken from the fp32 chain itself.
//
// Rows and planes are scaled by powers of two (no sign changes) and split into
// two bf16 terms, x = xh + xl + ex with |ex| <= 2^-18 |x|.  xh rh and xh rl + xl
// rh are accumulated apart in fp32.  Against the exact product the sum S of
// the two is off by at most
//   3 (1 + 2^-7) 2^-18 ||x|| ||r||   the terms left out (Cauchy-Schwarz)
//   + (D + 16) 2^-23 ||x|| ||r||     the additions of xh rh, each within 2^-23 of
//                                    a partial sum (twice rounding to nearest;
//                                    those of the smaller products are 2^-8 of that;
//                                    an instruction's 16 together measured within
//                                    2.9 2^-23 of its terms' sizes, test_gpu_bounds.py),
// and k_srp_dense_mfma's fp32 chain by at most D 2^-23 ||x|| ||r||.  Where |S|
// exceeds the sum of these (kFilter), S, the exact product and the chain have
// one sign.  The other signs (about 1 in 1000 for Gaussian planes at D = 256),
// and those of planes whose scale lets the chain under- or overflow, are listed
// per wave and worked out by k_srp_dense_settle with the chain's own instructions in
// the chain's own order, so the bits are k_srp_dense_mfma's, every one.  A wave with
// more open signs than its list holds (a row of such a scale is enough) stops
// there, and its block takes its rows through the chain as k_srp_dense_mfma does
// (100,000 x 256 x 1024, one row in 32 such: 709 us, 599 by k_srp_dense_mfma alone;
// 1463 when the settling kernel took them).
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int D>
constexpr float kFilter = 3.1f / 262144.f + float(2 * D + 32) / 8388608.f;
// exponents of a row's and a plane's norm for which the chain neither overflows
// (products and partial sums below 2.25 2^120) nor loses more than kFilter has to
// spare where it underflows (2 D 2^-126 against 2^-22 of 2^-94)
constexpr int kRowLo = -70, kRowHi = 70, kPlaneLo = -24, kPlaneHi = 50;
constexpr uint32_t kOpenCol = (1u << 26) - 1;  // an open sign: row in the wave << 27 | sign of S << 26 | plane

// Scale of a vector with largest element mx: the power of two 2^-e that takes
// its norm into [0.75, 1.5), found from the sum of squares of the elements
// scaled by `first` (a power of two that takes mx into [1, 2)).  ok: e is in
// [LO, HI] (false for zero, infinite or NaN).
__device__ inline float first_scale(float mx) { return mx > 0.f && mx < INFINITY ? ldexpf(1.f, -ilogbf(mx)) : 1.f; }
template <int LO, int HI>
__device__ inline float norm_scale(float mx, float first, float sumsq, float &norm, bool &ok) {
  ok = mx > 0.f && mx < INFINITY && sumsq < INFINITY;
  if (!ok) { norm = 0.f; return 1.f; }
  const float n = sqrtf(sumsq);                       // of the elements times `first`: in [1, 2 sqrt(D))
  const int e = ilogbf(n * (4.f / 3.f));
  norm = ldexpf(n, -e) * (1.f + 1.f / 1024.f);        // (covers the rounding of the sum of squares)
  const int total = e + ilogbf(mx);
  ok = total >= LO && total <= HI;
  return ok ? ldexpf(1.f, -total) : 1.f;
}

// Planes for the filter, one block per 32 of them: the scaled bf16 terms in
// the order the matrix instruction takes them, Bf[tile][k / 16][term][lane] (8
// values: plane lane % 32, k % 16 = 8 (lane / 32) ..), their scaled norms (NaN
// where every sign has to be settled, -1 for a plane of zeros, whose signs all are
// known), and the planes by rows for the chain.
template <int D>
__global__ __launch_bounds__(256) void k_srp_planes(const float *R, int32_t n_bits, uint4 *Bf, float *norms, float *Rt) {
  __shared__ float s[D][33];
  __shared__ float s_scale[32], s_part[8][32];
  const int col0 = int(blockIdx.x) * 32, j = threadIdx.x % 32, part = threadIdx.x / 32;
  for (int i = threadIdx.x; i < D * 32; i += 256) s[i / 32][i % 32] = R[size_t(i / 32) * n_bits + col0 + i % 32];
  __syncthreads();
  // plane j's largest element, then its sum of squares, by 8 threads
  float mx = 0.f, sum = 0.f;
  for (int d = part; d < D; d += 8) {
    const float v = fabsf(s[d][j]);
    mx = v == v ? fmaxf(mx, v) : INFINITY;   // (NaN: refused as infinite)
  }
  s_part[part][j] = mx;
  __syncthreads();
  for (int q = 0; q < 8; ++q) mx = fmaxf(mx, s_part[q][j]);
  const float f = first_scale(mx);
  for (int d = part; d < D; d += 8) { const float v = s[d][j] * f; sum += v * v; }
  __syncthreads();
  s_part[part][j] = sum;
  __syncthreads();
  if (part == 0) {
    for (int q = 1; q < 8; ++q) sum += s_part[q][j];
    float norm;
    bool ok;
    s_scale[j] = norm_scale<kPlaneLo, kPlaneHi>(mx, f, sum, norm, ok);
    norms[col0 + j] = ok ? norm : mx == 0.f ? -1.f : __builtin_nanf("");
  }
  __syncthreads();
  for (int i = threadIdx.x; i < D * 32; i += 256) Rt[size_t(col0) * D + i] = s[i % D][i / D];
  for (int i = threadIdx.x; i < D / 16 * 64; i += 256) {
    const int kb = i / 64, lane = i % 64, j = lane & 31, k0 = 16 * kb + 8 * (lane >> 5);
    bf16x8 hi, lo;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float v = s[k0 + q][j] * s_scale[j];
      hi[q] = __bf16(v);
      lo[q] = __bf16(v - float(hi[q]));
    }
    uint4 *to = Bf + (size_t(blockIdx.x) * (D / 16) + kb) * 128 + lane;
    to[0] = __builtin_bit_cast(uint4, hi);
    to[64] = __builtin_bit_cast(uint4, lo);
  }
}

struct FilterArgs {   // (k_srp_dense_filter's only argument: at the start of its argument segment)
  const float *X;
  int64_t n_rows;
  const float *R;
  const uint4 *Bf;
  const float *norms;
  uint32_t *out, *open, *n_open;
  int32_t n_bits, n_splits, word_major, cap;
};

// Block = 4 waves = 128 rows, each wave's 32 rows held as bf16 terms in
// registers; tile by tile of 32 planes (the split's share of them), the terms of the
// next tile are copied to LDS while a tile's products run.  Bound by the
// matrix cores: 1M rows, 1024 planes, D = 256 are 1.61e12 operations in three products,
// 1.43 ms or 1.13e15 a second (what a large bf16 product reaches on this card);
// with the settling and the planes' preparation 1.76 ms, against 4.09 ms of
// k_srp_dense_mfma (131e12 a second of the 157e12 that fp32 instructions allow).
template <int D>
__global__ __launch_bounds__(256, 2) void k_srp_dense_filter(FilterArgs fa) {
  const float *const X = fa.X, *const norms = fa.norms;
  const int64_t n_rows = fa.n_rows;
  const uint4 *const Bf = fa.Bf;
  const int32_t n_bits = fa.n_bits, n_splits = fa.n_splits, word_major = fa.word_major, cap = fa.cap;
  uint32_t *const out = fa.out, *const open = fa.open, *const n_open = fa.n_open;
  constexpr int KB = D / 16;
  __shared__ union {
    uint4 b[2][KB * 128];
    float r[2][D * 32];   // (dense_chain)
  } s_u;
  auto &s_b = s_u.b;
  __shared__ uint32_t s_over[2][4];
  const int lane = lane_id(), wv = threadIdx.x >> 6, h = lane >> 5, i = lane & 31;
  const int64_t rb = blockIdx.x / unsigned(n_splits);
  const int sp = int(blockIdx.x % unsigned(n_splits)), W = n_bits / 32;
  const int t0 = int(int64_t(sp) * W / n_splits), t1 = int(int64_t(sp + 1) * W / n_splits);
  const int64_t row0 = rb * 128 + wv * 32, region = (rb * 4 + wv) * n_splits + sp;
  auto stage = [&](int tile, int b) {   // wave wv copies its quarter of the tile's fragments
#pragma unroll
    for (int u = 0; u < KB / 2; ++u) {
      const int at = (u * 4 + wv) * 64;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(Bf + size_t(tile) * KB * 128 + at + lane),
                                       (__attribute__((address_space(3))) void *)(s_b[b] + at), 16, 0, 0);
    }
  };
  stage(t0, 0);
  bf16x8 xh[KB], xl[KB];
  float xmax;
  uint32_t zeros;   // rows of zeros: a sign of 1 with every finite plane
  bool over;        // more open signs than the list holds (wave-uniform)
  {
    float x[KB][8];
    const bool in = row0 + i < n_rows;
    const float4 *src = reinterpret_cast<const float4 *>(X + size_t(in ? row0 + i : 0) * D + 8 * h);
    float mx = 0.f, sum = 0.f;
    bool num = true;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const float4 u = src[4 * kb], v = src[4 * kb + 1];
      const float t[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        x[kb][q] = t[q];
        mx = fmaxf(mx, fabsf(t[q]));
        num = num && t[q] == t[q];
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float f = first_scale(mx);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int q = 0; q < 8; ++q) { const float v = x[kb][q] * f; sum += v * v; }
    sum += __shfl_xor(sum, 32);
    float norm;
    bool ok;
    float scale = norm_scale<kRowLo, kRowHi>(mx, f, sum, norm, ok);
    ok = ok && num && in;
    const bool other = __shfl_xor(int(ok), 32) != 0;
    ok = ok && other;
    // a row whose scale lets the chain under- or overflow: every sign open, n_bits
    // of them, which no list holds
    zeros = uint32_t(__ballot(in && num && mx == 0.f) & __ballot(in && num && mx == 0.f) >> 32);
    over = __ballot(in && !ok && !((zeros >> i) & 1u)) != 0;
    xmax = ok ? norm : 0.f;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) xmax = fmaxf(xmax, __shfl_xor(xmax, o));
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float v = x[kb][q] * scale;
        xh[kb][q] = __bf16(v);
        xl[kb][q] = __bf16(v - float(xh[kb][q]));
      }
  }
  const float bound = kFilter<D> * xmax;
  float norm = norms[t0 * 32 + i];   // of this lane's plane (the next tile's is requested with its fragments)
  uint32_t n = 0;   // open signs of the wave (wave-uniform)
  uint32_t *list = open + size_t(region) * cap;
  if (lane == 0) s_over[0][wv] = s_over[1][wv] = over;
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the copies to LDS have arrived
  __syncthreads();
  for (int tile = t0; tile < t1; ++tile) {
    const int b = (tile - t0) & 1;
    // all four over (as of the tile before, so that all waves find the same)
    if (over && (s_over[b ^ 1][0] & s_over[b ^ 1][1] & s_over[b ^ 1][2] & s_over[b ^ 1][3])) break;
    if (tile + 1 < t1) stage(tile + 1, b ^ 1);
    const float T = bound * norm;
    norm = norms[min(tile + 1, t1 - 1) * 32 + i];
    floatx16 ah = {}, al = {};
    // (the fragments of a step are read while the step before it multiplies;
    // left to itself the compiler reads them right before their use)
    uint4 bh = s_b[b][lane], bl = s_b[b][64 + lane];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      uint4 nh = bh, nl = bl;
      if (kb + 1 < KB) {
        nh = s_b[b][(kb + 1) * 128 + lane];
        nl = s_b[b][(kb + 1) * 128 + 64 + lane];
      }
      __builtin_amdgcn_sched_barrier(0);
      al = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl[kb], __builtin_bit_cast(bf16x8, bh), al, 0, 0, 0);
      ah = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[kb], __builtin_bit_cast(bf16x8, bh), ah, 0, 0, 0);
      al = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[kb], __builtin_bit_cast(bf16x8, bl), al, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      bh = nh;
      bl = nl;
    }
    // value v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4 of the wave, plane l % 32
    uint32_t word = 0;
    bool sure = true;
    {
      uint64_t neg[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        ah[v] += al[v];
        neg[v] = __ballot(ah[v] < 0.f);
        sure = sure && fabsf(ah[v]) > T;
      }
      write_rows(word, neg, std::make_integer_sequence<int, 16>{});
      word = ~word;
    }
    const int64_t r = row0 + i;
    if (lane < 32 && r < n_rows) {
      if (word_major) out[size_t(tile) * n_rows + r] = word;
      else out[size_t(r) * W + tile] = word;
    }
    if (zeros != 0 && T == T) {   // (rows of zeros, finite planes: known)
      uint32_t z = zeros;
      asm volatile("" : "+s"(z));   // (worked out here: 16 masks kept for it would not fit the scalar registers)
      const uint32_t zh = z >> (4 * h);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if ((zh >> (8 * (v >> 2) + (v & 3))) & 1u) ah[v] = INFINITY;
    }
    if (__ballot(!sure)) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v >> 2) + 4 * h + (v & 3);
        const bool mine = !(fabsf(ah[v]) > T) && row0 + row < n_rows;
        const uint64_t mask = __ballot(mine);
        if (mask == 0) continue;
        const uint32_t at = n + lanes_below(mask);
        if (mine && at < uint32_t(cap))
          list[at] = uint32_t(row) << 27 | uint32_t(!(ah[v] < 0.f)) << 26 | uint32_t(tile * 32 + i);
        n += uint32_t(__popcll(mask));
      }
    }
    over = over || n > uint32_t(cap);
    if (over && lane == 0) s_over[b][wv] = 1;
    // buffer b ^ 1 was last read before the barrier that ended the previous tile
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }
  if (lane == 0) {
    n_open[region] = over ? 0 : n;
    s_over[0][wv] = over;
  }
  __syncthreads();
  if (s_over[0][0] | s_over[0][1] | s_over[0][2] | s_over[0][3]) {   // block-uniform
    // (a rare path: its arguments are read from the argument segment here, not held
    // in scalar registers through the loop)
    const auto *kp = (const char __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kp));
    const auto *ap = (const FilterArgs __attribute__((address_space(4))) *)kp;
    const int32_t nb = ap->n_bits;
    const int64_t rows0 = int64_t(blockIdx.x / unsigned(ap->n_splits)) * 128 + wv * 32;
    dense_chain<D, false>(ap->X, ap->n_rows, ap->R, nb, ap->word_major, ap->out, rows0, int(int64_t(sp) * (nb / 32) / ap->n_splits),
                          int(int64_t(sp + 1) * (nb / 32) / ap->n_splits), over, s_u.r);
  }
}

// Four steps of k_srp_dense_mfma's chain.
__device__ inline floatx16 chain4(floatx16 acc, const float4 &a, const float4 &b) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
  return acc;
}

// The open signs of four waves' lists, 32 at a time: open sign t as row t and
// plane t of the chain's own matrix product, whose value (t, t) is its sign's.
// The 64 vectors of a batch go through LDS in chunks of 2 C elements (C of
// either half, the order of the chain), read 64 bytes at a time; four blocks to
// a CU cover the reads.  (Rows and planes read by the lanes that multiply them:
// 64 lines per load, 0.57 ms for 1M rows, 1024 planes, D = 256.  Copies straight to
// LDS gave wrong values now and then when read after the wave's own wait
// alone, without a barrier.)
template <int D>
__global__ __launch_bounds__(256) void k_srp_dense_settle(const float *X, int64_t n_rows, const float *Rt,
                                                             int32_t n_bits, int32_t n_splits, int32_t word_major,
                                                             uint32_t *out, const uint32_t *open,
                                                             const uint32_t *n_open, int32_t cap, int64_t n_regions) {
  constexpr int HD = D / 2, C = 16, NC = HD / C;
  constexpr int NL = 8;   // loads per chunk: 8 vectors each, 8 lanes of 16 bytes to a vector
  // [vector][piece]: vectors 0..31 rows, 32..63 planes; piece p (p < 4: of the
  // first half) of vector v sits at p ^ (v % 8), so that 8 vectors' reads of one
  // piece spread over the banks
  __shared__ float4 s_v[4][64 * 8];
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), h = lane >> 5, i = lane & 31;
  const int W = n_bits / 32, my_v = 4 * (i >> 3) + (i & 3), my_h = (i >> 2) & 1;
  const int64_t reg0 = int64_t(blockIdx.x) * 4;
  uint32_t cnt[4], total = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    cnt[q] = reg0 + q < n_regions ? n_open[reg0 + q] : 0u;
    total += cnt[q];
  }
  auto word_at = [&](int64_t row, int w) -> uint32_t * {
    return word_major ? out + size_t(w) * n_rows + row : out + size_t(row) * W + w;
  };
  for (uint32_t e0 = 32u * wv; e0 < total; e0 += 128) {   // wave-uniform
    const bool act = e0 + i < total;
    uint32_t k = act ? e0 + i : e0;   // entry k of the lists one after another
    int q = 0;
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      if (q == x && k >= cnt[x]) { k -= cnt[x]; ++q; }
    }
    const uint32_t e = open[size_t(reg0 + q) * cap + k];
    const int64_t row = (reg0 + q) / n_splits * 32 + (e >> 27);
    const uint32_t col = e & kOpenCol;
    // load u: vectors 8 u + lane / 8
    const int piece = (lane & 7) ^ (lane >> 3), off = (piece >> 2) * HD + (piece & 3) * 4;
    const float *src[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int v = (8 * u + (lane >> 3)) & 31;
      if (u < NL / 2) src[u] = X + size_t(__shfl(row, v)) * D + off;
      else src[u] = Rt + size_t(uint32_t(__shfl(int(col), v))) * D + off;
    }
    floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int c = 0; c < NC; ++c) {
      float4 st[NL];
#pragma unroll
      for (int u = 0; u < NL; ++u) st[u] = *reinterpret_cast<const float4 *>(src[u] + c * C);
#pragma unroll
      for (int u = 0; u < NL; ++u) s_v[wv][64 * u + lane] = st[u];
      wave_lds_sync();
#pragma unroll
      for (int s = 0; s < C / 4; ++s) {
        const int at = (4 * h + s) ^ (i & 7);
        acc = chain4(acc, s_v[wv][8 * i + at], s_v[wv][8 * (32 + i) + at]);
      }
      wave_lds_sync();
    }
    float d = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) d = my_v == v ? acc[v] : d;
    // (a word's signs may sit in several lanes: only those that change it do, atomically)
    if (act && h == my_h && uint32_t(d >= 0.f) != ((e >> 26) & 1u)) atomicXor(word_at(row, int(col >> 5)), 1u << (col & 31));
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int launch_minhash(blsh_ctx *ctx, const int64_t *offsets, const uint32_t *elems, int64_t n_sets, const uint32_t *a,
                   const uint32_t *b, int n_hashes, uint32_t *out, hipStream_t s) {
  const int hpl = (n_hashes + kWave - 1) / kWave;
  const int64_t nb = std::min<int64_t>((n_sets + 3) / 4, int64_t(ctx->n_cu) * 32);
  LaunchScope ls(ctx, s, "minhash_sigs");
#define BLSH_MH(N) if (hpl <= N) { hipLaunchKernelGGL(k_minhash<N>, dim3(nb), dim3(256), 0, s, offsets, elems, n_sets, a, b, n_hashes, out, ctx->d_status); return hipGetLastError() == hipSuccess ? BLSH_OK : BLSH_EDEVICE; }
  // (hashes per lane: the next of these, so that little is done for padding)
  BLSH_MH(1) BLSH_MH(2) BLSH_MH(3) BLSH_MH(4) BLSH_MH(5) BLSH_MH(6) BLSH_MH(7) BLSH_MH(8) BLSH_MH(10) BLSH_MH(12) BLSH_MH(16)
#undef BLSH_MH
  return fail(BLSH_EINVAL, "minhash: n_hashes %d > 1024", n_hashes);
}

constexpr size_t kSrpTableMaxBytes = size_t(16) << 30;
constexpr int64_t kSrpRows = int64_t(1) << 22;   // rows per launch (8 slices of 64 lanes each: 2^31 work-items)
// Fewest rows per launch: 20,000 rows of 100 terms, entries drawn, 256 at a time 5.3
// ms, 32 at a time 34 ms, and 11.5 with every bit worked out.
constexpr int64_t kSrpFewest = 256;

int launch_srp_sparse(blsh_ctx *ctx, const int64_t *offsets, const uint32_t *indices, const float *values,
                      int64_t n_rows, int64_t dim, int n_bits, uint64_t seed, bool word_major, bool q16,
                      uint32_t *out, hipStream_t s) {
  if (n_bits > 2048) return fail(BLSH_EINVAL, "srp (sparse): n_bits %d > 2048", n_bits);
  // two quads per lane with the table (16-byte loads) when they fill a wave; drawn
  // entries go one quad per lane (more waves)
  const uint32_t k0 = uint32_t(seed), k1 = uint32_t(seed >> 32);
  // a table of plane entries pays when terms repeat: more nonzeros than twice the dimension
  int64_t nnz = 0;
  BLSH_HIP(hipMemcpyAsync(&nnz, offsets + n_rows, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  BLSH_HIP(hipStreamSynchronize(s));
  // workspace: the table, a byte per term, and the masks of as many rows' open
  // bits as one launch takes.  What does not fit (a workspace fixed smaller, or
  // not enough device memory): first fewer rows at a time, then no table (entries
  // drawn per nonzero), then no masks (every bit worked out): the same bits each time.
  auto align = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t mask_row = size_t(n_bits / 32) * 4;
  const size_t table_bytes = align(size_t(std::max<int64_t>(dim, 0)) * size_t(n_bits) * sizeof(int16_t));
  const size_t used_bytes = align(size_t(std::max<int64_t>(dim, 0)));
  const int64_t most = std::min<int64_t>(n_rows, kSrpRows), fewest = std::min<int64_t>(n_rows, kSrpFewest);
  bool use_table = dim > 0 && nnz > 2 * dim && table_bytes <= kSrpTableMaxBytes;
  size_t table_room = use_table ? table_bytes + used_bytes : 0;
  int64_t chunk = most;   // rows per launch; 0: no masks
  if (ctx->ws_fixed) {
    if (table_room + mask_row * size_t(fewest) > ctx->ws_bytes) {
      use_table = false;
      table_room = 0;
    }
    chunk = std::min<int64_t>(most, int64_t((ctx->ws_bytes - table_room) / mask_row));
    if (chunk < fewest) chunk = 0;
  } else {
    int rc;
    while ((rc = ensure_workspace(ctx, table_room + mask_row * size_t(chunk))) == BLSH_ENOMEM) {
      (void)hipGetLastError();
      if (chunk > fewest) {
        chunk = std::max(fewest, chunk / 8);
      } else if (use_table) {
        use_table = false;
        table_room = 0;
        chunk = most;
      } else {
        chunk = 0;
      }
    }
    if (rc) return rc;
  }
  // A few short rows are settled at once, one launch for two: 1000 rows of 3 terms at 64
  // bits 28.5 us against 30.4, of 1 at 2048 29.6 / 31.5 (400 of 4 at 2048 36.5 / 31.7; 4000
  // of 2 at 64 37 / 31; 30 of 20 at 512 42 / 31).
  if (!use_table && n_rows <= int64_t(ctx->n_cu) * 4 && nnz <= 4 * n_rows && nnz * n_bits <= int64_t(1) << 21) chunk = 0;
  int16_t *table = static_cast<int16_t *>(ctx->ws);
  uint8_t *used = static_cast<uint8_t *>(ctx->ws) + table_bytes;
  uint32_t *open = reinterpret_cast<uint32_t *>(static_cast<char *>(ctx->ws) + table_room);
  LaunchScope ls(ctx, s, "srp_sparse");
  if (use_table) {
    // the codes of the terms that occur
    const unsigned gz = unsigned(std::min<int64_t>((dim + 255) / 256, 4096));
    hipLaunchKernelGGL(k_fill_u8, dim3(gz), dim3(256), 0, s, used, dim);
    const unsigned gm = unsigned(std::min<int64_t>((nnz + 255) / 256, 8192));
    hipLaunchKernelGGL(k_srp_mark, dim3(gm), dim3(256), 0, s, indices, nnz, dim, used);
    // (fewer than 64 terms to a wave where that would leave SIMDs without one)
    const int per = int(std::max<int64_t>(1, std::min<int64_t>(kWave, dim / (int64_t(ctx->n_cu) * 32))));
    const int64_t tb = (dim + per * 4 - 1) / (per * 4);
    hipLaunchKernelGGL(k_srp_table, dim3(unsigned(std::min<int64_t>(tb, int64_t(ctx->n_cu) * 64))), dim3(256), 0, s, dim,
                       n_bits, k0, k1, used, table, per);
  }
  const int qpl = use_table && n_bits > 256 ? 2 : 1;
  const int n_slices = (n_bits / 4 + kWave * qpl - 1) / (kWave * qpl);
  const float err = kUnit * kFastErr + (use_table ? 0.5f : 0.f) + (q16 ? kUnit / 8192.f : 0.f);
  const bool filter = chunk > 0;
  for (int64_t r0 = 0, r1; r0 < n_rows; r0 = r1) {
    r1 = std::min(n_rows, r0 + (filter ? chunk : kSrpRows));
    if (filter)
      hipLaunchKernelGGL((!use_table ? k_srp_sparse<false, 1> : qpl == 2 ? k_srp_sparse<true, 2> : k_srp_sparse<true, 1>),
                         dim3(unsigned((r1 - r0 + 3) / 4 * n_slices)), dim3(256), 0, s, offsets, indices, values, n_rows,
                         r0, r1, n_bits, n_slices, k0, k1, int(word_major), out, open, table, dim, err);
    // (fewer rows to a block where 32 would leave CUs without one)
    const int per = int(std::max<int64_t>(1, std::min<int64_t>(kSettleRows, (r1 - r0) / (int64_t(ctx->n_cu) * (filter ? 4 : 32)))));
    hipLaunchKernelGGL(q16 ? k_srp_settle<true> : k_srp_settle<false>, dim3(unsigned((r1 - r0 + per - 1) / per)),
                       dim3(256), 0, s, offsets, indices, values, n_rows, r0, r1, per, n_bits, k0, k1, int(word_major),
                       out, filter ? open : nullptr);
  }
  return hipGetLastError() == hipSuccess ? BLSH_OK : BLSH_EDEVICE;
}

// Where the filtered product is the faster one.  Its planes are prepared and
// its open signs settled by two small kernels, about 15 us beside the main one,
// but it splits the planes over blocks when rows alone do not fill the chip:
// from 512 planes (and 2^15 plane elements) on it wins at any number of rows
// (us, plain / filtered: 1000 x 256 x 1024 144 / 31; 20,000 x 128 x 512 41 / 36; 40,000 x
// 64 x 512 41 / 30) but, for the least of these, about one block to a CU (30,000 x 64 x
// 512: 26 / 28); with 128 planes from 2^32 multiply-adds on (300,000 x 128 x 128: 94 / 81;
// 100,000 x 128 x 128: 42 / 41; 300,000 x 32 x 256: 52 / 52).
static bool filter_pays(const blsh_ctx *ctx, int64_t n_rows, int64_t dim, int64_t n_bits) {
  const int64_t cu_rows = int64_t(ctx->n_cu) * 128;   // a block to a CU
  if (n_bits >= 512 && dim * n_bits >= (1 << 15))
    return n_bits >= 1024 || dim * n_bits >= (1 << 16) || n_rows <= cu_rows / 2 || n_rows > cu_rows;
  return n_bits >= 128 && double(n_rows) * double(dim) * double(n_bits) >= 4294967296.0;
}
constexpr int kOpenShare = 256;   // a wave's list holds 1 in kOpenShare of its signs (Gaussian planes leave 1 in 1000 open)

template <int D>
static int launch_srp_filter(blsh_ctx *ctx, const float *X, int64_t n_rows, const float *R, int n_bits, bool word_major,
                             uint32_t *out, hipStream_t s, bool *done) {
  *done = false;
  const int W = n_bits / 32;
  const int64_t rb = (n_rows + 127) / 128;
  // rows alone may not fill the chip: split the planes too, as far as all blocks
  // run at once (registers allow 2 to a CU with 256 columns, 3 with 128, else 4;
  // 20,000 x 64 x 512 in 1099 blocks 30 us, in 942 25)
  const int64_t want = int64_t(ctx->n_cu) * (D == 256 ? 2 : D == 128 ? 3 : 4) / rb;
  const int splits = int(std::max<int64_t>(1, std::min<int64_t>(want, W / 2)));
  const int64_t regions = rb * 4 * splits;
  const int cap = std::max(32, 32 * (n_bits / splits) / kOpenShare);
  auto align = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t b_bf = align(size_t(n_bits) * D * 4), b_rt = align(size_t(n_bits) * D * 4), b_n = align(size_t(n_bits) * 4),
               b_cnt = align(size_t(regions) * 4), b_open = align(size_t(regions) * cap * 4);
  const size_t need = b_bf + b_rt + b_n + b_cnt + b_open;
  if (need > ctx->ws_bytes) {
    if (ctx->ws_fixed) return BLSH_OK;
    if (ensure_workspace(ctx, need) != BLSH_OK) {
      (void)hipGetLastError();
      return BLSH_OK;
    }
  }
  char *p = static_cast<char *>(ctx->ws);
  uint4 *Bf = reinterpret_cast<uint4 *>(p);
  float *Rt = reinterpret_cast<float *>(p + b_bf), *norms = reinterpret_cast<float *>(p + b_bf + b_rt);
  uint32_t *cnt = reinterpret_cast<uint32_t *>(p + b_bf + b_rt + b_n), *open = cnt + b_cnt / 4;
  LaunchScope ls(ctx, s, "srp_dense_mfma");
  hipLaunchKernelGGL(k_srp_planes<D>, dim3(W), dim3(256), 0, s, R, n_bits, Bf, norms, Rt);
  const FilterArgs fa{X, n_rows, R, Bf, norms, out, open, cnt, n_bits, splits, int32_t(word_major), cap};
  hipLaunchKernelGGL(k_srp_dense_filter<D>, dim3(unsigned(rb * splits)), dim3(256), 0, s, fa);
  hipLaunchKernelGGL(k_srp_dense_settle<D>, dim3(unsigned((regions + 3) / 4)), dim3(256), 0, s, X, n_rows, Rt, n_bits,
                     splits, int(word_major), out, open, cnt, cap, regions);
  *done = true;
  return hipGetLastError() == hipSuccess ? BLSH_OK : BLSH_EDEVICE;
}

int launch_srp_dense(blsh_ctx *ctx, const float *X, int64_t n_rows, int64_t dim, const float *R, int n_bits,
                     bool word_major, uint32_t *out, hipStream_t s) {
  const int64_t nb = (n_rows + 127) / 128;
  // a call under capture keeps to the plain kernel: it neither grows the
  // workspace nor leaves its address in a graph
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (filter_pays(ctx, n_rows, dim, n_bits) && uint32_t(n_bits) <= kOpenCol &&
      hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) {
    bool done = false;
    int rc = BLSH_OK;
#define BLSH_DF(DD) if (dim == DD) rc = launch_srp_filter<DD>(ctx, X, n_rows, R, n_bits, word_major, out, s, &done);
    BLSH_DF(32) BLSH_DF(64) BLSH_DF(128) BLSH_DF(256)
#undef BLSH_DF
    if (rc || done) return rc;
  }
  LaunchScope ls(ctx, s, "srp_dense_mfma");
#define BLSH_DN(DD) if (dim == DD) { hipLaunchKernelGGL(k_srp_dense_mfma<DD>, dim3(nb), dim3(256), 0, s, X, n_rows, R, n_bits, int(word_major), out); return hipGetLastError() == hipSuccess ? BLSH_OK : BLSH_EDEVICE; }
  BLSH_DN(32) BLSH_DN(64) BLSH_DN(128) BLSH_DN(256)
#undef BLSH_DN
  return fail(BLSH_EINVAL, "srp (dense): dim must be 32, 64, 128 or 256 (got %lld)", (long long)dim);
}

}  // namespace blsh
