// Grouping of key occurrences by row id: a stable least-significant-digit radix sort of
// (row id, segment id) pairs, hand-written for wave64 and a 160 KB LDS.
//
// Paper: the push of Algorithm 1 updates each referenced parameter once per
// mini-batch, so the occurrences of one key must be brought together before
// their gradients can be summed (the "union of the referenced parameters" of
// Section 2.3, here formed on the GPU).  Row ids are dense small integers
// (ceil(log2 R) bits), so sorting them costs half the passes of sorting the
// 64-bit keys.
//
// One pass = three launches, two for short lists:
//   k_sort_hist    per-chunk digit histogram           -> hist[digit][chunk] (wide digits: hist[chunk][digit])
//   k_sort_scan    per digit: exclusive scan over chunks, digit totals
//   k_sort_scatter per chunk: for each sub-tile, rank elements
//                  per digit inside each wave with ballots (stable), counting-
//                  sort the sub-tile in LDS, then write each digit's run to
//                  its place; runs are contiguous, so the writes coalesce.
// A sub-tile is 256 * ITEMS elements.  Long lists take ITEMS = 16 (long runs, few histograms; bound by memory:
// 39 M elements of 24 bits 817 us, 887 with 8); short ones are bound by the ranking chain of one sub-tile on an idle
// chip and take fewer: 300 k elements 53 us with 16, 41 with 4; 1.25 M 65 with 16, 58 with 8.
// Lists of few chunks do without the scan: every scatter block adds up the histograms before its own while its elements
// are on their way (two passes of 8 bits: 1000 elements 16.8 -> 13.3 us, 32 k 20.3 -> 16.4, 64 k 20.6 -> 19.1, 73 k 20.7 ->
// 21.1; two of 10 bits: 4 k 20.2 -> 16.5, 8 k 20.6 -> 18.6, 16 k 21.0 -> 23.1; of 11 bits: 1000 20.2 -> 15.0, 4 k 21.3 -> 21.2).
// (Also measured, and not gaining: the scan done by the last block of every 16 or 32 chunks to end; blocks of 1024 threads, whose
// lists have fewer chunks.)
// Digits have 8 bits, or 10 or 11 where that saves a pass and the list is short.  A pass of a short list costs its
// three launches and their chains rather than bytes, so fewer passes win: 20-bit keys, 73 k elements 32 -> 25 us,
// 400 k 42 -> 36, 800 k 51 -> 44; 22-bit keys, 175 k 35 -> 33, 400 k 43 -> 40.  Long lists lose by it: a sub-tile then
// leaves runs of one or two elements per digit (2.5 M elements, 20 bits 77 -> 83 us, 22 bits 78 -> 96).  Three wide
// passes instead of four, for keys of more than 24 bits, pay for still shorter lists only: 26 bits, 20 k 42 -> 35, 73 k
// 43 -> 40, 175 k 45 -> 48, 300 k 52 -> 56.  Wide digits keep their histograms as [chunk][digit], which a block writes
// and reads coalesced.  (All sizes, both sides of each line: profiles/sort_sizes.txt.)
#pragma once
#include <algorithm>

#include "common.h"

namespace ctr {

constexpr u32 SORT_ITEMS_4_MAX = 300000, SORT_ITEMS_8_MAX = 1600000;  // elements
constexpr u32 SORT_10_BITS_MAX = 1000000, SORT_11_BITS_MAX = 500000, SORT_3_WIDE_PASSES_MAX = 100000;
// most chunks of 1024 elements that a scatter block adds up itself, for digits of 8, 10 and 11 bits
constexpr u32 SORT_SHORT_CHUNKS = 64, SORT_SHORT_CHUNKS_10 = 8, SORT_SHORT_CHUNKS_11 = 3;
#ifndef CTR_SORT_MAX_CHUNKS
#define CTR_SORT_MAX_CHUNKS 4096
#endif
constexpr int SORT_MAX_CHUNKS = CTR_SORT_MAX_CHUNKS;
static_assert(SORT_MAX_CHUNKS % BLOCK == 0, "k_sort_scan");
constexpr int RADIX = 256;
#ifndef CTR_HIST_COPIES
#define CTR_HIST_COPIES 4
#endif
constexpr int HIST_COPIES = CTR_HIST_COPIES;  // power of two

struct SortGeom {
  u32 n;            // elements
  u32 n_chunks;     // blocks of the histogram / scatter launches
  u32 chunk_elems;  // multiple of 256 * items
  u32 items;        // elements per thread of a sub-tile: 4, 8 or 16
};

// The histograms of a list's first pass, taken beside the pooling by blocks of its launch behind n_pool_blocks of them
// (a launch of its own costs 3 to 6 us); n_pool_blocks 0: there is none.  rows: hist[chunk][digit].
struct SortFirst {
  u32 n_pool_blocks, digit_mask, log2_radix, rows;
  SortGeom geo;
  u32* hist;
};

constexpr u32 SORT_FIRST_WORDS = 4096;  // LDS: 16 histograms of 256 digits, 4 of 1024, 2 of 2048

// row_of: the row of an entry of the list.
template <class RowOf>
__device__ __forceinline__ void sort_first_hist(const SortFirst& f, u32 chunk, const u32* __restrict__ entries, u32* lds,
                                                const RowOf& row_of) {
  const u32 radix = 1u << f.log2_radix;
  for (u32 i = threadIdx.x; i < SORT_FIRST_WORDS; i += BLOCK) lds[i] = 0;
  __syncthreads();
  const u32 beg = chunk * f.geo.chunk_elems, end = min(beg + f.geo.chunk_elems, f.geo.n);
  u32* mine = lds + (((u32)wave_id() * 4 + ((u32)lane_id() & 3u)) >> (f.log2_radix - 8)) * radix;
  for (u32 e = beg + threadIdx.x * 4; e < end; e += BLOCK * 4) {
    u32 d[4];
    if (e + 4 <= end) {
      const uint4 v = *reinterpret_cast<const uint4*>(entries + e);
      d[0] = row_of(v.x); d[1] = row_of(v.y); d[2] = row_of(v.z); d[3] = row_of(v.w);
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] &= f.digit_mask;
      // see k_sort_hist
      const u32 ref = (u32)__builtin_amdgcn_readfirstlane((int)d[0]);
      u32 n_ref = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        n_ref += (u32)__popcll(__ballot(d[i] == ref));
        if (d[i] != ref) atomicAdd(&mine[d[i]], 1u);
      }
      if (lane_id() == __ffsll((long long)__ballot(true)) - 1) atomicAdd(&mine[ref], n_ref);
    } else {
      for (u32 j = e; j < end; ++j) atomicAdd(&mine[row_of(entries[j]) & f.digit_mask], 1u);
    }
  }
  __syncthreads();
  for (u32 d = threadIdx.x; d < radix; d += BLOCK) {
    u32 total = 0;
    for (u32 i = d; i < SORT_FIRST_WORDS; i += radix) total += lds[i];
    f.hist[f.rows ? chunk * radix + d : d * f.geo.n_chunks + chunk] = total;
  }
}

// ROWS: hist[chunk][digit], otherwise hist[digit][chunk].
template <int R, bool ROWS>
__global__ void __launch_bounds__(BLOCK)
k_sort_hist(const DevHeader* hdr, const u32* __restrict__ keys, SortGeom geo, u32 shift, u32 digit_mask,
            u32* __restrict__ hist) {
  const u32 beg = blockIdx.x * geo.chunk_elems;  // multiple of 1024, so 16-byte aligned
  const u32 end = min(beg + geo.chunk_elems, geo.n);
  const u32 status = hdr->status, e0 = beg + threadIdx.x * 4;
  uint4 k4 = {0u, 0u, 0u, 0u};  // of the thread's first step; the next one's are requested while a step is counted
  if (e0 + 4 <= end) k4 = *reinterpret_cast<const uint4*>(keys + e0);
  requested();
  if (status) return;
  // COPIES histograms per wave, chosen by lane: a popular digit (row ids of popular keys share
  // their high bits) would otherwise serialise all 64 lanes on one LDS address
  constexpr int COPIES = R == RADIX ? HIST_COPIES : 1;
  __shared__ u32 h[4 * COPIES][R];
#pragma unroll
  for (int i = 0; i < 4 * COPIES; ++i)
#pragma unroll
    for (int q = 0; q < R / BLOCK; ++q) h[i][q * BLOCK + threadIdx.x] = 0;
  __syncthreads();
  u32* mine = h[wave_id() * COPIES + (lane_id() & (COPIES - 1))];
  for (u32 e = e0; e < end; e += BLOCK * 4) {
    if (e + 4 <= end) {
      const u32 d0 = (k4.x >> shift) & digit_mask, d1 = (k4.y >> shift) & digit_mask;
      const u32 d2 = (k4.z >> shift) & digit_mask, d3 = (k4.w >> shift) & digit_mask;
      if (e + BLOCK * 4 + 4 <= end) k4 = *reinterpret_cast<const uint4*>(keys + e + BLOCK * 4);
      // the digit of the wave's first key is counted with ballots (one add for the whole wave):
      // under a popular digit that takes most of the keys away from the LDS atomics
      const u32 ref = (u32)__builtin_amdgcn_readfirstlane((int)d0);
      const u32 n_ref = (u32)(__popcll(__ballot(d0 == ref)) + __popcll(__ballot(d1 == ref)) +
                              __popcll(__ballot(d2 == ref)) + __popcll(__ballot(d3 == ref)));
      if (d0 != ref) atomicAdd(&mine[d0], 1u);
      if (d1 != ref) atomicAdd(&mine[d1], 1u);
      if (d2 != ref) atomicAdd(&mine[d2], 1u);
      if (d3 != ref) atomicAdd(&mine[d3], 1u);
      if (lane_id() == __ffsll((long long)__ballot(true)) - 1) atomicAdd(&mine[ref], n_ref);  // first lane that is here
    } else {
      for (u32 j = e; j < end; ++j) atomicAdd(&mine[(keys[j] >> shift) & digit_mask], 1u);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < R / BLOCK; ++q) {
    const u32 d = q * BLOCK + threadIdx.x;
    u32 total = 0;
#pragma unroll
    for (int i = 0; i < 4 * COPIES; ++i) total += h[i][d];
    hist[ROWS ? blockIdx.x * R + d : d * geo.n_chunks + blockIdx.x] = total;
  }
}

// grid = RADIX blocks; block d turns hist[d][0..n_chunks) into exclusive prefix sums.  A thread's entries (PER at most, 1 for
// lists of up to 256 chunks) stay in registers.
template <u32 PER>
__global__ void __launch_bounds__(BLOCK)
k_sort_scan(const DevHeader* hdr, u32* __restrict__ hist, u32 n_chunks, u32* __restrict__ digit_total) {
  __shared__ u32 lds[4];
  u32* row = hist + blockIdx.x * n_chunks;
  const u32 per = PER == 1 ? 1u : (n_chunks + BLOCK - 1) / BLOCK;  // consecutive entries per thread
  const u32 c0 = threadIdx.x * per;
  const u32 n = c0 < n_chunks ? min(per, n_chunks - c0) : 0u;
  u32 v[PER], s = 0, total;
  const u32 status = hdr->status;
#pragma unroll
  for (u32 i = 0; i < PER; ++i) v[i] = i < n ? row[c0 + i] : 0u;
  requested();
  if (status) return;
#pragma unroll
  for (u32 i = 0; i < PER; ++i) s += v[i];
  u32 ex = block_exclusive_scan(s, lds, total);
#pragma unroll
  for (u32 i = 0; i < PER; ++i) {
    if (i < n) row[c0 + i] = ex;
    ex += v[i];
  }
  if (threadIdx.x == 0) digit_total[blockIdx.x] = total;
}

// The same for hist[chunk][digit]: a block takes 16 neighbouring digits, 16 groups of threads a share of the chunks, of
// which the entries stay in registers.
constexpr u32 SCAN_WIDE_PER = 32;
__global__ void __launch_bounds__(BLOCK)
k_sort_scan_wide(const DevHeader* hdr, u32* __restrict__ hist, u32 n_chunks, u32 radix, u32* __restrict__ digit_total) {
  __shared__ u32 sums[16][16];
  const u32 in = threadIdx.x & 15u, group = threadIdx.x >> 4, d = blockIdx.x * 16 + in;
  const u32 per = (n_chunks + 15) / 16, c0 = min(group * per, n_chunks), n = min(per, n_chunks - c0);
  u32* at = hist + c0 * radix + d;
  u32 v[SCAN_WIDE_PER], s = 0;
  const u32 status = hdr->status;
#pragma unroll
  for (u32 i = 0; i < SCAN_WIDE_PER; ++i) v[i] = i < n ? at[i * radix] : 0u;
  requested();
  if (status) return;
#pragma unroll
  for (u32 i = 0; i < SCAN_WIDE_PER; ++i) s += v[i];
  sums[group][in] = s;
  __syncthreads();
  u32 ex = 0, total = 0;
#pragma unroll
  for (u32 g = 0; g < 16; ++g) {
    const u32 v = sums[g][in];
    if (g < group) ex += v;
    total += v;
  }
#pragma unroll
  for (u32 i = 0; i < SCAN_WIDE_PER; ++i) {
    if (i < n) at[i * radix] = ex;
    ex += v[i];
  }
  if (group == 0) digit_total[d] = total;
}

// SCANNED: hist holds the prefix sums of a scan launch, [digit][chunk] or, of wide digits, [chunk][digit]; otherwise the
// counts, [chunk][digit], of few chunks, which every block adds up itself.
template <int ITEMS, int R, bool SCANNED>
__global__ void __launch_bounds__(BLOCK)
k_sort_scatter(const DevHeader* hdr, const u32* __restrict__ keys_in, const u32* __restrict__ vals_in,
               u32* __restrict__ keys_out, u32* __restrict__ vals_out, SortGeom geo, u32 shift,
               u32 digit_mask, const u32* __restrict__ hist, const u32* __restrict__ digit_total) {
  constexpr int TILE = BLOCK * ITEMS, DIGITS = R / BLOCK;  // digits a thread owns: DIGITS neighbouring ones
  constexpr int BITS = __builtin_ctz(R);
  __shared__ u32 scan_lds[4];
  __shared__ u32 whist[4][R];  // per-wave digit counts, then per-wave local bases
  __shared__ u32 delta[R];     // global position of a digit's first element of the sub-tile - its sub-tile position
  __shared__ u32 lkeys[TILE];
  __shared__ u32 lvals[TILE];

  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const u32 chunk_beg = blockIdx.x * geo.chunk_elems;
  const u32 chunk_end = min(chunk_beg + geo.chunk_elems, geo.n);
  u32 k[ITEMS], v[ITEMS];
  const auto request = [&](u32 sub) {  // waves own consecutive quarters of a sub-tile
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const u32 at = sub + w * (TILE / 4) + i * WAVE + lane;
      k[i] = at < chunk_end ? keys_in[at] : 0u;
      v[i] = at < chunk_end ? vals_in[at] : 0u;
    }
  };
  const u32 status = hdr->status;
  u32 gbase[DIGITS], count[DIGITS];  // gbase: next global position of the thread's digits for this chunk
  request(chunk_beg);
  if constexpr (SCANNED) {
#pragma unroll
    for (int q = 0; q < DIGITS; ++q) {
      const u32 d = tid * DIGITS + q;
      count[q] = digit_total[d];
      gbase[q] = hist[R == RADIX ? d * geo.n_chunks + blockIdx.x : blockIdx.x * R + d];
    }
  } else {
#pragma unroll
    for (int q = 0; q < DIGITS; ++q) count[q] = gbase[q] = 0;
    constexpr u32 SIDE = 32 / DIGITS;  // chunks requested together
    for (u32 c0 = 0; c0 < geo.n_chunks; c0 += SIDE) {
      u32 h[SIDE][DIGITS];
#pragma unroll
      for (u32 i = 0; i < SIDE; ++i)
#pragma unroll
        for (int q = 0; q < DIGITS; ++q) h[i][q] = c0 + i < geo.n_chunks ? hist[(c0 + i) * R + tid * DIGITS + q] : 0u;
#pragma unroll
      for (u32 i = 0; i < SIDE; ++i)
#pragma unroll
        for (int q = 0; q < DIGITS; ++q) {
          count[q] += h[i][q];
          gbase[q] += c0 + i < blockIdx.x ? h[i][q] : 0u;
        }
    }
  }
  requested();
  if (status) return;
  {
    u32 sum = 0, total;
#pragma unroll
    for (int q = 0; q < DIGITS; ++q) sum += count[q];
    u32 ex = block_exclusive_scan(sum, scan_lds, total);
#pragma unroll
    for (int q = 0; q < DIGITS; ++q) {
      gbase[q] += ex;
      ex += count[q];
    }
  }
  const u64 lanes_below = (1ull << lane) - 1ull;

  for (u32 sub = chunk_beg; sub < chunk_end; sub += TILE) {
    const u32 n_valid = min((u32)TILE, chunk_end - sub);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < DIGITS; ++q) whist[i][q * BLOCK + tid] = 0;
    __syncthreads();

    u32 rank[ITEMS];
    volatile u32* my_hist = whist[w];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const u32 local = w * (TILE / 4) + i * WAVE + lane;
      const bool valid = local < n_valid;
      const u32 d = (k[i] >> shift) & digit_mask;  // 0 for lanes past the end (k = 0)
      // lanes whose digit equals mine: for every bit, the ballot of that bit XNOR my bit (m is
      // 0 or ~0); the disagreements are OR-ed per 32-bit half, lanes past the end masked at the end
      u32 diff_lo = 0, diff_hi = 0;
#pragma unroll
      for (int b = 0; b < BITS; ++b) {
        const u32 m = (u32)__builtin_amdgcn_sbfe((int)d, b, 1);
        const u64 bal = __builtin_amdgcn_ballot_w64(m != 0u);
        diff_lo |= (u32)bal ^ m;
        diff_hi |= (u32)(bal >> 32) ^ m;
      }
      const u64 same = __ballot(valid) & ~(((u64)diff_hi << 32) | diff_lo);
      // lanes of `same` hold digit d; the lowest of them bumps the wave's counter
      const int leader = __ffsll((long long)same) - 1;
      u32 before = 0;
      if (valid && lane == leader) {
        before = my_hist[d];
        my_hist[d] = before + (u32)__popcll(same);
      }
      before = __shfl(before, leader < 0 ? 0 : leader, WAVE);
      rank[i] = before + (u32)__popcll(same & lanes_below);
    }
    __syncthreads();

    {  // digit-major, wave-minor exclusive scan of the counts
      u32 sum = 0, total;
#pragma unroll
      for (int q = 0; q < DIGITS; ++q) {
        const int d = tid * DIGITS + q;
        sum += whist[0][d] + whist[1][d] + whist[2][d] + whist[3][d];
      }
      u32 at = block_exclusive_scan(sum, scan_lds, total);
#pragma unroll
      for (int q = 0; q < DIGITS; ++q) {
        const int d = tid * DIGITS + q;
        const u32 c0 = whist[0][d], c1 = whist[1][d], c2 = whist[2][d], c3 = whist[3][d];
        delta[d] = gbase[q] - at;
        gbase[q] += c0 + c1 + c2 + c3;
        whist[0][d] = at;
        whist[1][d] = at += c0;
        whist[2][d] = at += c1;
        whist[3][d] = at += c2;
        at += c3;
      }
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const u32 local = w * (TILE / 4) + i * WAVE + lane;
      if (local < n_valid) {
        const u32 d = (k[i] >> shift) & digit_mask;
        const u32 pos = whist[w][d] + rank[i];
        lkeys[pos] = k[i];
        lvals[pos] = v[i];
      }
    }
    if (sub + TILE < chunk_end) request(sub + TILE);
    __syncthreads();

    for (u32 j = tid; j < n_valid; j += BLOCK) {
      const u32 kk = lkeys[j];
      const u32 pos = delta[(kk >> shift) & digit_mask] + j;
      keys_out[pos] = kk;
      vals_out[pos] = lvals[j];
    }
    // the barriers of the next iteration order these reads of the LDS lists before their next writes
  }
}

// ---------------------------------------------------------------- host side

// How a list of n elements is cut into the chunks the sort's launches work on.
constexpr SortGeom sort_geom(u64 n, u32 items, u64 max_chunks) {
  SortGeom g{};
  g.items = items;
  const u64 tile = (u64)BLOCK * g.items, tiles = (n + tile - 1) / tile;
  const u64 chunks = std::min<u64>(std::max<u64>(tiles, 1), max_chunks);
  const u64 per = (n + chunks - 1) / chunks;
  const u64 chunk_elems = std::max<u64>(((per + tile - 1) / tile) * tile, tile);
  g.n = (u32)n;
  g.chunk_elems = (u32)chunk_elems;
  g.n_chunks = (u32)std::max<u64>((n + chunk_elems - 1) / chunk_elems, 1);
  return g;
}
inline SortGeom sort_geom(u64 n) {
  return sort_geom(n, n <= SORT_ITEMS_4_MAX ? 4u : n <= SORT_ITEMS_8_MAX ? 8u : 16u, SORT_MAX_CHUNKS);
}

// Words of `hist`: the histograms of SORT_MAX_CHUNKS chunks of RADIX digits.
constexpr size_t SORT_HIST_WORDS = (size_t)RADIX * SORT_MAX_CHUNKS;

// Geometry of a list of n elements that takes digits of `bits` (10 or 11) bits.
constexpr bool sort_takes_wide(u64 n, u32 bits) { return n <= (bits == 10 ? SORT_10_BITS_MAX : SORT_11_BITS_MAX); }
constexpr SortGeom sort_geom_wide(u64 n, u32 bits) {
  return sort_geom(n, n <= SORT_ITEMS_4_MAX ? 4u : 8u, (SORT_HIST_WORDS >> bits) - 1);
}
// the most chunks: of the longest list, and of the longest one that takes 4 elements per thread
constexpr bool sort_scan_wide_holds(u64 n, u32 bits) { return sort_geom_wide(n, bits).n_chunks <= 16 * SCAN_WIDE_PER; }
static_assert(sort_scan_wide_holds(SORT_10_BITS_MAX, 10) && sort_scan_wide_holds(SORT_11_BITS_MAX, 11) &&
                  sort_scan_wide_holds(SORT_ITEMS_4_MAX, 10) && sort_scan_wide_holds(SORT_ITEMS_4_MAX, 11),
              "k_sort_scan_wide keeps SCAN_WIDE_PER entries per thread");

// Words of `hist` that a list of n elements uses, whatever its keys, and the order of a push's n_spans spans.
inline size_t sort_hist_words(u64 n, u64 n_spans) {
  size_t words = (size_t)RADIX * std::max(sort_geom(n).n_chunks, sort_geom(n_spans).n_chunks);
  for (u32 bits : {10u, 11u})
    if (sort_takes_wide(n, bits)) words = std::max(words, ((size_t)sort_geom_wide(n, bits).n_chunks + 1) << bits);
  return words;
}

// One pass over the digit (key >> shift) & digit_mask; counted: its histograms have been taken.
inline void sort_pass_enqueue(const DevHeader* hdr, const u32* keys_in, const u32* vals_in, u32* keys_out, u32* vals_out,
                              const SortGeom& geo, u32 shift, u32 digit_mask, u32* hist, u32* digit_total, bool counted,
                              hipStream_t st) {
  if (!counted) hipLaunchKernelGGL((k_sort_hist<RADIX, false>), dim3(geo.n_chunks), dim3(BLOCK), 0, st, hdr, keys_in, geo, shift, digit_mask, hist);
  if (geo.n_chunks <= BLOCK)
    hipLaunchKernelGGL(k_sort_scan<1>, dim3(RADIX), dim3(BLOCK), 0, st, hdr, hist, geo.n_chunks, digit_total);
  else if (geo.n_chunks <= 4 * BLOCK)
    hipLaunchKernelGGL(k_sort_scan<4>, dim3(RADIX), dim3(BLOCK), 0, st, hdr, hist, geo.n_chunks, digit_total);
  else
    hipLaunchKernelGGL(k_sort_scan<SORT_MAX_CHUNKS / BLOCK>, dim3(RADIX), dim3(BLOCK), 0, st, hdr, hist, geo.n_chunks, digit_total);
#define CTR_SORT_SCATTER(ITEMS, R, SCANNED)                                                                        \
  hipLaunchKernelGGL((k_sort_scatter<ITEMS, R, SCANNED>), dim3(geo.n_chunks), dim3(BLOCK), 0, st, hdr, keys_in, vals_in,      \
                     keys_out, vals_out, geo, shift, digit_mask, hist, digit_total)
  if (geo.items == 4) CTR_SORT_SCATTER(4, RADIX, true);
  else if (geo.items == 8) CTR_SORT_SCATTER(8, RADIX, true);
  else CTR_SORT_SCATTER(16, RADIX, true);
}

// A pass of wide digits (R = 1024 or 2048; the digit totals stand behind the histograms).
template <int R>
inline void sort_pass_wide_enqueue(const DevHeader* hdr, const u32* keys_in, const u32* vals_in, u32* keys_out,
                                   u32* vals_out, const SortGeom& geo, u32 shift, u32 digit_mask, u32* hist, bool counted,
                                   hipStream_t st) {
  u32* digit_total = hist + (size_t)R * geo.n_chunks;
  if (!counted) hipLaunchKernelGGL((k_sort_hist<R, true>), dim3(geo.n_chunks), dim3(BLOCK), 0, st, hdr, keys_in, geo, shift, digit_mask, hist);
  hipLaunchKernelGGL(k_sort_scan_wide, dim3(R / 16), dim3(BLOCK), 0, st, hdr, hist, geo.n_chunks, (u32)R, digit_total);
  if (geo.items == 4) CTR_SORT_SCATTER(4, R, true);
  else CTR_SORT_SCATTER(8, R, true);
}

// A pass without a scan, of a list of few chunks (4 elements per thread).
template <int R>
inline void sort_pass_short_enqueue(const DevHeader* hdr, const u32* keys_in, const u32* vals_in, u32* keys_out,
                                    u32* vals_out, const SortGeom& geo, u32 shift, u32 digit_mask, u32* hist, bool counted,
                                    hipStream_t st) {
  const u32* digit_total = nullptr;
  if (!counted) hipLaunchKernelGGL((k_sort_hist<R, true>), dim3(geo.n_chunks), dim3(BLOCK), 0, st, hdr, keys_in, geo, shift, digit_mask, hist);
  CTR_SORT_SCATTER(4, R, false);
}
#undef CTR_SORT_SCATTER

// How a list of n elements is sorted by the low key_bits bits of its keys.
struct SortPlan {
  u32 passes, log2_radix, key_bits;
  bool scanned;  // with a scan launch per pass
  SortGeom geo;
  u32 bits(u32 pass, u32 shift) const { return (key_bits - shift + (passes - pass) - 1) / (passes - pass); }  // spread evenly
  bool rows() const { return log2_radix != 8 || !scanned; }  // hist[chunk][digit]
};

inline SortPlan sort_plan(u64 n, u32 key_bits) {
  SortPlan p;
  const u32 wide_bits = key_bits > 20 ? 11u : 10u;
  p.key_bits = key_bits;
  p.passes = (key_bits + 7) / 8;
  const u32 wide_passes = (key_bits + wide_bits - 1) / wide_bits;
  const bool wide = wide_passes < p.passes && sort_takes_wide(n, wide_bits) && (wide_passes < 3 || n <= SORT_3_WIDE_PASSES_MAX);
  if (wide) p.passes = wide_passes;
  p.log2_radix = wide ? wide_bits : 8;
  p.geo = wide ? sort_geom_wide(n, wide_bits) : sort_geom(n);
  p.scanned = p.geo.n_chunks > (!wide ? SORT_SHORT_CHUNKS : wide_bits == 10 ? SORT_SHORT_CHUNKS_10 : SORT_SHORT_CHUNKS_11);
  return p;
}

// The part of the first pass that the pooling launch takes over.
inline SortFirst sort_first(const SortPlan& p, u32* hist, u32 n_pool_blocks) {
  return {n_pool_blocks, (1u << p.bits(0, 0)) - 1u, p.log2_radix, p.rows() ? 1u : 0u, p.geo, hist};
}

// Sorts the (key, value) pairs as planned, between the two pairs of arrays; returns which of them (0 = a, 1 = b) holds the
// result.  counted: the first pass's histograms have been taken (sort_first).
inline u32 sort_enqueue(const DevHeader* hdr, const u32* keys_in, const u32* vals_in, u32* const (&keys)[2],
                        u32* const (&vals)[2], const SortPlan& plan, bool counted, u32* hist, u32* digit_total,
                        hipStream_t st) {
  u32 shift = 0;
  for (u32 p = 0; p < plan.passes; ++p, counted = false) {
    const u32 bits = plan.bits(p, shift), mask = (1u << bits) - 1u;
#define CTR_SORT_PASS(KIND, R) \
  sort_pass_##KIND##_enqueue<R>(hdr, keys_in, vals_in, keys[p & 1], vals[p & 1], plan.geo, shift, mask, hist, counted, st)
    if (plan.log2_radix == 8 && plan.scanned)
      sort_pass_enqueue(hdr, keys_in, vals_in, keys[p & 1], vals[p & 1], plan.geo, shift, mask, hist, digit_total, counted, st);
    else if (plan.log2_radix == 8) CTR_SORT_PASS(short, RADIX);
    else if (plan.log2_radix == 10 && plan.scanned) CTR_SORT_PASS(wide, 1024);
    else if (plan.log2_radix == 10) CTR_SORT_PASS(short, 1024);
    else if (plan.scanned) CTR_SORT_PASS(wide, 2048);
    else CTR_SORT_PASS(short, 2048);
#undef CTR_SORT_PASS
    keys_in = keys[p & 1];
    vals_in = vals[p & 1];
    shift += bits;
  }
  return (plan.passes - 1) & 1;
}

}  // namespace ctr
