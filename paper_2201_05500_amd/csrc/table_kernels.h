// Key index (open addressing, insert-on-miss), row creation and the gather + per-segment sum.
//
// Paper: the per-GPU HBM hash table of Section 2.3 that holds the working
// parameters; Algorithm 1's insert_into_hash_table and pull steps; the state a
// new row starts from is Algorithm 2's "Initialize" line (m = 0, v = eps).
#pragma once
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "sort_kernels.h"

namespace ctr {


// ---------------------------------------------------------------- table creation

// keep_step_count: the number of accepted pushes (step count of the bias-corrected update) survives.
__global__ void k_table_clear(DevHeader* hdr, Slot* slots, u64 n_slots, u32* row_state, u64 n_rows_cap,
                              u32 keep_step_count) {
  const u64 tid = (u64)blockIdx.x * BLOCK + threadIdx.x;
  const u64 stride = (u64)gridDim.x * BLOCK;
  const bool count = tid == HDR_WORD_N_PUSH || (tid >= HDR_WORD_BC && tid < HDR_WORD_BC + 8);  // and the next push's factors
  if (tid < 64 && !(keep_step_count && count)) reinterpret_cast<u32*>(hdr)[tid] = 0;
  for (u64 i = tid; i < n_slots; i += stride) {
    Slot s;
    s.key = KEY_EMPTY;
    s.row = ROW_PENDING;
    s.first_p = 0xFFFFFFFFu;
    slots[i] = s;
  }
  for (u64 i = tid; i < n_rows_cap; i += stride) row_state[i] = 0;
}

// ---------------------------------------------------------------- probe / tentative insert

// One thread per key occurrence (a block takes a tile of 256 * items consecutive ones):
// linear probing from hash(key).  A hit on a committed slot yields the row id.  A miss claims
// the first free slot with a 64-bit compare-and-swap; the row id of such a slot is assigned
// later, so the occurrence records the slot index instead, lowers the slot's first_p to its
// own position (the smallest position wins: new rows are numbered in order of first
// occurrence) and is appended to its tile's list of pending occurrences (counted in LDS, so no
// global atomic is shared between blocks).  The same launch checks the CSR offsets.
constexpr int PROBE_MAX_ITEMS = 8;  // occurrences per thread: 8 for large batches, 1 for small ones (host's choice)
// ranking of new keys (below)
constexpr u32 RANK_TILE = PROBE_MAX_ITEMS * BLOCK;  // 2048 occurrences: a whole number of probe tiles of any size
constexpr u32 RANK_WORDS = RANK_TILE / 32;
constexpr u32 RANK_GROUP = 256;  // tiles: 39 M occurrences have 75 groups
constexpr u32 RANK_GROUP_STRIDE = 32;  // words: a group's count has a cache line to itself, because atomics on one
                                       // line are served one after the other (39 M occurrences: 19 k of them on
                                       // 5 lines took 60 of k_rank_count's 84 us)

__global__ void __launch_bounds__(BLOCK)
k_probe_insert(DevHeader* hdr, Slot* slots, u32 slot_mask, const u64* __restrict__ keys, u32 n_keys,
               const u32* __restrict__ offsets, u32 n_seg, u32* __restrict__ occ_row,
               u32* __restrict__ pend_list, u32* __restrict__ tile_pending, u32 items,
               u32* __restrict__ group_count, u32 n_groups) {
  const u32 tile0 = blockIdx.x * (BLOCK * items);
  u64 key = KEY_EMPTY;  // the thread's next occurrence: requested one ahead
  if (tile0 + threadIdx.x < n_keys) key = keys[tile0 + threadIdx.x];
  const bool refused = hdr->status != 0;  // an earlier call failed: this pull is a no-op
  requested();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    hdr->live = refused ? 0u : 1u;
    hdr->batch_ok = 0;
    hdr->n_rows_base = hdr->n_rows;
  }
  if (refused) return;
  if (blockIdx.x * BLOCK + threadIdx.x < n_groups) group_count[(blockIdx.x * BLOCK + threadIdx.x) * RANK_GROUP_STRIDE] = 0;
  __shared__ u32 n_pend;
  if (threadIdx.x == 0) n_pend = 0;
  __syncthreads();
  const int lane = lane_id();

#pragma unroll 1
  for (u32 it = 0; it < items; ++it) {
    const u32 p = tile0 + it * BLOCK + threadIdx.x;
    if (offsets != nullptr && p <= n_seg) {  // (a working-set load has no segments)
      const u32 a = offsets[p];
      bool bad = (p == 0 && a != 0);
      if (p == n_seg)
        bad = bad || (a != n_keys);
      else
        bad = bad || (offsets[p + 1] < a);
      if (bad) atomicOr(&hdr->pull_err, ST_INVAL);
    }

    const u64 this_key = key;
    if (it + 1 < items && p + BLOCK < n_keys) key = keys[p + BLOCK];
    bool pending = false;
    if (p < n_keys) {
      const u64 key = this_key;
      u32 out = OCC_INVALID;
      if (key == KEY_EMPTY) {
        atomicOr(&hdr->pull_err, ST_BADKEY);
      } else {
        u32 h = (u32)hash_key(key) & slot_mask;
        bool found = false;
        u32 r = ROW_PENDING;
        for (u32 probe = 0; probe <= slot_mask; ++probe) {
          // One plain (cacheable) 16-byte load brings key and row id in a single request.  Slots
          // only ever go from free to taken inside this launch, so the worst a stale copy can
          // show is "free", and the compare-and-swap below then returns the key that is really
          // there; rows are assigned between launches, never inside this one, so a slot taken
          // during this launch has no row yet.
          const uint4 raw = *reinterpret_cast<const uint4*>(&slots[h]);
          u64 k = ((u64)raw.y << 32) | raw.x;
          r = raw.z;
          if (k == KEY_EMPTY) {
            const u64 old = atomicCAS(&slots[h].key, KEY_EMPTY, key);
            k = (old == KEY_EMPTY) ? key : old;
            r = ROW_PENDING;
          }
          if (k == key) {
            found = true;
            break;
          }
          h = (h + 1) & slot_mask;
          if ((probe & 63u) == 63u && (ld_relaxed(&hdr->pull_err) & ST_FULL)) break;
        }
        if (!found) {  // every slot holds another key: more distinct keys than slots
          atomicOr(&hdr->pull_err, ST_FULL);
        } else {
          if (r == ROW_PENDING) {
            // a popular new key has millions of occurrences: only those that can still lower
            // the minimum go to the atomic unit, the rest see a smaller value and pass
            if (ld_relaxed(&slots[h].first_p) > p) atomicMin(&slots[h].first_p, p);
            out = OCC_PEND_FLAG | h;
            pending = true;
          } else {
            out = r;
          }
        }
      }
      occ_row[p] = out;
    }

    // every lane of the wave is here again: one LDS atomic per wave reserves list entries
    const u64 bal = __ballot(pending);
    if (bal) {
      const int leader = __ffsll((long long)bal) - 1;
      u32 base = 0;
      if (lane == leader) base = atomicAdd(&n_pend, (u32)__popcll(bal));
      base = __shfl(base, leader, WAVE);
      if (pending) pend_list[tile0 + base + (u32)__popcll(bal & ((1ull << lane) - 1ull))] = p;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && tile0 < n_keys) tile_pending[blockIdx.x] = n_pend;  // blocks past the keys only check offsets
}

// ---------------------------------------------------------------- ranking of new keys

// New rows are numbered in order of first occurrence, so the launches below need a prefix sum over the whole
// batch.  They are two: one that finds and counts the first occurrences, per rank tile and per group of
// RANK_GROUP tiles, and one in which every tile that has any adds up the counts of the groups before its own and
// of the tiles before it in its group by itself (a few hundred words that sit in L2).  A launch that only waits for
// the one before costs 4.5 us, and in mid-training almost no tile has new keys: with flags, counts, scan, assignment,
// row creation and the patching of pending occurrences in launches of their own they were a fifth of a step of 73 k
// keys.  (No spin-waits: they would need block tickets, and 8 ns per ticket is more than the launch.)

// Orders the LDS accesses of a wave's lanes with each other (a wave's LDS accesses are executed in order: only the
// compiler has to keep them so).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Over the pending occurrences of a rank tile's probe tiles: finds those that are the first occurrence of their
// (new) key, leaves them as a bitmap (written only where there are any) and their number.
// Bound by its chain of dependent loads (count, list, entry, slot), so a thread's chains run side by side.
// ITEMS = 1, the probe tiles of small batches (256 occurrences): a block per rank tile, a thread takes one entry of
// each of its 8 probe tiles.  ITEMS = 8, those of large ones (2048): a wave per rank tile and no block barrier - with
// a block each, 39 M occurrences are 19 k blocks, ten rounds of the chip.
template <int ITEMS>
__global__ void __launch_bounds__(BLOCK)
k_rank_count(DevHeader* hdr, const Slot* __restrict__ slots, const u32* __restrict__ occ_row,
             const u32* __restrict__ pend_list, const u32* __restrict__ tile_pending, u32 n_probe_tiles, u32 n_tiles,
             u32* __restrict__ first_bits, u32* __restrict__ tile_count, u32* __restrict__ group_count) {
  constexpr bool BY_WAVE = ITEMS != 1;
  constexpr u32 PROBE_TILE = BLOCK * ITEMS, PER = RANK_TILE / PROBE_TILE;
  __shared__ u32 lds[BY_WAVE ? BLOCK / WAVE : 1][RANK_WORDS];
  const u32 tile = BY_WAVE ? (blockIdx.x * BLOCK + threadIdx.x) / WAVE : blockIdx.x;
  u32* bits = lds[BY_WAVE ? wave_id() : 0];
  const u32 p0 = tile * RANK_TILE, live = hdr->live;
  u32 cnt[PER], any = 0;
#pragma unroll
  for (u32 t = 0; t < PER; ++t) cnt[t] = tile * PER + t < n_probe_tiles ? tile_pending[tile * PER + t] : 0u;
  requested();
  if (!live) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    hdr->pull_seen = hdr->pull_err;
    hdr->pull_err = 0;
  }
  if (tile >= n_tiles) return;  // uniform over the block or the wave
#pragma unroll
  for (u32 t = 0; t < PER; ++t) any |= cnt[t];
  if (any == 0) {
    if (threadIdx.x == 0 || (BY_WAVE && lane_id() == 0)) tile_count[tile] = 0;
    return;
  }
  // list entries at[i] of the tile's part of pend_list; those that are a first occurrence set their bit
  constexpr u32 CHAINS = BY_WAVE ? 4 : PER;
  const auto mark = [&](const u32 (&at)[CHAINS], const bool (&take)[CHAINS]) {
    u32 p[CHAINS], slot[CHAINS];
    bool first[CHAINS];
#pragma unroll
    for (u32 i = 0; i < CHAINS; ++i) p[i] = take[i] ? pend_list[p0 + at[i]] : p0;
#pragma unroll
    for (u32 i = 0; i < CHAINS; ++i) slot[i] = take[i] ? occ_row[p[i]] & ~OCC_PEND_FLAG : 0u;
#pragma unroll
    for (u32 i = 0; i < CHAINS; ++i) first[i] = take[i] && slots[slot[i]].first_p == p[i];
#pragma unroll
    for (u32 i = 0; i < CHAINS; ++i)
      if (first[i]) atomicOr(&bits[(p[i] - p0) >> 5], 1u << (p[i] & 31u));
  };
  u32 at[CHAINS];
  bool take[CHAINS];
  const u32 lane = (u32)lane_id();
  if constexpr (BY_WAVE) {
    bits[lane] = 0;
    wave_lds_fence();
    for (u32 i0 = lane; i0 - lane < cnt[0]; i0 += CHAINS * WAVE) {
#pragma unroll
      for (u32 i = 0; i < CHAINS; ++i) {
        at[i] = i0 + i * WAVE;
        take[i] = at[i] < cnt[0];
      }
      mark(at, take);
    }
    wave_lds_fence();
  } else {
    if (threadIdx.x < RANK_WORDS) bits[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (u32 i = 0; i < CHAINS; ++i) {
      at[i] = i * PROBE_TILE + threadIdx.x;
      take[i] = threadIdx.x < cnt[i];
    }
    mark(at, take);
    __syncthreads();
    if (threadIdx.x >= RANK_WORDS) return;
  }
  const u32 w = bits[lane];
  first_bits[tile * RANK_WORDS + lane] = w;
  const u32 total = wave_sum((u32)__popc(w));
  if (lane == 0) {
    tile_count[tile] = total;
    if (total) atomicAdd(&group_count[tile / RANK_GROUP * RANK_GROUP_STRIDE], total);
  }
}
static_assert(RANK_WORDS == WAVE, "a lane of one wave holds a word of a rank tile's bitmap");

// Writes columns 4 c .. 4 c + 3 of a new row's initial state, in every replica.
__device__ __forceinline__ void init_row(u32 row, u64 key, u32 c, float* values, u64 replica_stride, u32 n_replicas,
                                         float* vhat, u32 D, u32 rf, u64 seed_mul, float scale, float v0) {
  f4 x, z, e;
  x.x = init_value(seed_mul, key, 4 * c + 0, scale);
  x.y = init_value(seed_mul, key, 4 * c + 1, scale);
  x.z = init_value(seed_mul, key, 4 * c + 2, scale);
  x.w = init_value(seed_mul, key, 4 * c + 3, scale);
  z.x = z.y = z.z = z.w = 0.0f;
  e.x = e.y = e.z = e.w = v0;
  for (u32 j = 0; j < n_replicas; ++j) {
    float* b = values + j * replica_stride + (u64)row * rf + 4 * c;
    stg4(b, x);
    if (rf == 3 * D) {
      stg4(b + D, z);
      stg4(b + 2 * D, e);
    } else {
      stg4(b + D, e);
    }
  }
  if (vhat) stg4(vhat + (u64)row * D + 4 * c, e);
}

// Commits the pull or undoes it, and gives the first occurrence of every new key its row: the row id (rows in
// use + first occurrences before it), the key of the row and its initial state in every replica:
// x = init(key, d); first moment 0 (rows that have one); second moment / AdaGrad accumulator = v0 (eps per
// Algorithm 2's "Initialize", 0 for the bias-corrected form); shared denominator = v0.  When the pull failed
// (an error of the probe, or more rows than the table has), clearing exactly the slots claimed by this pull
// restores the index as it was.  rf = floats per row (3*D with a first moment, 2*D without); init_rows = 0: the
// caller writes the state of every row of the batch itself (a working-set load).
// A rank tile's new rows are dealt evenly to `parts` waves (rank_parts below), without block barriers: one wave per
// tile where the batch is large (a tile has a dozen new rows in mid-training, and what counts is how few rounds of
// the chip the tiles take), many where a small batch of unseen keys would otherwise write its rows from a few compute
// units.  (First pull of 4096 keys, 256 columns, 8 replicas: a block of 256 threads per tile 574 us for numbering and
// rows, so 33; 73 k keys of 64 columns 98 and 29.)
template <int LPR>
__global__ void __launch_bounds__(BLOCK)
k_rank_assign(DevHeader* hdr, Slot* slots, const u64* __restrict__ keys, u32* __restrict__ occ_row,
              const u32* __restrict__ first_bits, const u32* __restrict__ tile_count,
              const u32* __restrict__ group_count, u32 n_tiles, u32 parts, u64 capacity_rows,
              u64* __restrict__ row_key, u32 init_rows, float* values, u64 replica_stride, u32 n_replicas, float* vhat,
              u32 D, u32 rf, u64 seed_mul, float scale, float v0) {
  const u32 wave = (blockIdx.x * BLOCK + threadIdx.x) / WAVE, lane = (u32)lane_id();
  const u32 tile = wave / parts, part = wave % parts, live = hdr->live;
  const u32 in_tile = tile < n_tiles ? tile_count[tile] : 0u;
  requested();
  if (!live) return;
  if (in_tile == 0 && wave != 0) return;
  u32 before = 0, total = 0;  // first occurrences in the tiles before this one, in all tiles
  const u32 n_groups = (n_tiles + RANK_GROUP - 1) / RANK_GROUP, group = tile / RANK_GROUP;
  for (u32 t = lane; t < n_groups; t += WAVE) {
    const u32 c = group_count[t * RANK_GROUP_STRIDE];
    total += c;
    if (t < group) before += c;
  }
  for (u32 t = group * RANK_GROUP + lane; t < tile; t += WAVE) before += tile_count[t];
  before = wave_sum(before);
  total = wave_sum(total);
  const u32 base = hdr->n_rows_base;
  const u32 err = hdr->pull_seen | ((u64)base + total > capacity_rows ? ST_FULL : 0u);
  if (wave == 0 && lane == 0) {  // read by later launches only
    hdr->n_unique = 0;
    hdr->status = err;
    hdr->batch_ok = err ? 0u : 1u;
    hdr->n_new = err ? 0u : total;
    if (!err) hdr->n_rows = base + total;
  }
  // this wave's share: the tile's new rows first .. first + own, the occurrences of which it lists in LDS
  const u32 first = (u32)((u64)in_tile * part / parts), own = (u32)((u64)in_tile * (part + 1) / parts) - first;
  if (own == 0) return;
  __shared__ unsigned short lists[BLOCK / WAVE][RANK_TILE];
  unsigned short* list = lists[wave_id()];
  u32 word = first_bits[tile * RANK_WORDS + lane];
  for (u32 rank = wave_inclusive_scan((u32)__popc(word)) - (u32)__popc(word) - first; word; word &= word - 1, ++rank)
    if (rank < own) list[rank] = (unsigned short)(lane * 32u + (u32)__builtin_ctz(word));
  wave_lds_fence();
  const u32 row0 = base + before + first, p0 = tile * RANK_TILE;
#pragma unroll 4
  for (u32 i = lane; i < own; i += WAVE) {
    const u32 p = p0 + list[i];
    Slot* s = &slots[occ_row[p] & ~OCC_PEND_FLAG];
    if (err) {
      s->first_p = 0xFFFFFFFFu;
      s->key = KEY_EMPTY;
    } else {
      s->row = row0 + i;
      occ_row[p] = row0 + i;  // the first occurrence is resolved here, the others by whoever reads them next
      row_key[row0 + i] = keys[p];
    }
  }
  if (err || !init_rows) return;
  const u32 c = lane % LPR;
  if (c * 4 >= D) return;
#pragma unroll 2
  for (u32 i = lane / LPR; i < own; i += WAVE / LPR)
    init_row(row0 + i, keys[p0 + list[i]], c, values, replica_stride, n_replicas, vhat, D, rf, seed_mul, scale, v0);
}

// Large batches (probe tiles of 2048 occurrences): the initial state of the rows the pull created, in a launch of its
// own behind the numbering, 4.5 us of a step of milliseconds.  Rows are written grid-wide in ascending order, which
// keeps the stores of the whole chip in one window of the table, where a wave per rank tile writes one stream each:
// 39 M occurrences, 64 columns, 5.8 M new rows: numbering and rows 1545 us in one launch, 276 + 864 in two; 90 k new
// rows: 32 and 18 + 13.
template <int LPR>
__global__ void __launch_bounds__(BLOCK)
k_init_rows(const DevHeader* hdr, const u64* __restrict__ row_key, float* values, u64 replica_stride, u32 n_replicas,
            float* vhat, u32 D, u32 rf, u64 seed_mul, float scale, float v0) {
  if (hdr->status) return;
  const u32 n_new = hdr->n_new, row_base = hdr->n_rows_base, groups = gridDim.x * (BLOCK / LPR), c = threadIdx.x % LPR;
  if (c * 4 >= D) return;
  for (u32 i = (blockIdx.x * BLOCK + threadIdx.x) / LPR; i < n_new; i += groups)
    init_row(row_base + i, row_key[row_base + i], c, values, replica_stride, n_replicas, vhat, D, rf, seed_mul, scale, v0);
}

// Waves per rank tile of k_rank_assign: RANK_WAVES in all, half of what the chip holds at once, as long as a wave
// still has a few of the tile's rows if all of them are new.  (Waves of tiles without new rows end after one load.)
constexpr u32 RANK_WAVES = 4096, RANK_MAX_PARTS = 256;
inline u32 rank_parts(u32 n_tiles) {
  return n_tiles == 0 ? 1u : std::min(std::max(RANK_WAVES / n_tiles, 1u), RANK_MAX_PARTS);
}

// Row of an occurrence as the probe left it: a row id, or a slot whose row has been assigned since.
__device__ __forceinline__ u32 resolve_row(u32 entry, const Slot* __restrict__ slots) {
  return (entry & OCC_PEND_FLAG) ? slots[entry & ~OCC_PEND_FLAG].row : entry;
}

// ---------------------------------------------------------------- working-set load / collection

// After the keys of a working set have been looked up or inserted (occ_row[p] leads to the row of keys[p]):
// overwrites the state of those rows, in every replica, with the values supplied by the caller
// (the shared denominator, where there is one, is set to v).  m_src may be null for rows without
// a first moment.
template <int LPR>
__global__ void k_load_rows(const DevHeader* hdr, const u32* __restrict__ occ_row, const Slot* __restrict__ slots,
                            u32 n, float* values,
                            u64 replica_stride, u32 n_replicas, float* vhat, u32 D, u32 rf,
                            const float* __restrict__ x_src, const float* __restrict__ m_src,
                            const float* __restrict__ v_src) {
  if (hdr->status) return;
  const u64 p64 = ((u64)blockIdx.x * BLOCK + threadIdx.x) / LPR;  // n * LPR threads can pass 2^32
  const u32 c = threadIdx.x % LPR;
  if (p64 >= n || c * 4 >= D) return;
  const u32 p = (u32)p64;
  const u32 row = resolve_row(occ_row[p], slots);
  const f4 x = ldg4(x_src + (u64)p * D + 4 * c);
  const f4 v = ldg4(v_src + (u64)p * D + 4 * c);
  f4 m = {0.0f, 0.0f, 0.0f, 0.0f};
  if (rf == 3 * D) m = ldg4(m_src + (u64)p * D + 4 * c);
  for (u32 j = 0; j < n_replicas; ++j) {
    float* b = values + j * replica_stride + (u64)row * rf + 4 * c;
    stg4(b, x);
    if (rf == 3 * D) {
      stg4(b + D, m);
      stg4(b + 2 * D, v);
    } else {
      stg4(b + D, v);
    }
  }
  if (vhat) stg4(vhat + (u64)row * D + 4 * c, v);
}

// Lookup without insert for every occurrence of a batch (prediction): occ_row[p] = row of keys[p],
// or OCC_INVALID if the key is not in the table.  Checks keys and offsets like the training probe;
// what it finds goes to pull_err, which the pooling kernel folds into the status (k_lookup_commit, where there are
// no segments to pool).
__global__ void __launch_bounds__(BLOCK)
k_lookup(DevHeader* hdr, const Slot* __restrict__ slots, u32 slot_mask, const u64* __restrict__ keys, u32 n_keys,
         const u32* __restrict__ offsets, u32 n_seg, u32* __restrict__ occ_row) {
  const u32 p = blockIdx.x * BLOCK + threadIdx.x, status = hdr->status;
  const u32 a = p <= n_seg ? offsets[p] : 0u, b = p < n_seg ? offsets[p + 1] : n_keys;
  const u64 key = p < n_keys ? keys[p] : KEY_EMPTY;
  requested();
  if (status) return;
  if (p <= n_seg && ((p == 0 && a != 0) || (p == n_seg ? a != n_keys : b < a))) atomicOr(&hdr->pull_err, ST_INVAL);
  if (p >= n_keys) return;
  u32 out = OCC_INVALID;
  if (key == KEY_EMPTY) {
    atomicOr(&hdr->pull_err, ST_BADKEY);
  } else {
    u32 h = (u32)hash_key(key) & slot_mask;
    for (u32 probe = 0; probe <= slot_mask; ++probe) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&slots[h]);  // key and row id in one request
      const u64 k = ((u64)raw.y << 32) | raw.x;
      if (k == key) {
        out = raw.z;
        break;
      }
      if (k == KEY_EMPTY) break;
      h = (h + 1) & slot_mask;
    }
  }
  occ_row[p] = out;
}

// True if the table refuses calls or the lookup before this launch failed; the failure becomes the table's status.
// pull_err stays as it is beside a status: other blocks read it, and whatever clears the status clears both.
// (In a launch of its own this cost 4.5 us, a tenth of a prediction for 8 requests.)
__device__ __forceinline__ bool lookup_failed(DevHeader* hdr, u32 status, u32 err) {
  if (!status && err && blockIdx.x == 0 && threadIdx.x == 0) hdr->status = err;
  return status || err;
}

__global__ void k_lookup_commit(DevHeader* hdr) { (void)lookup_failed(hdr, hdr->status, hdr->pull_err); }

// Pure lookup (no insert) of n keys and copy of their rows of one replica to dense arrays; a key
// that is not in the table gets found = 0 and zeros.
// Bound by HBM: a row is read once and written once, so both sides carry the non-temporal hint, and a
// slot's key and row id come in one request (10.9 M keys of 64-wide rows, 16.7 GB: 3.89 -> 3.57 ms,
// 4.7 TB/s, the rate of a streaming copy; 16-wide rows, 8 x 2.7 M keys: 2.27 -> 2.07 ms).
template <int LPR>
__global__ void k_collect_rows(const DevHeader* hdr, const Slot* __restrict__ slots, u32 slot_mask,
                               const u64* __restrict__ keys, u32 n, const float* __restrict__ values, u32 D,
                               u32 rf, float* __restrict__ x_dst, float* __restrict__ m_dst,
                               float* __restrict__ v_dst, u32* __restrict__ found) {
  const u64 p64 = ((u64)blockIdx.x * BLOCK + threadIdx.x) / LPR;  // n * LPR threads can pass 2^32
  const u32 c = threadIdx.x % LPR, status = hdr->status;
  if (p64 >= n) return;
  const u32 p = (u32)p64;
  const u64 key = keys[p];
  requested();
  if (status) return;
  u32 row = ROW_PENDING;
  if (key != KEY_EMPTY) {
    u32 h = (u32)hash_key(key) & slot_mask;
    for (u32 probe = 0; probe <= slot_mask; ++probe) {  // every lane of the group walks the same slots
      const uint4 raw = *reinterpret_cast<const uint4*>(&slots[h]);  // key and row id in one request
      const u64 k = ((u64)raw.y << 32) | raw.x;
      if (k == key) {
        row = raw.z;
        break;
      }
      if (k == KEY_EMPTY) break;
      h = (h + 1) & slot_mask;
    }
  }
  const bool hit = row != ROW_PENDING;
  if (c == 0 && found) found[p] = hit ? 1u : 0u;
  if (c * 4 >= D) return;
  f4 x = {0.0f, 0.0f, 0.0f, 0.0f}, m = x, v = x;
  if (hit) {
    const float* b = values + (u64)row * rf + 4 * c;
    x = ldg4_stream(b);
    if (rf == 3 * D) {
      m = ldg4_stream(b + D);
      v = ldg4_stream(b + 2 * D);
    } else {
      v = ldg4_stream(b + D);
    }
  }
  if (x_dst) stg4_stream(x_dst + (u64)p * D + 4 * c, x);
  if (m_dst) stg4_stream(m_dst + (u64)p * D + 4 * c, m);
  if (v_dst) stg4_stream(v_dst + (u64)p * D + 4 * c, v);
}

// ---------------------------------------------------------------- gather + per-segment sum

// pooled[g, :] = sum over the segment's occurrences of x[row, :], in CSR order, binary32 inside a batch of 4
// consecutive occurrences and binary64 across batches, rounded once (error <= 3 * 2^-24 * sum |x|).  A row is
// rf floats and starts with x; a group of LPR lanes (a lane owns 4 consecutive columns) sums a segment.
// On the way a training pull records the segment of every occurrence (the push needs it) and replaces
// "slot, row assigned later" entries by the row (the sort reads them).  Two kernels:
//  * k_pool, for large batches, is bound by the rate of L2 requests (two 128-byte lines per gathered row), so
//    everything else is kept off that path: a block stages the boundaries and up to POOL_STAGED row ids of its
//    POOL_NS * POOL_ROUNDS segments per group in LDS with coalesced loads, and the segment ids leave coalesced (found
//    by binary search in the staged boundaries).  A group sums two segments at a time: up to 8 row loads in flight.
//    (With room for 6 ids per segment only, and broadcast loads in blocks that have more, 300000 segments of 32
//    columns: 8 ids each 42 us, now 33; 12 ids 55 and 42; 30 ids 121 and 79.)
//  * k_pool_small, for grids that leave the chip mostly idle, is bound by its chain of dependent loads: one
//    segment per group, no barrier, nothing staged (pool_segment).  16384 segments of 8 columns: 17.1 us with k_pool,
//    6.3 here; at 10 M segments of 64 columns the unstaged form costs 1.38 against 1.31 ms.
#ifndef CTR_POOL_NT_OUT
#define CTR_POOL_NT_OUT 1  // the pooled output (written once, read by the next stage) leaves with the non-temporal hint
#endif
constexpr u32 POOL_NS = 2;      // k_pool: segments a group works on at once
constexpr u32 POOL_ROUNDS = 2;  // such pairs per group
constexpr u32 POOL_MIN_BLOCKS = 1024;  // grids of k_pool below this go to k_pool_small
constexpr u32 POOL_STAGED = 4096;  // row ids a block of k_pool stages: 16 KB, with which eight blocks still fit a CU

// OUT: 1 = fp32 output, 2 = bf16 output, 3 = both; + 4 = lookup-only input, where an occurrence may have
// no row (compile-time, so the common fp32-only training kernel carries none of the other cases).
template <int OUT>
__device__ __forceinline__ void pool_store(u64 g, u32 D, u32 c, d4 acc, float* __restrict__ pooled,
                                           bf16_t* __restrict__ pooled_bf16) {
  const f4 o = {(float)acc.x, (float)acc.y, (float)acc.z, (float)acc.w};
  const u64 at = g * D + 4 * c;
#if CTR_POOL_NT_OUT
  if constexpr (OUT & 1) stg4_stream(pooled + at, o);
#else
  if constexpr (OUT & 1) stg4(pooled + at, o);
#endif
  if constexpr (OUT & 2) stg4_bf16(pooled_bf16 + at, o);  // the fp32 value, rounded again
}

// Adds a batch of 4 gathered rows to a segment's sum (padded entries add +0.0).
__device__ __forceinline__ void pool_add4(const f4 (&xv)[4], d4& acc) {
  f4 f = xv[0];
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    f.x += xv[i].x; f.y += xv[i].y; f.z += xv[i].z; f.w += xv[i].w;
  }
  acc.x += (double)f.x; acc.y += (double)f.y; acc.z += (double)f.z; acc.w += (double)f.w;
}

// Sum of one segment by its group of LPR lanes, the row ids straight from memory.  From 4 lanes on in windows of one id
// per lane: one coalesced load brings LPR ids, which shuffles hand out, where a broadcast load per occurrence would be
// a request each (30000 segments of 100 ids, 128 columns: 116 -> 96 us).  RESOLVE: entries whose row was assigned after the
// probe are replaced on the way, and the segment id is recorded for every occurrence.
template <int LPR, bool LOOKUP, bool RESOLVE>
__device__ __forceinline__ d4 pool_segment(u32 g, u32 beg, u32 end, u32* __restrict__ occ_row,
                                           const Slot* __restrict__ slots, u32* __restrict__ seg_of,
                                           const float* __restrict__ values, u32 D, u32 rf, u32 c) {
  const bool col_ok = c * 4 < D;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  // occurrences k .. k + 3, as far as they are the segment's; what `meanwhile` does comes behind the requests
  const auto add4 = [&](const u32 (&r)[4], u32 k, const auto& meanwhile) {
    f4 xv[4];
#pragma unroll
    for (u32 i = 0; i < 4; ++i) {
      xv[i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
      bool take = k + i < end && col_ok;
      if constexpr (LOOKUP) take = take && r[i] != OCC_INVALID;  // absent keys add nothing
      if (take) xv[i] = ldg4(values + (u64)r[i] * rf + 4 * c);
    }
    meanwhile();
    pool_add4(xv, acc);
  };
  if constexpr (LPR >= 4) {
    for (u32 k0 = beg; k0 < end; k0 += LPR) {
      const bool mine = k0 + c < end;
      u32 entry = mine ? occ_row[k0 + c] : 0u;
      if constexpr (RESOLVE) {
        if (entry & OCC_PEND_FLAG) occ_row[k0 + c] = entry = resolve_row(entry, slots);
      }
#pragma unroll 1
      for (u32 k = 0; k < LPR && k0 + k < end; k += 4) {
        u32 r[4];
#pragma unroll
        for (u32 i = 0; i < 4; ++i) r[i] = __shfl(entry, (int)(k + i), LPR);
        add4(r, k0 + k, [&]() {
          if constexpr (RESOLVE) {
            if (k == 0 && mine) seg_of[k0 + c] = g;
          }
        });
      }
    }
  } else {
    for (u32 k = beg; k < end; k += 4) {
      u32 r[4];
#pragma unroll
      for (u32 i = 0; i < 4; ++i) r[i] = k + i < end ? occ_row[k + i] : 0u;
      // All four are waited for here: the waits that the branches below would bring come where an address takes the register
      // of an id, for everything in flight, rows and stores of segment ids (20 segments of 200 ids: 8 columns 96.0 -> 52.6
      // us, 4 columns 50.2).
      asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
      if constexpr (RESOLVE) {
#pragma unroll
        for (u32 i = 0; i < 4; ++i)
          if (k + i < end && (r[i] & OCC_PEND_FLAG)) occ_row[k + i] = r[i] = resolve_row(r[i], slots);
      }
      add4(r, k, [&]() {
        if constexpr (RESOLVE) {
#pragma unroll
          for (u32 i = 0; i < 4; ++i)  // lane i % LPR writes entry i
            if (k + i < end && i % LPR == c) seg_of[k + i] = g;
        }
      });
    }
  }
  return acc;
}

// True for the blocks of a training pull's pooling launch that count digits instead (SortFirst).
__device__ __forceinline__ bool pool_takes_hist(const DevHeader* hdr, const u32* occ_row, const Slot* __restrict__ slots,
                                                const SortFirst& first, u32* lds) {
  if (first.n_pool_blocks == 0 || blockIdx.x < first.n_pool_blocks) return false;
  if (hdr->status) return true;
  // an entry is the same row before and after a pooling block has put the row in the place of its slot
  sort_first_hist(first, blockIdx.x - first.n_pool_blocks, occ_row, lds, [&](u32 entry) { return resolve_row(entry, slots); });
  return true;
}
static_assert(SORT_FIRST_WORDS <= POOL_STAGED, "the histograms fit where the pooling stages its row ids");

template <int LPR, int OUT>
__device__ __forceinline__ void pool_body(DevHeader* hdr, u32* occ_row,
                                          const Slot* __restrict__ slots, u32* __restrict__ seg_of,
                                          const u32* __restrict__ offsets, u32 n_seg,
                                          const float* __restrict__ values, u32 D, u32 rf,
                                          float* __restrict__ pooled, bf16_t* __restrict__ pooled_bf16,
                                          const SortFirst& first) {
  constexpr bool LOOKUP = (OUT & 4) != 0;
  constexpr u32 GROUPS = BLOCK / LPR;
  constexpr u32 TILE = GROUPS * POOL_NS * POOL_ROUNDS;
  __shared__ u32 off_lds[TILE + 1];
  __shared__ u32 row_lds[POOL_STAGED];
  if (!LOOKUP && pool_takes_hist(hdr, occ_row, slots, first, row_lds)) return;
  const u32 tile_g0 = blockIdx.x * TILE;
  const u32 tile_n = __builtin_amdgcn_readfirstlane(min(TILE, n_seg - tile_g0));
  // before requested(), behind which they are vector loads, one after the other, of a line that every wave of a large grid asks
  // for (lookup of 8.3 M segments of one id, 36 columns as bf16: 409 -> 381 us)
  const u32 status = hdr->status, err = LOOKUP ? hdr->pull_err : 0u;
  const u32 off0 = threadIdx.x <= tile_n ? offsets[tile_g0 + threadIdx.x] : 0u;
  requested();
  if (LOOKUP ? lookup_failed(hdr, status, err) : status != 0) return;
  if (threadIdx.x <= tile_n) off_lds[threadIdx.x] = off0;
  for (u32 i = threadIdx.x + BLOCK; i <= tile_n; i += BLOCK) off_lds[i] = offsets[tile_g0 + i];
  __syncthreads();

  const u32 P0 = __builtin_amdgcn_readfirstlane(off_lds[0]), P1 = __builtin_amdgcn_readfirstlane(off_lds[tile_n]);
  // A thread takes AHEAD occurrences at a time: requests them together, then the slots of those that are pending, then
  // searches their segments side by side.
  const auto stage = [&](auto ahead) {
    constexpr u32 AHEAD = decltype(ahead)::value;
    for (u32 p0 = P0 + threadIdx.x; p0 < P1; p0 += AHEAD * BLOCK) {
      u32 entry[AHEAD];
      bool pending[AHEAD];
#pragma unroll
      for (u32 i = 0; i < AHEAD; ++i) entry[i] = p0 + i * BLOCK < P1 ? occ_row[p0 + i * BLOCK] : 0u;
      if constexpr (!LOOKUP) {
#pragma unroll
        for (u32 i = 0; i < AHEAD; ++i) {
          pending[i] = (entry[i] & OCC_PEND_FLAG) != 0;
          entry[i] = resolve_row(entry[i], slots);
        }
      }
      u32 seg[AHEAD] = {};  // last l with off[l] <= p (skips empty segments)
      if constexpr (!LOOKUP) {
#pragma unroll
        for (u32 step = TILE / 2; step > 0; step >>= 1)
#pragma unroll
          for (u32 i = 0; i < AHEAD; ++i)
            if (seg[i] + step < tile_n && off_lds[seg[i] + step] <= p0 + i * BLOCK) seg[i] += step;
      }
#pragma unroll
      for (u32 i = 0; i < AHEAD; ++i) {
        const u32 p = p0 + i * BLOCK;
        if (p >= P1) break;
        if (p - P0 < POOL_STAGED) row_lds[p - P0] = entry[i];
        if constexpr (!LOOKUP) {
          if (pending[i]) occ_row[p] = entry[i];
          seg_of[p] = tile_g0 + seg[i];
        }
      }
    }
  };
  if (P1 - P0 <= BLOCK)  // uniform over the block
    stage(std::integral_constant<u32, 1>());
  else if (P1 - P0 <= 2 * BLOCK)
    stage(std::integral_constant<u32, 2>());
  else
    stage(std::integral_constant<u32, 4>());
  __syncthreads();

  const u32 grp = threadIdx.x / LPR, c = threadIdx.x % LPR;
  const bool col_ok = c * 4 < D;
  if (P1 - P0 > POOL_STAGED) {  // uniform over the block: segments much longer than usual
    for (u32 l = grp; l < tile_n; l += GROUPS) {
      const d4 acc = pool_segment<LPR, LOOKUP, false>(0u, off_lds[l], off_lds[l + 1], occ_row, slots, seg_of, values, D, rf, c);
      if (col_ok) pool_store<OUT>((u64)tile_g0 + l, D, c, acc, pooled, pooled_bf16);
    }
    return;
  }
#pragma unroll
  for (u32 rnd = 0; rnd < POOL_ROUNDS; ++rnd) {
    u32 beg[POOL_NS], end[POOL_NS];
    d4 acc[POOL_NS];
    u32 maxlen = 0;
#pragma unroll
    for (u32 s = 0; s < POOL_NS; ++s) {
      const u32 l = (rnd * POOL_NS + s) * GROUPS + grp;
      beg[s] = l < tile_n ? off_lds[l] : P0;
      end[s] = l < tile_n ? off_lds[l + 1] : P0;
      acc[s] = d4{0.0, 0.0, 0.0, 0.0};
      maxlen = max(maxlen, end[s] - beg[s]);
    }
    for (u32 k = 0; k < maxlen; k += 4) {
      u32 r[POOL_NS][4];  // all ids are read before the first row is requested
      f4 xv[POOL_NS][4];
#pragma unroll
      for (u32 s = 0; s < POOL_NS; ++s)
#pragma unroll
        for (u32 i = 0; i < 4; ++i) r[s][i] = row_lds[min(beg[s] + k + i, P1 - 1u) - P0];
#pragma unroll
      for (u32 s = 0; s < POOL_NS; ++s)
#pragma unroll
        for (u32 i = 0; i < 4; ++i) {
          xv[s][i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
          bool take = beg[s] + k + i < end[s] && col_ok;
          if constexpr (LOOKUP) take = take && r[s][i] != OCC_INVALID;  // absent keys add nothing
          if (take) xv[s][i] = ldg4(values + (u64)r[s][i] * rf + 4 * c);
        }
#pragma unroll
      for (u32 s = 0; s < POOL_NS; ++s) pool_add4(xv[s], acc[s]);
    }
#pragma unroll
    for (u32 s = 0; s < POOL_NS; ++s) {
      const u32 l = (rnd * POOL_NS + s) * GROUPS + grp;
      if (l < tile_n && col_ok) pool_store<OUT>((u64)tile_g0 + l, D, c, acc[s], pooled, pooled_bf16);
    }
  }
}

template <int LPR, int OUT>
__device__ __forceinline__ void pool_small_body(DevHeader* hdr, u32* __restrict__ occ_row,
                                                const Slot* __restrict__ slots, u32* __restrict__ seg_of,
                                                const u32* __restrict__ offsets, u32 n_seg,
                                                const float* __restrict__ values, u32 D, u32 rf,
                                                float* __restrict__ pooled, bf16_t* __restrict__ pooled_bf16,
                                                const SortFirst& first) {
  constexpr bool LOOKUP = (OUT & 4) != 0;
  if constexpr (!LOOKUP) {
    __shared__ u32 lds[SORT_FIRST_WORDS];
    if (pool_takes_hist(hdr, occ_row, slots, first, lds)) return;
  }
  const u32 g = (blockIdx.x * BLOCK + threadIdx.x) / LPR, c = threadIdx.x % LPR;
  const u32 status = hdr->status, err = LOOKUP ? hdr->pull_err : 0u;
  const u32 beg = g < n_seg ? offsets[g] : 0u, end = g < n_seg ? offsets[g + 1] : 0u;
  requested();
  if (LOOKUP ? lookup_failed(hdr, status, err) : status != 0) return;
  if (g >= n_seg) return;
  const d4 acc = pool_segment<LPR, LOOKUP, !LOOKUP>(g, beg, end, occ_row, slots, seg_of, values, D, rf, c);
  if (c * 4 < D) pool_store<OUT>(g, D, c, acc, pooled, pooled_bf16);
}

#define CTR_POOL_ARGS                                                                                       \
  DevHeader *hdr, u32 *__restrict__ occ_row, const Slot *__restrict__ slots, u32 *__restrict__ seg_of, \
      const u32 *__restrict__ offsets, u32 n_seg, const float *__restrict__ values, u32 D, u32 rf,          \
      float *__restrict__ pooled, bf16_t *__restrict__ pooled_bf16, SortFirst first
#define CTR_DEFINE_POOL(NAME, OUT)                                                                           \
  template <int LPR>                                                                                         \
  __global__ void __launch_bounds__(BLOCK) NAME(CTR_POOL_ARGS) {                                             \
    pool_body<LPR, OUT>(hdr, occ_row, slots, seg_of, offsets, n_seg, values, D, rf, pooled, pooled_bf16, first);    \
  }                                                                                                          \
  template <int LPR>                                                                                         \
  __global__ void __launch_bounds__(BLOCK) NAME##_small(CTR_POOL_ARGS) {                                     \
    pool_small_body<LPR, OUT>(hdr, occ_row, slots, seg_of, offsets, n_seg, values, D, rf, pooled, pooled_bf16, first); \
  }
CTR_DEFINE_POOL(k_pool, 1)
CTR_DEFINE_POOL(k_pool_bf16, 2)
CTR_DEFINE_POOL(k_pool_both, 3)
CTR_DEFINE_POOL(k_pool_lookup, 5)
CTR_DEFINE_POOL(k_pool_lookup_bf16, 6)
CTR_DEFINE_POOL(k_pool_lookup_both, 7)

}  // namespace ctr
