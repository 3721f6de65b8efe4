// bf16 x bf16 -> fp32 matrix product on the gfx950 matrix cores, hand-written for the dense tower.
//
// Paper: Algorithm 1's train_mini-batch step on the network of Section 2.1 - the three products of
// a fully connected layer (forward Z = H W, weight gradient dW = H^T dZ, input gradient
// dH = dZ W^T).  They are the only dense contractions of the training step.
//
// C[M x N] (row-major, N contiguous) = A[M x K] B[K x N].  Either operand may be stored with the
// contraction index contiguous ("k-contiguous": A as M rows of K, B as N rows of K) or with its
// other index contiguous (A as K rows of M, B as K rows of N); the three products of a row-major
// layer need three of the four combinations, and none of them needs a transposed copy in memory.
//
// Two kernels share the way operands travel.  The contraction runs in steps of 64.  An operand's tile of a step goes
// straight from memory to LDS (buffer loads with an LDS destination, 16 bytes per lane: no staging registers and no LDS
// write instructions), several steps ahead of its use; a wave waits for its own loads by count, the workgroup by a
// barrier.  A k-contiguous operand lies in LDS as rows of 64 k values and is read as the 16-byte fragments the matrix
// instruction takes; one with its other index contiguous lies as rows of that index, and the LDS transpose read
// (ds_read_b64_tr_b16) turns 4 k x 16 values into k-contiguous fragments on the way out.  The 16-byte chunks of a row are
// swizzled so that neither read has bank conflicts; the load's destination is linear in the lane, so it is the lane's
// source address that is permuted (inside a line of memory).
// k_gemm_large takes 256 x 256 tiles, k_gemm_tiles smaller ones for products that have few of those.
// A long contraction with few output tiles (the weight gradients) is split along K over several
// workgroups; each writes its fp32 partial tile, and a second launch adds the partials in a fixed
// order and applies the epilogue, so results do not depend on scheduling.  A result has the same bits whatever the tile:
// every element is the sum of its ranges' sums (gemm_sum_ranges), each accumulated along k by the same matrix instruction.
// All dimensions are multiples of 8 (16-byte vectors never straddle an edge).  Rows beyond the matrices are read from
// their first ones (they only feed elements of C that are never stored), k beyond a range as zeros.
#pragma once
#include <algorithm>
#include <cmath>

#include "common.h"

namespace ctr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr u32 GEMM_BM = 256, GEMM_BN = 256, GEMM_BK = 64;
constexpr u32 GEMM_GROUP_M = 8;  // tile rows walked together (operand reuse in L2)

// what happens to a finished element of C
enum GemmEpilogue : int {
  EPI_F32 = 0,             // C32[m, n] = acc
  EPI_BIAS_RELU_BF16 = 1,  // C16[m, n] = bf16(max(acc + bias[n], 0))       (forward: the next activation)
  EPI_BF16 = 2,            // C16[m, n] = bf16(acc)
  EPI_RELU_MASK_BF16 = 3,  // C16[m, n] = bf16(mask[m, n] > 0 ? acc : 0)    (input gradient through a ReLU)
  EPI_PARTIAL = 4,         // internal: partial[split][m][n] = acc (a split contraction)
  EPI_F32_STREAM = 5       // internal: EPI_F32 with the non-temporal hint
};

struct GemmArgs {
  const bf16_t* A;
  const bf16_t* B;
  u32 lda, ldb;  // elements between consecutive rows of the operand as stored
  u32 M, N, K;
  u32 n_split, k_per_split;  // K is cut into n_split ranges of k_per_split (a multiple of GEMM_BK)
  u32 k_per_sum;             // k_gemm_tiles: the length of the ranges whose sums are taken on their own
  u32 tiles_m, tiles_n;
  float* C32;
  bf16_t* C16;
  u32 ldc;
  const float* bias;   // EPI_BIAS_RELU_BF16
  const bf16_t* mask;  // EPI_RELU_MASK_BF16, laid out like C
  float* partial;      // n_split > 1: [n_split][M][N] fp32
  int epilogue;
};

// Epilogue on 4 consecutive columns of one row (n a multiple of 4; C, mask and partial rows are 16-byte
// aligned because every dimension is a multiple of 8).
__device__ __forceinline__ void gemm_emit4(const GemmArgs& g, int epilogue, u32 m, u32 n, f4 v, u32 split) {
  if (epilogue == EPI_PARTIAL) {
    stg4(g.partial + ((u64)split * g.M + m) * g.N + n, v);
    return;
  }
  const u64 i = (u64)m * g.ldc + n;
  if (epilogue == EPI_F32) {
    stg4(g.C32 + i, v);
  } else if (epilogue == EPI_F32_STREAM) {
    stg4_stream(g.C32 + i, v);
  } else if (epilogue == EPI_BIAS_RELU_BF16) {
    const f4 b = ldg4(g.bias + n);
    stg4_bf16(g.C16 + i, f4{fmaxf(v.x + b.x, 0.0f), fmaxf(v.y + b.y, 0.0f), fmaxf(v.z + b.z, 0.0f), fmaxf(v.w + b.w, 0.0f)});
  } else if (epilogue == EPI_BF16) {
    stg4_bf16(g.C16 + i, v);
  } else {
    const ushort4 a = *reinterpret_cast<const ushort4*>(g.mask + i);
    stg4_bf16(g.C16 + i, f4{from_bf16(a.x) > 0.0f ? v.x : 0.0f, from_bf16(a.y) > 0.0f ? v.y : 0.0f,
                             from_bf16(a.z) > 0.0f ? v.z : 0.0f, from_bf16(a.w) > 0.0f ? v.w : 0.0f});
  }
}

// ---------------------------------------------------------------- operand tiles

// What the loads of an operand may touch: its first byte and its size (below 4 GiB).  A lane whose offset is out of
// range brings zeros.
struct GemmBuffer {
  const bf16_t* p;
  u32 bytes;
};
constexpr u32 GEMM_NOWHERE = 0xFFFFFFF0u;  // out of range of every operand
// `lines` rows as stored, `in_line` elements of each are the operand's
__device__ __forceinline__ GemmBuffer gemm_buffer(const bf16_t* p, u32 ld, u32 lines, u32 in_line) {
  return {p, ((lines - 1u) * ld + in_line) * 2u};
}

#define CTR_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))

// 64 x 16 bytes from memory to 1 KB of LDS: lane i's, from byte lane_off + off of the operand, to dst + 16 i.
__device__ __forceinline__ void gemm_to_lds(const GemmBuffer& b, char* dst, u32 lane_off, u32 off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)b.p, 0, b.bytes, 0x00020000),
                                           CTR_LDS(void, dst), 16, lane_off, off, 0, 0);
}

// All but the last N of the wave's loads (and stores) are done; their data is in LDS.
template <int N>
__device__ __forceinline__ void gemm_wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// This wave's LDS reads are done: behind a barrier, others may overwrite what they read.
__device__ __forceinline__ void gemm_wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// The bare barrier: __syncthreads() would wait for every load in flight.
__device__ __forceinline__ void gemm_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The tile of R rows (of A; columns of B) x 64 k of an operand, carried by WAVES waves with N loads each.  A load brings
// 1 KB of the tile's LDS image: 8 rows of 64 k, or LINES k of R values.
// Swizzle: chunk c of a row lies at c ^ (row & 7) ^ (row / 8 & 1) (k-contiguous: 16 lanes, whom the 64 banks serve together,
// read one chunk of 16 rows, two rows to the banks; with row & 7 alone rows r and r + 8 met: 40 % of the LDS clocks of the
// 16384 x 1024 x 19200 product were conflicts, profiles/gemm_counters.txt); at c ^ 4 (k & 3) or, with rows of 128 bytes,
// c ^ 4 (k / 2 & 1) (otherwise: 32 lanes read 64 bytes of 4 consecutive k).
template <int R, bool KC, int WAVES>
struct GemmTile {
  static constexpr u32 N = R / 8 / WAVES, CHUNKS = KC ? 8 : R / 8, LINES = 64 / CHUNKS;
  static_assert(N % 2 == 0, "load j of every wave begins at a row whose (row / 8 & 1) is j's");
  u32 lane_off[KC ? 2 : 1];  // from the load's first byte to this lane's 16, of even and odd loads
  u32 line_bytes, row0, total, w;
  __device__ __forceinline__ GemmTile(u32 wave, u32 ld, u32 rows_total, u32 first_row)
      : line_bytes(2u * ld), row0(first_row), total(rows_total), w(wave) {
    const u32 lane = (u32)lane_id(), line = lane / CHUNKS, pos = lane % CHUNKS;
    if constexpr (KC) {
      lane_off[0] = line * line_bytes + (pos ^ line) * 16;
      lane_off[1] = line * line_bytes + (pos ^ line ^ 1u) * 16;
    } else {
      const u32 row = row0 + (pos ^ swizzle(line)) * 8;
      lane_off[0] = line * line_bytes + (row < total ? row : 0u) * 2u;
    }
  }
  static __device__ __forceinline__ u32 swizzle(u32 k) { return R == 64 ? (k >> 1 & 1u) << 2 : (k & 3u) << 2; }
  __device__ __forceinline__ u32 load_off(u32 j, u32 k0) const {
    if constexpr (KC) {
      const u32 row = row0 + (w * N + j) * 8;  // all 8 rows are the matrix's or none is
      return (row < total ? row : 0u) * line_bytes + k0 * 2;
    } else {
      return (k0 + (w * N + j) * LINES) * line_bytes;
    }
  }
  // requests k0 .. k0 + 63; INSIDE: all below k_end
  template <bool INSIDE>
  __device__ __forceinline__ void request(char* tile, const GemmBuffer& b, u32 k0, u32 k_end) const {
    char* dst = tile + w * N * 1024;
#pragma unroll
    for (u32 j = 0; j < N; ++j) {
      if constexpr (INSIDE) {
        gemm_to_lds(b, dst + j * 1024, lane_off[KC ? j & 1 : 0], load_off(j, k0));
      } else {
        const u32 lane = (u32)lane_id(), line = lane / CHUNKS;
        const u32 k = k0 + (KC ? ((lane % CHUNKS) ^ line ^ (j & 1u)) * 8 : (w * N + j) * LINES + line);
        gemm_to_lds(b, dst + j * 1024, (lane_off[KC ? j & 1 : 0] + load_off(j, k0)) | (k < k_end ? 0u : GEMM_NOWHERE), 0);
      }
    }
  }
  __device__ __forceinline__ void request(char* tile, const GemmBuffer& b, u32 k0, u32 k_end) const {
    if (k0 + GEMM_BK <= k_end)
      request<true>(tile, b, k0, k_end);
    else
      request<false>(tile, b, k0, k_end);
  }
  // the matrix instruction's fragment of rows row .. row + 31 (row a multiple of 32), k = 16 kk .. 16 kk + 15: lane l holds
  // row l % 32, 8 k from 8 (l / 32) on
  static __device__ __forceinline__ bf16x8 fragment(const char* tile, u32 row, u32 kk) {
    const u32 l = (u32)lane_id();
    if constexpr (KC) {
      return *reinterpret_cast<const bf16x8*>(tile + (row + (l & 31u)) * 128 + (((2 * kk) ^ ((l >> 5) ^ (l & 7u) ^ (l >> 3 & 1u))) << 4));
    } else {
      // 16 lanes take 4 k x 16 rows: lane 4 t + q addresses rows 4 q .. 4 q + 3 of k = t and receives row 4 t + q
      const u32 g = l >> 4, j = l & 15u, chunk = row / 8 + 2 * (g & 1u) + (j >> 1 & 1u);
      const char* p = tile + (16 * kk + 8 * (g >> 1) + (j >> 2)) * (2 * R) + ((chunk ^ swizzle(j >> 2)) << 4) + (j & 1u) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(CTR_LDS(s16x4, p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(CTR_LDS(s16x4, p + 4 * 2 * R));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

// Work item -> range of K and tile.  Workgroups are dealt to the 8 XCDs round-robin: ids are re-numbered so that one XCD
// gets a contiguous range, and tile rows are walked in groups so that the tiles an L2 sees at about the same time share
// their operand panels.
struct GemmItem {
  u32 m0, n0, split, k_begin, k_end;
  __device__ __forceinline__ GemmItem(const GemmArgs& g, u32 tile, u32 block) {
    const u32 tiles = g.tiles_m * g.tiles_n, total = tiles * g.n_split;
    u32 id = block;
    if (total % 8u == 0u) id = (block % 8u) * (total / 8u) + block / 8u;
    const u32 tid = id % tiles, group_size = GEMM_GROUP_M * g.tiles_n, first_m = (tid / group_size) * GEMM_GROUP_M;
    const u32 gm = min(GEMM_GROUP_M, g.tiles_m - first_m);
    m0 = __builtin_amdgcn_readfirstlane((first_m + (tid % group_size) % gm) * tile);
    n0 = __builtin_amdgcn_readfirstlane(((tid % group_size) / gm) * tile);
    split = id / tiles;
    k_begin = split * g.k_per_split;
    k_end = min(g.K, k_begin + g.k_per_split);
  }
};

// A 32 x 32 block of accumulators (register r of a lane is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32) to
// rows of `stride` floats in LDS.
__device__ __forceinline__ void gemm_block_to_lds(float* region, u32 stride, const f32x16& c, u32 lane) {
#pragma unroll
  for (u32 r = 0; r < 16; ++r) region[(8 * (r / 4) + 4 * (lane >> 5) + r % 4) * stride + (lane & 31u)] = c[r];
}
// Orders a wave's LDS accesses for the compiler (in hardware they are in order).
__device__ __forceinline__ void gemm_wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- tiles of 64 and 128

// T x T tiles, 4 waves (2 x WN, WN = 2) of T/2 x T/2 or 8 (WN = 4) of 64 x 32, a ring of S steps in LDS.  One barrier per step:
// it says that the step's tiles have landed for every wave and that the step before has been read by all, whose place
// the step S - 1 ahead is requested into.
// A work item that takes all ranges of its contraction folds each finished one into `sum`, one that takes a single range
// leaves it for k_gemm_reduce.
// A step of T = 128 takes 0.5 us on a CU that has one item, against 0.21 of matrix instructions; the arrival of its 32 KB alone
// takes 0.30 (45 bytes a clock into one CU's LDS), whatever is in flight: neither more steps in the ring nor fragments read a
// step ahead gain (both measured).  Two workgroups of T = 128 fit a CU with S = 2; where there is one at most per CU, its
// latency shows, and 8 waves with S = 4 are faster (4096 x 1024 x 3200: 40 -> 35 us; 16384 x 512 x 1024, two per CU: 28 with 8
// waves, 23 with 4).
// Through registers, with transposes of 8 x 8 blocks in them, these took (us -> now): 1000 x 400 x 624 8.4 -> 6.5;
// 4096 x 1024 x 3200 60 -> 35; 4096 x 512 x 1024 14.2 -> 10.3; 16384 x 512 x 1024 30 -> 23; 3200 x 1024 x 4096 64 -> 42;
// 8 x 1024 x 19200 17.5 -> 15.2.
// `rd` and `wr` are different steps of the ring (the restrict qualifiers say so: without them every fragment read would
// wait for all requests in flight).
template <int T, int WN, class TA, class TB>
__device__ __forceinline__ void gemm_tiles_step(const char* __restrict__ rd, char* __restrict__ wr, const TA& ta, const TB& tb,
                                                const GemmBuffer& ba, const GemmBuffer& bb, u32 k_next, u32 k_end, u32 wm,
                                                u32 wn, f32x16 (&acc)[T / 64][T / WN / 32]) {
  constexpr u32 FM = T / 64, FN = T / WN / 32;
  ta.request(wr, ba, k_next, k_end);
  tb.request(wr + T * 128, bb, k_next, k_end);
  bf16x8 a[4][FM], b[4][FN];
#pragma unroll
  for (u32 kk = 0; kk < 4; ++kk) {
#pragma unroll
    for (u32 i = 0; i < FM; ++i) a[kk][i] = TA::fragment(rd, wm * (T / 2) + i * 32, kk);
#pragma unroll
    for (u32 i = 0; i < FN; ++i) b[kk][i] = TB::fragment(rd + T * 128, wn * (T / WN) + i * 32, kk);
  }
#pragma unroll
  for (u32 kk = 0; kk < 4; ++kk)
#pragma unroll
    for (u32 mi = 0; mi < FM; ++mi)
#pragma unroll
      for (u32 ni = 0; ni < FN; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][mi], b[kk][ni], acc[mi][ni], 0, 0, 0);
}

template <int T, int S>
constexpr u32 gemm_tiles_lds() { return S * 2 * T * 128; }

template <int T, int WN, int S, bool A_KC, bool B_KC>
__device__ __forceinline__ void gemm_tiles_body(char* lds, u32 block, const bf16_t* __restrict__ Ap,
                                                const bf16_t* __restrict__ Bp, const GemmArgs& g) {
  constexpr int WAVES = 2 * WN;
  constexpr u32 FM = T / 64, FN = T / WN / 32, STEP = 2 * T * 128, RING = gemm_tiles_lds<T, S>();
  const GemmItem it(g, T, block);
  const u32 n_steps = (it.k_end - it.k_begin + GEMM_BK - 1) / GEMM_BK;  // the last one may reach beyond k_end
  const u32 w = (u32)__builtin_amdgcn_readfirstlane(wave_id()), lane = (u32)lane_id(), wm = w / WN, wn = w % WN;
  typedef GemmTile<T, A_KC, WAVES> TA;
  typedef GemmTile<T, B_KC, WAVES> TB;
  const TA ta(w, g.lda, g.M, it.m0);
  const TB tb(w, g.ldb, g.N, it.n0);
  const GemmBuffer ba = gemm_buffer(Ap, g.lda, A_KC ? g.M : g.K, A_KC ? g.K : g.M);
  const GemmBuffer bb = gemm_buffer(Bp, g.ldb, B_KC ? g.N : g.K, B_KC ? g.K : g.N);
#pragma unroll
  for (u32 s = 0; s + 1 < S; ++s) {
    ta.request(lds + s * STEP, ba, it.k_begin + s * GEMM_BK, it.k_end);
    tb.request(lds + s * STEP + T * 128, bb, it.k_begin + s * GEMM_BK, it.k_end);
  }
  f32x16 acc[FM][FN], sum[FM][FN];
#pragma unroll
  for (u32 mi = 0; mi < FM; ++mi)
#pragma unroll
    for (u32 ni = 0; ni < FN; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = sum[mi][ni][r] = 0.0f;
  const auto fold = [&]() {
#pragma unroll
    for (u32 mi = 0; mi < FM; ++mi)
#pragma unroll
      for (u32 ni = 0; ni < FN; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sum[mi][ni][r] += acc[mi][ni][r];
          acc[mi][ni][r] = 0.0f;
        }
  };
  u32 left = g.k_per_sum / GEMM_BK;  // steps until the range ends
  u32 rd = 0, wr = (S - 1) * STEP;
  for (u32 s = 0; s < n_steps; ++s) {
    gemm_wait_loads<(S - 2) * (TA::N + TB::N)>();  // steps behind the last one are requested, too: the count stays
    gemm_wait_reads();  // of the step before: its products have them already
    gemm_barrier();
    if (left == 0) {
      fold();
      left = g.k_per_sum / GEMM_BK;
    }
    --left;
    gemm_tiles_step<T, WN>(lds + rd, lds + wr, ta, tb, ba, bb, it.k_begin + (s + S - 1) * GEMM_BK, it.k_end, wm, wn, acc);
    wr = rd;
    rd = rd + STEP == RING ? 0 : rd + STEP;
  }
  fold();

  // sums to rows through LDS, each wave in its own region: nothing is in flight and everything has been read
  gemm_wait_loads<0>();
  __syncthreads();
  constexpr u32 ROWS = T / 2, COLS = T / WN, LANES = COLS / 4;  // lanes that read back one row
  static_assert(WAVES * ROWS * COLS * sizeof(float) <= RING, "a region for each wave");
  float* region = reinterpret_cast<float*>(lds) + w * (ROWS * COLS);
#pragma unroll
  for (u32 mi = 0; mi < FM; ++mi)
#pragma unroll
    for (u32 ni = 0; ni < FN; ++ni) gemm_block_to_lds(region + mi * 32 * COLS + ni * 32, COLS, sum[mi][ni], lane);
  gemm_wave_fence();
  const int epilogue = g.n_split > 1 ? (int)EPI_PARTIAL : g.epilogue;
  const u32 n = it.n0 + wn * COLS + (lane % LANES) * 4;
  for (u32 row = lane / LANES; row < ROWS; row += WAVE / LANES) {
    const u32 m = it.m0 + wm * ROWS + row;
    const f4 v = *reinterpret_cast<const f4*>(region + row * COLS + (lane % LANES) * 4);
    if (m < g.M && n < g.N) gemm_emit4(g, epilogue, m, n, v, it.split);
  }
}

template <int T, int WN, int S, bool A_KC, bool B_KC>
__global__ void __launch_bounds__(128 * WN, 2)
k_gemm_tiles(const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Bp, GemmArgs g) {
  __shared__ __align__(16) char lds[gemm_tiles_lds<T, S>()];
  gemm_tiles_body<T, WN, S, A_KC, B_KC>(lds, blockIdx.x, Ap, Bp, g);
}

// ---------------------------------------------------------------- tiles of 256

// 8 waves (2 x 4), two per SIMD, one workgroup per CU.  A step's tiles are four units of 128 rows x 64 k (A0 A1 B0 B1, 16 KB
// each), two steps fit beside each other.  A wave's share of C is 64 x 32 of each of the four quadrants A_i B_j (128
// accumulator registers), and a step is four phases of one quadrant each:
//   phase   reads the fragments of   multiplies   requests (into the place of the unit read two phases before)
//     0     B0                       A0 B0        A1 of the next step
//     1     B1                       A0 B1        A0 of the step after that
//     2     A1                       A1 B1        B0
//     3     A0 of the next step      A1 B0        B1
// so every unit is requested six phases before it is read: 12 loads of a wave in flight, no LDS beyond the two steps.
// A phase has two halves, reads and requests | products, with a barrier behind each, and waves 4..7 run one half behind
// waves 0..3: on every SIMD one wave multiplies while the other reads.  The barriers carry all the order there is:
//   * a unit read in phase p + 1 was waited for (by count: 5 units may be in flight) by every wave in its first half of
//     phase p, and a barrier lies between;
//   * a unit's place is overwritten by requests of phase p + 2 at the earliest, and every wave waits for its reads of phase p
//     at the end of that phase.
// The forward product keeps the matrix cores busy 88 % of its clocks, at the 1.5 GHz that the chip's power leaves them
// (counters: profiles/gemm_counters.txt), the weight gradient 69 % (300 tiles in 4 ranges are 4.7 rounds of the chip, and their
// partial sums are stored), the input gradient 56 % (16 steps per tile: its first requests and stores).
// With 4 waves of 128 x 128, operands through registers and one step in flight
// the products of a layer of 19200 x 1024 and 16384 samples took (us -> now) 752 -> 460 forward (1.40 PFLOP/s), 930 -> 600
// weight gradient, 790 -> 605 input gradient (event pairs; 1.26 GB of fp32 leave: with the non-temporal hint, 690 without, 540 if
// nothing is stored).  Workgroups that walk several tiles and request the next one's units before they store: no gain.
constexpr u32 LARGE_UNIT = 128 * 128, LARGE_STEP = 4 * LARGE_UNIT;
constexpr u32 LARGE_A0 = 0, LARGE_A1 = LARGE_UNIT, LARGE_B0 = 2 * LARGE_UNIT, LARGE_B1 = 3 * LARGE_UNIT;
constexpr u32 LARGE_BLOCK = 512;

template <bool A_KC, bool B_KC>
struct LargeWork {
  typedef GemmTile<128, A_KC, 8> TA;
  typedef GemmTile<128, B_KC, 8> TB;
  TA a0, a1;
  TB b0, b1;
  GemmBuffer ba, bb;
  u32 k_end, wm, wn;
  bf16x8 fa0[4][2], fa1[4][2], fb0[4], fb1[4];
  f32x16 c[2][2][2];  // quadrant i, j: 2 blocks of 32 x 32
};

// `rd` is the unit read, `wr` the one requested, never the same (see gemm_tiles_step); k0: this step's first k.
template <int PHASE, bool INSIDE, bool A_KC, bool B_KC>
__device__ __forceinline__ void large_read_request(const char* __restrict__ rd, char* __restrict__ wr, LargeWork<A_KC, B_KC>& t,
                                                   u32 k0) {
  typedef LargeWork<A_KC, B_KC> W;
#pragma unroll
  for (u32 kk = 0; kk < 4; ++kk) {
    if constexpr (PHASE == 0) t.fb0[kk] = W::TB::fragment(rd, t.wn * 32, kk);
    if constexpr (PHASE == 1) t.fb1[kk] = W::TB::fragment(rd, t.wn * 32, kk);
#pragma unroll
    for (u32 i = 0; i < 2; ++i) {
      if constexpr (PHASE == 2) t.fa1[kk][i] = W::TA::fragment(rd, t.wm * 64 + i * 32, kk);
      if constexpr (PHASE == 3) t.fa0[kk][i] = W::TA::fragment(rd, t.wm * 64 + i * 32, kk);
    }
  }
  if constexpr (PHASE == 0) t.a1.template request<INSIDE>(wr, t.ba, k0 + GEMM_BK, t.k_end);
  if constexpr (PHASE == 1) t.a0.template request<INSIDE>(wr, t.ba, k0 + 2 * GEMM_BK, t.k_end);
  if constexpr (PHASE == 2) t.b0.template request<INSIDE>(wr, t.bb, k0 + 2 * GEMM_BK, t.k_end);
  if constexpr (PHASE == 3) t.b1.template request<INSIDE>(wr, t.bb, k0 + 2 * GEMM_BK, t.k_end);
}

template <int PHASE, bool INSIDE, bool A_KC, bool B_KC>
__device__ __forceinline__ void large_phase(char* lds, u32 buf, LargeWork<A_KC, B_KC>& t, u32 k0) {
  constexpr u32 RD = PHASE == 0 ? LARGE_B0 : PHASE == 1 ? LARGE_B1 : PHASE == 2 ? LARGE_A1 : LARGE_A0;
  constexpr u32 WR = PHASE == 0 ? LARGE_A1 : PHASE == 1 ? LARGE_A0 : PHASE == 2 ? LARGE_B0 : LARGE_B1;
  large_read_request<PHASE, INSIDE>(lds + (PHASE == 3 ? buf ^ LARGE_STEP : buf) + RD,
                                    lds + (PHASE == 0 ? buf ^ LARGE_STEP : buf) + WR, t, k0);
  gemm_wait_loads<10>();
  gemm_barrier();
  __builtin_amdgcn_s_setprio(1);
  const bf16x8(&fa)[4][2] = PHASE < 2 ? t.fa0 : t.fa1;
  const bf16x8(&fb)[4] = (PHASE == 0 || PHASE == 3) ? t.fb0 : t.fb1;
  f32x16(&c)[2] = t.c[PHASE / 2][(PHASE == 0 || PHASE == 3) ? 0 : 1];
#pragma unroll
  for (u32 kk = 0; kk < 4; ++kk)
#pragma unroll
    for (u32 i = 0; i < 2; ++i) c[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i], fb[kk], c[i], 0, 0, 0);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
  gemm_wait_reads();
  gemm_barrier();
}

template <bool INSIDE, bool A_KC, bool B_KC>
__device__ __forceinline__ void large_step(char* lds, u32 buf, LargeWork<A_KC, B_KC>& t, u32 k0) {
  large_phase<0, INSIDE>(lds, buf, t, k0);
  large_phase<1, INSIDE>(lds, buf, t, k0);
  large_phase<2, INSIDE>(lds, buf, t, k0);
  large_phase<3, INSIDE>(lds, buf, t, k0);
}

template <bool A_KC, bool B_KC>
__global__ void __launch_bounds__(LARGE_BLOCK, 2)
k_gemm_large(const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Bp, GemmArgs g) {
  __shared__ __align__(16) char lds[2 * LARGE_STEP + 8 * 4096];  // two steps; a 32 x 32 block of C for each wave
  const GemmItem it(g, 256, blockIdx.x);
  const u32 n_steps = (it.k_end - it.k_begin + GEMM_BK - 1) / GEMM_BK, n_full = (it.k_end - it.k_begin) / GEMM_BK;
  const u32 w = (u32)__builtin_amdgcn_readfirstlane(wave_id());
  LargeWork<A_KC, B_KC> t{{w, g.lda, g.M, it.m0}, {w, g.lda, g.M, it.m0 + 128}, {w, g.ldb, g.N, it.n0},
                          {w, g.ldb, g.N, it.n0 + 128},
                          gemm_buffer(Ap, g.lda, A_KC ? g.M : g.K, A_KC ? g.K : g.M),
                          gemm_buffer(Bp, g.ldb, B_KC ? g.N : g.K, B_KC ? g.K : g.N), it.k_end, w >> 2, w & 3u};
  // in the order in which they are read: two loads each
  t.a0.request(lds + LARGE_A0, t.ba, it.k_begin, it.k_end);
  t.b0.request(lds + LARGE_B0, t.bb, it.k_begin, it.k_end);
  t.b1.request(lds + LARGE_B1, t.bb, it.k_begin, it.k_end);
  t.a1.request(lds + LARGE_A1, t.ba, it.k_begin, it.k_end);
  t.a0.request(lds + LARGE_STEP + LARGE_A0, t.ba, it.k_begin + GEMM_BK, it.k_end);
  t.b0.request(lds + LARGE_STEP + LARGE_B0, t.bb, it.k_begin + GEMM_BK, it.k_end);
  t.b1.request(lds + LARGE_STEP + LARGE_B1, t.bb, it.k_begin + GEMM_BK, it.k_end);
#pragma unroll
  for (u32 q = 0; q < 8; ++q)
#pragma unroll
    for (u32 r = 0; r < 16; ++r) t.c[q >> 2][q >> 1 & 1][q & 1][r] = 0.0f;
  gemm_wait_loads<10>();
  gemm_barrier();
#pragma unroll
  for (u32 kk = 0; kk < 4; ++kk)
#pragma unroll
    for (u32 i = 0; i < 2; ++i)
      t.fa0[kk][i] = LargeWork<A_KC, B_KC>::TA::fragment((const char*)lds + LARGE_A0, t.wm * 64 + i * 32, kk);
  gemm_wait_reads();
  if (w >= 4) gemm_barrier();  // half a phase behind from here on
  u32 buf = 0, s = 0;
  for (; s + 2 < n_full; ++s, buf ^= LARGE_STEP) large_step<true>(lds, buf, t, it.k_begin + s * GEMM_BK);
#pragma unroll 1
  for (; s < n_steps; ++s, buf ^= LARGE_STEP) large_step<false>(lds, buf, t, it.k_begin + s * GEMM_BK);
  if (w < 4) gemm_barrier();
  gemm_wait_loads<0>();  // requests beyond the last step

  const int epilogue = g.n_split > 1 ? (int)EPI_PARTIAL : g.epilogue;
  float* region = reinterpret_cast<float*>(lds + 2 * LARGE_STEP) + w * 1024;
  u32 l = (u32)lane_id();
  asm volatile("" : "+v"(l));  // so that the stores' addresses are not kept in registers through the loop
#pragma unroll
  for (u32 q = 0; q < 8; ++q) {
    const u32 i = q >> 2, block = q >> 1 & 1, j = q & 1;  // the two halves of 128 columns after each other
    gemm_block_to_lds(region, 32, t.c[i][j][block], l);
    gemm_wave_fence();
    const u32 m = it.m0 + i * 128 + t.wm * 64 + block * 32 + (l >> 3), n = it.n0 + j * 128 + t.wn * 32 + (l & 7u) * 4;
#pragma unroll
    for (u32 r = 0; r < 32; r += 8) {
      const f4 v = *reinterpret_cast<const f4*>(region + (r + (l >> 3)) * 32 + (l & 7u) * 4);
      if (m + r < g.M && n < g.N) gemm_emit4(g, epilogue, m + r, n, v, it.split);
    }
    gemm_wave_fence();
  }
}

// Second launch of a split product: adds the partial tiles in the order of the splits and applies the epilogue.
// SIDE partials are requested together behind the first: 8 where the chip is full of threads, which then wait for memory, all 31
// of a small product, which waits for its chain of requests (8 x 1024 outputs, 30 partials: 4.5 -> 4.3 us by the kernel's own
// clock, a prediction of 8 requests with such products 37.5 -> 36.0), unless 8 are all there are (8 x 1024 x 2160, 9 partials,
// both launches: 6.6 us with 8, 7.4 with 32; 10 partials 7.35 and 7.4; 20 9.2 and 8.3).
constexpr u32 GEMM_REDUCE_FEW = 64 * 1024;  // threads
template <u32 SIDE>
__global__ void __launch_bounds__(BLOCK) k_gemm_reduce(GemmArgs g) {
  const u64 i4 = ((u64)blockIdx.x * BLOCK + threadIdx.x) * 4;  // 4 consecutive columns of one row
  const u64 mn = (u64)g.M * g.N;
  if (i4 >= mn) return;
  f4 s = ldg4(g.partial + i4);
  for (u32 sp = 1; sp < g.n_split; sp += SIDE) {
    f4 p[SIDE];
#pragma unroll
    for (u32 j = 0; j < SIDE; ++j) p[j] = ldg4(g.partial + min(sp + j, g.n_split - 1u) * mn + i4);
#pragma unroll
    for (u32 j = 0; j < SIDE; ++j)
      if (sp + j < g.n_split) {
        s.x += p[j].x; s.y += p[j].y; s.z += p[j].z; s.w += p[j].w;
      }
  }
  gemm_emit4(g, g.epilogue, (u32)(i4 / g.N), (u32)(i4 % g.N), s, 0);
}

// ---------------------------------------------------------------- host side

// The ranges of K whose sums are taken on their own and then added in order: a property of the product's size, so
// that its result does not depend on how it is executed.  The cut is the one that minimises (rounds of 256
// workgroups with 256 x 256 tiles) x (contraction steps per work item + a fixed cost per item) + the cost of adding
// the partials, within the scratch there is for them.  The ranges decide the bits of a result, so the prices here stay those of
// the kernels that they were first made for (3 us per step of a tile; GEMM_TILE_COSTS has what a step takes now).
struct GemmRanges {
  u32 n, length;  // length: a multiple of GEMM_BK
};

inline GemmRanges gemm_sum_ranges(u32 M, u32 N, u32 K, size_t partial_capacity) {
  const double tiles = (double)((M + GEMM_BM - 1) / GEMM_BM) * ((N + GEMM_BN - 1) / GEMM_BN), cus = 256.0;
  const u32 k_steps = (K + GEMM_BK - 1) / GEMM_BK;
  double best = 0.0;
  u32 n = 1;
  for (u32 s = 1; s <= 32 && s <= k_steps; ++s) {
    const u32 steps_per = (k_steps + s - 1) / s;
    if (s > 1 && steps_per < 4) break;
    const size_t need = s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
    if (need > partial_capacity) break;
    const double rounds = (double)(u64)((tiles * s + cus - 1) / cus);
    // unit: one contraction step of one tile (then 3 us); fixed cost per item ~2 steps; the partials move
    // (s + 1) x M x N x 4 bytes at ~4 TB/s
    const double cost = rounds * (steps_per + 2.0) + (s > 1 ? (s + 1.0) * M * N * 4.0 / 4e12 / 3e-6 : 0.0);
    if (s == 1 || cost < best) {
      best = cost;
      n = s;
    }
  }
  const u32 steps_per = (k_steps + n - 1) / n;
  return {(k_steps + steps_per - 1) / steps_per, steps_per * GEMM_BK};  // no empty range at the end
}

// How a product is cut into work items: the tile, and whether an item takes one range of the contraction or all.
struct GemmPlan {
  u32 tile, tiles_m, tiles_n, n_split, k_per_split, k_per_sum;
  double cost;  // estimated time, us
};

// Times the plan is made from, in us, fitted to sweeps over tile and split of the products of towers at batches of 8 to
// 16384 (profiles/gemm_tiles.txt, which ctr_debug_mlp_gemm can measure again).  A step of a large tile is 1.5 us whatever
// the others do.  Smaller tiles share a CU: a step of T = 128 takes 0.62 us with 8 waves while every CU has one item at most,
// 0.8 with two on a few CUs and 1.1 with two on all of them, where the L2s feed the tiles.
// An item of T = 64 behind another costs its stores even where the contraction has a step or two: 1.5 us (priced at 1.0, outputs
// of 35 MB took that tile: 14584 x 600 x 8 16.6 us, 14.3 with T = 128).  A split product's second launch is 2.4 us (priced at 3.2,
// contractions of 13 to 16 steps stayed whole: 176 x 24 x 848 7.7 us, 6.7 split).  Over the 972 products of 160 random towers what
// is taken is 0.3 % behind the fastest, 9 of them by more than 10 % (with the former two prices 0.7 %, 36).
constexpr u32 GEMM_CUS = 256;
constexpr double GEMM_SECOND_LAUNCH = 2.4;
struct GemmTileCost {
  u32 tile, per_cu;              // work items a CU takes at once
  double fixed;                  // launch, first requests and epilogue of a work item
  double step_few;               // a contraction step where no CU has two items
  double step1, step_two, step2; // ... of the last round: one item per CU at most, two on some, two on all
  double next;                   // an item that follows another one
};
constexpr GemmTileCost GEMM_TILE_COSTS[3] = {
    {256, 1, 8.0, 1.5, 1.5, 1.5, 1.5, 9.0},
    {128, 2, 5.0, 0.62, 0.72, 0.8, 1.1, 3.0},
    {64, 2, 3.4, 0.28, 0.28, 0.45, 0.45, 1.5},
};
// fp32 outputs from here on (the last-level cache's size) are stored with the non-temporal hint: 1.26 GB 690 -> 605 us; 52 MB
// 33.1 and 32.4, but there the next kernel still finds them.
constexpr u64 GEMM_STREAM_BYTES = 256ull << 20;

inline GemmPlan gemm_plan_one(const GemmTileCost& c, bool split, const GemmRanges& ranges, u32 M, u32 N, u32 K) {
  GemmPlan p;
  p.tile = c.tile;
  p.tiles_m = (M + c.tile - 1) / c.tile;
  p.tiles_n = (N + c.tile - 1) / c.tile;
  p.n_split = split ? ranges.n : 1;
  p.k_per_sum = ranges.length;
  p.k_per_split = split ? ranges.length : ranges.length * ranges.n;
  const u64 items = (u64)p.tiles_m * p.tiles_n * p.n_split, per_round = (u64)GEMM_CUS * c.per_cu;
  const u64 full = items / per_round, rest = items % per_round;
  const u32 steps = (std::min(K, p.k_per_split) + GEMM_BK - 1) / GEMM_BK;
  const double both = rest > GEMM_CUS ? (double)(rest - GEMM_CUS) / GEMM_CUS : 0.0;  // share of the CUs with two items
  const double rest_step = rest == 0 ? 0.0 : rest > GEMM_CUS ? c.step_two + both * (c.step2 - c.step_two) : full ? c.step1 : c.step_few;
  p.cost = c.fixed + steps * (full * c.step2 + rest_step) + (full + (rest ? 1 : 0) - 1.0) * c.next;
  if (p.n_split > 1) p.cost += GEMM_SECOND_LAUNCH + (p.n_split + 1.0) * M * N * 4.0 / 5e6;  // the partials move at about 5 TB/s
  return p;
}

inline GemmPlan gemm_plan(u32 M, u32 N, u32 K, size_t partial_capacity) {
  const GemmRanges ranges = gemm_sum_ranges(M, N, K, partial_capacity);
  GemmPlan best = gemm_plan_one(GEMM_TILE_COSTS[0], true, ranges, M, N, K);
  for (int i = 1; i < 3; ++i)
    for (bool split : {false, true}) {
      const GemmPlan p = gemm_plan_one(GEMM_TILE_COSTS[i], split, ranges, M, N, K);
      if (p.cost < best.cost) best = p;
    }
  return best;
}

// Two products in one launch of tiles of 64, the second unsplit: estimated time, us, and the first one's plan.  A product
// that leaves the chip idle costs its chain of steps, whatever runs beside it.
inline double gemm_pair_plan(u32 M1, u32 N1, u32 K1, u32 M2, u32 N2, u32 K2, size_t partial_capacity, GemmPlan* first,
                             GemmPlan* second) {
  const GemmTileCost& c = GEMM_TILE_COSTS[2];
  const GemmRanges r1 = gemm_sum_ranges(M1, N1, K1, partial_capacity), r2 = gemm_sum_ranges(M2, N2, K2, partial_capacity);
  *second = gemm_plan_one(c, false, r2, M2, N2, K2);
  double best = 0.0;
  for (bool split : {false, true}) {
    if (split && r1.n == 1) break;
    const GemmPlan p = gemm_plan_one(c, split, r1, M1, N1, K1);
    const double items1 = (double)p.tiles_m * p.tiles_n * p.n_split, items2 = (double)second->tiles_m * second->tiles_n;
    const double steps1 = (std::min(K1, p.k_per_split) + GEMM_BK - 1) / GEMM_BK, steps2 = (K2 + GEMM_BK - 1) / GEMM_BK;
    const double at_once = (double)GEMM_CUS * c.per_cu, more = std::max(0.0, std::ceil((items1 + items2) / at_once) - 1.0);
    const double work = (items1 * steps1 + items2 * steps2) / at_once * c.step2 + more * c.next;
    const double cost = c.fixed + std::max(std::max(steps1, steps2) * c.step_few, work) +
                        (split ? (p.n_split + 1.0) * M1 * N1 * 4.0 / 5e6 : 0.0);
    if (!split || cost < best) {
      best = cost;
      *first = p;
    }
  }
  return best;
}

// The plan with the given tile (64, 128 or 256) and with one work item per range of the contraction or one for all;
// false if there is no such kernel (the large tile takes one range per item).
inline bool gemm_plan_forced(u32 M, u32 N, u32 K, size_t partial_capacity, u32 tile, bool split, GemmPlan* p) {
  const GemmRanges ranges = gemm_sum_ranges(M, N, K, partial_capacity);
  for (const GemmTileCost& c : GEMM_TILE_COSTS)
    if (c.tile == tile && (tile != 256 || split || ranges.n == 1)) {
      *p = gemm_plan_one(c, split, ranges, M, N, K);
      return true;
    }
  return false;
}

inline void gemm_set_plan(GemmArgs& g, const GemmPlan& p, float* partial) {
  g.tiles_m = p.tiles_m;
  g.tiles_n = p.tiles_n;
  g.n_split = p.n_split;
  g.k_per_split = p.k_per_split;
  g.k_per_sum = p.k_per_sum;
  g.partial = partial;
}

// Enqueues C = A B as planned (operands, sizes, outputs and epilogue fields of `g` filled in by the caller).
// keep_partial: the sums of a split product are left in `partial`, [range][m][n], for a later launch to add.
inline hipError_t gemm_launch(bool a_kc, bool b_kc, GemmArgs g, const GemmPlan& p, float* partial, bool keep_partial,
                              hipStream_t st) {
  gemm_set_plan(g, p, partial);
  // an output that no cache holds leaves without displacing the operands
  if (g.epilogue == EPI_F32 && (u64)g.M * g.N * sizeof(float) >= GEMM_STREAM_BYTES) g.epilogue = EPI_F32_STREAM;
  const u32 grid = p.tiles_m * p.tiles_n * p.n_split;
  const int layout = (a_kc ? 2 : 0) | (b_kc ? 1 : 0);
#define CTR_GEMM_LAUNCH(KERNEL, THREADS, ...)                                                                               \
  switch (layout) {                                                                                                        \
    case 3: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ true, true>), dim3(grid), dim3(THREADS), 0, st, g.A, g.B, g); break;    \
    case 2: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ true, false>), dim3(grid), dim3(THREADS), 0, st, g.A, g.B, g); break;   \
    case 1: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ false, true>), dim3(grid), dim3(THREADS), 0, st, g.A, g.B, g); break;   \
    default: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ false, false>), dim3(grid), dim3(THREADS), 0, st, g.A, g.B, g); break; \
  }
#define CTR_GEMM_PARAMS(...) __VA_ARGS__,
  if (p.tile == 256) {
    CTR_GEMM_LAUNCH(k_gemm_large, LARGE_BLOCK, )
  } else if (p.tile == 128 && grid <= GEMM_CUS) {
    CTR_GEMM_LAUNCH(k_gemm_tiles, 512, CTR_GEMM_PARAMS(128, 4, 4))
  } else if (p.tile == 128) {
    CTR_GEMM_LAUNCH(k_gemm_tiles, 256, CTR_GEMM_PARAMS(128, 2, 2))
  } else {
    CTR_GEMM_LAUNCH(k_gemm_tiles, 256, CTR_GEMM_PARAMS(64, 2, 4))
  }
#undef CTR_GEMM_LAUNCH
#undef CTR_GEMM_PARAMS
  if (g.n_split > 1 && !keep_partial) {
    const u64 mn = (u64)g.M * g.N;
    const dim3 blocks((u32)((mn / 4 + BLOCK - 1) / BLOCK));
    if (mn / 4 <= GEMM_REDUCE_FEW && g.n_split > 9)
      hipLaunchKernelGGL(k_gemm_reduce<32>, blocks, dim3(BLOCK), 0, st, g);
    else
      hipLaunchKernelGGL(k_gemm_reduce<8>, blocks, dim3(BLOCK), 0, st, g);
  }
  return hipGetLastError();
}

inline bool gemm_args_ok(bool a_kc, bool b_kc, const GemmArgs& g) {
  if (g.M == 0 || g.N == 0 || g.K == 0) return false;
  if ((g.M | g.N | g.K | g.lda | g.ldb) % 8u != 0u) return false;
  // lanes address an operand with 32-bit byte offsets
  const u64 a_bytes = 2ull * g.lda * (a_kc ? g.M : g.K), b_bytes = 2ull * g.ldb * (b_kc ? g.N : g.K);
  return a_bytes < (1ull << 32) && b_bytes < (1ull << 32);
}

// partial: fp32 scratch of partial_capacity bytes for split products.
inline hipError_t gemm_enqueue(bool a_kc, bool b_kc, const GemmArgs& g, float* partial, size_t partial_capacity,
                               hipStream_t st) {
  if (!gemm_args_ok(a_kc, b_kc, g)) return hipErrorInvalidValue;
  return gemm_launch(a_kc, b_kc, g, gemm_plan(g.M, g.N, g.K, partial ? partial_capacity : 0), partial, false, st);
}

}  // namespace ctr
