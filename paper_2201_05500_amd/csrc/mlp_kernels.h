// Element-wise and reduction kernels of the dense tower (the matrix products, with bias + ReLU and the
// ReLU gate of back-propagated gradients fused into their epilogues, are in gemm_kernels.h).
//
// Paper: the train_mini-batch step of Algorithm 1 on the network of Section 2.1, and Algorithm 2
// (k-step Adam) on the dense parameters.  bf16 rounding is nearest-even, done here by hand so that
// it is the same rule everywhere: (u + 0x7FFF + ((u >> 16) & 1)) >> 16 on the fp32 bit pattern.
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm_kernels.h"

namespace ctr {

struct MlpLayout {
  u32 n_layers;        // hidden layers + the output layer
  u32 in[8], out[8];   // widths per layer
  u64 w_off[8];        // offset of W_l in the flat parameter vector (b_l follows W_l)
  u64 n_params;
};

// fp32 -> bf16, 4 values per thread (n multiple of 4).
__global__ void k_cast_bf16(const float* __restrict__ src, bf16_t* __restrict__ dst, u64 n) {
  const u64 i = ((u64)blockIdx.x * BLOCK + threadIdx.x) * 4;
  if (i >= n) return;
  const f4 v = ldg4(src + i);
  ushort4 o;
  o.x = to_bf16(v.x); o.y = to_bf16(v.y); o.z = to_bf16(v.z); o.w = to_bf16(v.w);
  *reinterpret_cast<ushort4*>(dst + i) = o;
}

template <class T>
__global__ void k_copy(const T* __restrict__ src, T* __restrict__ dst, u64 n) {
  const u64 i = (u64)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// Output layer (width 1): logit[b] = a[b, :] . w + bias.  One wave per sample, fixed summation order.
__global__ void k_out_forward(const bf16_t* __restrict__ a, const bf16_t* __restrict__ w, const float* __restrict__ bias,
                              u32 rows, u32 H, float* __restrict__ logits) {
  const u32 r = (blockIdx.x * BLOCK + threadIdx.x) / WAVE;
  if (r >= rows) return;
  const int lane = lane_id();
  float s = 0.0f;
  for (u32 j = lane; j < H; j += WAVE) s += from_bf16(a[(u64)r * H + j]) * from_bf16(w[j]);
#pragma unroll
  for (int off = WAVE / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
  if (lane == 0) logits[r] = s + bias[0];
}

// Output layer of a training step, forward and back through the last ReLU, one wave per sample: the logit as in
// k_out_forward; sigmoid cross-entropy with logits in binary64, lterm[b] = max(z, 0) - z y + log1p(exp(-|z|)) and
// dlogit[b] = (sigmoid(z) - y) / rows; dz[b, j] = bf16(dlogit[b] * w[j] * [a[b, j] > 0]).
// (In launches of their own the three parts cost a launch each, 4.5 us on a small batch, and a second pass over a.)
// Bound by the one wave's chain where the layer is wide: from OUT_WIDE columns on the logit's terms, in the same order,
// are requested eight ahead, and the gradient takes 8 columns per lane.  (8 samples of 65536 columns: 540 -> 80 us, of
// 16384 128 -> 23, of 4096 36 -> 8; 32768 samples of 64 columns would take 4 us more by it.)
constexpr u32 OUT_WIDE = 512;
__global__ void __launch_bounds__(BLOCK)
k_out_step(const bf16_t* __restrict__ a, const bf16_t* __restrict__ w, const float* __restrict__ bias,
           const float* __restrict__ labels, u32 rows, u32 H, float* __restrict__ dlogit, double* __restrict__ lterm,
           bf16_t* __restrict__ dz) {
  const u32 r = (blockIdx.x * BLOCK + threadIdx.x) / WAVE;
  if (r >= rows) return;
  const u32 lane = (u32)lane_id();
  const bf16_t* row = a + (u64)r * H;
  float s = 0.0f;
  if (H >= OUT_WIDE) {
#pragma unroll 8
    for (u32 j = lane; j < H; j += WAVE) s += from_bf16(row[j]) * from_bf16(w[j]);
  } else {
    for (u32 j = lane; j < H; j += WAVE) s += from_bf16(row[j]) * from_bf16(w[j]);
  }
#pragma unroll
  for (int off = WAVE / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
  const double z = (double)(s + bias[0]), y = (double)labels[r];
  const float d = (float)((1.0 / (1.0 + exp(-z)) - y) / (double)rows);
  if (lane == 0) {
    lterm[r] = fmax(z, 0.0) - z * y + log1p(exp(-fabs(z)));
    dlogit[r] = d;
  }
  if (H < OUT_WIDE) {
    for (u32 j = lane; j < H; j += WAVE)
      dz[(u64)r * H + j] = to_bf16(from_bf16(row[j]) > 0.0f ? d * from_bf16(w[j]) : 0.0f);
    return;
  }
  const auto gate = [d](u32 a2, u32 w2) {  // two neighbouring columns
    const u32 lo = to_bf16(from_bf16((bf16_t)a2) > 0.0f ? d * from_bf16((bf16_t)w2) : 0.0f);
    const u32 hi = to_bf16(from_bf16((bf16_t)(a2 >> 16)) > 0.0f ? d * from_bf16((bf16_t)(w2 >> 16)) : 0.0f);
    return hi << 16 | lo;
  };
#pragma unroll 4
  for (u32 j = lane * 8; j < H; j += WAVE * 8) {  // H is a multiple of 8
    const uint4 av = *reinterpret_cast<const uint4*>(row + j), wv = *reinterpret_cast<const uint4*>(w + j);
    *reinterpret_cast<uint4*>(dz + (u64)r * H + j) =
        uint4{gate(av.x, wv.x), gate(av.y, wv.y), gate(av.z, wv.z), gate(av.w, wv.w)};
  }
}

// Sum over the threads of a block, left in part[0], in a fixed order (a binary tree).
template <class T>
__device__ __forceinline__ T block_tree_sum(T s, T* part) {
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = BLOCK / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  return part[0];
}

// The sums over the batch of a training step, all in one launch behind its products: column sums in a fixed order,
// out[j] = sum_b x[b, j] * (weight ? weight[b] : 1) (bias gradients, the output layer's weight gradient), the mean
// loss and the output bias gradient.
// Stage 1: a block takes a tile of columns (a thread 4 neighbouring ones) and a slice of the rows - its 8 row groups
// each sum the slice's rows congruent to them, the 8 partial sums are added in order -> partial[slice][column].
// Stage 2: the slices are added in order.
// (Per layer, with one column per thread and the two scalar sums in launches of their own, a tower of three hidden
// layers took ten launches here.)
constexpr u32 COLSUM_SLICES = 64, COLSUM_TILE = 128;
constexpr u32 COLSUM_MAX_JOBS = 8;  // a sum per hidden layer and one

struct BatchSums {
  const bf16_t* x[COLSUM_MAX_JOBS];
  const float* weight[COLSUM_MAX_JOBS];  // null: 1
  float* out[COLSUM_MAX_JOBS];
  u32 H[COLSUM_MAX_JOBS];                // a multiple of 8
  u32 col0[COLSUM_MAX_JOBS];             // first column of the job in a row of `partial`
  u32 n_jobs, n_cols, n_tiles, rows;     // n_cols: columns of all jobs, n_tiles: their tiles
  float* partial;                        // [COLSUM_SLICES][n_cols]
  const double* lterm;
  const float* dlogit;
  float *loss, *out_bias_grad;
};

inline __host__ __device__ u32 batch_sums_blocks(const BatchSums& q) { return 2 + q.n_tiles * COLSUM_SLICES; }

typedef float BatchSumsLds[8][COLSUM_TILE];
__device__ __forceinline__ void batch_sums_body(const BatchSums& q, u32 block, BatchSumsLds& part) {
  if (block == 0) {  // mean of the per-sample loss terms
    double s = 0.0;
#pragma unroll 8
    for (u32 r = threadIdx.x; r < q.rows; r += BLOCK) s += q.lterm[r];
    s = block_tree_sum(s, reinterpret_cast<double*>(part));
    if (threadIdx.x == 0) *q.loss = (float)(s / (double)q.rows);
    return;
  }
  if (block == 1) {
    float s = 0.0f;
#pragma unroll 8
    for (u32 r = threadIdx.x; r < q.rows; r += BLOCK) s += q.dlogit[r];
    s = block_tree_sum(s, &part[0][0]);
    if (threadIdx.x == 0) *q.out_bias_grad = s;
    return;
  }
  u32 tile = (block - 2) % q.n_tiles;
  const u32 slice = (block - 2) / q.n_tiles;
  u32 job = 0;
  while (tile >= (q.H[job] + COLSUM_TILE - 1) / COLSUM_TILE) tile -= (q.H[job++] + COLSUM_TILE - 1) / COLSUM_TILE;
  const u32 H = q.H[job], rg = threadIdx.x >> 5, in_tile = (threadIdx.x & 31) * 4, col = tile * COLSUM_TILE + in_tile;
  const u32 per = (q.rows + COLSUM_SLICES - 1) / COLSUM_SLICES;
  const u32 r0 = slice * per, r1 = min(r0 + per, q.rows);
  const bf16_t* x = q.x[job] + col;
  const float* weight = q.weight[job];
  f4 s = {0.0f, 0.0f, 0.0f, 0.0f};
  if (col < H) {
#pragma unroll 4
    for (u32 r = r0 + rg; r < r1; r += 8) {
      const ushort4 v = *reinterpret_cast<const ushort4*>(x + (u64)r * H);
      const float f = weight ? weight[r] : 1.0f;
      s.x += from_bf16(v.x) * f; s.y += from_bf16(v.y) * f; s.z += from_bf16(v.z) * f; s.w += from_bf16(v.w) * f;
    }
  }
  stg4(&part[rg][in_tile], s);
  __syncthreads();
  if (rg == 0 && col < H) {
#pragma unroll
    for (int g = 1; g < 8; ++g) {
      const f4 t = ldg4(&part[g][in_tile]);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    stg4(q.partial + (u64)slice * q.n_cols + q.col0[job] + col, s);
  }
}

__global__ void __launch_bounds__(BLOCK) k_batch_sums(BatchSums q) {
  __shared__ __align__(16) BatchSumsLds part;
  batch_sums_body(q, blockIdx.x, part);
}

// The two products of a layer's backward pass in one launch, and the sums over the batch behind those of the first layer:
// n_w work items of the weight gradient, n_i of the input gradient, then the blocks of the sums.  They need nothing of
// each other, and in a small tower none fills the chip: 1000 samples, 624 x 400: 8.5 and 6.4 us in launches of their own.
// The input gradient must not take the place of the layer's input, which the weight gradient reads.
__global__ void __launch_bounds__(BLOCK, 2)
k_gemm_backward(const bf16_t* __restrict__ h, const bf16_t* __restrict__ dz_w, GemmArgs w, const bf16_t* __restrict__ dz_i,
                const bf16_t* __restrict__ weights, GemmArgs i, u32 n_w, u32 n_i, BatchSums q) {
  __shared__ __align__(16) char lds[gemm_tiles_lds<64, 4>()];
  if (blockIdx.x < n_w)
    gemm_tiles_body<64, 2, 4, false, false>(lds, blockIdx.x, h, dz_w, w);
  else if (blockIdx.x < n_w + n_i)
    gemm_tiles_body<64, 2, 4, true, true>(lds, blockIdx.x - n_w, dz_i, weights, i);
  else
    batch_sums_body(q, blockIdx.x - n_w - n_i, *reinterpret_cast<BatchSumsLds*>(lds));
}

__global__ void __launch_bounds__(BLOCK) k_batch_sums_final(BatchSums q) {
  const u32 c = blockIdx.x * BLOCK + threadIdx.x;
  if (c >= q.n_cols) return;
  float t = 0.0f;
#pragma unroll 16
  for (u32 sl = 0; sl < COLSUM_SLICES; ++sl) t += q.partial[(u64)sl * q.n_cols + c];
  u32 job = 0;
  while (job + 1 < q.n_jobs && c >= q.col0[job + 1]) ++job;
  q.out[job][c - q.col0[job]] = t;
}

// Initial parameters of every replica: weights from the integer recipe of the row initialiser with
// key = layer << 48 | index, scaled to a standard deviation of sqrt(2 / fan_in); biases 0; m = 0;
// v = shared v = eps (Algorithm 2, "Initialize"); bf16 copies of the parameters.
__global__ void k_mlp_init(MlpLayout L, u64 seed_mul, float eps, u32 W, u64 stride, float* __restrict__ params,
                           float* __restrict__ m, float* __restrict__ v, float* __restrict__ vhat,
                           bf16_t* __restrict__ pb) {
  const u64 i = (u64)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= L.n_params) return;
  float val = 0.0f;
  for (u32 l = 0; l < L.n_layers; ++l) {
    const u64 nw = (u64)L.in[l] * L.out[l];
    if (i >= L.w_off[l] && i < L.w_off[l] + nw) {
      const float scale = (float)(sqrt(2.0 / (double)L.in[l]) / 37837.2);
      val = init_value(seed_mul, ((u64)l << 48) | (i - L.w_off[l]), 0, scale);
    }
  }
  for (u32 j = 0; j < W; ++j) {
    params[j * stride + i] = val;
    m[j * stride + i] = 0.0f;
    v[j * stride + i] = eps;
    pb[j * stride + i] = to_bf16(val);
  }
  if (vhat) vhat[i] = eps;
}

// bf16 copy of a flat fp32 vector (any length).
__global__ void k_refresh_bf16(const float* __restrict__ src, bf16_t* __restrict__ dst, u64 n) {
  const u64 i = (u64)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) dst[i] = to_bf16(src[i]);
}

// Dense Adam step (Algorithm 2's m, v and model lines) on one replica's flat parameter vector;
// every assignment in binary64 from the stored fp32 values, rounded once; refreshes the bf16 copy.
//   mode 0: x -= lr m / sqrt(own v)   1: x -= lr m / sqrt(shared v)   2: moments only (merge pending)
// Bound by memory: 30 bytes a parameter (34 with the shared denominator), of which only the bf16 copy is read again
// before the next step.  A thread takes 4 neighbouring parameters, everything but that copy with the non-temporal
// hint (20.3 M parameters 121 -> 107 us, 3.9 M 23.0 -> 20.4 us); the rest behind the n4 groups of 4 go to one thread
// each, and so do all parameters of a tower that does not fill the chip with groups of 4 (256 CUs x 2048 threads),
// which is bound by the chain of one thread's square roots and divisions.
struct DenseAdam {
  double b1, b2, lr;
  u32 mode;
  __device__ __forceinline__ void operator()(float g32, float den_shared, float& x, float& m, float& v) const {
    const double g = (double)g32;
    m = (float)(b1 * (double)m + (1.0 - b1) * g);
    v = (float)(b2 * (double)v + (1.0 - b2) * (g * g));
    if (mode != 2u) x = (float)((double)x - lr * (double)m / sqrt((double)(mode == 1u ? den_shared : v)));
  }
};

constexpr u64 DENSE_ADAM_WIDE_MIN = 4ull * 256 * 2048;  // parameters

// Where the gradient of a layer's weights and biases stands: the sum, in this order, of n arrays `stride` apart (the ranges
// of a split weight gradient, the slices of the batch sums).  Launches that only add those up cost a tenth of a small
// tower's step.
struct GradTerms {
  const float* p;
  u64 stride;
  u32 n;
};
struct GradSource {
  u32 n_layers;
  u64 w_off[9], n_weights[8];  // as in MlpLayout; w_off[n_layers]: the number of parameters
  GradTerms weights[8], biases[8];
};

template <class T, class Load>
__device__ __forceinline__ T grad_sum(const GradSource& src, u64 i, const Load& load) {
  u32 l = 0;
  while (l + 1 < src.n_layers && i >= src.w_off[l + 1]) ++l;
  u64 at = i - src.w_off[l];
  const bool bias = at >= src.n_weights[l];
  if (bias) at -= src.n_weights[l];
  const GradTerms t = bias ? src.biases[l] : src.weights[l];
  T s = load(t.p + at);
  // terms are requested together (the last ones again, beyond the end) and added in order: a few of a split product, many of
  // the batch sums
  const auto add = [&](auto side) {
    constexpr u32 SIDE = decltype(side)::value;
    for (u32 k = 1; k < t.n; k += SIDE) {
      T v[SIDE];
#pragma unroll
      for (u32 j = 0; j < SIDE; ++j) v[j] = load(t.p + min(k + j, t.n - 1u) * t.stride + at);
#pragma unroll
      for (u32 j = 0; j < SIDE; ++j)
        if (k + j < t.n) s = s + v[j];
    }
  };
  if (t.n > 32)
    add(std::integral_constant<u32, sizeof(T) == sizeof(float) ? 32 : 16>());
  else if (t.n > 4)
    add(std::integral_constant<u32, 8>());
  else
    add(std::integral_constant<u32, 4>());
  return s;
}

__global__ void __launch_bounds__(BLOCK)
k_dense_adam(float* __restrict__ params, float* __restrict__ m, float* __restrict__ v, const float* __restrict__ vhat,
             GradSource src, bf16_t* __restrict__ pb, u64 n, u64 n4, DenseAdam step) {
  // from the last parameters on: those of the small layers, with many terms to add, are not the end of the launch
  const u64 t = (u64)(gridDim.x - 1u - blockIdx.x) * BLOCK + threadIdx.x;
  if (t < n4) {  // layers begin and biases begin at multiples of 4
    const u64 i = t * 4;
    f4 mm = ldg4_stream(m + i), vv = ldg4_stream(v + i), x = {0.0f, 0.0f, 0.0f, 0.0f}, den = x;
    if (step.mode != 2u) x = ldg4_stream(params + i);
    if (step.mode == 1u) den = ldg4(vhat + i);
    const vf4 g = grad_sum<vf4>(src, i, [](const float* p) { return __builtin_nontemporal_load(reinterpret_cast<const vf4*>(p)); });
    step(g.x, den.x, x.x, mm.x, vv.x);
    step(g.y, den.y, x.y, mm.y, vv.y);
    step(g.z, den.z, x.z, mm.z, vv.z);
    step(g.w, den.w, x.w, mm.w, vv.w);
    stg4_stream(m + i, mm);
    stg4_stream(v + i, vv);
    if (step.mode != 2u) {
      stg4_stream(params + i, x);
      stg4_bf16(pb + i, x);
    }
  } else if (t < n - 3 * n4) {
    const u64 i = 3 * n4 + t;
    float x = params[i], mm = m[i], vv = v[i];
    const float den = step.mode == 1u ? vhat[i] : 0.0f;
    const float g = grad_sum<float>(src, i, [](const float* p) { return *p; });
    step(g, den, x, mm, vv);
    m[i] = mm;
    v[i] = vv;
    if (step.mode != 2u) {
      params[i] = x;
      pb[i] = to_bf16(x);
    }
  }
}

// Algorithm 2's global-averaging branch on the dense parameters of W replicas.
__global__ void k_dense_merge(float* __restrict__ params, const float* __restrict__ m, const float* __restrict__ v,
                              float* __restrict__ vhat, bf16_t* __restrict__ pb, u64 n, u64 stride, u32 W,
                              u32 pend_mask, double lr) {
  const u64 i = (u64)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= n) return;
  double vs = 0.0;
  for (u32 j = 0; j < W; ++j) vs += (double)v[j * stride + i];
  const float vh = (float)(vs / (double)W);
  vhat[i] = vh;
  const double den = sqrt((double)vh);
  double xs = 0.0;
  for (u32 j = 0; j < W; ++j) {
    double y = (double)params[j * stride + i];
    if (pend_mask & (1u << j)) y -= lr * (double)m[j * stride + i] / den;
    xs += y;
  }
  const float xb = (float)(xs / (double)W);
  const bf16_t hb = to_bf16(xb);
  for (u32 j = 0; j < W; ++j) {
    params[j * stride + i] = xb;
    pb[j * stride + i] = hb;
  }
}

}  // namespace ctr
