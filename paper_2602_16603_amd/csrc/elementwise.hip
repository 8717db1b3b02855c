// HBM-bound operators of the prefill layer: the start of a task, RMSNorm, rotary embedding
// with paged KV-cache write, SiLU(gate)*up.  All are coalesced, 16-byte-vectorised and do their
// arithmetic in fp32 (FlowPrefill Section 2.1: "FFN and residual connections"; the operators
// between the five core operators of Section 5.1).
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace fp {

template <typename T> using vec8 = T __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------------------------------
// RMSNorm: out = x * rsqrt(mean(x^2) + eps) * gain.  One 256-thread workgroup per token row;
// the row stays in registers between the sum-of-squares pass and the scaling pass (one HBM
// read), for rows up to 256*8*kMaxVec elements; longer rows are re-read.
// ------------------------------------------------------------------------------------------
constexpr int kNormMaxVec = 4;   // 256 threads * 8 elems * 4 = 8192 columns held in registers

// One row by one workgroup.  START: `row` is the task's input in the storage type, and the widened row
// goes to `x`, the fp32 residual stream.
template <typename T, typename IN, bool START>
__device__ __forceinline__ void rmsnorm_row(const IN* __restrict__ row, const T* __restrict__ gain, T* __restrict__ orow,
                                            float* __restrict__ x, int64_t d, float eps) {
  __shared__ float partial[4];
  const int tid = threadIdx.x;
  const int64_t n8 = d / 8;
  f32x8 held[kNormMaxVec];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kNormMaxVec; ++i) {
    int64_t c = tid + (int64_t)i * 256;
    if (c < n8) {
      held[i] = Vec8<IN>::load(row + c * 8);
      if (START) Vec8<float>::store(x + c * 8, held[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += held[i][e] * held[i][e];
    }
  }
  for (int64_t c = tid + (int64_t)kNormMaxVec * 256; c < n8; c += 256) {
    f32x8 v = Vec8<IN>::load(row + c * 8);
    if (START) Vec8<float>::store(x + c * 8, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) partial[tid >> 6] = ss;
  __syncthreads();
  float total = partial[0] + partial[1] + partial[2] + partial[3];
  float inv = 1.0f / sqrtf(total / (float)d + eps);
#pragma unroll
  for (int i = 0; i < kNormMaxVec; ++i) {
    int64_t c = tid + (int64_t)i * 256;
    if (c < n8) {
      f32x8 g = Vec8<T>::load(gain + c * 8);
      f32x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = held[i][e] * inv * g[e];
      Vec8<T>::store(orow + c * 8, o);
    }
  }
  for (int64_t c = tid + (int64_t)kNormMaxVec * 256; c < n8; c += 256) {
    f32x8 v = Vec8<IN>::load(row + c * 8);
    f32x8 g = Vec8<T>::load(gain + c * 8);
    f32x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[e] * inv * g[e];
    Vec8<T>::store(orow + c * 8, o);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ x,
                                                      const T* __restrict__ gain,
                                                      T* __restrict__ out, int64_t d, float eps) {
  rmsnorm_row<T, float, false>(x + (int64_t)blockIdx.x * d, gain, out + (int64_t)blockIdx.x * d, nullptr, d, eps);
}

void launch_rmsnorm(int dtype, const float* x, const void* gain, void* out, int64_t t, int64_t d,
                    float eps, hipStream_t s) {
  if (t == 0) return;
  dim3 grid((unsigned)t);
  if (dtype == 1)
    launch_kernel(rmsnorm_kernel<bf16>, grid, 256, 0, s, x, (const bf16*)gain, (bf16*)out, d, eps);
  else
    launch_kernel(rmsnorm_kernel<float>, grid, 256, 0, s, x, (const float*)gain, (float*)out, d, eps);
}

// ------------------------------------------------------------------------------------------
// Everything a task needs on the device before its first GEMM, in one launch: the batch's metadata from pinned host
// memory (16 bytes per thread, the first workgroups), hidden_in widened into the fp32 residual stream, and
// the first layer's attention RMSNorm of the same rows (one workgroup per token), with the bits of the separate
// operator.  Separately these are an upload and two kernels, the second re-reading the residual: 67 us of kernels
// at 8192 x 4096, 49 here, and two launches fewer for a short request.
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void task_start_kernel(const T* __restrict__ in, float* __restrict__ x,
                                                         const T* __restrict__ gain, T* __restrict__ out, int64_t d,
                                                         float eps, const u32x4* __restrict__ meta_in,
                                                         u32x4* __restrict__ meta_out, int64_t n_meta, int meta_blocks) {
  if ((int)blockIdx.x < meta_blocks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_meta) meta_out[i] = meta_in[i];
    return;
  }
  const int64_t at = (int64_t)(blockIdx.x - meta_blocks) * d;
  rmsnorm_row<T, T, true>(in + at, gain, out + at, x + at, d, eps);
}

void launch_task_start(int dtype, const void* in, float* x, const void* gain, void* out, int64_t t, int64_t d, float eps,
                       const int32_t* meta_in, int32_t* meta_out, int64_t n_ints, hipStream_t s) {
  const int64_t n_meta = (n_ints + 3) / 4;
  const int meta_blocks = (int)((n_meta + 255) / 256);
  dim3 grid((unsigned)(meta_blocks + t));
  if (grid.x == 0) return;
  if (dtype == 1)
    launch_kernel(task_start_kernel<bf16>, grid, 256, 0, s, (const bf16*)in, x, (const bf16*)gain, (bf16*)out, d, eps,
                                                 (const u32x4*)meta_in, (u32x4*)meta_out, n_meta, meta_blocks);
  else
    launch_kernel(task_start_kernel<float>, grid, 256, 0, s, (const float*)in, x, (const float*)gain, (float*)out, d, eps,
                                                  (const u32x4*)meta_in, (u32x4*)meta_out, n_meta, meta_blocks);
}

// ------------------------------------------------------------------------------------------
// SiLU(gate) * up : gu [T, 2F] -> out [T, F]; gate = columns [0,F), up = columns [F,2F).
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void silu_mul_kernel(const T* __restrict__ gu,
                                                       T* __restrict__ out, int64_t t, int64_t f) {
  const int64_t f8 = f / 8;
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= t * f8) return;
  int64_t r = i / f8, c = i - r * f8;
  const T* row = gu + r * 2 * f;
  f32x8 g = Vec8<T>::load(row + c * 8);
  f32x8 u = Vec8<T>::load(row + f + c * 8);
  f32x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = silu_mul_f32(g[e], u[e]);
  Vec8<T>::store(out + r * f + c * 8, o);
}

void launch_silu_mul(int dtype, const void* gu, void* out, int64_t t, int64_t f, hipStream_t s) {
  int64_t n = t * (f / 8);
  if (n == 0) return;
  dim3 grid((unsigned)((n + 255) / 256));
  if (dtype == 1)
    launch_kernel(silu_mul_kernel<bf16>, grid, 256, 0, s, (const bf16*)gu, (bf16*)out, t, f);
  else
    launch_kernel(silu_mul_kernel<float>, grid, 256, 0, s, (const float*)gu, (float*)out, t, f);
}

// ------------------------------------------------------------------------------------------
// Rotary embedding + paged KV-cache write, one launch.
//   the first n_kv_items workgroups: one (sequence, logical block) each -- copy the raw values of
//                                 that block's new tokens into the V pool
//                                 [layer][block][Hkv][D][16] (transposed inside the block so the
//                                 attention kernel can read 8 consecutive keys of one channel
//                                 as a 16-byte MFMA operand); they take longest and go first;
//   the following T workgroups:   one token each -- rotate its Hq query heads in place in the
//                                 qkv buffer, rotate its Hkv key heads and store them into the
//                                 K pool [layer][block][Hkv][16][D].
// Pair (j, j+D/2) is rotated by angle pos * theta^(-2j/D); cos/sin come from a table computed in
// fp64 on the host.
// ------------------------------------------------------------------------------------------
// PARTS: a short request's projection was cut over K and its fp32 partial sums are added up here, in index order and
// rounded to the storage type -- the bits of the stand-alone reduction, one launch and one pass over qkv less.
template <typename T, bool PARTS>
__device__ __forceinline__ f32x8 qkv_load8(const T* __restrict__ qkv, const float* __restrict__ part, int64_t at, int64_t slab, int parts) {
  if (!PARTS) return Vec8<T>::load(qkv + at);
  f32x8 acc = Vec8<float>::load(part + at);
  for (int z = 1; z < parts; ++z) {
    const f32x8 v = Vec8<float>::load(part + z * slab + at);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += v[e];
  }
  return __builtin_convertvector(__builtin_convertvector(acc, vec8<T>), f32x8);
}

template <typename T, bool PARTS>
__global__ __launch_bounds__(256) void rope_kvwrite_kernel(
    T* __restrict__ qkv, const float* __restrict__ rope_cos, const float* __restrict__ rope_sin,
    int n_q_heads, int n_kv_heads, int head_dim, int64_t kv_num_blocks, int layer,
    T* __restrict__ k_pool, T* __restrict__ v_pool, int n_tokens,
    const int32_t* __restrict__ tok_seq, const int32_t* __restrict__ tok_pos,
    const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ cached_lens,
    const int32_t* __restrict__ block_tables, int max_blocks,
    const int32_t* __restrict__ kv_items, const float* __restrict__ part, int parts) {
  const int tid = threadIdx.x;
  const int half = head_dim / 2;
  const int64_t width = (int64_t)(n_q_heads + 2 * n_kv_heads) * head_dim;
  const int n_kv_items = (int)gridDim.x - n_tokens;
  const int64_t slab = n_tokens * width;
  if ((int)blockIdx.x >= n_kv_items) {
    const int t = (int)blockIdx.x - n_kv_items;
    const int s = tok_seq[t];
    const int pos = tok_pos[t];
    const int64_t blk = block_tables[(int64_t)s * max_blocks + pos / kKvBlock];
    T* row = qkv + (int64_t)t * width;
    const float* cs = rope_cos + (int64_t)pos * half;
    const float* sn = rope_sin + (int64_t)pos * half;
    const int per_head = half / 8;
    const int units = (n_q_heads + n_kv_heads) * per_head;
    for (int u = tid; u < units; u += 256) {
      const int h = u / per_head;
      const int j = (u - h * per_head) * 8;
      T* base = row + (int64_t)h * head_dim;
      const int64_t at = t * width + (int64_t)h * head_dim + j;
      f32x8 a = qkv_load8<T, PARTS>(qkv, part, at, slab, parts);
      f32x8 b = qkv_load8<T, PARTS>(qkv, part, at + half, slab, parts);
      f32x8 c = Vec8<float>::load(cs + j);
      f32x8 sv = Vec8<float>::load(sn + j);
      f32x8 ra, rb;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ra[e] = a[e] * c[e] - b[e] * sv[e];
        rb[e] = b[e] * c[e] + a[e] * sv[e];
      }
      if (h < n_q_heads) {
        Vec8<T>::store(base + j, ra);
        Vec8<T>::store(base + half + j, rb);
      } else {
        const int kh = h - n_q_heads;
        T* dst = k_pool + ((((int64_t)layer * kv_num_blocks + blk) * n_kv_heads + kh) * kKvBlock +
                           (pos % kKvBlock)) * head_dim;
        Vec8<T>::store(dst + j, ra);
        Vec8<T>::store(dst + half + j, rb);
      }
    }
    return;
  }
  // ---- value block role ----
  const int item = blockIdx.x;
  const int s = kv_items[2 * item];
  const int lb = kv_items[2 * item + 1];
  const int cached = cached_lens[s];
  const int seq_lo = cu_seqlens[s];
  const int n_new = cu_seqlens[s + 1] - seq_lo;
  const int64_t blk = block_tables[(int64_t)s * max_blocks + lb];
  const int p_lo = max(lb * kKvBlock, cached);
  const int p_hi = min(lb * kKvBlock + kKvBlock, cached + n_new);
  const int units = n_kv_heads * head_dim / 8;
  const int64_t v_off = (int64_t)(n_q_heads + n_kv_heads) * head_dim;
  if (PARTS) {                                       // half a block of 8 channels per thread: the sums are loads enough
    for (int u2 = tid; u2 < 2 * units; u2 += 256) {
      const int h = u2 / units, u = u2 - h * units;
      const int kh = u / (head_dim / 8);
      const int d0 = (u - kh * (head_dim / 8)) * 8;
      T* dst = v_pool + (((int64_t)layer * kv_num_blocks + blk) * n_kv_heads + kh) *
                            ((int64_t)head_dim * kKvBlock) + (int64_t)d0 * kKvBlock + 8 * h;
      const int first = lb * kKvBlock + 8 * h;
      if (first >= p_hi || first + 8 <= p_lo) continue;
      int64_t at[8];
      f32x8 acc[8];
#pragma unroll
      for (int tk = 0; tk < 8; ++tk) {
        const int p = min(max(first + tk, p_lo), p_hi - 1);
        at[tk] = (seq_lo + (p - cached)) * width + v_off + kh * head_dim + d0;
        acc[tk] = Vec8<float>::load(part + at[tk]);
      }
      for (int z = 1; z < parts; ++z)
#pragma unroll
        for (int tk = 0; tk < 8; ++tk) {
          const f32x8 v = Vec8<float>::load(part + z * slab + at[tk]);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[tk][e] += v[e];
        }
      const bool all = first >= p_lo && first + 8 <= p_hi;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        vec8<T> piece;
#pragma unroll
        for (int tk = 0; tk < 8; ++tk) piece[tk] = static_cast<T>(acc[tk][e]);
        if (all) {
          *reinterpret_cast<vec8<T>*>(dst + e * kKvBlock) = piece;
        } else {
#pragma unroll
          for (int tk = 0; tk < 8; ++tk)
            if (first + tk >= p_lo && first + tk < p_hi) dst[e * kKvBlock + tk] = piece[tk];
        }
      }
    }
    return;
  }
  for (int u = tid; u < units; u += 256) {
    const int kh = u / (head_dim / 8);
    const int d0 = (u - kh * (head_dim / 8)) * 8;
    T* dst = v_pool + (((int64_t)layer * kv_num_blocks + blk) * n_kv_heads + kh) *
                          ((int64_t)head_dim * kKvBlock) + (int64_t)d0 * kKvBlock;
    // All tokens' loads are in flight together.  A half of the block's 16 slots leaves as whole 16-byte pieces
    // where all of it is new; slots of tokens that are not new keep what they hold.
    vec8<T> v[kKvBlock];
#pragma unroll
    for (int tk = 0; tk < kKvBlock; ++tk) {
      const int p = min(max(lb * kKvBlock + tk, p_lo), p_hi - 1);
      const int64_t trow = seq_lo + (p - cached);
      v[tk] = *reinterpret_cast<const vec8<T>*>(qkv + trow * width + v_off + kh * head_dim + d0);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int first = lb * kKvBlock + 8 * h;
      if (first >= p_lo && first + 8 <= p_hi) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          vec8<T> piece;
#pragma unroll
          for (int tk = 0; tk < 8; ++tk) piece[tk] = v[8 * h + tk][e];
          *reinterpret_cast<vec8<T>*>(dst + e * kKvBlock + 8 * h) = piece;
        }
      } else {
#pragma unroll
        for (int tk = 0; tk < 8; ++tk)
          if (first + tk >= p_lo && first + tk < p_hi) {
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[e * kKvBlock + 8 * h + tk] = v[8 * h + tk][e];
          }
      }
    }
  }
}

void launch_rope_kvwrite(int dtype, void* qkv, const float* rope_cos, const float* rope_sin,
                         const Geometry& g, const BatchMeta& m, int layer, void* k_pool,
                         void* v_pool, const float* part, int parts, hipStream_t s) {
  if (m.n_tokens == 0) return;
  dim3 grid((unsigned)(m.n_tokens + m.n_kv_items));
  if (dtype == 1 && parts > 0)
    launch_kernel(rope_kvwrite_kernel<bf16, true>, grid, 256, 0, s,
        (bf16*)qkv, rope_cos, rope_sin, g.n_q_heads, g.n_kv_heads, g.head_dim, g.kv_num_blocks,
        layer, (bf16*)k_pool, (bf16*)v_pool, m.n_tokens, m.tok_seq, m.tok_pos, m.cu_seqlens,
        m.cached_lens, m.block_tables, m.max_blocks, m.kv_items, part, parts);
  else if (dtype == 1)
    launch_kernel(rope_kvwrite_kernel<bf16, false>, grid, 256, 0, s,
        (bf16*)qkv, rope_cos, rope_sin, g.n_q_heads, g.n_kv_heads, g.head_dim, g.kv_num_blocks,
        layer, (bf16*)k_pool, (bf16*)v_pool, m.n_tokens, m.tok_seq, m.tok_pos, m.cu_seqlens,
        m.cached_lens, m.block_tables, m.max_blocks, m.kv_items, nullptr, 0);
  else
    launch_kernel(rope_kvwrite_kernel<float, false>, grid, 256, 0, s,
        (float*)qkv, rope_cos, rope_sin, g.n_q_heads, g.n_kv_heads, g.head_dim, g.kv_num_blocks,
        layer, (float*)k_pool, (float*)v_pool, m.n_tokens, m.tok_seq, m.tok_pos, m.cu_seqlens,
        m.cached_lens, m.block_tables, m.max_blocks, m.kv_items, nullptr, 0);
}

// ------------------------------------------------------------------------------------------
// Gather one sequence's keys/values of one layer from the paged pools into contiguous
// [len, Hkv, D] buffers (what a prefill instance hands to a decode instance, and what the
// parity tests compare).  D/4 threads per (16-token block, kv head, K or V): for V (blockIdx.y = 0) each
// transposes 8 channels x 8 tokens of the slab [D][16] in registers, so both sides move 16 bytes at a
// time; for K it copies eight pieces of the slab.  Moves 4 bytes per element and is bound by HBM (one thread per 8 channels of a token,
// picking 2-byte values out of the V slab: 57 us for 16384 tokens of 8 heads x 128, 134 MB; now 25).
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void kv_gather_kernel(const T* __restrict__ k_pool,
                                                        const T* __restrict__ v_pool,
                                                        T* __restrict__ k_out, T* __restrict__ v_out,
                                                        int len, int n_kv_heads, int head_dim,
                                                        int64_t kv_num_blocks, int layer,
                                                        const int32_t* __restrict__ table) {
  const int per_slab = head_dim / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t slab = i / per_slab;
  const int sub = (int)(i - slab * per_slab);
  const int lb = (int)(slab / n_kv_heads), kh = (int)(slab - (int64_t)lb * n_kv_heads);
  const int p0 = lb * kKvBlock;
  if (p0 >= len) return;
  const int64_t blk = table[lb];
  const int64_t base = (((int64_t)layer * kv_num_blocks + blk) * n_kv_heads + kh) *
                       ((int64_t)head_dim * kKvBlock);
  const int64_t row = (int64_t)n_kv_heads * head_dim;
  const int64_t dst = (int64_t)p0 * row + (int64_t)kh * head_dim;
  const int half = sub & 1, d0 = (sub >> 1) * 8;
  vec8<T> v[8];
  if (blockIdx.y == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      v[e] = *reinterpret_cast<const vec8<T>*>(v_pool + base + (int64_t)(d0 + e) * kKvBlock + half * 8);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      vec8<T> o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = v[e][t];
      if (p0 + half * 8 + t < len) *reinterpret_cast<vec8<T>*>(v_out + dst + (half * 8 + t) * row + d0) = o;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = *reinterpret_cast<const vec8<T>*>(k_pool + base + (int64_t)(t * per_slab + sub) * 8);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int at = (t * per_slab + sub) * 8;         // element of the K slab [16][D]
      const int slot = at / head_dim;
      if (p0 + slot < len) *reinterpret_cast<vec8<T>*>(k_out + dst + slot * row + (at - slot * head_dim)) = v[t];
    }
  }
}

void launch_kv_gather(int dtype, const void* k_pool, const void* v_pool, void* k_out, void* v_out,
                      int len, const Geometry& g, int layer, const int32_t* table_dev,
                      hipStream_t s) {
  if (len == 0) return;
  const int64_t n = (int64_t)((len + kKvBlock - 1) / kKvBlock) * g.n_kv_heads * (g.head_dim / 4);
  dim3 grid((unsigned)((n + 255) / 256), 2);
  if (dtype == 1)
    launch_kernel(kv_gather_kernel<bf16>, grid, 256, 0, s, (const bf16*)k_pool, (const bf16*)v_pool,
                                                (bf16*)k_out, (bf16*)v_out, len, g.n_kv_heads,
                                                g.head_dim, g.kv_num_blocks, layer, table_dev);
  else
    launch_kernel(kv_gather_kernel<float>, grid, 256, 0, s, (const float*)k_pool, (const float*)v_pool,
                                                 (float*)k_out, (float*)v_out, len, g.n_kv_heads,
                                                 g.head_dim, g.kv_num_blocks, layer, table_dev);
}

}  // namespace fp
