// Causal variable-length grouped-query attention over the paged KV cache in fp32 (debug path): FlowPrefill Eq. (2)
// with the causal mask and KV-cache reuse of Section 3.1; operator `attn` of Section 5.1.  Compiled with NaN
// semantics, unlike the bf16 kernel: this is the path on which a NaN is looked for.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace fp {

// ------------------------------------------------------------------------------------------
// fp32 kernel (debug path) on v_mfma_f32_16x16x4_f32, fp32 online softmax.  One workgroup = 4 waves = 64
// query rows of one head, 16 rows per wave; keys come one 16-token cache block at a time.  Scores are
// computed transposed, S^T = K Q^T, so a lane owns one query (lane % 16) and the four keys 4 (lane / 16)
// + (0..3) of the block -- which is what the B operand of O^T += V^T P^T wants when step r of four takes
// key 4 q + r of lane quarter q: the probabilities go from the accumulators into the next product as
// they are, and the A operand is four consecutive keys of one channel, one 16-byte piece of the V pool.
// K, Q and V fragments come straight from global memory (the four waves share them through L1 and L2);
// the next block's keys are requested before this block's softmax.
// A masked probability is an exact zero, which is enough as long as the value beside it is finite.  In a block that
// holds keys some of the wave's queries do not see, slots that none of them sees (behind the sequence they hold what an
// earlier request left) therefore enter as zeros, and if any other value is not finite, the block's products are formed
// one key at a time and only for the queries that see the key.  300 tokens, 32 heads of 128: 33 us,
// 798 us with one wave per (token, head) on plain FMAs; the walk over the key blocks bounds it.
// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void attn_f32_kernel(
    const float* __restrict__ qkv, const float* __restrict__ k_pool, const float* __restrict__ v_pool,
    float* __restrict__ o, int n_q_heads, int n_kv_heads, int64_t kv_num_blocks, int layer,
    const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ cached_lens,
    const int32_t* __restrict__ block_tables, int max_blocks, const int32_t* __restrict__ attn_items,
    float scale) {
  constexpr int C = D / 16;                          // 16-channel blocks
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, quad = lane >> 4;
  const int head = blockIdx.x % n_q_heads, kvh = head / (n_q_heads / n_kv_heads);
  const int rest = blockIdx.x / n_q_heads;
  const int s = attn_items[kAttnItemInts * (rest >> 2)];
  const int q0 = attn_items[kAttnItemInts * (rest >> 2) + 1] * 256 + (rest & 3) * 64 + wave * 16;
  const int seq_lo = cu_seqlens[s], n_new = cu_seqlens[s + 1] - seq_lo, cached = cached_lens[s];
  if (q0 >= n_new) return;                           // whole wave; no barrier below
  const int64_t width = (int64_t)(n_q_heads + 2 * n_kv_heads) * D;
  const int32_t* bt = block_tables + (int64_t)s * max_blocks;
  const int64_t block_elems = (int64_t)n_kv_heads * kKvBlock * D;
  const int64_t head_elems = ((int64_t)layer * kv_num_blocks * n_kv_heads + kvh) * (kKvBlock * D);
  const int qpos = cached + q0 + col;
  const int last_key = cached + min(q0 + 15, n_new - 1);   // that any query of the wave sees
  const int n_blocks = last_key / kKvBlock + 1;

  f32x4 qf[C], kf[C], acc[C];
  {
    const float* src = qkv + (int64_t)(seq_lo + min(q0 + col, n_new - 1)) * width + head * D + 4 * quad;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      qf[c] = *reinterpret_cast<const f32x4*>(src + c * 16);
      acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  auto load_keys = [&](int b) __attribute__((always_inline)) {
    const float* src = k_pool + head_elems + (int64_t)bt[b] * block_elems + col * D + 4 * quad;
#pragma unroll
    for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const f32x4*>(src + c * 16);
  };
  load_keys(0);
  float m = -INFINITY, l = 0.f;
  for (int b = 0; b < n_blocks; ++b) {
    f32x4 vf[C];
    const float* vsrc = v_pool + head_elems + (int64_t)bt[b] * block_elems + col * kKvBlock + 4 * quad;
#pragma unroll
    for (int c = 0; c < C; ++c) vf[c] = *reinterpret_cast<const f32x4*>(vsrc + c * (16 * kKvBlock));
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], sc, 0, 0, 0);
    if (b + 1 < n_blocks) load_keys(b + 1);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = b * kKvBlock + 4 * quad + r <= qpos ? sc[r] * scale : -INFINITY;
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx);                // finite from the first block on: key 0 is visible to all
    const float alpha = __expf(m - m_new);
    float p[4], sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __expf(sc[r] - m_new);
      sum += p[r];
    }
    l = l * alpha + sum;                             // this lane's keys only; the quarters are added at the end
    m = m_new;
    bool finite = true;
    if (b * kKvBlock + kKvBlock - 1 > cached + q0) {   // (wave-uniform)
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          vf[c][r] = b * kKvBlock + 4 * quad + r <= last_key ? vf[c][r] : 0.f;
          finite = finite && fabsf(vf[c][r]) < INFINITY;
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c][r] *= alpha;
    if (__all(finite)) {
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][r], p[r], acc[c], 0, 0, 0);
    } else {
      // This lane's accumulators are channels 16 c + 4 quad + (0..3) of query `col`.
      const float* rows = v_pool + head_elems + (int64_t)bt[b] * block_elems + 4 * quad * kKvBlock;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        for (int kq = 0; kq < 4; ++kq) {
          const int key = 4 * kq + r;
          const float pk = __shfl(p[r], 16 * kq + col);
          if (b * kKvBlock + key <= qpos) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[c][i] = fmaf(pk, rows[(16 * c + i) * kKvBlock + key], acc[c][i]);
          }
        }
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (q0 + col < n_new) {
    float* dst = o + (int64_t)(seq_lo + q0 + col) * n_q_heads * D + head * D + 4 * quad;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      f32x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = acc[c][r] / l;
      *reinterpret_cast<f32x4*>(dst + c * 16) = v;
    }
  }
}

template <int D>
static void launch_attn_f32(const float* qkv, const float* k_pool, const float* v_pool, float* o,
                            const Geometry& g, const BatchMeta& m, int layer, hipStream_t s) {
  dim3 grid((unsigned)((int64_t)m.n_attn_items * 4 * g.n_q_heads));   // 64 of an item's 256 query rows each
  launch_kernel(attn_f32_kernel<D>, grid, 256, 0, s, qkv, k_pool, v_pool, o, g.n_q_heads, g.n_kv_heads, g.kv_num_blocks, layer,
                                          m.cu_seqlens, m.cached_lens, m.block_tables, m.max_blocks, m.attn_items,
                                          1.0f / sqrtf((float)D));
}

void launch_attention_f32(const float* qkv, const float* k_pool, const float* v_pool, float* o, const Geometry& g,
                          const BatchMeta& m, int layer, hipStream_t s) {
  switch (g.head_dim) {
    case 16: launch_attn_f32<16>(qkv, k_pool, v_pool, o, g, m, layer, s); break;
    case 32: launch_attn_f32<32>(qkv, k_pool, v_pool, o, g, m, layer, s); break;
    case 64: launch_attn_f32<64>(qkv, k_pool, v_pool, o, g, m, layer, s); break;
    default: launch_attn_f32<128>(qkv, k_pool, v_pool, o, g, m, layer, s); break;
  }
}

}  // namespace fp
