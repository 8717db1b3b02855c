// Mixture-of-experts FFN support (FlowPrefill Section 7, "Mixture-of-Experts (MoE) models": the
// `gate` operator -- a gated router -- and the `experts` operator -- several expert FFNs).
// Router: softmax over all experts of h W_r^T, the top_k most probable experts per token (ties:
// lower index), probabilities renormalised over the selected ones.  The expert FFNs run as two
// grouped GEMMs over per-expert row ranges (the first gathers the routed tokens' activations by
// index; the second one's rows are then combined, weighted, into the residual stream).  The arithmetic of a token never depends on
// where in an expert's row range it lands, so the (atomic, run-to-run varying) slot order does not reach the
// results.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace fp {

// Router: Q tokens per wave: probabilities, top_k selection, renormalised weights.  n_experts <= 256 (lane l holds experts l,
// l+64, l+128, l+192), top_k <= 8.  A selection step is a chain -- the wave's maximum by DPP, then the first lane that holds it by
// ballot (ties: lower index) -- so a wave runs the chains of its tokens side by side (29 us with one after the other on
// LDS-shuffle reductions).  Every chosen (token, expert) pair also takes a rank among the workgroup's pairs of
// that expert (an LDS counter), and the workgroup leaves its per-expert counts in
// block_counts[block][expert]: the row plan below needs no global atomics (65536 of them on 128
// addresses cost more than the rest of the operator).
// The selections are bound by instruction issue, so they are spread over the CUs as far as the plan's walk over the workgroups'
// counts allows (kFusedPlanBlocks of them): below 2048 tokens workgroups of 8, two per wave, up to 8192 of 32, four per wave, then
// 64.  The gate operator, us, against workgroups of 16 and 64, four tokens per wave: 16 tokens 22.2 -> 19.2, 200 25.6 -> 21.5, 590
// 26 -> 22.8, 1000 27.9 -> 25.2, 1700 30 -> 28.3, 2100 35.3 -> 31.8, 4096 37.5 -> 33.8, 8192 47.6 -> 45.  (Workgroups of 16 from
// 2048 to 4096 tokens: not measured.)
__host__ __device__ inline int route_tokens_per_block(int64_t n_tokens) { return n_tokens < 2048 ? 8 : n_tokens <= 8192 ? 32 : 64; }
inline int route_tokens_per_wave(int64_t n_tokens) { return n_tokens < 2048 ? 2 : 4; }   // (four waves or more)

template <int CTRL, int ROWS> __device__ __forceinline__ float max_dpp(float v) {   // lanes without a source keep v
  const int u = __builtin_bit_cast(int, v);
  return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, CTRL, ROWS, 0xf, false)));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = max_dpp<0x111, 0xf>(v);                       // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has the row's maximum
  v = max_dpp<0x112, 0xf>(v);
  v = max_dpp<0x114, 0xf>(v);
  v = max_dpp<0x118, 0xf>(v);
  v = max_dpp<0x142, 0xa>(v);                       // row_bcast 15 into rows 1 and 3, row_bcast 31 into rows 2 and 3
  v = max_dpp<0x143, 0xc>(v);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

template <int Q>
__global__ __launch_bounds__(1024) void moe_route_kernel(const float* __restrict__ logits,
                                                         int32_t* __restrict__ ids,
                                                         float* __restrict__ wts,
                                                         int32_t* __restrict__ rank_in_block,
                                                         int32_t* __restrict__ block_counts,
                                                         int n_tokens, int n_experts, int top_k) {
  __shared__ int hist[256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x < 256) hist[threadIdx.x] = 0;     // (256 threads or more)
  __syncthreads();
  const int t0 = (blockIdx.x * (blockDim.x >> 6) + wave) * Q;   // (a token past the end repeats the last one and is not written)
  float p[Q][4];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane + 64 * i;
      p[q][i] = e < n_experts ? logits[(int64_t)min(t0 + q, n_tokens - 1) * n_experts + e] : -INFINITY;
    }
  float total[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const float mx = wave_max_dpp(fmaxf(fmaxf(p[q][0], p[q][1]), fmaxf(p[q][2], p[q][3])));
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[q][i] = lane + 64 * i < n_experts ? expf(p[q][i] - mx) : -1.0f;   // -1: never selected
      sum += fmaxf(p[q][i], 0.f);
    }
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[q][i] = p[q][i] >= 0.f ? p[q][i] * inv : -1.0f;
    total[q] = mx == INFINITY ? NAN : 0.f;          // a logit of +inf: the softmax, and with it every weight, is NaN
  }
  // Lane j (< 8) of the wave keeps choice j of every token.
  float my_p[Q];
  int my_e[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) { my_p[q] = 0.f; my_e[q] = 0; }
#pragma unroll
  for (int j = 0; j < kMaxChoices; ++j) {
    if (j >= top_k) break;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float best = wave_max_dpp(fmaxf(fmaxf(p[q][0], p[q][1]), fmaxf(p[q][2], p[q][3])));
      int e = -1;
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const uint64_t holds = __ballot(p[q][i] == best);
        e = holds ? 64 * i + __ffsll((unsigned long long)holds) - 1 : e;
      }
      if (e < 0 || e >= n_experts) e = 0;             // (only infinities or NaN among the logits leave none in range)
      total[q] += best;
      if (lane == j) { my_p[q] = best; my_e[q] = e; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (lane + 64 * i == e) p[q][i] = -1.0f;                    // taken
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (t0 + q < n_tokens && lane < top_k) {
      const int64_t at = (int64_t)(t0 + q) * top_k + lane;
      const float norm = 1.0f / total[q];
      ids[at] = my_e[q];
      wts[at] = my_p[q] * norm;
      rank_in_block[at] = atomicAdd(&hist[my_e[q]], 1);
    }
  __syncthreads();
  if (threadIdx.x < n_experts) block_counts[(int64_t)blockIdx.x * n_experts + threadIdx.x] = hist[threadIdx.x];
}

// Row offset of expert e among all experts' rows (256 threads, thread e of an expert with `total` rows; all of them call), and, if `table`,
// the grouped GEMMs' row-tile table: groups[0] = row tiles, then {expert, first row, rows} per tile of tile_rows rows.
__device__ __forceinline__ int expert_rows(int total, int e, int n_experts, int tile_rows, bool table, int32_t* __restrict__ groups) {
  __shared__ int s_rows[4], s_tiles[4];
  // The 256-row tile multiplies only the multiple of 32 rows that a tile has: an expert's rows are spread evenly over as
  // few tiles as hold them (520 rows: three tiles of 192, where 256 + 256 + 8 are three full ones and the last is bound by
  // the latency of its k-tiles however few rows it has).
  int rows = tile_rows;
  if (tile_rows == 256 && total > 0) {
    const int n = (total + 255) / 256;
    rows = ((total + n - 1) / n + 31) / 32 * 32;
  }
  // Exclusive prefix sums of rows and of tiles over the experts: within a wave by shuffles, across the four waves
  // through LDS (one thread walking all experts took 5 us).
  const int tiles = (total + rows - 1) / rows;
  int off = total, first = tiles;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(off, d), f = __shfl_up(first, d);
    if ((e & 63) >= d) { off += o; first += f; }
  }
  if ((e & 63) == 63) { s_rows[e >> 6] = off; s_tiles[e >> 6] = first; }
  __syncthreads();
  off -= total;
  first -= tiles;
  for (int w = 0; w < (e >> 6); ++w) { off += s_rows[w]; first += s_tiles[w]; }
  if (table && e == 0) groups[0] = s_tiles[0] + s_tiles[1] + s_tiles[2] + s_tiles[3];
  if (table && e < n_experts)
    for (int m = 0; m < total; m += rows, ++first) {
      groups[1 + 3 * first] = e;
      groups[2 + 3 * first] = off + m;
      groups[3 + 3 * first] = min(rows, total - m);
    }
  return off;
}


// One workgroup: per-expert totals and row offsets, the route workgroups' counts turned into
// their first row inside each expert's range (in place), and the grouped GEMMs' row-tile table.
//   plan[0 .. E) offsets;   groups[0] = row tiles, then {expert, first row, rows} per tile of tile_rows rows
__global__ __launch_bounds__(256) void moe_plan_kernel(int32_t* __restrict__ plan,
                                                       int32_t* __restrict__ block_counts,
                                                       int32_t* __restrict__ groups, int n_experts,
                                                       int n_blocks, int tile_rows) {
  const int e = threadIdx.x;
  int total = 0;
  if (e < n_experts)
    for (int b0 = 0; b0 < n_blocks; b0 += 16) {    // 16 loads in flight, then their prefix, then 16 stores
      int c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        c[i] = b0 + i < n_blocks ? block_counts[(int64_t)(b0 + i) * n_experts + e] : 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (b0 + i < n_blocks) block_counts[(int64_t)(b0 + i) * n_experts + e] = total;
        total += c[i];
      }
    }
  const int off = expert_rows(total, e, n_experts, tile_rows, true, groups);
  if (e < n_experts) plan[e] = off;
}

// One thread per (token, choice): the pair's row = expert's offset + its route workgroup's first
// row for that expert + its rank there; leaves the row in slot_of and the token in row_token[row]
// (the index the grouped GEMM gathers the activations by -- they are never copied).
__global__ __launch_bounds__(256) void moe_index_kernel(const int32_t* __restrict__ ids,
                                                        const int32_t* __restrict__ plan,
                                                        const int32_t* __restrict__ block_counts,
                                                        int32_t* __restrict__ slot_of,
                                                        int32_t* __restrict__ row_token, int n_pairs,
                                                        int top_k, int n_experts, int tokens_per_block) {
  const int pair = blockIdx.x * 256 + threadIdx.x;
  if (pair >= n_pairs) return;
  const int token = pair / top_k;
  const int e = ids[pair];
  const int slot = plan[e] + block_counts[(int64_t)(token / tokens_per_block) * n_experts + e] + slot_of[pair];
  slot_of[pair] = slot;
  row_token[slot] = token;
}

// Both of the above in one launch for up to kFusedPlanBlocks route workgroups: workgroup b adds up the counts itself (four threads per
// expert, each a quarter of the route workgroups) and places the pairs of route workgroup b; the first one writes the table.  A launch
// and the gap before it less: gate and experts_up together, us, 16 tokens 101 -> 98, 590 tokens 162 -> 160, 4096 299 -> 296, 16000
// 741 -> 733.  Every workgroup reads all counts, so their number squared bounds it: beyond the line the two kernels.
constexpr int kFusedPlanBlocks = 256;
__global__ __launch_bounds__(1024) void moe_plan_index_kernel(const int32_t* __restrict__ ids,
                                                              const int32_t* __restrict__ block_counts,
                                                              int32_t* __restrict__ slot_of, int32_t* __restrict__ row_token,
                                                              int32_t* __restrict__ groups, int n_pairs, int top_k, int n_experts,
                                                              int n_blocks, int tokens_per_block, int tile_rows) {
  __shared__ int s_total[4][256], s_before[4][256], s_base[256];
  const int e = threadIdx.x & 255, part = threadIdx.x >> 8;
  const int lo = n_blocks * part / 4, hi = n_blocks * (part + 1) / 4;
  int total = 0, before = 0;
  if (e < n_experts)
    for (int b0 = lo; b0 < hi; b0 += 16) {           // 16 loads in flight
      int c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = b0 + i < hi ? block_counts[(int64_t)(b0 + i) * n_experts + e] : 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        total += c[i];
        before += b0 + i < (int)blockIdx.x ? c[i] : 0;
      }
    }
  s_total[part][e] = total;
  s_before[part][e] = before;
  __syncthreads();
  total = s_total[0][e] + s_total[1][e] + s_total[2][e] + s_total[3][e];
  before = s_before[0][e] + s_before[1][e] + s_before[2][e] + s_before[3][e];
  // (Four waves' prefix sums; the other twelve repeat them, since everybody calls.)
  const int off = expert_rows(total, e, n_experts, tile_rows, blockIdx.x == 0 && part == 0, groups);
  if (part == 0) s_base[e] = off + before;
  __syncthreads();
  const int per_block = tokens_per_block * top_k, first = blockIdx.x * per_block;
  for (int i = threadIdx.x; i < per_block && first + i < n_pairs; i += 1024) {
    const int pair = first + i;
    const int slot = s_base[ids[pair]] + slot_of[pair];
    slot_of[pair] = slot;
    row_token[slot] = pair / top_k;
  }
}

// x[t] += sum_j wts[t][j] * y[slot_of[t][j]], j ascending, fp32.  Bound by its bytes (8192 tokens of 2048, 8 choices: 402 MB);
// a thread requests the rows of all choices together instead of slot, weight and row one after the other, and
// past the caches, since nobody reads them again.  experts_down with it, us, 30B-A3B shape: 16 tokens 46.6 -> 45.2, 590 90 -> 88.8,
// 8192 331 -> 326.5, 16000 572 -> 566.
__global__ __launch_bounds__(256) void moe_combine_kernel(float* __restrict__ x,
                                                          const bf16* __restrict__ y,
                                                          const int32_t* __restrict__ slot_of,
                                                          const float* __restrict__ wts, int64_t n_tokens,
                                                          int top_k, int d) {
  const int64_t d8 = d / 8;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_tokens * d8) return;
  const int64_t t = i / d8, c = i - t * d8;
  f32x8 acc = Vec8<float>::load(x + t * d + c * 8);
  bf16x8 v[kMaxChoices];
  float w[kMaxChoices];
#pragma unroll
  for (int j = 0; j < kMaxChoices; ++j)
    if (j < top_k) {
      const int64_t at = t * top_k + j;
      w[j] = wts[at];
      v[j] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(y + (int64_t)slot_of[at] * d + c * 8));
    }
#pragma unroll
  for (int j = 0; j < kMaxChoices; ++j)
    if (j < top_k)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = fmaf(w[j], static_cast<float>(v[j][e]), acc[e]);
  Vec8<float>::store(x + t * d + c * 8, acc);
}

int moe_route_blocks(int64_t n_tokens) {
  const int per = route_tokens_per_block(n_tokens);
  return (int)((n_tokens + per - 1) / per);
}

// Selection, row plan and index (up to kFusedPlanBlocks route workgroups; beyond, launch_moe_index has the index left to do).
void launch_moe_route(const float* logits, int32_t* ids, float* wts, int32_t* slot_of, int32_t* plan,
                      int32_t* block_counts, int32_t* groups, int32_t* row_token, int64_t n_tokens, int n_experts, int top_k,
                      int tile_rows, hipStream_t s) {
  const int n_blocks = moe_route_blocks(n_tokens), per_block = route_tokens_per_block(n_tokens);
  const int q = route_tokens_per_wave(n_tokens);
  launch_kernel(q == 2 ? moe_route_kernel<2> : moe_route_kernel<4>, dim3((unsigned)n_blocks), per_block / q * 64, 0, s,
      logits, ids, wts, slot_of, block_counts, (int)n_tokens, n_experts, top_k);
  if (n_blocks <= kFusedPlanBlocks)
    launch_kernel(moe_plan_index_kernel, dim3((unsigned)n_blocks), 1024, 0, s,
        ids, block_counts, slot_of, row_token, groups, (int)(n_tokens * top_k),
                                                                    top_k, n_experts, n_blocks, per_block, tile_rows);
  else
    launch_kernel(moe_plan_kernel, 1, 256, 0, s, plan, block_counts, groups, n_experts, n_blocks, tile_rows);
}

void launch_moe_index(const int32_t* ids, const int32_t* plan, const int32_t* block_counts,
                      int32_t* slot_of, int32_t* row_token, int64_t n_tokens, int top_k, int n_experts,
                      hipStream_t s) {
  if (moe_route_blocks(n_tokens) <= kFusedPlanBlocks) return;    // done with the plan
  const int64_t pairs = n_tokens * top_k;
  launch_kernel(moe_index_kernel, dim3((unsigned)((pairs + 255) / 256)), 256, 0, s, ids, plan, block_counts, slot_of, row_token,
                                                                        (int)pairs, top_k, n_experts,
                                                                        route_tokens_per_block(n_tokens));
}

void launch_moe_combine(float* x, const void* y, const int32_t* slot_of, const float* wts,
                        int64_t n_tokens, int top_k, int d, hipStream_t s) {
  const int64_t n = n_tokens * (d / 8);
  launch_kernel(moe_combine_kernel, dim3((unsigned)((n + 255) / 256)), 256, 0, s, x, (const bf16*)y, slot_of, wts, n_tokens,
                                                                       top_k, d);
}

}  // namespace fp
