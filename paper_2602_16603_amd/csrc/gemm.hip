// Dense projections of the prefill layer: C[M,N] = A[M,K] * W[N,K]^T (both operands K-major),
// FlowPrefill Eq. (1) and the operators qkv_proj / o_proj / gate_up_proj / down_proj of
// Section 5.1.  bf16 path: MFMA tiles with fp32 accumulation, operands staged through LDS by DMA (the
// large-tile and the ring kernel, on 16x16x32) or through registers (the kernel for any operand
// address, on 32x32x16).  fp32 path (debug): MFMA tiles in fp32 throughout.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_plan.h"
#include "kernels.h"
#include "launch.h"

namespace fp {

// ------------------------------------------------------------------------------------------
// Workgroup -> output tile mapping.  Hardware deals consecutive workgroup ids round-robin over
// the 8 XCDs, each with its own L2.  The map gives every XCD a contiguous run of logical tiles
// and walks that run in column-panels of `kGroupM` tile rows, so the ~32 tiles an XCD has in
// flight share a small set of A row-panels and W row-panels in its L2.
// ------------------------------------------------------------------------------------------
constexpr int kXcds = 8;
constexpr int kGroupM = 8;

// EVEN: panels of equally many tile rows, at most kGroupM (the large kernel, whose L2 warm-up wants sharers in every panel; to
// the others it makes no difference or costs: 4261 x 992 x 4888 on 128-row tiles 85 -> 92 us, 4859 x 1992 x 5832 with its K
// tail 142 -> 150).  Returns the panel's rows.
template <bool EVEN = false>
__device__ __forceinline__ int tile_of_workgroup(int wg, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int xcd = wg % kXcds;
  const int local = wg / kXcds;
  const int base = total / kXcds, rem = total % kXcds;
  const int logical = xcd * base + min(xcd, rem) + local;
  const int groups = (tiles_m + kGroupM - 1) / kGroupM, rows = EVEN ? (tiles_m + groups - 1) / groups : kGroupM;
  const int per_group = rows * tiles_n;
  const int group = logical / per_group;
  const int in_group = logical - group * per_group;
  const int gm = min(rows, tiles_m - group * rows);
  tm = group * rows + in_group % gm;
  tn = in_group / gm;
  return gm;
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA GEMM for operands at any address (register-staged loads).  WGM x WGN waves; each wave
// owns a (BM/WGM)x(BN/WGN) block of 32x32 MFMA accumulators.  SWIGLU: the 64 W rows of a wave's two column blocks are
// 32 gate rows and the up rows of the same 32 outputs.  K is consumed 64 at a time.  LDS rows hold 64 bf16 = eight 16-byte chunks.  The
// gfx950 LDS has 64 four-byte banks (256 B per clock for reads); a ds_read_b128 is served one
// half-wave after the other and a half-wave costs max(2, most lanes on one 16-byte bank group)
// clocks.  Two consecutive 128-byte rows fill one bank period, so chunk c of row r is stored at
// chunk position c ^ ((r >> 1) & 7): the 32 rows a half-wave reads then put exactly two lanes on
// every bank group (measured: full rate, against half rate with key r & 7).
// ------------------------------------------------------------------------------------------
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // 16 bytes at any bf16's address

// up > 0 (SwiGLU): rows 64 u + (0..31) of the tile are rows row0 + 32 u + (0..31) of src, the next 32 lie `up` rows on.
template <int ROWS, int NT>
__device__ __forceinline__ void load_tile_global(const bf16* __restrict__ src, int64_t ld,
                                                 int row0, int row_max, int k0, int K, int tid,
                                                 u32x4 (&regs)[ROWS * 8 / NT], int up = 0) {
#pragma unroll
  for (int i = 0; i < ROWS * 8 / NT; ++i) {
    const int c = tid + i * NT;
    const int row = c >> 3, ch = c & 7;
    const int64_t grow = up ? min(row0 + (row >> 6) * 32 + (row & 31), row_max) + (int64_t)((row >> 5) & 1) * up
                            : min(row0 + row, row_max);
    const int k = k0 + ch * 8;
    if (k < K)
      regs[i] = *reinterpret_cast<const u32x4_any*>(src + grow * ld + k);
    else
      regs[i] = u32x4{0, 0, 0, 0};
  }
}

template <int ROWS, int NT>
__device__ __forceinline__ void store_tile_lds(bf16* dst, int tid, const u32x4 (&regs)[ROWS * 8 / NT]) {
#pragma unroll
  for (int i = 0; i < ROWS * 8 / NT; ++i) {
    const int c = tid + i * NT;
    const int row = c >> 3, ch = c & 7;
    *reinterpret_cast<u32x4*>(dst + row * kBK + ((ch ^ ((row >> 1) & 7)) << 3)) = regs[i];
  }
}

template <int BM, int BN, int WGM, int WGN, bool RESID, bool SWIGLU = false>
__global__ __launch_bounds__(WGM * WGN * 64) void gemm_bf16_kernel(const bf16* __restrict__ A,
                                                           const bf16* __restrict__ W,
                                                           void* __restrict__ Cout, int M, int N,
                                                           int K, int tiles_m, int tiles_n) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16* sA = reinterpret_cast<bf16*>(smem_raw);            // [2][BM*64]
  bf16* sB = sA + 2 * BM * kBK;                            // [2][BN*64]

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  int tile_m, tile_n;
  tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * (SWIGLU ? BN / 2 : BN);   // (SWIGLU: N is the number of outputs)
  const int up = SWIGLU ? N : 0;
  static_assert(!SWIGLU || (WTN == 64 && !RESID));

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  u32x4 ra[BM * 8 / NT], rb[BN * 8 / NT];
  const int kt_count = (K + kBK - 1) / kBK;
  load_tile_global<BM, NT>(A, K, m0, M - 1, 0, K, tid, ra);
  load_tile_global<BN, NT>(W, K, n0, N - 1, 0, K, tid, rb, up);
  store_tile_lds<BM, NT>(sA, tid, ra);
  store_tile_lds<BN, NT>(sB, tid, rb);
  __syncthreads();

  const int frag_row = lane & 31, frag_half = lane >> 5;
  for (int kt = 0; kt < kt_count; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < kt_count) {
      load_tile_global<BM, NT>(A, K, m0, M - 1, (kt + 1) * kBK, K, tid, ra);
      load_tile_global<BN, NT>(W, K, n0, N - 1, (kt + 1) * kBK, K, tid, rb, up);
    }
    const bf16* cA = sA + cur * BM * kBK;
    const bf16* cB = sB + cur * BN * kBK;
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8 fa[TM], fb[TN];
      const int ch = kk * 2 + frag_half;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WTM + i * 32 + frag_row;
        fa[i] = *reinterpret_cast<const bf16x8*>(cA + row * kBK + ((ch ^ ((row >> 1) & 7)) << 3));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * WTN + j * 32 + frag_row;
        fb[j] = *reinterpret_cast<const bf16x8*>(cB + row * kBK + ((ch ^ ((row >> 1) & 7)) << 3));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < kt_count) {
      store_tile_lds<BM, NT>(sA + (cur ^ 1) * BM * kBK, tid, ra);
      store_tile_lds<BN, NT>(sB + (cur ^ 1) * BN * kBK, tid, rb);
    }
    __syncthreads();
  }

  // Epilogue.  Accumulator register r of lane l is C[8*(r/4) + 4*(l/32) + r%4][l%32] of its
  // 32x32 block: the 32 lanes of a half-wave write 32 consecutive columns of one row.
  if constexpr (SWIGLU) {
    const int n = n0 + wn * 32 + frag_row;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
        if (m < M && n < N)
          reinterpret_cast<bf16*>(Cout)[(int64_t)m * N + n] =
              static_cast<bf16>(silu_mul_f32(static_cast<float>(static_cast<bf16>(acc[i][0][r])),
                                             static_cast<float>(static_cast<bf16>(acc[i][1][r]))));
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WTN + j * 32 + frag_row;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * frag_half + (r & 3);
        if (m < M && n < N) {
          if (RESID) {
            float* c = reinterpret_cast<float*>(Cout) + (int64_t)m * N + n;
            *c = *c + acc[i][j][r];
          } else {
            reinterpret_cast<bf16*>(Cout)[(int64_t)m * N + n] = static_cast<bf16>(acc[i][j][r]);
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA GEMM, one wave per SIMD (the fast path; K % 64 == 0, or KTAIL below).
//
// 256x256 output tile, K consumed 64 at a time, 256 threads = 4 waves, one per SIMD, each with the
// whole 512-register budget: a wave owns a 128x128 block of the tile, 8x8 accumulators of 16x16 =
// 256 accumulator registers, multiplied with v_mfma_f32_16x16x32_bf16 (on random operands the
// register-only loop of this instruction sustains 2.0-2.1 PFLOP/s where 32x32x16 sustains
// 1.8-1.9: the chip is power limited and the smaller accumulator costs less energy per FLOP).
// The wave's instruction stream is software-pipelined by k-step (32 of K = 64 MFMAs = 1024
// matrix-pipe cycles): every LDS fragment read of the next k-step and every global load sits
// alone behind an MFMA, inside the 16 cycles the matrix pipe is busy with it; one s_barrier per
// k-tile.  The loop body is straight-line code on purpose: the compiler keeps the 256
// accumulators in place in the accumulation registers only while no control flow crosses them, so
// "nothing left to fetch" is expressed through an empty buffer descriptor, never through a branch.
//
// Global -> LDS goes through the DMA path (buffer_load_dwordx4 ... lds: no VGPR staging, no
// ds_write).  A DMA instruction writes lane i's 16 bytes at base + 16*i, i.e. one wave fills
// eight consecutive 128-byte LDS rows; the LDS swizzle is obtained by permuting which 16-byte
// global chunk each lane fetches.  Two LDS stages (A and W, 32 KB each per stage; less high or narrow tiles have three, below) as four
// separate __shared__ arrays, so that the compiler can tell that DMA in flight to one stage does
// not alias LDS reads of the other (otherwise it would serialise them with vmcnt(0)).  Wave w
// fetches rows [64w, 64w+64) of both operands, 16 instructions per k-tile, all in the k-step after
// the barrier that frees the stage; the other k-step gives them time to land.  Operand panels are addressed through raw buffer descriptors
// sized to the valid rows, so row tails of A and W read as zero.
//
// L2 warm-up.  The 32 workgroups running on one XCD share operand panels (8 tile rows x 4 tile
// columns under tile_of_workgroup), run in step, and would all ask the XCD's L2 for the same
// 128-byte lines within a few hundred cycles: one request misses and every sharer's request
// queues behind that miss (measured: 480 cycles average L2 read latency in gate_up_proj, 3300
// cycles per k-tile in down_proj).  Instead each workgroup asks for its share of the lines three
// k-tiles ahead of the DMA -- every 4th row of its A panel (wave 0) and every 8th row of its W
// panel (wave 1; every 4th or 2nd where fewer row tiles share it), the shares rotating with the k-tile -- with a
// one-dword-per-lane load into a dummy LDS pad, so the DMA requests of all sharers find the line resident (2180-2240 cycles per
// k-tile for both projections).  The pad load is the last VMEM instruction before the wave's
// wait, which therefore asks for "all but one" and never blocks on it.
// ------------------------------------------------------------------------------------------
constexpr int kWaitVm0 = 0x0F70;   // s_waitcnt vmcnt(0)           (expcnt/lgkmcnt untouched)
constexpr int kWaitVm1 = 0x0F71;   // s_waitcnt vmcnt(1)
template <int N> constexpr int wait_vm() { return 0x0F70 | (N & 15) | ((N >> 4) << 14); }   // s_waitcnt vmcnt(N)
constexpr int kWaitLgkm0 = 0xC07F; // s_waitcnt lgkmcnt(0)         (vmcnt/expcnt untouched)
constexpr int kWarmAhead = 3;      // k-tiles between the L2 warm-up load and the DMA of the same lines

typedef float f32x4_acc __attribute__((ext_vector_type(4)));
template <int MI, int NJ>
struct W4Frags {     // MFMA operands of one k-step (32 of K): MI 16-row blocks of A and NJ of W
  bf16x8 a[MI];
  bf16x8 b[NJ];
};

// Raw buffer descriptor over `bytes` bytes at `base` (stride 0, 32-bit offsets, reads past the
// end return zero -- which is how row tails of A and W are zero-filled -- and writes past the end
// are dropped).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// NT: non-temporal, for lines that one workgroup reads and nobody after it.
constexpr int kAuxNonTemporal = 2;                 // of a buffer instruction: the nt bit
template <bool NT = false>
__device__ __forceinline__ void w4_dma(__amdgpu_buffer_rsrc_t r, bf16* lds_rows, uint32_t voff, int kbyte) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds_rows, 16, voff, kbyte, 0, NT ? kAuxNonTemporal : 0);
}

// One k-step: MI NJ MFMAs from `cur` (A block s against the NJ W blocks, s = 0 .. MI - 1; MI = 8: the 256-row
// tile described here, less: the row tiles of few rows of the grouped launches; NJ = 8: 256 columns, NJ = 4: the 128-column
// tile of short requests, with half the W fragments and DMA instructions in the same slots).  Every other
// instruction sits alone behind an MFMA: the fragment reads of the next k-step (EARLY: all in its first half,
// for the k-step that ends at the barrier, so that the wait in front of the barrier finds them done; else
// spread over the k-step), in the order of their first use (all of W, then the A blocks); and D0 .. D1 - 1 of the wave's
// MI + NJ DMA instructions (its A rows, then its W rows, 8 rows of 128 bytes each), evenly over the k-step: the CU takes one per 16
// cycles from its four waves together.
// The MFMA is written as inline assembly to accumulate in place: the compiler leaves the
// destination of this 4-pass instruction free to differ from its accumulator input, which
// overflows the completely used accumulation registers (the 8-pass 32x32x16 is tied by itself).
// No accumulator is touched twice within MI NJ MFMAs, and LDS results reach the operands through
// the s_waitcnt the compiler places for the asm inputs, so no software-managed hazard arises.
enum { kReadsNone, kReadsSpread, kReadsEarly };
template <int READS, int D0, int D1, int MI, int NJ, bool NT = false>
__device__ __forceinline__ void w4_block(f32x4_acc (&acc)[MI][NJ], const W4Frags<MI, NJ>& cur, W4Frags<MI, NJ>& nxt,
                                         const bf16* rA, const bf16* rB, int pch,
                                         __amdgpu_buffer_rsrc_t rs_a, __amdgpu_buffer_rsrc_t rs_w, bf16* dA,
                                         bf16* dB, const uint32_t (&voff_a)[MI], const uint32_t (&voff)[8], int kbyte) {
  constexpr int kSpread = (MI + NJ + MI - 1) / MI;    // per A block, so that MI blocks place all of them
  constexpr int kReads = READS == kReadsNone ? 0 : READS == kReadsSpread ? kSpread : kSpread < NJ / 2 ? 2 * kSpread : NJ;
  constexpr int kTwice = D1 > D0 ? 2 * (D1 - D0) : 1;
  static_assert(kSpread <= NJ && 0 <= D0 && D0 <= D1 && D1 <= MI + NJ);
#pragma unroll
  for (int s = 0; s < MI; ++s) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[s][j]) : "v"(cur.b[j]), "v"(cur.a[s]));
      if (j < kReads) {
        const int r = s * kReads + j;
        if (r < NJ) nxt.b[r] = *reinterpret_cast<const bf16x8*>(rB + r * 16 * kBK + pch);
        else if (r < NJ + MI) nxt.a[r - NJ] = *reinterpret_cast<const bf16x8*>(rA + (r - NJ) * 16 * kBK + pch);
      }
#pragma unroll
      for (int d = D0; d < D1; ++d) {
        // (256 rows by 256 columns: two behind the second half of every A block, 0.3 % faster than one behind every fourth MFMA)
        const int slot = D1 - D0 == 16 ? 4 + (d / 2) * 8 + d % 2 * 2 : (2 * (d - D0) + 1) * MI * NJ / kTwice;
        if (slot != s * NJ + j) continue;
        if (d < MI) w4_dma(rs_a, dA + d * 8 * kBK, voff_a[d], kbyte);
        else w4_dma<NT>(rs_w, dB + (d - MI) * 8 * kBK, voff[d - MI], kbyte);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

__device__ __forceinline__ void w4_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// EPI selects the epilogue: bf16 store, fp32 residual read-modify-write, (split-K) fp32 partial
// sums to a workspace [split][M][N] that splitk_reduce_kernel adds up in a fixed order, or the
// fused SwiGLU: W is [2N][K] = [gate rows | up rows], the tile covers 128 FFN columns, the 128 W
// rows a wave multiplies are 64 gate rows followed by the 64 up rows of the same columns, so its
// accumulator blocks [i][0..1] and [i][2..3] are gate and up of the same output elements, and the
// output [M][N] is silu(bf16(gate)) * bf16(up) -- the values, rounding included, that the
// separate gate_up GEMM + silu_mul operators produce, without the [M][2N] round trip through HBM.
enum { kEpiBf16 = 0, kEpiResidual = 1, kEpiPartial = 2, kEpiSwiGLU = 3 };

//
// GROUPED (mixture-of-experts): the launch covers many independent problems that share N and K.
// groups[0] = number of row tiles; entry i (three ints from groups[1 + 3 i]) = {expert, first
// row, rows (<= 256)}: the tile multiplies rows [first, first + rows) of A with expert's weight
// matrix (W holds the experts' matrices back to back) into the same rows of C.  The grid is sized
// for the worst case on the host; workgroups past groups[0] row tiles return at once.
// With a_rows != null the rows of A are GATHERED: row r of the launch's row space is row a_rows[r]
// of A (the tokens routed to an expert, fetched by the DMA from where they lie -- no gathered copy
// of the activations is ever written); the kernel's M argument then holds the number of rows of A.
//
// An expert of a few dozen to a few hundred rows does not fill 256-row tiles: the kernel holds the tile on 64, 96, .. 256
// rows and takes the one that a row tile's rows fit (the plan spreads an expert's rows evenly over its tiles: moe_plan_kernel).
// What bounds these launches is the latency of their lines rather than MFMAs (15 % fewer of those gave 4 % at 8192
// tokens): W panels come from HBM for one to three row tiles, so every (expert, column tile) starts at another k-tile, as
// in the kernel for few rows below, and the L2 warm-up asks for more of them.  30B-A3B shape, us, experts_up / experts_down
// (with the combine): 2000 tokens 244 / 141 -> 193 / 132 (even tiles 232 / 133), 5000 tokens 340 / 252 -> 303 / 231 (314 / 240),
// 8192 tokens 429 / 343 -> 395 / 328 (425 / 341), 16000 tokens 720 / 605 -> 675 / 582.  (The switch over seven bodies spills 15 to 20
// scalar registers, none of them inside a loop over k.)
//
// NJ = 4: the tile is half as wide (128 W rows per stage, wave tile 128 x 64).  A request of a few
// hundred tokens has one or two row tiles: the narrow tile doubles the number of output tiles, so
// the chip is occupied with half as many K ranges -- half the fp32 partial sums through memory,
// and the fused gate_up projection of a 256-token request needs no K ranges at all (measured: a
// 256-token request through the 8B-shaped stack 7.3 -> 6.5 ms; from three row tiles on the MFMAs
// bound the launch and the wide tile's operand reuse wins).  Such a launch streams its weights from
// HBM, every line for one or two workgroups only, and what a CU gets is its bytes in flight per
// latency: the narrow tile's stages are three (144 KB, filled two to three k-tiles ahead) instead of two with
// L2 warm-up.  Cold weights, 256 tokens of the 8B shape: gate_up 81 -> 71 us, down 48 -> 44;
// 512 tokens: down 74 -> 66.  (Three stages of the 256-row wide tile would take 192 KB.)
//
// STREAM (NJ = 4, one row tile, not cut): W is loaded non-temporally, as in the kernel for few rows below.  Narrow uncut tiles
// may start at another k-tile (start_groups).
//
// Three stages (the narrow tile, and the wide one up to 160 rows, where they fit): half of a k-tile's DMA is issued in either k-step.  A CU
// takes one DMA instruction per 16 cycles from its four waves, so all of a k-tile's in one k-step took longer than that k-step's
// MFMAs on every tile but 256 x 256 (64 x 16 cycles there, as many as its MFMAs); with two stages the other k-step is what
// they have to land in, and they are spread evenly (224 rows: 2100 -> 2040 cycles a k-tile).  Cold, us, with the heights chosen anew:
// 600 x 14336 x 4096 SwiGLU 133 -> 122, 777 149 -> 145, 1300 x 6144 x 4096 66 -> 58, 1500 x 27648 x 5120 SwiGLU 632 -> 583.
//
// ROWS: the tile on 96, 128, .. 256 rows, the same sums in the same order.  What an uncut launch of few
// rounds of tiles loses is its last, partly filled round and the padding of its last row tile; another height often
// comes out better (large_tile_rows).
//
// KTAIL (256-column tile, not cut): K is not a multiple of 64; its last K % 64 columns (a multiple of 8) follow the
// main loop as one more k-tile, not pipelined, whose missing 16-byte chunks are fetched from outside the
// descriptors (K < 64: there is nothing else; the prologue's k-tile 0 is overwritten unread).  K rows then start at odd multiples
// of 16 bytes, which the DMA does not mind.  8192 x 8192 x 2056: 408 us on register-staged 128x128 tiles, 265 here (1.04 PFLOP/s;
// rows that straddle lines cost the rest).
template <int EPI, bool GROUPED = false, int NJ = 8, bool KTAIL = false, int ROWS = 256, bool STREAM = false>
__global__ __launch_bounds__(256) void gemm_bf16_w4_kernel(const bf16* __restrict__ A,
                                                           const bf16* __restrict__ W,
                                                           void* __restrict__ Cout, int M, int N,
                                                           int K, int tiles_m, int tiles_n,
                                                           int kt_per_split, int start_groups,
                                                           const int32_t* __restrict__ groups,
                                                           const int32_t* __restrict__ a_rows) {
  constexpr bool RESID = EPI == kEpiResidual;
  constexpr bool SWIGLU = EPI == kEpiSwiGLU;
  constexpr int WR = 32 * NJ;                        // W rows per stage (256 or 128)
  constexpr int Q = WR / 4;                          // of which each wave fetches this many
  constexpr int BM = ROWS, BN = SWIGLU ? WR / 2 : WR;   // output rows and columns per tile
  constexpr bool kStarts = NJ == 4 && (EPI == kEpiBf16 || SWIGLU);   // may start at another k-tile than 0
  static_assert(BM % 32 == 0 && BM <= 256 && (!GROUPED || BM == 256) && (!STREAM || kStarts));
  __shared__ __attribute__((aligned(1024))) bf16 sA0[BM * kBK];
  __shared__ __attribute__((aligned(1024))) bf16 sA1[BM * kBK];
  __shared__ __attribute__((aligned(1024))) bf16 sB0[(WR > BM ? WR : BM) * kBK];   // (as large as an A stage: the epilogue
  __shared__ __attribute__((aligned(1024))) bf16 sB1[(NJ == 8 ? 256 : WR) * kBK];   //  stages its wave's outputs through the first four)
  constexpr bool kThree = NJ == 4 || (ROWS <= 160 && !GROUPED && !KTAIL);         // stages: three where they fit, else two
  __shared__ __attribute__((aligned(1024))) bf16 sA2[kThree ? BM * kBK : 8];
  __shared__ __attribute__((aligned(1024))) bf16 sB2[kThree ? WR * kBK : 8];
  __shared__ __attribute__((aligned(256))) uint32_t sWarm[NJ == 8 ? 4 * 64 : 4];   // landing pad of the L2 warm-up loads

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;           // 2 x 2 waves, wave tile 16 MI x WR/2 (SwiGLU: 16 MI x WR/4 outputs)
  int tile_m, tile_n, share_m, rot = 0, w_sharers = 2;
  bool shared = true;                                // somebody else reads these rows of W
  int a_total_rows = 0;
  const int n_tiles = tiles_m * tiles_n;
  const int split = GROUPED ? 0 : blockIdx.x / n_tiles;   // which K range (0 unless split-K)
  if (GROUPED) {
    // Consecutive workgroup ids go to the 8 XCDs in turn, each with its own L2.  Every XCD takes a
    // contiguous run of the row-tile table (row tiles of one expert are neighbours in it) and walks
    // it row tile by row tile, all column tiles of a row tile in a row: the workgroups an XCD has
    // in flight then share the A panel of their row tile (all column tiles) and the W panels of
    // their expert (its two or three row tiles) through that L2, instead of each fetching both
    // panels from the fabric.
    const int n_row_tiles = groups[0];
    const int quota = (n_row_tiles + kXcds - 1) / kXcds;
    const int in_xcd = blockIdx.x / kXcds;
    const int ti = (blockIdx.x % kXcds) * quota + in_xcd / tiles_n;
    if (in_xcd / tiles_n >= quota || ti >= n_row_tiles) return;   // whole workgroup, before any barrier
    const int expert = groups[1 + 3 * ti], first = groups[2 + 3 * ti];
    a_total_rows = M;                                // gathered mode: the caller passes the rows of A here
    M = groups[3 + 3 * ti];
    if (a_rows) a_rows += first;                     // row r of the tile is row a_rows[r] of A
    else A += (int64_t)first * K;
    W += (int64_t)expert * (SWIGLU ? 2 : 1) * N * K;
    Cout = reinterpret_cast<char*>(Cout) + (int64_t)first * N * (EPI == kEpiBf16 || SWIGLU ? 2 : 4);
    tile_m = 0;
    tile_n = in_xcd % tiles_n;
    share_m = ti;
    rot = (expert * tiles_n + tile_n) % (K / kBK);
    shared = (ti > 0 && groups[1 + 3 * (ti - 1)] == expert) || (ti + 1 < n_row_tiles && groups[1 + 3 * (ti + 1)] == expert);
  } else {
    w_sharers = tile_of_workgroup<!KTAIL>(blockIdx.x - split * n_tiles, tiles_m, tiles_n, tile_m, tile_n);
    share_m = tile_m;
    if (kStarts) rot = k_start(tile_n * BN, K, start_groups) / kBK;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  // The tile itself, on 32 MI rows.
  auto tile = [&](auto mi) __attribute__((always_inline)) {
  constexpr int MI = decltype(mi)::value;
  const int kt_first = split * kt_per_split;
  const int kt_count = min(kt_per_split, K / kBK - kt_first);
  const int kbyte0 = kt_first * kBK * 2;
  auto kbyte = [&](int u) __attribute__((always_inline)) {   // of k-tile u of this workgroup
    return kbyte0 + (!GROUPED && !kStarts ? u : u + rot >= kt_count ? u + rot - kt_count : u + rot) * kBK * 2;
  };

  // DMA sources.  Wave w fetches LDS rows [8 MI w, 8 MI w + 8 MI) of A and [Q w, Q w + Q) of W, 8 rows per instruction;
  // voff[j] is lane's byte offset inside the wave's panel for instruction j (the same for A
  // and W: both have K as row stride): row 8j + lane/8, 16-byte chunk (lane%8) ^ swizzle key.
  uint32_t voff[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int row = j * 8 + (lane >> 3);
    const int ch = (lane & 7) ^ ((row >> 1) & 7);
    voff[j] = (uint32_t)((row * K + ch * 8) * 2);
  }
  // A rows of the same lanes: the same offsets, unless the rows are gathered (then absolute
  // offsets into all of A, rows past the tile's end pointing outside the descriptor).
  uint32_t voff_a[MI];
#pragma unroll
  for (int j = 0; j < MI; ++j) {                     // (8 MI w is not a multiple of 16 where MI and w are odd)
    const int row = j * 8 + (lane >> 3);
    const int ch = (lane & 7) ^ (((8 * MI * wave + row) >> 1) & 7);
    voff_a[j] = MI % 2 ? (uint32_t)((row * K + ch * 8) * 2) : voff[j];
  }
  const bool gathered = GROUPED && a_rows != nullptr;
  if (gathered) {
#pragma unroll
    for (int j = 0; j < MI; ++j) {
      const int row = 8 * MI * wave + j * 8 + (lane >> 3);          // tile_m = 0 in grouped launches
      const int ch = (lane & 7) ^ ((row >> 1) & 7);
      const int src = row < M ? a_rows[row] : -1;
      voff_a[j] = src >= 0 ? (uint32_t)((src * K + ch * 8) * 2) : kOffOutOfRange;
    }
  }
  // Plain: W rows n0 + Q w ..; SwiGLU: LDS rows 2Q wn + (0..Q-1) are gate rows n0 + Q wn + (0..Q-1),
  // rows 2Q wn + Q + (0..Q-1) the up rows N + the same -- waves 2*wn and 2*wn+1 fetch them.
  const int w_col0 = SWIGLU ? n0 + Q * (wave >> 1) : n0 + Q * wave;
  const int64_t w_row0 = SWIGLU ? (int64_t)(wave & 1) * N + w_col0 : w_col0;
  const int a_panel_rows = __builtin_amdgcn_readfirstlane(min(8 * MI, max(0, M - m0 - 8 * MI * wave)));
  const int w_rows = __builtin_amdgcn_readfirstlane(min(Q, max(0, N - w_col0)));
  const __amdgpu_buffer_rsrc_t rsrc_a =
      gathered ? panel_rsrc(A, (uint32_t)(a_total_rows * K * 2))
               : panel_rsrc(A + (int64_t)(m0 + 8 * MI * wave) * K, (uint32_t)(a_panel_rows * K * 2));
  const __amdgpu_buffer_rsrc_t rsrc_w = panel_rsrc(W + w_row0 * K, (uint32_t)(w_rows * K * 2));
  const __amdgpu_buffer_rsrc_t rsrc_none = panel_rsrc(A, 0u);
  bf16* const dA0 = sA0 + 8 * MI * wave * kBK;
  bf16* const dA1 = sA1 + 8 * MI * wave * kBK;
  bf16* const dA2 = sA2 + 8 * MI * wave * kBK;
  bf16* const dB0 = sB0 + Q * wave * kBK;
  bf16* const dB1 = sB1 + Q * wave * kBK;
  bf16* const dB2 = sB2 + Q * wave * kBK;

  // L2 warm-up sources: wave 0 lane l -> A row 4l + share, wave 1 lane l (below 256 / shares) -> W-stage row shares l +
  // share (SwiGLU: stage row r is gate row n0 + Q*(r/2Q) + r%Q, or the up row N + that, for
  // r%2Q >= Q).  The share is added through the scalar offset.
  uint32_t* const warm = sWarm + 64 * wave;
  const int warm_rows_a = __builtin_amdgcn_readfirstlane(min(BM, M - m0));
  const int warm_rows_w = __builtin_amdgcn_readfirstlane(SWIGLU ? N + min(BN, N - n0) : min(BN, N - n0));
  const __amdgpu_buffer_rsrc_t rsrc_warm_a = panel_rsrc(A + (int64_t)m0 * K, (uint32_t)(warm_rows_a * K * 2));
  const __amdgpu_buffer_rsrc_t rsrc_warm_w = panel_rsrc(W + (int64_t)n0 * K, (uint32_t)(warm_rows_w * K * 2));
  // As many shares of W as workgroups to ask for them (warm_shares).
  // Grouped launches: a W panel is shared by the two or three row tiles of its expert only, so there waves 1 and 2 ask
  // for every other row of it, and nobody where the expert has one tile; gathered rows of A have an address each, and
  // their shares do not rotate (8192 tokens of the 30B-A3B shape: experts_up 409 -> 396 us, experts_down 335 -> 329).
  const int w_shares = warm_shares(w_sharers);
  const bool warm_up = GROUPED ? shared : !kThree || warm_three_stages(K, SWIGLU);
  const __amdgpu_buffer_rsrc_t rsrc_warm = !warm_up ? rsrc_none
                                           : wave == 0 ? (gathered ? rsrc_a : rsrc_warm_a)
                                           : w_shares > 0 && (wave == 1 || (w_shares == 2 && wave == 2)) ? rsrc_warm_w : rsrc_none;
  const int warm_mask = wave == 0 ? 3 : max(w_shares, 1) - 1;
  const int warm_id = wave == 0 ? (tile_n & 3) : (share_m & warm_mask);
  const int warm_step = gathered && wave == 0 ? 0 : K * 2;
  uint32_t voff_warm;
  {
    const int r0 = (lane + (wave == 2 ? 64 : 0)) * w_shares;   // waves 1 and 2: W-stage row of this lane's share 0
    const int64_t wrow = SWIGLU ? (int64_t)((r0 / Q) & 1) * N + Q * (r0 / (2 * Q)) + (r0 % Q) : r0;
    voff_warm = wave == 0 ? (uint32_t)(lane * 4 * K * 2) : r0 < WR ? (uint32_t)(wrow * K * 2) : kOffOutOfRange;
    if (gathered && wave == 0) {
      const int row = 4 * lane + warm_id;
      voff_warm = row < M ? (uint32_t)(a_rows[row] * K * 2) : kOffOutOfRange;
    }
  }

  // MFMA fragment addresses: lane reads row (lane%16) of each 16-row block, k-chunk 4*ks + lane/16
  // of k-step ks, at its swizzled position.
  const int frag_row = lane & 15, quad = lane >> 4;
  const int key = (lane >> 1) & 7;
  const int pch0 = ((0 + quad) ^ key) << 3, pch1 = ((4 + quad) ^ key) << 3;
  const bf16* const rA0 = sA0 + (wm * 16 * MI + frag_row) * kBK;
  const bf16* const rA1 = sA1 + (wm * 16 * MI + frag_row) * kBK;
  const bf16* const rA2 = sA2 + (wm * 16 * MI + frag_row) * kBK;
  const bf16* const rB2 = sB2 + (wn * (WR / 2) + frag_row) * kBK;
  const bf16* const rB0 = sB0 + (wn * (WR / 2) + frag_row) * kBK;
  const bf16* const rB1 = sB1 + (wn * (WR / 2) + frag_row) * kBK;

// `last`: the last k-tile of the trip, which exists (the compiler does not always see that those before it do).
#define W4_WARM(u, last)                                                                                      \
  __builtin_amdgcn_raw_ptr_buffer_load_lds((u) <= (last) || (u) < kt_count ? rsrc_warm : rsrc_none,           \
                                           (__attribute__((address_space(3))) void*)warm, 4, voff_warm,       \
                                           kbyte(u) + ((warm_id - (u)) & warm_mask) * warm_step, 0, 0)
  f32x4_acc acc[MI][NJ];
  W4Frags<MI, NJ> f0, f1;
  if constexpr (!kThree) {
    // Prologue: k-tile 0 into stage 0 (awaited), k-tile 1 into stage 1 (in flight), then one warm-up
    // load, so that "all but one" is the right wait from the first barrier on.
#pragma unroll
    for (int s = 0; s < MI; ++s) w4_dma(rsrc_a, dA0 + s * 8 * kBK, voff_a[s], kbyte(0));
#pragma unroll
    for (int s = 0; s < NJ; ++s) w4_dma(rsrc_w, dB0 + s * 8 * kBK, voff[s], kbyte(0));
    {
      const __amdgpu_buffer_rsrc_t ra1 = kt_count > 1 ? rsrc_a : rsrc_none, rw1 = kt_count > 1 ? rsrc_w : rsrc_none;
#pragma unroll
      for (int s = 0; s < MI; ++s) w4_dma(ra1, dA1 + s * 8 * kBK, voff_a[s], kbyte(1));
#pragma unroll
      for (int s = 0; s < NJ; ++s) w4_dma(rw1, dB1 + s * 8 * kBK, voff[s], kbyte(1));
    }
    W4_WARM(kWarmAhead - 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    // Cleared while the first k-tile is on its way.
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) asm volatile("" : "+a"(acc[i][j]));   // materialise the zeros here, not at first use
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm<MI + NJ + 1>());   // all but k-tile 1 and the warm-up load
    w4_barrier();
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (s < NJ) f0.b[s] = *reinterpret_cast<const bf16x8*>(rB0 + s * 16 * kBK + pch0);
      if (s < MI) f0.a[s] = *reinterpret_cast<const bf16x8*>(rA0 + s * 16 * kBK + pch0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // k-tile t on stage c (the other stage: o).  On entry f0 holds k-step 0 of tile t and tile t+1 is
    // in flight to stage o.  k-step 0 reads k-step 1's fragments; then everything but the last
    // warm-up load must have landed; the barrier tells all waves that tile t+1 is complete and stage
    // c is free; k-step 1 (fed from registers) refills stage c with tile t+2, asks for the wave's
    // share of tile t+3's lines, and starts reading tile t+1.
#define W4_TILE(first, x, last, c, o)                                                                         \
  {                                                                                                           \
    const int t2_ = (first) + (x) + 2;                                                                        \
    const bool more_ = (x) + 2 <= (last) || t2_ < kt_count;                                                   \
    w4_block<kReadsEarly, 0, 0, MI, NJ>(acc, f0, f1, rA##c, rB##c, pch1, rsrc_none, rsrc_none, dA##c, dB##c, voff_a, voff, 0); \
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);                                                                   \
    __builtin_amdgcn_s_waitcnt(kWaitVm1);                                                                     \
    w4_barrier();                                                                                             \
    w4_block<kReadsSpread, 0, MI + NJ, MI, NJ>(acc, f1, f0, rA##o, rB##o, pch0, more_ ? rsrc_a : rsrc_none, \
                      more_ ? rsrc_w : rsrc_none, dA##c, dB##c, voff_a, voff, kbyte(t2_)); \
    W4_WARM((first) + (x) + kWarmAhead, (first) + (last));                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                                        \
    }
    // Eight k-tiles per trip: the taken branch at the end of a trip costs the matrix pipe about 200
    // cycles.
    int t = 0;
    for (; t + 7 < kt_count; t += 8) {
      W4_TILE(t, 0, 7, 0, 1);
      W4_TILE(t, 1, 7, 1, 0);
      W4_TILE(t, 2, 7, 0, 1);
      W4_TILE(t, 3, 7, 1, 0);
      W4_TILE(t, 4, 7, 0, 1);
      W4_TILE(t, 5, 7, 1, 0);
      W4_TILE(t, 6, 7, 0, 1);
      W4_TILE(t, 7, 7, 1, 0);
    }
    for (; t + 1 < kt_count; t += 2) {
      W4_TILE(t, 0, 1, 0, 1);
      W4_TILE(t, 1, 1, 1, 0);
    }
    if (t < kt_count) W4_TILE(t, 0, 0, 0, 1);
#undef W4_TILE
    if constexpr (KTAIL) {
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      w4_barrier();                            // both stages are free
      const int left = K - kt_count * kBK, kb = kt_count * kBK * 2;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = ((lane & 7) ^ (((s * 8 + (lane >> 3)) >> 1) & 7)) * 8;
        w4_dma(rsrc_a, dA0 + s * 8 * kBK, k < left ? voff_a[s] : kOffOutOfRange, kb);
        w4_dma(rsrc_w, dB0 + s * 8 * kBK, k < left ? voff[s] : kOffOutOfRange, kb);
      }
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      w4_barrier();
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        f0.b[s] = *reinterpret_cast<const bf16x8*>(rB0 + s * 16 * kBK + pch0);
        f0.a[s] = *reinterpret_cast<const bf16x8*>(rA0 + s * 16 * kBK + pch0);
      }
      __builtin_amdgcn_sched_barrier(0);
      w4_block<kReadsEarly, 0, 0, MI, NJ>(acc, f0, f1, rA0, rB0, pch1, rsrc_none, rsrc_none, dA0, dB0, voff_a, voff, 0);
      w4_block<kReadsNone, 0, 0, MI, NJ>(acc, f1, f0, rA0, rB0, pch0, rsrc_none, rsrc_none, dA0, dB0, voff_a, voff, 0);
    }
  } else {
    // Three stages, filled two to three k-tiles ahead, half of a k-tile's DMA in either k-step: k-tiles 0, 1 and the first half of 2
    // are requested here and k-tile 0 awaited.
    constexpr int HALF = (MI + NJ) / 2;
#define W4_FETCH(u, c, n)                                                                                     \
  {                                                                                                           \
    const __amdgpu_buffer_rsrc_t ra_ = (u) < kt_count ? rsrc_a : rsrc_none, rw_ = (u) < kt_count ? rsrc_w : rsrc_none; \
    _Pragma("unroll") for (int s = 0; s < MI && s < (n); ++s) w4_dma(ra_, dA##c + s * 8 * kBK, voff_a[s], kbyte(u)); \
    _Pragma("unroll") for (int s = 0; s < NJ && s < (n) - MI; ++s) w4_dma<STREAM>(rw_, dB##c + s * 8 * kBK, voff[s], kbyte(u)); \
  }
    W4_FETCH(0, 0, MI + NJ);
    W4_FETCH(1, 1, MI + NJ);
    W4_FETCH(2, 2, HALF);
#undef W4_FETCH
    constexpr int WARM = NJ == 8;                    // (the narrow tile asks for nothing ahead)
    if (WARM) W4_WARM(3, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) asm volatile("" : "+a"(acc[i][j]));
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm<MI + NJ + HALF + WARM>());   // all but k-tiles 1 and 2 and the warm-up load
    w4_barrier();
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (s < NJ) f0.b[s] = *reinterpret_cast<const bf16x8*>(rB0 + s * 16 * kBK + pch0);
      if (s < MI) f0.a[s] = *reinterpret_cast<const bf16x8*>(rA0 + s * 16 * kBK + pch0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // As above (p: the stage before c), but k-step 0 asks for the second half of k-tile t + 2, which may still be in flight at the barrier,
    // and k-step 1 for the first half of t + 3.
#define W4_TILE(first, x, last, c, o, p)                                                                      \
  {                                                                                                           \
    const int t2_ = (first) + (x) + 2, t3_ = t2_ + 1;                                                         \
    const bool more2_ = (x) + 2 <= (last) || t2_ < kt_count, more3_ = (x) + 3 <= (last) || t3_ < kt_count;    \
    w4_block<kReadsEarly, HALF, MI + NJ, MI, NJ, STREAM>(acc, f0, f1, rA##c, rB##c, pch1, more2_ ? rsrc_a : rsrc_none, \
                      more2_ ? rsrc_w : rsrc_none, dA##p, dB##p, voff_a, voff, kbyte(t2_));           \
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);                                                                   \
    __builtin_amdgcn_s_waitcnt(wait_vm<MI + NJ + WARM>());                                                    \
    w4_barrier();                                                                                             \
    w4_block<kReadsSpread, 0, HALF, MI, NJ, STREAM>(acc, f1, f0, rA##o, rB##o, pch0, more3_ ? rsrc_a : rsrc_none, \
                      more3_ ? rsrc_w : rsrc_none, dA##c, dB##c, voff_a, voff, kbyte(t3_));           \
    if (WARM) W4_WARM((first) + (x) + kWarmAhead + 1, (first) + (last));                                                                       \
    __builtin_amdgcn_sched_barrier(0);                                                                        \
  }
    int t = 0;
    for (; t + 5 < kt_count; t += 6) {
      W4_TILE(t, 0, 5, 0, 1, 2);
      W4_TILE(t, 1, 5, 1, 2, 0);
      W4_TILE(t, 2, 5, 2, 0, 1);
      W4_TILE(t, 3, 5, 0, 1, 2);
      W4_TILE(t, 4, 5, 1, 2, 0);
      W4_TILE(t, 5, 5, 2, 0, 1);
    }
    for (; t + 2 < kt_count; t += 3) {
      W4_TILE(t, 0, 2, 0, 1, 2);
      W4_TILE(t, 1, 2, 1, 2, 0);
      W4_TILE(t, 2, 2, 2, 0, 1);
    }
    if (t < kt_count) W4_TILE(t, 0, 0, 0, 1, 2);
    if (t + 1 < kt_count) W4_TILE(t, 1, 1, 1, 2, 0);
  }
#undef W4_TILE
#undef W4_WARM
  __builtin_amdgcn_s_waitcnt(kWaitVm0);      // the trailing (empty) DMA writes have landed
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  w4_barrier();                              // before the stages are reused for the epilogue
  // The compiler does not know that the assembly above writes the accumulators with MFMA latency:
  // keep the first read of them away from the last MFMA by more than any such hazard asks for
  // (the waits and the barrier above already take longer; this makes it independent of them).
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

  // Epilogue.  The MFMAs take the W fragment as their row operand, so each 16x16 accumulator is a
  // block of C^T: accumulator [i][j] of lane l holds output row m = 16i + l%16 and the four
  // consecutive columns n = 16j + 4*(l/16) + (0..3).  The wave stages its block through its own
  // 32 KB of the (now idle) LDS stages so that global memory sees whole row segments of 128-256
  // bytes.  Global accesses go through a buffer descriptor over the wave's valid rows (rows past M
  // fall outside it, columns past N get an out-of-range offset): no branches, so the stores -- and
  // the residual reads, 16 row segments at a time -- are in flight together instead of one after
  // the other.
  // (The lane's number is made anew here: computed from the first one, the epilogue's addresses would be hoisted above the
  // main loop and spilled.)
  int lane_out = lane;
  asm volatile("" : "+v"(lane_out));
  const int row_out = lane_out & 15, quad_out = lane_out >> 4;
  bf16* region = wave == 0 ? sA0 : wave == 1 ? sA1 : wave == 2 ? sB0 : NJ == 8 ? sB1 : sA2;
  const int rows_valid = __builtin_amdgcn_readfirstlane(min(16 * MI, max(0, M - m0 - wm * 16 * MI)));
  if (SWIGLU) {
    // Accumulators [i][0..NJ/2-1] are gate, [i][NJ/2..NJ-1] up of outputs n0 + (WR/4)*wn + (0..WR/4-1):
    // staged as [128 rows][CH = NJ chunks of 8 bf16], chunk c of row r at position c ^ ((r>>1) & (CH-1)).
    constexpr int CH = NJ;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row = i * 16 + row_out;
      const int rkey = (row >> 1) & (CH - 1);
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) {
        bf16x4 v;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const float g = static_cast<float>(static_cast<bf16>(acc[i][j][b]));
          const float u = static_cast<float>(static_cast<bf16>(acc[i][NJ / 2 + j][b]));
          v[b] = static_cast<bf16>(silu_mul_f32(g, u));
        }
        *reinterpret_cast<bf16x4*>(region + row * (CH * 8) + (((2 * j + (quad_out >> 1)) ^ rkey) << 3) + 4 * (quad_out & 1)) = v;
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);     // own wave's LDS writes have landed; no other wave touches the region
    bf16* cb = reinterpret_cast<bf16*>(Cout) + (int64_t)(m0 + wm * 16 * MI) * N;
    const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cb, (uint32_t)(rows_valid * N * 2));
    const int col = n0 + wn * (CH * 8) + (lane_out % CH) * 8;
    const uint32_t cbyte = col < N ? (uint32_t)(((lane_out / CH) * N + col) * 2) : kOffOutOfRange;
#pragma unroll
    for (int it = 0; it < MI * CH / 4; ++it) {
      const int idx = lane_out + it * 64;
      const int row = idx / CH, ch = idx % CH;
      const u32x4 v = *reinterpret_cast<const u32x4*>(region + row * (CH * 8) + ((ch ^ ((row >> 1) & (CH - 1))) << 3));
      __builtin_amdgcn_raw_buffer_store_b128(v, rc, cbyte, it * (64 / CH) * N * 2, 0);
    }
  } else if (EPI == kEpiBf16) {
    // [128 rows][CH = 2 NJ chunks of 8 bf16], chunk c of row r at position c ^ (r & (CH-1)).
    // The experts' outputs go past the L2, which the neighbours' panels want: with the combine, 30B-A3B shape, us, 1700 tokens 129 -> 125,
    // 8192 336.5 -> 331, 16000 596 -> 577.  (Not those of gate_up, which the next kernel reads: 1700 tokens 183 -> 177, but 4096
    // 272 -> 275; nor a dense projection's: no change.)
    constexpr int CH = 2 * NJ;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row = i * 16 + row_out;
      const int rkey = row & (CH - 1);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        bf16x4 v;
#pragma unroll
        for (int b = 0; b < 4; ++b) v[b] = static_cast<bf16>(acc[i][j][b]);
        *reinterpret_cast<bf16x4*>(region + row * (CH * 8) + (((2 * j + (quad_out >> 1)) ^ rkey) << 3) + 4 * (quad_out & 1)) = v;
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    bf16* cb = reinterpret_cast<bf16*>(Cout) + (int64_t)(m0 + wm * 16 * MI) * N;
    const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cb, (uint32_t)(rows_valid * N * 2));
    const int col = n0 + wn * (CH * 8) + (lane_out % CH) * 8;
    const uint32_t cbyte = col < N ? (uint32_t)(((lane_out / CH) * N + col) * 2) : kOffOutOfRange;
#pragma unroll
    for (int it = 0; it < MI * CH / 4; ++it) {
      const int idx = lane_out + it * 64;
      const int row = idx / CH, ch = idx % CH;
      const u32x4 v = *reinterpret_cast<const u32x4*>(region + row * (CH * 8) + ((ch ^ (row & (CH - 1))) << 3));
      __builtin_amdgcn_raw_buffer_store_b128(v, rc, cbyte, it * (64 / CH) * N * 2, GROUPED ? kAuxNonTemporal : 0);
    }
  } else {
    // fp32 residual (read-modify-write) or split-K partial (plain store into this split's [M][N]
    // slab): two passes of 64 columns, staged as [128 rows][16 chunks of 4 floats], chunk c of row r
    // at position c ^ (r & 15).
    float* stage = reinterpret_cast<float*>(region);
    float* cf = reinterpret_cast<float*>(Cout) + (EPI == kEpiPartial ? (int64_t)split * M * N : 0) +
                (int64_t)(m0 + wm * 16 * MI) * N;
    const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cf, (uint32_t)(rows_valid * N * 4));
    const int col0 = n0 + wn * (WR / 2) + (lane_out & 15) * 4;
#pragma unroll
    for (int jp = 0; jp < NJ / 4; ++jp) {
      const int col = col0 + jp * 64;
      const uint32_t cbyte = col < N ? (uint32_t)(((lane_out >> 4) * N + col) * 4) : kOffOutOfRange;   // N % 8 == 0: quads all-in or all-out
      f32x4 x[16];
      if (RESID) {
#pragma unroll
        for (int it = 0; it < (MI < 4 ? 4 * MI : 16); ++it)
          x[it] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, cbyte, it * 4 * N * 4, 0));
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int row = i * 16 + row_out;
        const int rkey = row & 15;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          f32x4 v;
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = acc[i][jp * 4 + jj][b];
          *reinterpret_cast<f32x4*>(stage + row * 64 + (((jj * 4 + quad_out) ^ rkey) << 2)) = v;
        }
      }
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
#pragma unroll
      for (int h = 0; h < (MI + 3) / 4; ++h) {
        if (RESID && h == 1) {
#pragma unroll
          for (int it = 0; it < 4 * MI - 16; ++it)
            x[it] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, cbyte, (16 + it) * 4 * N * 4, 0));
        }
#pragma unroll
        for (int it = 0; it < (4 * MI - 16 * h < 16 ? 4 * MI - 16 * h : 16); ++it) {
          const int idx = lane_out + (h * 16 + it) * 64;
          const int row = idx >> 4, ch = idx & 15;
          f32x4 v = *reinterpret_cast<const f32x4*>(stage + row * 64 + ((ch ^ (row & 15)) << 2));
          if (RESID) {
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] += x[it][b];
          }
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rc, cbyte, (h * 16 + it) * 4 * N * 4, 0);
        }
      }
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);   // the stage is rewritten by the next pass
    }
  }
  };
  if constexpr (GROUPED) {
    switch ((M + 31) / 32) {
      case 1: case 2: tile(std::integral_constant<int, 2>{}); break;
      case 3: tile(std::integral_constant<int, 3>{}); break;
      case 4: tile(std::integral_constant<int, 4>{}); break;
      case 5: tile(std::integral_constant<int, 5>{}); break;
      case 6: tile(std::integral_constant<int, 6>{}); break;
      case 7: tile(std::integral_constant<int, 7>{}); break;
      default: tile(std::integral_constant<int, 8>{}); break;
    }
  } else {
    tile(std::integral_constant<int, BM / 32>{});
  }
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA GEMM on small tiles (16 MI = 32, 64 or 128 rows, 64 NJ columns; any K % 8 == 0).  Its main use is a
// launch of few rows, which reads every weight once from HBM for a handful of MFMAs, so the weights'
// stream is all there is to it; it also takes most of what has too few 256-row tiles to occupy the chip,
// and of odd K (gemm_plan.h).
// 256 threads = 4 waves side by side along N; every wave multiplies all rows by its 16 NJ columns with
// v_mfma_f32_16x16x32_bf16, in the k order of the kernel above (the same bits, unless grouped or cut; both start columns at the
// same k).  K is consumed KT at a time through a ring of S LDS stages, separate arrays filled by DMA S - 1 k-tiles ahead; the loop
// body has no branch and always runs a multiple of S k-tiles (behind the last one there is nothing to fetch and
// zeros to multiply), since with a branch between stages the compiler waits for all DMA before a read.
// LDS rows hold KT bf16, 16-byte chunk c of row r at c ^ ((r >> 1) & 7) (KT = 64) or c ^ (r & 15)
// (KT = 128): a half-wave's 16 rows x 2 chunks put two lanes on every bank group.
// Grouped: workgroups start at different k and read W non-temporally, so that the stream leaves the activations in the L2: the
// experts' projections of the 30B-A3B shape, cold, us: 16 tokens 87 -> 80 and 55 -> 49, 590 tokens 164 -> 147 and 97 -> 92 (with the
// combine).  Not the experts' gate_up on 128 rows, which loses by the hint from 70 rows per expert on (96 rows of 8 experts [4096 14336]
// 390 us, 377 without; of 64 [4096 1536] 345 and 331) and gains less below (50 rows: 367 and 371, 314 and 320).
// K ranges start at different k as it is, and gain nothing by more starts (50 x 5120 x 27648 57 us, 73 with them); by the hint, of
// up to 64 rows: 16 rows of 4096 x 14336 24.6 -> 22.3, 6144 x 4096 14.3 -> 13.1, 50 rows of 4096 x 14336 27.1 -> 25.5, 5120 x
// 27648 57 -> 53.8, short K no change.  (Not the large kernel's: 256 x 4096 x 14336 45 -> 44, but 100 x 4096 x 4096 16 -> 19, 256
// x 5120 x 2048 19.5 -> 23.)
// STREAM (uncut launches of one row tile, the W of all of them read once): the same two, the start by start_groups, which
// keeps the fused projection and the plain one on one order of sums.  The hint by itself: 50 rows of [14336 outputs 4096]
// 52.5 -> 49.3 us, 27648 x 5120 110 -> 103; with the starts 41.2, and 256 rows on the 128-column tile 68.2 -> 60.4.
// Not on 128 rows here: 27648 x 5120 125 -> 126.7.
// ------------------------------------------------------------------------------------------
template <int KT> __device__ __forceinline__ int ring_chunk(int chunk, int row) {
  return KT == 128 ? chunk ^ (row & 15) : chunk ^ ((row >> 1) & 7);
}

template <bool NT = false>
__device__ __forceinline__ void ring_dma(const bf16* base, uint32_t bytes, bf16* lds, uint32_t voff, int kbyte) {
  w4_dma<NT>(panel_rsrc(base, bytes), lds, voff, kbyte);
}

template <int MI, int NJ, int KT, int S, int EPI, bool GROUPED, bool STREAM = false>
__global__ __launch_bounds__(256) void gemm_bf16_ring_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                                 void* __restrict__ Cout, int M, int N, int K,
                                                                 int tiles_m, int tiles_n, int kt_per_split, int start_groups,
                                                                 const int32_t* __restrict__ groups,
                                                                 const int32_t* __restrict__ a_rows) {
  constexpr bool SWIGLU = EPI == kEpiSwiGLU;
  constexpr int BM = 16 * MI, WR = 64 * NJ;          // rows of A and of W per stage
  constexpr int BN = SWIGLU ? WR / 2 : WR;           // output columns per tile
  constexpr int CPR = KT / 8;                        // 16-byte chunks per LDS row
  constexpr int RPI = 64 / CPR;                      // rows per DMA instruction
  constexpr int IA = BM / RPI / 4, IW = WR / RPI / 4;   // DMA instructions per wave and stage
  constexpr int STAGE = (BM + WR) * KT;
  constexpr bool kNonTemporal = STREAM || (GROUPED && !(SWIGLU && MI == 8));   // W (above)
  static_assert(BM % (4 * RPI) == 0 && S >= 2 && S <= 4 && (!SWIGLU || NJ % 2 == 0));
  __shared__ __attribute__((aligned(1024))) bf16 s0[STAGE];
  __shared__ __attribute__((aligned(1024))) bf16 s1[STAGE];
  __shared__ __attribute__((aligned(1024))) bf16 s2[S > 2 ? STAGE : 8];
  __shared__ __attribute__((aligned(1024))) bf16 s3[S > 3 ? STAGE : 8];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile_m = 0, tile_n, a_total_rows = M, rot = 0;
  const int split = GROUPED ? 0 : blockIdx.x / (tiles_m * tiles_n);
  const int64_t slab = (int64_t)split * M * N;       // of the partial sums
  if (GROUPED) {                                     // (the order of gemm_bf16_w4_kernel)
    const int n_row_tiles = groups[0];
    const int quota = (n_row_tiles + kXcds - 1) / kXcds;
    const int in_xcd = blockIdx.x / kXcds;
    const int ti = (blockIdx.x % kXcds) * quota + in_xcd / tiles_n;
    if (in_xcd / tiles_n >= quota || ti >= n_row_tiles) return;   // whole workgroup, before any barrier
    const int expert = groups[1 + 3 * ti], first = groups[2 + 3 * ti];
    M = groups[3 + 3 * ti];
    if (a_rows) a_rows += first;
    else A += (int64_t)first * K;
    W += (int64_t)expert * (SWIGLU ? 2 : 1) * N * K;
    Cout = reinterpret_cast<char*>(Cout) + (int64_t)first * N * 2;
    tile_n = in_xcd % tiles_n;
    // Experts' matrices lie at multiples of the HBM channels' period, and workgroups in step would ask a few
    // channels for the same columns of all of them: every (expert, column tile) starts at another k-tile
    // (experts_up of the 30B-A3B shape, 590 tokens 183 -> 164 us, 16 tokens 100 -> 89).  The start depends on
    // nothing else, so neither do a row's bits among these tiles; the 256-row tile's columns are others, so a batch of
    // more than 96 rows per expert rounds differently.
    rot = (expert * tiles_n + tile_n) % ((K + KT - 1) / KT);
  } else {
    tile_n = blockIdx.x - split * (tiles_m * tiles_n);
    if (tiles_m > 1) tile_of_workgroup(tile_n, tiles_m, tiles_n, tile_m, tile_n);
    const int m0 = tile_m * BM;
    A += (int64_t)m0 * K;
    Cout = reinterpret_cast<char*>(Cout) + ((int64_t)m0 * N + slab) * (EPI == kEpiBf16 || SWIGLU ? 2 : 4);
    M = min(BM, M - m0);
    if (STREAM && EPI != kEpiPartial) rot = k_start(tile_n * BN, K, start_groups) / KT;
  }
  const int n0 = tile_n * BN;
  const int k_first = split * kt_per_split * kBK;    // (K ranges are counted in k-tiles of 64)
  const int k_count = min(kt_per_split * kBK, K - k_first);
  const bool gathered = GROUPED && a_rows != nullptr;

  // DMA sources: instruction i of this wave fills LDS rows RPI (IA wave + i) .. (A), RPI (IW wave + i) .. (W).
  // W stage row r is row n0 + r; SwiGLU: rows 32 u .. + 15 of a wave's share are gate rows, the next 16 the up
  // rows of the same outputs (unit u = r / 32 covers outputs n0 + 16 u ..).
  uint32_t off_a[IA], off_w[IW];
  int k_a[IA], k_w[IW];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int row = RPI * (IA * wave + i) + lane / CPR;
    k_a[i] = ring_chunk<KT>(lane % CPR, row) * 8;
    int src = row < M ? row : -1;
    if (gathered && src >= 0) src = a_rows[row];
    off_a[i] = src >= 0 ? (uint32_t)((src * K + k_a[i]) * 2) : kOffOutOfRange;
  }
#pragma unroll
  for (int i = 0; i < IW; ++i) {
    const int row = RPI * (IW * wave + i) + lane / CPR;
    k_w[i] = ring_chunk<KT>(lane % CPR, row) * 8;
    const int col = n0 + (SWIGLU ? (row >> 5) * 16 + (row & 15) : row);
    const int src = SWIGLU ? ((row >> 4) & 1) * N + col : col;
    off_w[i] = col < N ? (uint32_t)(((src - n0) * K + k_w[i]) * 2) : kOffOutOfRange;
  }
  const bf16* const panel_a = A + k_first;
  const bf16* const panel_w = W + (int64_t)n0 * K + k_first;
  const uint32_t bytes_a = (uint32_t)(((gathered ? a_total_rows : M) * K - k_first) * 2);
  const uint32_t bytes_w = (uint32_t)((((SWIGLU ? N : 0) + min(BN, N - n0)) * K - k_first) * 2);
  const int kt_count = (k_count + KT - 1) / KT;
  auto fetch = [&](int t, bf16* s) __attribute__((always_inline)) {
    int left = k_count - t * KT;                     // behind the last k-tile every chunk is out of range
    if ((GROUPED || STREAM) && left > 0) {
      t = t + rot >= kt_count ? t + rot - kt_count : t + rot;
      left = k_count - t * KT;
    }
#pragma unroll
    for (int i = 0; i < IA; ++i)
      ring_dma(panel_a, bytes_a, s + RPI * (IA * wave + i) * KT, k_a[i] < left ? off_a[i] : kOffOutOfRange, t * KT * 2);
#pragma unroll
    for (int i = 0; i < IW; ++i)
      ring_dma<kNonTemporal>(panel_w, bytes_w, s + (BM + RPI * (IW * wave + i)) * KT, k_w[i] < left ? off_w[i] : kOffOutOfRange, t * KT * 2);
  };

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int frag_row = lane & 15, quad = lane >> 4;
  auto step = [&](int t, const bf16* s, bf16* next) __attribute__((always_inline)) {
    fetch(t + S - 1, next);                          // the stage every wave finished before the last barrier
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KT / 32; ++ks) {
      bf16x8 fa[MI], fw[NJ];
      const int at = ring_chunk<KT>(4 * ks + quad, frag_row) * 8;   // (16-row blocks: the block's first row does not change it)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        fw[j] = *reinterpret_cast<const bf16x8*>(s + (BM + 16 * (NJ * wave + j) + frag_row) * KT + at);
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(s + (16 * i + frag_row) * KT + at);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j], fa[i], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);          // this wave is done with the stage ...
    __builtin_amdgcn_s_waitcnt(wait_vm<(S - 2) * (IA + IW)>());   // ... and its share of the next one has landed
    w4_barrier();
  };
  fetch(0, s0);
  if (S > 2) fetch(1, s1);
  if (S > 3) fetch(2, s2);
  __builtin_amdgcn_s_waitcnt(wait_vm<(S - 2) * (IA + IW)>());
  w4_barrier();
  for (int t = 0; t * KT < k_count; t += S) {
    step(t, s0, S == 2 ? s1 : S == 3 ? s2 : s3);
    step(t + 1, s1, s0);
    if (S > 2) step(t + 2, s2, s1);
    if (S > 3) step(t + 3, s3, s2);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);              // the last (empty) fetches

  // Accumulator [i][j] of a lane holds output row 16 i + lane % 16 and the four columns 4 (lane / 16) +
  // (0..3) of the wave's j-th 16: stored as they are, 32 to 64 bytes of a row at a time (few rows: the output is
  // a small part of what moves).
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = 16 * i + frag_row;
    if (m >= M) continue;
    if (SWIGLU) {
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) {
        const int n = n0 + 16 * (NJ / 2 * wave + j) + 4 * quad;
        if (n >= N) continue;                        // N % 8 == 0: all four or none
        bf16x4 v;
#pragma unroll
        for (int b = 0; b < 4; ++b)
          v[b] = static_cast<bf16>(silu_mul_f32(static_cast<float>(static_cast<bf16>(acc[i][2 * j][b])),
                                                static_cast<float>(static_cast<bf16>(acc[i][2 * j + 1][b]))));
        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Cout) + (int64_t)m * N + n) = v;
      }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = n0 + 16 * (NJ * wave + j) + 4 * quad;
        if (n >= N) continue;
        if (EPI == kEpiBf16) {
          bf16x4 v;
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = static_cast<bf16>(acc[i][j][b]);
          *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Cout) + (int64_t)m * N + n) = v;
        } else {
          float* c = reinterpret_cast<float*>(Cout) + (int64_t)m * N + n;
          f32x4 v = acc[i][j];
          if (EPI == kEpiResidual) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(c);
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] += x[b];
          }
          *reinterpret_cast<f32x4*>(c) = v;
        }
      }
    }
  }
}

// Split-K reduction: out[m][n] = sum over splits (in index order: deterministic) of the fp32
// partials, added into the fp32 residual or rounded to bf16.  One thread per 8 outputs.
template <bool RESID>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part,
                                                            void* __restrict__ out, int64_t mn8,
                                                            int64_t mn, int splits) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= mn8) return;
  f32x8 acc = Vec8<float>::load(part + i * 8);
  for (int z = 1; z < splits; ++z) {
    const f32x8 v = Vec8<float>::load(part + z * mn + i * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += v[e];
  }
  if (RESID) {
    float* o = reinterpret_cast<float*>(out) + i * 8;
    const f32x8 x = Vec8<float>::load(o);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += x[e];
    Vec8<float>::store(o, acc);
  } else {
    Vec8<bf16>::store(reinterpret_cast<bf16*>(out) + i * 8, acc);
  }
}

// Split-K reduction of a gate_up projection fused with SiLU(gate)*up: part [splits][M][2F] fp32
// -> out [M][F].  Gate and up sums are rounded to bf16 first, so the result has the bits of
// splitk_reduce_kernel<false> into [M][2F] followed by the stand-alone silu_mul operator, without
// that intermediate.  One thread per 8 outputs.
__global__ __launch_bounds__(256) void splitk_reduce_swiglu_kernel(const float* __restrict__ part,
                                                                   bf16* __restrict__ out, int64_t m,
                                                                   int64_t f, int splits) {
  const int64_t f8 = f / 8;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m * f8) return;
  const int64_t r = i / f8, c = i - r * f8;
  const int64_t mn = m * 2 * f;
  const float* row = part + r * 2 * f + c * 8;
  f32x8 g = Vec8<float>::load(row), u = Vec8<float>::load(row + f);
  for (int z = 1; z < splits; ++z) {
    const f32x8 gz = Vec8<float>::load(row + z * mn), uz = Vec8<float>::load(row + z * mn + f);
#pragma unroll
    for (int e = 0; e < 8; ++e) { g[e] += gz[e]; u[e] += uz[e]; }
  }
  f32x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    o[e] = silu_mul_f32(static_cast<float>(static_cast<bf16>(g[e])), static_cast<float>(static_cast<bf16>(u[e])));
  Vec8<bf16>::store(out + r * f + c * 8, o);
}

// Split-K reduction of a residual projection fused with the RMSNorm that follows it: one
// 256-thread workgroup per token row adds the partial sums (in index order) and the residual,
// writes the new residual row, and normalises it from registers into h -- the arithmetic, in the
// order, of splitk_reduce_kernel<true> followed by the stand-alone RMSNorm operator, which then
// has nothing left to do.  Rows of up to kTailNormCols columns.
constexpr int kTailNormVec = 4;
constexpr int kTailNormCols = 256 * 8 * kTailNormVec;
__global__ __launch_bounds__(256) void splitk_reduce_norm_kernel(const float* __restrict__ part,
                                                                 float* __restrict__ x,
                                                                 const bf16* __restrict__ gain,
                                                                 bf16* __restrict__ h, int64_t mn, int n,
                                                                 int splits, float eps) {
  __shared__ float partial[4];
  const int tid = threadIdx.x;
  const int64_t at = (int64_t)blockIdx.x * n;
  const int n8 = n / 8;
  f32x8 held[kTailNormVec];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kTailNormVec; ++i) {
    const int c = tid + i * 256;
    if (c < n8) {
      const f32x8 xv = Vec8<float>::load(x + at + c * 8);
      f32x8 acc = Vec8<float>::load(part + at + c * 8);
      int z = 1;
      for (; z + 3 < splits; z += 4) {               // four loads in flight; added in index order
        const f32x8 v0 = Vec8<float>::load(part + z * mn + at + c * 8);
        const f32x8 v1 = Vec8<float>::load(part + (z + 1) * mn + at + c * 8);
        const f32x8 v2 = Vec8<float>::load(part + (z + 2) * mn + at + c * 8);
        const f32x8 v3 = Vec8<float>::load(part + (z + 3) * mn + at + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = ((acc[e] + v0[e]) + v1[e]) + v2[e] + v3[e];
      }
      for (; z < splits; ++z) {
        const f32x8 v = Vec8<float>::load(part + z * mn + at + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += v[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += xv[e];
      Vec8<float>::store(x + at + c * 8, acc);
      held[i] = acc;
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += acc[e] * acc[e];
    }
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) partial[tid >> 6] = ss;
  __syncthreads();
  const float total = partial[0] + partial[1] + partial[2] + partial[3];
  const float inv = 1.0f / sqrtf(total / (float)n + eps);
#pragma unroll
  for (int i = 0; i < kTailNormVec; ++i) {
    const int c = tid + i * 256;
    if (c < n8) {
      const f32x8 g = Vec8<bf16>::load(gain + c * 8);
      f32x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = held[i][e] * inv * g[e];
      Vec8<bf16>::store(h + at + c * 8, o);
    }
  }
}

// The large-tile kernels move their operands by buffer instructions, which want dwords, the ring kernel also by 8 and 16
// byte loads and stores; operands off either grid run on gemm_bf16_kernel.
static bool aligned_to(uintptr_t bytes, const void* a, const void* w, const void* c) {
  return (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(c)) % bytes == 0;
}

// SWIGLU: n outputs, w holds 2 n rows.
template <bool RESID, bool SWIGLU = false>
static void launch_bf16_any(const bf16* a, const bf16* w, void* c, int m, int n, int k, hipStream_t s) {
  constexpr int BM = 128, BN = 128, WGM = 2, WGN = 2, OUT = SWIGLU ? BN / 2 : BN;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + OUT - 1) / OUT;
  const size_t smem = (size_t)2 * (BM + BN) * kBK * sizeof(bf16);
  // Once per instantiation; a function-local static is initialised exactly once even when several
  // threads launch at the same time.
  static const hipError_t attr_set =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<BM, BN, WGM, WGN, RESID, SWIGLU>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  (void)attr_set;
  launch_kernel(gemm_bf16_kernel<BM, BN, WGM, WGN, RESID, SWIGLU>, dim3((unsigned)(tiles_m * tiles_n)), WGM * WGN * 64, smem, s,
      a, w, c, m, n, k, tiles_m, tiles_n);
}

// Few rows (gemm_plan.h's few_rows): columns per tile, k-tiles and stages by
// row count and epilogue, as measured on cold weights of the 8B shape (us, against the two-stage 256-row tile): up to
// 64 rows 64-column tiles of 128 k (256 bytes of a weight row at a time: HBM gives 4.9 TB/s to such pieces where 128-byte
// pieces get 4.2) -- 50 rows: qkv 22 -> 17, o 17 -> 12.6, down 40 -> 28; from 65 rows on the A tile weighs more and 128-column
// tiles of 64 k read it half as often.  SwiGLU: 128 W rows of 64 k, 75 -> 52 at 50 rows; from 3072 k on (LONG_K) 128 k at a time
// there too, through three stages for 64 rows (50 rows, outputs x k: 8192 x 3072 32.1 -> 29.8, 14336 x 6144 61.9 -> 59.5, 8192 x
// 8192 73 -> 69; 8192 x 2048 23.5 -> 23.8, 14336 x 1024 15.8 -> 16.7).
template <int MI, bool SWIGLU, bool LONG_K = false> struct RingTile {
  static constexpr bool kWide = SWIGLU || MI > 4;
  static constexpr int NJ = kWide ? 2 : 1, KT = kWide && !LONG_K ? 64 : 128, S = LONG_K && MI == 4 ? 3 : 4, BN = SWIGLU ? 32 * NJ : 64 * NJ;
};
struct KRanges {
  int per, used;      // k-tiles of 64 per range, ranges (every range has at least one k-tile)
};
static KRanges k_ranges(int k, int splits) {
  const int kt = (k + kBK - 1) / kBK, per = (kt + splits - 1) / splits;
  return {per, (kt + per - 1) / per};
}
// A CU holds one workgroup of the ring kernel: no more K ranges than it takes to occupy the 256 once.
template <int MI, int EPI>
static KRanges ring_ranges(int n, int k, int splits) {
  using T = RingTile<MI, EPI == kEpiSwiGLU>;
  return k_ranges(k, splits > 1 ? std::max(2, std::min(splits, 256 / ((n + T::BN - 1) / T::BN))) : 1);
}
template <int MI, int EPI, bool STREAM = false, bool LONG_K = false>
static int launch_ring(const bf16* a, const bf16* w, void* c, int m, int n, int k, int splits, hipStream_t s, int starts = 0) {
  using T = RingTile<MI, EPI == kEpiSwiGLU, LONG_K>;
  const int tiles_m = (m + 16 * MI - 1) / (16 * MI), tiles_n = (n + T::BN - 1) / T::BN;
  const KRanges r = ring_ranges<MI, EPI>(n, k, splits);
  launch_kernel(gemm_bf16_ring_kernel<MI, T::NJ, T::KT, T::S, EPI, false, STREAM>, dim3((unsigned)(tiles_m * tiles_n * r.used)), 256, 0, s,
      a, w, c, m, n, k, tiles_m, tiles_n, r.per, starts, nullptr, nullptr);
  return r.used;
}
// starts: uncut_starts.  Returns the number of K ranges launched (at most `splits`).
template <int EPI>
static int launch_few_rows(const bf16* a, const bf16* w, void* c, int m, int n, int k, int splits, int starts, hipStream_t s) {
  constexpr bool SWIGLU = EPI == kEpiSwiGLU, STREAM = EPI != kEpiResidual;
  if (SWIGLU && k >= 3072) {
    if (m <= 32) return launch_ring<2, EPI, STREAM, SWIGLU>(a, w, c, m, n, k, splits, s, starts);
    if (m <= 64) return launch_ring<4, EPI, STREAM, SWIGLU>(a, w, c, m, n, k, splits, s, starts);
  }
  if (m <= 32) return launch_ring<2, EPI, STREAM>(a, w, c, m, n, k, splits, s, starts);
  if (m <= 64) return launch_ring<4, EPI, STREAM>(a, w, c, m, n, k, splits, s, starts);
  return launch_ring<8, EPI>(a, w, c, m, n, k, splits, s);
}

static bool takes_small_tiles(int64_t m, int64_t n, int64_t k, size_t workspace_bytes);

// Small problems' fused gate_up: columns of W are gate and up of 64 outputs per tile.
bool gemm_swiglu_small(int dtype, int64_t m, int64_t f, int64_t k, size_t workspace_bytes) {
  return dtype == 1 && m > 0 && f % 8 == 0 && k % 8 == 0 && (f + 256) * k * 2 < (int64_t)kOffOutOfRange &&
         takes_small_tiles(m, 2 * f, k, workspace_bytes) && k <= (1 << 21) &&
         ((m + 31) / 32) * ((f + 63) / 64) <= INT32_MAX && swiglu_tile_rows(m, f, k) > 0;
}

void launch_gemm_swiglu_small(const void* a, const void* w_gate_up, void* out, int64_t m, int64_t f, int64_t k, hipStream_t s) {
  const bf16 *pa = (const bf16*)a, *pw = (const bf16*)w_gate_up;
  switch (swiglu_tile_rows(m, f, k)) {
    case 128: launch_ring<8, kEpiSwiGLU>(pa, pw, out, (int)m, (int)f, (int)k, 1, s); break;
    case 64: launch_ring<4, kEpiSwiGLU>(pa, pw, out, (int)m, (int)f, (int)k, 1, s); break;
    default: launch_ring<2, kEpiSwiGLU>(pa, pw, out, (int)m, (int)f, (int)k, 1, s); break;
  }
}

// The router has few outputs and as many rows as the task: 32-row tiles, logits stored in fp32 as they come (590
// x 128 x 2048: 52 -> 8 us).
void launch_router_gemm(const void* a, const void* w, float* logits, int64_t m, int64_t n, int64_t k, hipStream_t s) {
  launch_ring<2, kEpiPartial>((const bf16*)a, (const bf16*)w, logits, (int)m, (int)n, (int)k, 1, s);
}

// An uncut problem on the large tile, 256 columns (SwiGLU: 128 outputs) by as many rows as large_tile_rows says.
template <int EPI, int ROWS>
static void launch_large_rows(const bf16* a, const bf16* w, void* c, int m, int n, int k, int tiles_n, hipStream_t s) {
  const int tiles_m = (m + ROWS - 1) / ROWS;
  launch_kernel(gemm_bf16_w4_kernel<EPI, false, 8, false, ROWS>, dim3((unsigned)(tiles_m * tiles_n)), 256, 0, s,
      a, w, c, m, n, k, tiles_m, tiles_n, k / kBK, 0, nullptr, nullptr);
}
template <int EPI>
static void launch_large(const bf16* a, const bf16* w, void* c, int m, int n, int k, hipStream_t s) {
  const int tiles_n = EPI == kEpiSwiGLU ? (n + 127) / 128 : (n + 255) / 256;
  switch (large_tile_rows(m, tiles_n, k, EPI == kEpiResidual ? LargeEpilogue::kResidual
                                         : EPI == kEpiSwiGLU ? LargeEpilogue::kSwiGLU : LargeEpilogue::kBf16)) {
    case 128: launch_large_rows<EPI, 128>(a, w, c, m, n, k, tiles_n, s); break;
    case 160: launch_large_rows<EPI, 160>(a, w, c, m, n, k, tiles_n, s); break;
    case 192: launch_large_rows<EPI, 192>(a, w, c, m, n, k, tiles_n, s); break;
    case 224: launch_large_rows<EPI, 224>(a, w, c, m, n, k, tiles_n, s); break;
    default: launch_large_rows<EPI, 256>(a, w, c, m, n, k, tiles_n, s); break;
  }
}

// A problem of few row tiles, whose number the columns and K ranges were chosen by: as many, on as few rows as hold m.
// The launch is bound by its lines (W from HBM, A from the L2 for every column tile), so a row tile that is not padded to 256
// fetches less: 8B shape, cold, us: 140 tokens gate_up 58 -> 55.5, 270 tokens qkv 33 -> 28.5, down 55 -> 49, 560 tokens qkv 43.5 -> 41,
// down 84 -> 75; 300 tokens of the 32B shape down 145 -> 112.
template <int EPI, int NJ>
static void launch_even_rows(const bf16* a, const bf16* w, void* c, int m, int n, int k, int kt_per_split, int splits, int starts,
                             hipStream_t s) {
  constexpr int BN = EPI == kEpiSwiGLU ? 16 * NJ : 32 * NJ;
  const int tiles_m = (m + 255) / 256, tiles_n = (n + BN - 1) / BN;
  constexpr bool kUncut = NJ == 4 && (EPI == kEpiBf16 || EPI == kEpiSwiGLU);
  auto launch = [&](auto rows) {
    constexpr int ROWS = decltype(rows)::value;
    if (kUncut && tiles_m == 1)
      launch_kernel(gemm_bf16_w4_kernel<EPI, false, NJ, false, ROWS, kUncut>, dim3((unsigned)tiles_n), 256, 0, s,
          a, w, c, m, n, k, 1, tiles_n, kt_per_split, starts, nullptr, nullptr);
    else
      launch_kernel(gemm_bf16_w4_kernel<EPI, false, NJ, false, ROWS>, dim3((unsigned)(tiles_m * tiles_n * splits)), 256, 0, s,
          a, w, c, m, n, k, tiles_m, tiles_n, kt_per_split, starts, nullptr, nullptr);
  };
  const int rows = (m + tiles_m - 1) / tiles_m;
  constexpr bool kAnyNumber = NJ == 4;     // (else three row tiles or more)
  if (kAnyNumber && rows <= 96) launch(std::integral_constant<int, kAnyNumber ? 96 : 256>{});
  else if (kAnyNumber && rows <= 128) launch(std::integral_constant<int, kAnyNumber ? 128 : 256>{});
  else if (kAnyNumber && rows <= 160) launch(std::integral_constant<int, kAnyNumber ? 160 : 256>{});
  else if (rows <= 192) launch(std::integral_constant<int, 192>{});
  else if (rows <= 224) launch(std::integral_constant<int, 224>{});
  else launch(std::integral_constant<int, 256>{});
}

bool gemm_swiglu_fusable(int dtype, int64_t m, int64_t f, int64_t k) { return dtype == 1 && swiglu_fusable(m, f, k); }

void launch_gemm_swiglu(const void* a, const void* w_gate_up, void* out, int64_t m, int64_t f,
                        int64_t k, hipStream_t s) {
  if (!aligned_to(4, a, w_gate_up, out)) {
    launch_bf16_any<false, true>((const bf16*)a, (const bf16*)w_gate_up, out, (int)m, (int)f, (int)k, s);
    return;
  }
  const int nj = swiglu_nj(m, f);
  const bool few = swiglu_few_rows(m, f) && aligned_to(16, a, w_gate_up, out);
  const int starts = uncut_starts(m, 2 * f, k, nj, few);
  if (few) {
    launch_few_rows<kEpiSwiGLU>((const bf16*)a, (const bf16*)w_gate_up, out, (int)m, (int)f, (int)k, 1, starts, s);
    return;
  }
  if (nj == 8)
    launch_large<kEpiSwiGLU>((const bf16*)a, (const bf16*)w_gate_up, out, (int)m, (int)f, (int)k, s);
  else
    launch_even_rows<kEpiSwiGLU, 4>((const bf16*)a, (const bf16*)w_gate_up, out, (int)m, (int)f, (int)k, (int)(k / kBK), 1, starts, s);
}

size_t gemm_workspace_bytes(int dtype, int64_t m, int64_t n, int64_t k) {
  if (dtype != 1 || k % kBK != 0) return 0;
  const int s = w4_shape(m, n, k).splits;
  return s > 1 ? (size_t)s * m * n * sizeof(float) : 0;
}

template <int MI, int EPI>
static void launch_grouped_ring(const bf16* a, const bf16* w, void* c, int n, int k, const int32_t* groups,
                                    int max_row_tiles, const int32_t* a_rows, int m_arg, hipStream_t s) {
  // Stages such that two workgroups share a CU (up to 32 rows: no fewer than four), so that one's prologue and stores lie under the
  // other's k-tiles: worth more than a stage more.  30B-A3B shape, cold, us, experts_up on four stages: 64-row tiles (350 to 720
  // tokens) 140 -> 132, 160 -> 151, 128-row ones (850, 1200 tokens) 185 -> 171.5, 188 -> 175; experts_down (with the combine) on
  // 32-row tiles 49.2 -> 46 with four stages instead of three (16 tokens), 64-row ones 87 -> 81 with three instead of four.
  constexpr bool SWIGLU = EPI == kEpiSwiGLU;
  constexpr int NJ = 2, KT = 64, S = MI == 8 ? 2 : MI == 4 ? 3 : 4, BN = SWIGLU ? 32 * NJ : 64 * NJ;
  const int tiles_n = (n + BN - 1) / BN;
  launch_kernel(gemm_bf16_ring_kernel<MI, NJ, KT, S, EPI, true>, dim3((unsigned)((max_row_tiles + kXcds - 1) / kXcds * kXcds * tiles_n)), 256, 0, s,
      a, w, c, m_arg, n, k, max_row_tiles, tiles_n, k / kBK, 0, groups, a_rows);
}

void launch_gemm_grouped(const void* a, const void* w, void* c, int64_t n, int64_t k, int swiglu,
                         const int32_t* groups, int max_row_tiles, int tile_rows,
                         const int32_t* a_rows, int64_t a_total_rows, hipStream_t s) {
  if (tile_rows < 256) {
    auto few = [&](auto mi) {
      constexpr int MI = decltype(mi)::value;
      const int m = a_rows ? (int)a_total_rows : 0;
      if (swiglu) launch_grouped_ring<MI, kEpiSwiGLU>((const bf16*)a, (const bf16*)w, c, (int)n, (int)k, groups, max_row_tiles, a_rows, m, s);
      else launch_grouped_ring<MI, kEpiBf16>((const bf16*)a, (const bf16*)w, c, (int)n, (int)k, groups, max_row_tiles, a_rows, m, s);
    };
    if (tile_rows == 32) few(std::integral_constant<int, 2>{});
    else if (tile_rows == 64) few(std::integral_constant<int, 4>{});
    else few(std::integral_constant<int, 8>{});
    return;
  }
  const int tiles_n = (int)(swiglu ? (n + 127) / 128 : (n + 255) / 256);
  const dim3 grid((unsigned)((max_row_tiles + kXcds - 1) / kXcds * kXcds * tiles_n));   // a whole number of row tiles per XCD
  const int m_arg = a_rows ? (int)a_total_rows : 0;
  if (swiglu)
    launch_kernel(gemm_bf16_w4_kernel<kEpiSwiGLU, true>, grid, 256, 0, s, (const bf16*)a, (const bf16*)w, c, m_arg, (int)n,
                                                              (int)k, max_row_tiles, tiles_n, (int)(k / kBK), 0, groups, a_rows);
  else
    launch_kernel(gemm_bf16_w4_kernel<kEpiBf16, true>, grid, 256, 0, s, (const bf16*)a, (const bf16*)w, c, m_arg, (int)n,
                                                            (int)k, max_row_tiles, tiles_n, (int)(k / kBK), 0, groups, a_rows);
}

// tail: what follows the split-K reduction in the same kernel (kTailNone: nothing).
template <bool RESID, int NJ>
static void launch_bf16_w4(const bf16* a, const bf16* w, void* c, int m, int n, int k, int splits,
                           float* workspace, const GemmTail& tail, hipStream_t s) {
  const bool few = few_rows(m, n, k) && aligned_to(16, a, w, c);
  const int starts = RESID || splits > 1 ? 0 : uncut_starts(m, n, k, NJ, few);
  if (splits <= 1 && few) {
    launch_few_rows<RESID ? kEpiResidual : kEpiBf16>(a, w, c, m, n, k, 1, starts, s);
    return;
  }
  if (splits <= 1) {
    constexpr int EPI = RESID ? kEpiResidual : kEpiBf16;
    if constexpr (NJ == 8)
      launch_large<EPI>(a, w, c, m, n, k, s);
    else
      launch_even_rows<EPI, NJ>(a, w, c, m, n, k, k / kBK, 1, starts, s);
    return;
  }
  const KRanges r = k_ranges(k, splits);
  int used = r.used;
  if (few)
    used = launch_few_rows<kEpiPartial>(a, w, workspace, m, n, k, splits, 0, s);
  else
    launch_even_rows<kEpiPartial, NJ>(a, w, workspace, m, n, k, r.per, used, 0, s);
  if (tail.kind == kTailLeave) return;               // (gemm_left_ranges tells the caller how many ranges)
  const int64_t mn = (int64_t)m * n;
  if (RESID && tail.kind == kTailRmsNorm)
    launch_kernel(splitk_reduce_norm_kernel, dim3((unsigned)m), 256, 0, s, workspace, (float*)c, (const bf16*)tail.gain,
                                                               (bf16*)tail.out, mn, n, used, tail.eps);
  else if (!RESID && tail.kind == kTailSwiGLU)
    launch_kernel(splitk_reduce_swiglu_kernel, dim3((unsigned)(((int64_t)m * (n / 2) / 8 + 255) / 256)), 256, 0, s,
        workspace, (bf16*)tail.out, m, n / 2, used);
  else
    launch_kernel(splitk_reduce_kernel<RESID>, dim3((unsigned)((mn / 8 + 255) / 256)), 256, 0, s, workspace, c, mn / 8,
                                                                                     mn, used);
}

// ------------------------------------------------------------------------------------------
// fp32 GEMM (debug path) on v_mfma_f32_16x16x4_f32: products and sums in fp32, 256 FLOP per clock and
// CU.  256 threads = WM x 4 / WM waves, wave tile (16 TM) x (16 TN), K consumed 32 at a time through a ring
// of three LDS stages filled by DMA two to three k-tiles ahead (128-byte rows, chunk c of row r at position
// c ^ ((r >> 1) & 7): conflict-free for the 16-row fragment reads, as in the bf16 kernel).  The
// instruction takes one k per lane quarter; a lane reads four consecutive k of its row with one
// ds_read_b128 and step j of four multiplies the j-th of each quarter -- A and W are permuted over k
// alike.  Chunks past K are fetched from outside the descriptor, so they read as zero (K % 4 == 0).
// The matrix pipes bound it: 300 rows of the 8B shape's gate_up projection, several workgroups per CU, keep them busy 85 % of its
// cycles (at 2.3 GHz), down and o, one per CU, 75 %.  Against the plain FMA kernel below gate_up 2040 -> 568 us (132 TFLOP/s of
// 157, row padding included), down 2476 -> 317 us; f32_tile_rows chooses the tile.  Half a k-tile's fragments are read, and the
// next DMA issued, while the other half is multiplied: with both in front of their MFMAs, us, 16-row tiles 67 x 4096 x 14336 179
// -> 161, 80-row ones 300 x 4096 x 14336 330 -> 317, 64-row ones 300 x 28672 x 4096 580 -> 568, 128-row ones 1000 x 4096 x 4096
// 273 -> 261.  Waves side by side along N (WM = 1) for heights that are no multiple of 32.
// ------------------------------------------------------------------------------------------
constexpr int kFK = 32;

__device__ __forceinline__ void f32_dma(const float* panel, uint32_t bytes, float* lds_rows, uint32_t voff, int kbyte) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(panel_rsrc(panel, bytes), (__attribute__((address_space(3))) void*)lds_rows, 16,
                                           voff, kbyte, 0, 0);
}

template <int TM, int TN, int WM, bool RESID>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const float* __restrict__ A,
                                                            const float* __restrict__ W,
                                                            float* __restrict__ C, int M, int N, int K,
                                                            int tiles_m, int tiles_n) {
  constexpr int WN = 4 / WM, BM = 16 * TM * WM, BN = 16 * TN * WN;
  constexpr int IA = (BM + 31) / 32, IW = BN / 32;   // DMA instructions (8 rows of 128 bytes) per wave and k-tile
  constexpr int RA = 32 * IA;                        // rows of A per stage: BM, or 16 more, which are zeros
  constexpr int kWaitNewest = wait_vm<IA + IW>(), kWaitTwoNewest = wait_vm<2 * (IA + IW)>();   // all but the newest k-tile's, two
  static_assert(BN % 32 == 0 && 2 * (IA + IW) < 64);
  __shared__ __attribute__((aligned(1024))) float s0[(RA + BN) * kFK];
  __shared__ __attribute__((aligned(1024))) float s1[(RA + BN) * kFK];
  __shared__ __attribute__((aligned(1024))) float s2[(RA + BN) * kFK];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  int tile_m, tile_n;
  tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const float* const panel_a = A + (int64_t)m0 * K;
  const float* const panel_w = W + (int64_t)n0 * K;
  const uint32_t bytes_a = (uint32_t)(min(BM, M - m0) * K * 4), bytes_w = (uint32_t)(min(BN, N - n0) * K * 4);
  // Instruction i of this wave fills rows 8 (wave * IA + i) .. + 7; lane: row lane/8, chunk position lane%8.
  uint32_t off_a[IA], off_w[IW];
  int k_a[IA], k_w[IW];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int row = 8 * (wave * IA + i) + (lane >> 3);
    k_a[i] = 4 * ((lane & 7) ^ ((row >> 1) & 7));
    off_a[i] = row < BM ? (uint32_t)((row * K + k_a[i]) * 4) : kOffOutOfRange;
  }
#pragma unroll
  for (int i = 0; i < IW; ++i) {
    const int row = 8 * (wave * IW + i) + (lane >> 3);
    k_w[i] = 4 * ((lane & 7) ^ ((row >> 1) & 7));
    off_w[i] = (uint32_t)((row * K + k_w[i]) * 4);
  }
  const int kt_count = (K + kFK - 1) / kFK;
  // DMA instruction d of k-tile t (past the last k-tile every chunk is outside: nothing to fetch).
  auto fetch_one = [&](int t, float* s, int d) __attribute__((always_inline)) {
    const int left = K - t * kFK;
    if (d < IA) f32_dma(panel_a, bytes_a, s + 8 * (wave * IA + d) * kFK, k_a[d] < left ? off_a[d] : kOffOutOfRange, t * kFK * 4);
    else f32_dma(panel_w, bytes_w, s + (RA + 8 * (wave * IW + d - IA)) * kFK, k_w[d - IA] < left ? off_w[d - IA] : kOffOutOfRange, t * kFK * 4);
  };
  auto fetch = [&](int t, float* s) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < IA + IW; ++d) fetch_one(t, s, d);
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int frag_row = lane & 15, quad = lane >> 4;
  const int key = (frag_row >> 1) & 7;               // (16-row blocks: the block's first row does not change it)
  // Half a k-tile is 16 k, four per lane and fragment (TM of A, then TN of W).
  struct Half { f32x4 f[TM + TN]; };
  auto read_one = [&](const float* s, int kk, Half& h, int i) __attribute__((always_inline)) {
    const int at = ((kk * 4 + quad) ^ key) * 4;
    const int row = i < TM ? wm * 16 * TM + i * 16 : RA + wn * 16 * TN + (i - TM) * 16;
    h.f[i] = *reinterpret_cast<const f32x4*>(s + (row + frag_row) * kFK + at);
  };
  // The MFMAs of one half, and behind each of them, inside the cycles it takes, one of `n` reads and DMA instructions (in front of
  // the MFMAs 300 x 4096 x 14336 323 us, so 317).  Up to two accumulators, whose MFMAs wait for each other anyway: in front of
  // them (67 x 6144 x 4096 52.9 us, between them 57).
  auto multiply = [&](const Half& h, int n, auto&& other) __attribute__((always_inline)) {
    constexpr int kMfmas = 4 * TM * TN;
    constexpr bool kBetween = TM * TN > 2;
    static_assert(!kBetween || kMfmas >= TM + TN + IA + IW);
    if (!kBetween) {
#pragma unroll
      for (int x = 0; x < n; ++x) other(x);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = 0; m < kMfmas; ++m) {
      const int e = m / (TM * TN), i = m / TN % TM, j = m % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(h.f[TM + j][e], h.f[i][e], acc[i][j], 0, 0, 0);
      if (kBetween && m < n) other(m);
      if (kBetween || m == kMfmas - 1) __builtin_amdgcn_sched_barrier(0);
    }
  };
  Half h0, h1;
  // K-tile t on stage s, t + 1 on `next`.  On entry the first half's fragments are read (or on their way) and t + 1 and t + 2 in flight; at
  // the barrier this wave is done with the stage and its share of t + 1 has landed.
  auto step = [&](int t, float* s, const float* next) __attribute__((always_inline)) {
    multiply(h0, TM + TN, [&](int x) __attribute__((always_inline)) { read_one(s, 1, h1, x); });
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_waitcnt(kWaitNewest);
    w4_barrier();
    multiply(h1, TM + TN + IA + IW, [&](int x) __attribute__((always_inline)) {
      if (x < TM + TN) read_one(next, 0, h0, x);
      else fetch_one(t + 3, s, x - TM - TN);
    });
  };
  fetch(0, s0);
  fetch(1, s1);
  fetch(2, s2);
  __builtin_amdgcn_s_waitcnt(kWaitTwoNewest);
  w4_barrier();
#pragma unroll
  for (int x = 0; x < TM + TN; ++x) read_one(s0, 0, h0, x);
  for (int t = 0; t < kt_count; t += 3) {
    // Always three: up to two k-tiles of zeros at the end.  (With a branch between them the compiler
    // waits for all DMA before it reads a stage.)
    step(t, s0, s1);
    step(t + 1, s1, s2);
    step(t + 2, s2, s0);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);              // the last (empty) fetches

  // W is the row operand: accumulator [i][j] of a lane holds row m = 16 i + lane % 16 and the four
  // consecutive columns 16 j + 4 (lane / 16) + (0..3).
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm * 16 * TM + i * 16 + frag_row;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * 16 * TN + j * 16 + 4 * quad;
      if (m < M && n < N) {                          // N % 8 == 0: all four or none
        float* c = C + (int64_t)m * N + n;
        f32x4 v = acc[i][j];
        if (RESID) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(c);
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = x[b] + v[b];
        }
        *reinterpret_cast<f32x4*>(c) = v;
      }
    }
  }
}

template <int TM, int TN, int WM, bool RESID>
static void launch_f32_mfma(const float* a, const float* w, float* c, int m, int n, int k, hipStream_t s) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * (4 / WM);
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + BN - 1) / BN;
  launch_kernel(gemm_f32_mfma_kernel<TM, TN, WM, RESID>, dim3((unsigned)(tiles_m * tiles_n)), 256, 0, s,
      a, w, c, m, n, k, tiles_m, tiles_n);
}

template <bool RESID>
static void launch_f32(const float* a, const float* w, float* c, int64_t m, int64_t n, int64_t k, hipStream_t s) {
  switch (f32_tile_rows(m, n, k, RESID)) {
    case 16: launch_f32_mfma<1, 1, 1, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
    case 32: launch_f32_mfma<1, 2, 2, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
    case 48: launch_f32_mfma<3, 1, 1, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
    case 64: launch_f32_mfma<2, 2, 2, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
    case 80: launch_f32_mfma<5, 1, 1, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
    default: launch_f32_mfma<4, 4, 2, RESID>(a, w, c, (int)m, (int)n, (int)k, s); break;
  }
}

// ------------------------------------------------------------------------------------------
// fp32 GEMM for operands that are not 16-byte aligned or too long for 32-bit offsets: 64x64 tile, 256 threads, 4x4 outputs per
// thread, K step 16, plain FMAs.
// ------------------------------------------------------------------------------------------
template <bool RESID>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A,
                                                       const float* __restrict__ W,
                                                       float* __restrict__ C, int M, int N,
                                                       int K) {
  __shared__ float sA[16][64 + 1];
  __shared__ float sW[16][64 + 1];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + i * 256;          // 0..1023 = 64 rows x 16 k
      const int row = e >> 4, kk = e & 15;
      const int gm = m0 + row, gn = n0 + row, gk = k0 + kk;
      sA[kk][row] = (gm < M && gk < K) ? A[(int64_t)gm * K + gk] : 0.f;
      sW[kk][row] = (gn < N && gk < K) ? W[(int64_t)gn * K + gk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sA[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sW[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < M && n < N) {
        float* c = C + (int64_t)m * N + n;
        *c = RESID ? (*c + acc[i][j]) : acc[i][j];
      }
    }
}

// Problems whose tile small_problem_tile chooses.
static bool takes_small_tiles(int64_t m, int64_t n, int64_t k, size_t workspace_bytes) {
  return w4_plan(1, m, n, k, workspace_bytes).splits == 0;
}

bool gemm_tail_fusable(int dtype, int64_t m, int64_t n, int64_t k, size_t workspace_bytes, int tail_kind) {
  if (w4_plan(dtype, m, n, k, workspace_bytes).splits <= 1) return false;   // tails ride on the split-K reduction
  if (tail_kind == kTailRmsNorm) return n <= kTailNormCols;
  if (tail_kind == kTailSwiGLU) return n % 16 == 0;
  return tail_kind == kTailLeave;
}

int gemm_left_ranges(int dtype, int64_t m, int64_t n, int64_t k, size_t workspace_bytes) {
  W4Shape plan = w4_plan(dtype, m, n, k, workspace_bytes);
  if (plan.splits > 1) plan = w4_cut(m, n, k, false, plan);
  if (plan.splits <= 1) return 0;
  if (!few_rows(m, n, k)) return k_ranges((int)k, plan.splits).used;
  if (m <= 32) return ring_ranges<2, kEpiPartial>((int)n, (int)k, plan.splits).used;
  if (m <= 64) return ring_ranges<4, kEpiPartial>((int)n, (int)k, plan.splits).used;
  return ring_ranges<8, kEpiPartial>((int)n, (int)k, plan.splits).used;
}

template <bool RESID>
static void launch_small_problem(const bf16* a, const bf16* w, void* c, int m, int n, int k, hipStream_t s) {
  constexpr int EPI = RESID ? kEpiResidual : kEpiBf16;
  switch (aligned_to(16, a, w, c) ? small_problem_tile(m, n, k, RESID) : GemmTile::kAny128) {
    case GemmTile::kRing32: launch_ring<2, EPI>(a, w, c, m, n, k, 1, s); break;
    case GemmTile::kRing64: launch_ring<4, EPI>(a, w, c, m, n, k, 1, s); break;
    case GemmTile::kRing128: launch_ring<8, EPI>(a, w, c, m, n, k, 1, s); break;
    case GemmTile::kAny128: launch_bf16_any<RESID>(a, w, c, m, n, k, s); break;
    case GemmTile::kLarge: {
      const int tiles_m = (m + 255) / 256, tiles_n = (n + 255) / 256;
      launch_kernel(gemm_bf16_w4_kernel<EPI, false, 8, true>, dim3((unsigned)(tiles_m * tiles_n)), 256, 0, s,
          a, w, c, m, n, k, tiles_m, tiles_n, k / kBK, 0, nullptr, nullptr);
      break;
    }
  }
}

void launch_gemm(int dtype, const void* a, const void* w, void* c, int64_t m, int64_t n,
                 int64_t k, int residual, void* workspace, size_t workspace_bytes, hipStream_t s,
                 const GemmTail* tail) {
  if (m == 0 || n == 0) return;
  if (dtype == 0) {
    const uintptr_t address = reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(c);
    if (address % 16 == 0 && n % 4 == 0 && k % 4 == 0 && k <= (1 << 20) && (m + 31) / 32 * ((n + 63) / 64) <= INT32_MAX) {
      if (residual) launch_f32<true>((const float*)a, (const float*)w, (float*)c, m, n, k, s);
      else launch_f32<false>((const float*)a, (const float*)w, (float*)c, m, n, k, s);
      return;
    }
    dim3 grid((unsigned)((n + 63) / 64), (unsigned)((m + 63) / 64));
    if (residual)
      launch_kernel(gemm_f32_kernel<true>, grid, 256, 0, s, (const float*)a, (const float*)w, (float*)c,
                                                  (int)m, (int)n, (int)k);
    else
      launch_kernel(gemm_f32_kernel<false>, grid, 256, 0, s, (const float*)a, (const float*)w, (float*)c,
                                                   (int)m, (int)n, (int)k);
    return;
  }
  const bf16* pa = (const bf16*)a;
  const bf16* pw = (const bf16*)w;
  // K a multiple of 64 and enough 256x256 tiles (or enough K to split) to occupy the chip: the one-wave-per-SIMD DMA
  // kernel, split over K when the caller's workspace allows.  Otherwise the tile small_problem_tile chooses.  Operands
  // those do not take: the register-staged kernel on 128x128 tiles.
  W4Shape plan = w4_plan(dtype, m, n, k, workspace_bytes);
  const GemmTail none{};
  const GemmTail& tl = tail && gemm_tail_fusable(dtype, m, n, k, workspace_bytes, tail->kind) ? *tail : none;
  if (!aligned_to(4, a, w, c)) {
    // The tail (kTailLeave apart, which goes with operands of the runtime's own) as the operator it stands for.  A cut
    // problem's workspace has room for at least two fp32 [m][n]: the unfused gate_up projection goes there.
    if (residual) launch_bf16_any<true>(pa, pw, c, (int)m, (int)n, (int)k, s);
    else launch_bf16_any<false>(pa, pw, tl.kind == kTailSwiGLU ? workspace : c, (int)m, (int)n, (int)k, s);
    if (tl.kind == kTailRmsNorm) launch_rmsnorm(dtype, (const float*)c, tl.gain, tl.out, m, n, tl.eps, s);
    if (tl.kind == kTailSwiGLU) launch_silu_mul(dtype, workspace, tl.out, m, n / 2, s);
    return;
  }
  if (plan.splits > 1) plan = w4_cut(m, n, k, residual, plan);
  const int splits = plan.splits;
  if (splits == 1 && tl.kind == kTailSwiGLU) {       // not cut after all: the fused epilogue gives the same bits
    launch_gemm_swiglu(a, w, tl.out, m, n / 2, k, s);
    return;
  }
  if (splits >= 1 && plan.nj == 8) {
    if (residual) launch_bf16_w4<true, 8>(pa, pw, c, (int)m, (int)n, (int)k, splits, (float*)workspace, tl, s);
    else launch_bf16_w4<false, 8>(pa, pw, c, (int)m, (int)n, (int)k, splits, (float*)workspace, tl, s);
  } else if (splits >= 1) {
    if (residual) launch_bf16_w4<true, 4>(pa, pw, c, (int)m, (int)n, (int)k, splits, (float*)workspace, tl, s);
    else launch_bf16_w4<false, 4>(pa, pw, c, (int)m, (int)n, (int)k, splits, (float*)workspace, tl, s);
  } else if (residual) {
    launch_small_problem<true>(pa, pw, c, (int)m, (int)n, (int)k, s);
  } else {
    launch_small_problem<false>(pa, pw, c, (int)m, (int)n, (int)k, s);
  }
}

// ------------------------------------------------------------------------------------------
// Diagnostic: what the matrix pipes sustain on this chip with nothing else in the way -- a loop of
// v_mfma_f32_16x16x32_bf16 (the instruction of the GEMM; on random operands it sustains about 12 %
// more than v_mfma_f32_32x32x16_bf16, which attention uses) on 32 independent accumulators from
// registers, random operands (the data the pipes chew on changes the power they draw, and with it
// the clock), two waves per SIMD on every CU.  The GEMM and attention kernels are judged against
// this as well as against the vendor peak.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512) void mfma_ceiling_kernel(float* __restrict__ sink, int iters) {
  f32x4_acc acc[32];
#pragma unroll
  for (int i = 0; i < 32; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] = 0.f;
  bf16x8 a[4], b[8];
  uint32_t h = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
#pragma unroll
  for (int f = 0; f < 12; ++f) {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h = h * 1664525u + 1013904223u;
      v[e] = static_cast<bf16>((float)((h >> 8) & 0xFFFF) / 65536.0f - 0.5f);
    }
    if (f < 4) a[f] = v; else b[f - 4] = v;
  }
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        acc[i * 8 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i * 8 + j], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) s += acc[i][r];
  sink[(size_t)blockIdx.x * 512 + threadIdx.x] = s;
}

// Launches the loop on `blocks` workgroups of 8 waves; returns the FLOPs one launch performs.
double launch_mfma_ceiling(float* sink, int blocks, int iters, hipStream_t s) {
  mfma_ceiling_kernel<<<dim3((unsigned)blocks), 512, 0, s>>>(sink, iters);
  return (double)blocks * 8.0 * (double)iters * 32.0 * 2.0 * 16.0 * 16.0 * 32.0;
}

}  // namespace fp
