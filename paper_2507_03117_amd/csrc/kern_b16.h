// Product kernel for 16 x 16 blocks (the smallest block size of BLaST's block-size sweeps, Sec. 5).
//
// A 16-wide block is half the contraction depth of v_mfma_f32_16x16x32_bf16, so the unit of work is a PAIR of
// stored blocks of one block row: consecutive blocks of a row are consecutive in the value array, and the 64
// lanes' 16-byte operand pieces (lane l: block l/32 of the pair, row l%16, columns 8*((l/16)%2) ...) are
// exactly the pair's 1 KiB, one fully coalesced load.  The activation operand of the same instruction is, per
// lane, 16 bytes of one token row at the block's column: both operands go from global memory straight into the
// registers the matrix instruction reads - no LDS, no barrier, nothing to synchronise but the wave's own loads.
// The weight rows are the M side of the instruction, so a lane ends up with four consecutive output rows of one
// token: one 16-byte (fp32) or 8-byte (bf16) store per 16-token tile.
//
// A wave owns (block row, NS tiles of 16 tokens); the four waves of a workgroup take neighbouring token tiles of
// the same block row, so the pair's weights are fetched from the L2 once per workgroup.  What bounds the kernel is
// the vector memory path: every matrix instruction needs a fresh 1 KiB activation fragment (16 bytes per lane =
// 16 flop per byte loaded), where a 64-wide block shares one staged tile between 64 rows.  In a token-major
// tensor that fragment is 32 segments of 32 bytes in 32 different cache lines, and the L2 sends a whole 128-byte
// line for each: with activations stored in column groups of 16 features ([K/16][T][16]: the 16 tokens x 16
// features of a fragment are 512 consecutive bytes) the same fragment is eight whole lines.  The kernel reads
// and writes either layout; the MLP regroups X once (k_group16) and keeps H grouped from the start.
#pragma once
#include "kern_common.h"

namespace blast_dev {

typedef float f32x4_b16 __attribute__((ext_vector_type(4)));

template <int NS>
struct B16Frag {
  bf16x8 w;
  bf16x8 x[NS];
};

// Block column of this lane's block of the pair (kp, kp + 1) of a row that ends at ke (lanes of the second half
// repeat block kp when the row has no block kp + 1); 0 beyond the row.
__device__ __forceinline__ int b16_col(const MatDev& m, int kp, int ke) {
  if (kp >= ke) return 0;
  const int blk = kp + ((threadIdx.x & 63) >> 5);
  return m.col_idx[blk < ke ? blk : kp];
}

// Operands of the pair of blocks (kp, kp + 1), block column c per lane from b16_col.  Lanes of the second half
// hold zeros as their weights when the row has no block kp + 1.
template <int NS>
__device__ __forceinline__ void b16_load(const TileArgs& a, const MatDev& m, int kp, int ke, int64_t c,
                                         const int64_t (&xrow)[NS], int64_t cstride, B16Frag<NS>& f) {
  const int lane = threadIdx.x & 63;
  const int blk = kp + (lane >> 5);
  const bool valid = blk < ke;
  const int src = valid ? blk : kp;
  const int piece = ((lane >> 4) & 1) * 8;
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  const bf16x8 w = *reinterpret_cast<const bf16x8*>(m.vals + (int64_t)src * 256 + (lane & 15) * 16 + piece);
  f.w = valid ? w : zero;
#pragma unroll
  for (int s = 0; s < NS; ++s) f.x[s] = *reinterpret_cast<const bf16x8*>(a.X + xrow[s] + c * cstride + piece);
}

// The stored blocks of block row r of matrix m, two per matrix instruction: pairs pair0, pair0 + pstride, ... of
// the row.  The next pair's operands are on their way while the current pair is multiplied, and the block
// columns are read one pair further ahead (an operand's address depends on them).
template <int NS>
__device__ __forceinline__ void b16_row(const TileArgs& a, const MatDev& m, int r, const int64_t (&xrow)[NS],
                                        int64_t cstride, f32x4_b16 (&acc)[NS], int pair0 = 0, int pstride = 1) {
  const int ke = m.row_ptr[r + 1], step = 2 * pstride;
  int kp = m.row_ptr[r] + 2 * pair0;
  if (kp >= ke) return;
  B16Frag<NS> cur, nxt;
  int c_nxt = b16_col(m, kp + step, ke);
  b16_load<NS>(a, m, kp, ke, b16_col(m, kp, ke), xrow, cstride, cur);
  for (; kp < ke; kp += step) {
    const bool more = kp + step < ke;
    const int c_far = b16_col(m, kp + 2 * step, ke);
    if (more) b16_load<NS>(a, m, kp + step, ke, c_nxt, xrow, cstride, nxt);
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.w, cur.x[s], acc[s], 0, 0, 0);
    if (more) cur = nxt;
    c_nxt = c_far;
  }
}

// ---- activations in column groups of 16 features ---------------------------------------------------------------------
// There a fragment of 16 tokens is 512 consecutive bytes, and those of the wave's next tokens follow it: both operands are
// addressed as (descriptor, one 32-bit offset per lane, an immediate), which leaves the registers to the operands of
// several pairs and takes a column's 64-bit product off every pair.  Reads past the row's values (a row with an odd number
// of blocks) and past the last group return zeros; tokens past T of an inner group are those of the next group and are
// never stored.  1B-shaped MLP with 16-wide blocks at 90 %, microseconds a pass, before / now: 64 tokens 17.2 / 15.8, 128
// 18.4 / 16.9, 1000 49.2 / 42.5, 2048 79.2 / 71.8; at 500, where all waves are resident at once and the three launches'
// start-up is half of it, 29.0 / 28.4.  (Three or four pairs on their way instead of two: 43.0 and 43.5 at 1000.)
struct B16Row {
  int n;                            // pairs of this wave
  int cols;                         // lane 2 i + h: block column of block h of the wave's i-th pair, i < 32
  int k0, ke, pair0, pstride;
  __amdgpu_buffer_rsrc_t w;         // the values of the row's blocks
};

// Columns of up to 32 pairs from the wave's pair `first` on (a row that ends with a single block repeats it).
__device__ __forceinline__ int b16_cols(const MatDev& m, const B16Row& q, int first) {
  const int lane = threadIdx.x & 63;
  const int kp = q.k0 + 2 * (q.pair0 + (first + (lane >> 1)) * q.pstride), blk = kp + (lane & 1);
  return kp < q.ke ? m.col_idx[blk < q.ke ? blk : kp] : 0;
}

__device__ __forceinline__ B16Row b16_begin(const MatDev& m, int r, int pair0, int pstride) {
  B16Row q;
  q.k0 = ld_idx(m.row_ptr, r);
  q.ke = ld_idx(m.row_ptr, r + 1);
  q.pair0 = pair0;
  q.pstride = pstride;
  const int pairs = (q.ke - q.k0 + 1) >> 1;
  q.n = pairs > pair0 ? (pairs - pair0 + pstride - 1) / pstride : 0;
  q.cols = b16_cols(m, q, 0);
  q.w = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(m.vals) + (int64_t)q.k0 * 256, 0, (q.ke - q.k0) * 512, 0x00027000);
  return q;
}

// The wave's pairs of a block row, DEPTH of them on their way at a time (which number: see launch_b16_t).  x_off: byte offset of this
// lane's token row and half in a column group, group_bytes: from one group to the next.
template <int NS, int DEPTH>
__device__ __forceinline__ void b16_walk(const MatDev& m, B16Row& q, __amdgpu_buffer_rsrc_t x, uint32_t x_off,
                                         uint32_t group_bytes, f32x4_b16 (&acc)[NS]) {
  const int lane = threadIdx.x & 63;
  const int w_off = (lane >> 5) * 512 + (lane & 15) * 32 + ((lane >> 4) & 1) * 16;
  auto multiply = [&](const B16Frag<NS>& f) {
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w, f.x[s], acc[s], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // the loads that take these registers stay behind: no second set of them
  };
#pragma unroll 1
  for (int done = 0; done < q.n; done += 32) {
    if (done > 0) q.cols = b16_cols(m, q, done);
    const int n = q.n - done < 32 ? q.n - done : 32;
    B16Frag<NS> f[DEPTH];
    auto load = [&](int i, B16Frag<NS>& d) {
      const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane(q.cols, 2 * i) * group_bytes;
      const uint32_t c1 = (uint32_t)__builtin_amdgcn_readlane(q.cols, 2 * i + 1) * group_bytes;
      const uint32_t off = x_off + (lane < 32 ? c0 : c1);
      d.w = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                           q.w, w_off + (q.pair0 + (done + i) * q.pstride) * 1024, 0, 0));
#pragma unroll
      for (int s = 0; s < NS; ++s)
        d.x[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(x, off + s * 512, 0, 0));
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
      if (u < n) load(u, f[u]);
    int i = 0;
    // nothing is decided per pair while a whole round of loads lies ahead
#pragma unroll 1
    for (; i + 2 * DEPTH <= n; i += DEPTH) {
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        multiply(f[u]);
        load(i + u + DEPTH, f[u]);
      }
    }
#pragma unroll 1
    for (; i < n; i += DEPTH) {
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        if (i + u < n) multiply(f[u]);
        if (i + u + DEPTH < n) load(i + u + DEPTH, f[u]);
      }
    }
  }
}

// Adds the waves' partial sums; every wave calls it, wave 0 returns with the totals (added in wave order).
template <int NS, int NW>
__device__ __forceinline__ void b16_join(f32x4_b16 (&acc)[NS]) {
  __shared__ f32x4_b16 part[NW - 1][NS][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave != 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s) part[wave - 1][s][lane] = acc[s];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int w = 0; w < NW - 1; ++w) acc[s] += part[w][s][lane];
  }
}

// One wave = one (block row, 16 * NS tokens).  DUAL: two matrices with the same block rows, the output is
// bf16-or-fp32 act(W0 x) * (W1 x); POST: one matrix, the activation on its output.
// y_vec: the four rows of a lane can be stored with one 16-byte (fp32) / 8-byte (bf16) store (always so for a
// grouped output).
// SPLIT (decode token counts): the whole workgroup owns one (block row, token tile), its NW waves (4 or 16) deal
// the row's pairs among themselves and the partial sums meet in LDS - there are too few rows to fill the chip
// with a wave each, and a row walked by one wave is a chain of dependent loads.
// DEPTH > 0: X in column groups, b16_walk with that many pairs in flight; 0: either layout of X, b16_row.
template <bool DUAL, bool POST, int NS, bool SPLIT = false, int NW = 4, int DEPTH = 0>
__global__ __launch_bounds__(NW * 64, DEPTH ? 4 : 1) void k_spmm_b16(const TileArgs a, const int y_vec) {
  static_assert(SPLIT || NW == 4, "without SPLIT a workgroup is four independent waves");
  static_assert(!(POST && DUAL), "an activation on the output belongs to the single-matrix product");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t item = SPLIT ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
  const int rank = (int)(item / a.ntt), tt = (int)(item % a.ntt);
  if (rank >= a.nbr) return;  // (whole waves leave; with SPLIT the whole workgroup does)
  const int r = a.row_order ? a.row_order[rank] : rank;
  const int t0 = tt * 16 * NS;

  // element offset of this lane's token row in each tile (rows past the end read the last token), and the
  // distance between block columns: [T][K] or [K/16][T][16]
  const int64_t tstride = a.x_grp16 ? 16 : a.sxt, cstride = a.x_grp16 ? (int64_t)a.T * 16 : 16;
  int64_t xrow[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int t = t0 + s * 16 + (lane & 15);
    xrow[s] = (int64_t)(t < a.T ? t : a.T - 1) * tstride;
  }
  f32x4_b16 acc0[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc0[s] = f32x4_b16{0.f, 0.f, 0.f, 0.f};
  f32x4_b16 acc1[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc1[s] = f32x4_b16{0.f, 0.f, 0.f, 0.f};
  const int pair0 = SPLIT ? __builtin_amdgcn_readfirstlane(wave) : 0, pstride = SPLIT ? NW : 1;
  if constexpr (DEPTH > 0) {
    const uint32_t group_bytes = (uint32_t)a.T * 32u;
    const uint32_t x_off = (uint32_t)(t0 + (lane & 15)) * 32u + ((lane >> 4) & 1) * 16u;
    const __amdgpu_buffer_rsrc_t x = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.X), 0, (int)((uint32_t)(a.kdim >> 4) * group_bytes), 0x00027000);
    const int ru = __builtin_amdgcn_readfirstlane(r);
    B16Row q0 = b16_begin(a.m0, ru, pair0, pstride), q1{};
    if (DUAL) q1 = b16_begin(a.m1, ru, pair0, pstride);
    b16_walk<NS, DEPTH>(a.m0, q0, x, x_off, group_bytes, acc0);
    if (DUAL) b16_walk<NS, DEPTH>(a.m1, q1, x, x_off, group_bytes, acc1);
  } else {
    b16_row<NS>(a, a.m0, r, xrow, cstride, acc0, pair0, pstride);
    if (DUAL) b16_row<NS>(a, a.m1, r, xrow, cstride, acc1, pair0, pstride);
  }
  if (DUAL) {
    if (SPLIT) b16_join<NS, NW>(acc1);
    if (SPLIT) __syncthreads();  // the buffer is used again for the first matrix
    if (SPLIT) b16_join<NS, NW>(acc0);
    if (SPLIT && wave != 0) return;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc0[s][j] = apply_act(a.act, acc0[s][j]) * acc1[s][j];
  } else if (SPLIT) {
    b16_join<NS, NW>(acc0);
    if (wave != 0) return;
  }
  if (POST) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc0[s][j] = apply_act(a.act, acc0[s][j]);
  }

  // Result layout of the 16x16 instruction: lane -> token lane % 16, register j -> row 4 * (lane / 16) + j.
  const int64_t row0 = (int64_t)r * 16 + (lane >> 4) * 4;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int t = t0 + s * 16 + (lane & 15);
    if (t >= a.T) continue;
    if (y_vec) {
      const int64_t off = a.y_grp16 ? ((int64_t)r * a.T + t) * 16 + (lane >> 4) * 4 : (int64_t)t * a.syt + row0;
      if (a.y_bf16) {
        uint2 v;
        v.x = (uint32_t)f32_to_bf16_rne(acc0[s][0]) | ((uint32_t)f32_to_bf16_rne(acc0[s][1]) << 16);
        v.y = (uint32_t)f32_to_bf16_rne(acc0[s][2]) | ((uint32_t)f32_to_bf16_rne(acc0[s][3]) << 16);
        store_through(reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.Y) + off), v);
      } else {
        *reinterpret_cast<f32x4_b16*>(reinterpret_cast<float*>(a.Y) + off) = acc0[s];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t off = (int64_t)t * a.syt + (row0 + j) * a.syi;
        if (a.y_bf16)
          reinterpret_cast<uint16_t*>(a.Y)[off] = f32_to_bf16_rne(acc0[s][j]);
        else
          reinterpret_cast<float*>(a.Y)[off] = acc0[s][j];
      }
    }
  }
}

// Token-major activations [T][K] (row pitch ld) into column groups of 16 features, [K/16][T][16].  A workgroup
// turns 16 tokens x 128 features; a half-wave writes the 512 consecutive bytes of one (column group, 16 tokens).
__global__ __launch_bounds__(256) void k_group16(const uint16_t* __restrict__ X, int64_t ld, int T, int nbc,
                                                 uint16_t* __restrict__ Xg) {
  const int i = threadIdx.x;
  const int half = i & 1, t = (int)blockIdx.x * 16 + ((i >> 1) & 15), c = (int)blockIdx.y * 8 + (i >> 5);
  if (t >= T || c >= nbc) return;
  *reinterpret_cast<uint4*>(Xg + ((int64_t)c * T + t) * 16 + half * 8) =
      *reinterpret_cast<const uint4*>(X + (int64_t)t * ld + c * 16 + half * 8);
}

}  // namespace blast_dev
