// Product kernel for few output tiles: a few hundred tokens, few block rows (token-major, 16-byte aligned activations).
//
// The streaming kernel gives an output tile to one workgroup, which walks the block row in sequence; with fewer tiles
// than CUs that chain is the whole launch while most of the chip has nothing to do.  Here a workgroup of eight or four waves
// shares a tile of 64 rows x 64 tokens by the contraction: the row's stages (64 contraction indices, whole 128-byte lines
// of a block and of the activations) are dealt to the waves, each accumulates the whole tile from copies of its own, and
// the partial sums meet in LDS.  No barrier before that.
//  - A wave owns one 16 KiB stage in LDS.  Its fragments go to registers as soon as it has landed (64 of them), so that
//    the next stage is copied over it while they are multiplied: eight stages are in flight per CU.  One workgroup of eight
//    waves fits a CU, or two of four, for up to twice and three times as many tiles as CUs, of which one is multiplied
//    while the other adds up or waits for its indices (2048 x 2048 at 90 %, 64-wide, 700 tokens, 352 tiles: 7.2 -> 5.8 us;
//    4096 x 4096 at 90 %, 128-wide, 500 tokens, 512 tiles: 10.9 -> 9.4).
//  - Rows of a wave's tile alternate between the two matrix tiles, so that a lane ends up with two neighbouring rows of a
//    token, as in the streaming kernel.
//  - Both forms add up the same eight chains: each of four waves keeps two accumulators, of every other stage it is dealt,
//    and adds them before the sums meet, as of eight waves 0 and 4, 1 and 5, ... are; so a token's row is the same bits
//    whichever form the size of a call leads to.  (With one accumulator a wave: 0.1 to 0.6 us slower than with two on rows of
//    10 to 26 blocks, 459 to 1590 tokens, b = 64, and chains twice as long.)
// Relative error against 64 bits, one chain (streaming kernel) / four / eight chains: b = 64, 40 rows of 5, 449 tokens 9.7e-8
// / 6.5e-8 / 6.2e-8; 33 rows of 24, 640 tokens 2.3e-7 / 1.14e-7 / 8.8e-8; b = 128, 24 rows of 4, one of 50, 900 tokens 3.2e-7 /
// 1.54e-7 / 1.12e-7.  2048 x 8192 at 90 %, 256 tokens, decode kernel / this one: 0.9e-7 / 0.8e-7.
// Second product of the two-matrix MLP of 1600 and 6400 features at 80 %, 384 tokens: 17.0 us on the streaming kernel, 10.6.
// What bounds it: a tile asks the L1 for a byte per 32 flop, half the matrix peak at 64 bytes a clock; at these sizes the
// chain (indices, one trip per stage, the sums in LDS) is most of the launch.
#pragma once
#include "kern_common.h"
#include "kern_stream.h"
#include "split_rule.h"

namespace blast_dev {

template <int B, int NWAVES>
struct SplitCfg {
  static_assert(B == 64 || B == 128, "a stage is a whole 128-byte line deep");
  static constexpr int NW = NWAVES;
  static constexpr int SETS = 8 / NW;         // chains of a wave
  static constexpr int SB = 64;               // rows and tokens of the tile
  static constexpr int SUB = B / SB;          // tiles per block row
  static constexpr int KSL = B / 64;          // stages per stored block
  static constexpr int TILE = SB * 128;       // bytes of one operand of a stage
  static constexpr int NI = TILE / 1024;      // wave-wide copy instructions per operand
  static constexpr int STAGE = 2 * TILE;
  static constexpr size_t LDS_BYTES = (size_t)NW * STAGE;  // (the partial sums are as large)
  static_assert(sizeof(float) * 64 * 64 == STAGE, "a wave's sums go over its stage");
};

template <int B, bool POST, int NWAVES>
__global__ __launch_bounds__(64 * NWAVES, 2) void k_spmm_split(const TileArgs a, const int n_units, const int groups,
                                                               const int stride_log2) {
  using C = SplitCfg<B, NWAVES>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const SplitTile tile = split_tile(blockIdx.x, stride_log2, groups);
  const int unit = tile.unit;
  if (unit >= n_units) return;  // whole workgroup, before any barrier
  const int t0 = tile.group * C::SB;
  const int rank = unit / C::SUB, si = unit % C::SUB;
  const int r = a.row_order ? ld_idx(a.row_order, rank) : rank;
  const int kb = ld_idx(a.m0.row_ptr, r);
  const int stages = (ld_idx(a.m0.row_ptr, r + 1) - kb) * C::KSL;
  const int mine = stages > wave ? (stages - wave + C::NW - 1) / C::NW : 0;
  unsigned char* slot = smem + wave * C::STAGE;

  // Copy side: instruction q of an operand writes LDS bytes [q * 1024 + lane * 16, +16): tile row q * 8 + lane / 8, chunk
  // lane % 8; it fetches that chunk ^ the key of the lane that reads the row.
  uint32_t woff[C::NI], xoff[C::NI];
#pragma unroll
  for (int q = 0; q < C::NI; ++q) {
    const int row = q * 8 + (lane >> 3), chunk = lane & 7;
    woff[q] = (uint32_t)((si * C::SB + row) * (B * 2) + ((chunk ^ ((row >> 1) & 7)) << 4));
    const int t = t0 + row < a.T ? t0 + row : a.T - 1;  // rows past T are never stored
    xoff[q] = (uint32_t)t * (uint32_t)a.sxt * 2u + (uint32_t)((chunk ^ (row & 7)) << 4);
  }
  auto issue = [&](int s) {
    const int gs = wave + C::NW * s, q = kb + gs / C::KSL, slice = gs % C::KSL;
    const unsigned char* w = reinterpret_cast<const unsigned char*>(a.m0.vals) + (int64_t)q * (B * B * 2) + slice * 128;
    const unsigned char* x = reinterpret_cast<const unsigned char*>(a.X) + (int64_t)ld_idx(a.m0.col_idx, q) * (B * 2) + slice * 128;
#pragma unroll
    for (int i = 0; i < C::NI; ++i) BLAST_GLDS16(w + woff[i], slot + i * 1024);
#pragma unroll
    for (int i = 0; i < C::NI; ++i) BLAST_GLDS16(x + xoff[i], slot + C::TILE + i * 1024);
  };

  f32x16 acc[C::SETS][2][2];  // [chain][token half][even / odd rows]
#pragma unroll
  for (int set = 0; set < C::SETS; ++set)
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nj = 0; nj < 2; ++nj)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[set][mi][nj][v] = 0.0f;
  auto multiply = [&](int s, f32x16 (&sum)[2][2]) {
    __builtin_amdgcn_s_waitcnt(BLAST_VMCNT(0));
    asm volatile("" ::: "memory");
    bf16x8 fw[4][2], fx[4][2];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int chunk = ((2 * kk + lh) ^ (l32 & 7)) << 4;
        fw[kk][h] = *reinterpret_cast<const bf16x8*>(slot + (2 * l32 + h) * 128 + chunk);
        fx[kk][h] = *reinterpret_cast<const bf16x8*>(slot + C::TILE + (32 * h + l32) * 128 + chunk);
      }
    // the fragments are in registers before the next stage is copied over this one
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    if (s + 1 < mine) issue(s + 1);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
          sum[mi][nj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[kk][mi], fw[kk][nj], sum[mi][nj], 0, 0, 0);
    asm volatile("" ::: "memory");
  };
  if (mine > 0) issue(0);
#pragma unroll 1
  for (int s = 0; s < mine; s += C::SETS) {
    multiply(s, acc[0]);
    if constexpr (C::SETS == 2) {
      if (s + 1 < mine) multiply(s + 1, acc[1]);
    }
  }

  if constexpr (C::SETS == 2) {
    if (mine > 1) {
#pragma unroll
      for (int mh = 0; mh < 2; ++mh)
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[0][mh][nj][v] += acc[1][mh][nj][v];
    }
  }
  // Every wave's sums go over its own stage (nothing is in flight into it any more); then a wave owns 1 / NW of the tile:
  // 32 / NW tokens per lane, two rows each.
  float (*red)[64][64] = reinterpret_cast<float (*)[64][64]>(smem);
#pragma unroll
  for (int mh = 0; mh < 2; ++mh)
#pragma unroll
    for (int nj = 0; nj < 2; ++nj)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[wave][(mh * 2 + nj) * 16 + v][lane] = acc[0][mh][nj][v];
  __syncthreads();
  constexpr int PER = 32 / C::NW;  // registers of a lane's half of the tile (token half, v) that a wave owns
  const int mi = wave * PER / 16, v0 = wave * PER % 16;
  const int64_t row = (int64_t)r * B + si * C::SB + 2 * l32;
#pragma unroll
  for (int v = 0; v < PER; ++v) {
    // register v0 + v of a 32 x 32 tile: token 8 * ((v0 + v) / 4) + 4 * lh + v % 4
    const int t = t0 + 32 * mi + 2 * v0 + 8 * (v / 4) + 4 * lh + v % 4;
    if (t >= a.T) continue;
    float y[2];
#pragma unroll
    for (int nj = 0; nj < 2; ++nj) {
      const int id = (mi * 2 + nj) * 16 + v0 + v;
      float part[C::NW];  // (read before any is added: 0.15 us less than read pair by pair)
#pragma unroll
      for (int w = 0; w < C::NW; ++w) part[w] = red[w][id][lane];
      auto pair = [&](int w) { return C::SETS == 2 ? part[w] : part[w] + part[(w + 4) % C::NW]; };
      const float sum = ((pair(0) + pair(1)) + pair(2)) + pair(3);
      y[nj] = POST ? post_act(a.act, sum) : sum;
    }
    const int64_t off = (int64_t)t * a.syt + row * a.syi;
    typedef __bf16 Bf16Pair __attribute__((ext_vector_type(2)));
    typedef float F32Pair __attribute__((ext_vector_type(2)));
    if (a.y_bf16) {
      uint16_t* p = reinterpret_cast<uint16_t*>(a.Y) + off;
      if (a.y_pairs) {
        store_through(reinterpret_cast<Bf16Pair*>(p), Bf16Pair{static_cast<__bf16>(y[0]), static_cast<__bf16>(y[1])});
      } else {
        p[0] = f32_to_bf16_rne(y[0]);
        p[a.syi] = f32_to_bf16_rne(y[1]);
      }
    } else {
      float* p = reinterpret_cast<float*>(a.Y) + off;
      if (a.y_pairs) {
        store_through(reinterpret_cast<F32Pair*>(p), F32Pair{y[0], y[1]});
      } else {
        p[0] = y[0];
        p[a.syi] = y[1];
      }
    }
  }
}

}  // namespace blast_dev
