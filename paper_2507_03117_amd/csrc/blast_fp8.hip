// E5M2 entry points: quantisation of bf16 data and the block-sparse product on E5M2 operands
// (BLaST Sec. 5.2 runs the kernel in float8_e5m2 as well as in 16-bit types).
#include "blast_common.h"

#include "kern_common.h"
#include "kern_fp8.h"

using namespace blast_dev;

namespace {

template <int B, bool KSPLIT, bool CHUNK = false>
int launch_fp8(Fp8Args a, hipStream_t stream) {
  using C = Fp8Cfg<B>;
  static blast::DeviceFlags lds_set;
  int dev = 0;
  BLAST_HIP_TRY(hipGetDevice(&dev));
  if (!lds_set.test(dev)) {
    BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_spmm_fp8<B, KSPLIT, CHUNK>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES));
    lds_set.set(dev);
  }
  const int64_t tokens_per_group = KSPLIT ? 64 : 256;
  const int64_t groups = (a.T + tokens_per_group - 1) / tokens_per_group;
  const int64_t grid = ((int64_t)a.n_units + 7) / 8 * 8 * groups;
  if (grid <= 0) return BLAST_OK;
  if (grid > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  a.groups = (int)groups;
  if (CHUNK) {
    // rows cut into several chunks are accumulated: clear them first (the kernel of the bf16 path; it only
    // reads the output description, the row pointers and the plan)
    StreamArgs sa{};
    sa.t.m0.row_ptr = a.row_ptr;
    sa.t.Y = a.Y;
    sa.t.syt = a.ldy;
    sa.t.syi = 1;
    sa.t.T = a.T;
    sa.hdr = a.hdr;
    sa.chunk_row = a.chunk_row;
    sa.chunk_kb = a.chunk_kb;
    sa.chunk_ke = a.chunk_ke;
    k_zero_shared_rows<B><<<dim3((unsigned)(a.n_units / C::SUB), (unsigned)((a.T + 63) / 64)), dim3(256), 0, stream>>>(sa);
    BLAST_LAUNCH_CHECK("k_zero_shared_rows");
  }
  k_spmm_fp8<B, KSPLIT, CHUNK><<<dim3((unsigned)grid), dim3(256), C::LDS_BYTES, stream>>>(a);
  BLAST_LAUNCH_CHECK("k_spmm_fp8");
  return BLAST_OK;
}

int cu_count_fp8() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

// Many tokens: the streaming kernel of the bf16 product, instantiated for one-byte values.  A wave that copies the
// weights for its own 64 x 64 tile asks the L1 for 128 bytes per clock at the matrix peak, and the two 64-row halves
// of a 128-wide block, on different XCDs, each bring the block's activations across the fabric; shared by a workgroup,
// a 256-token x 128-row tile asks for 47, and the activations come once.  53248 x 16384, 95 % uniform, bf16 output,
// column groups: 1000 tokens 99.9 -> 85.9 us, 2048 tokens 227.5 -> 143.8 (1.24 PFLOP/s on stored blocks).  Bound there by the
// fabric: 348 MB read and 112 MB written in 86 us (rows pinned to XCDs instead of token tiles: 98.4).
template <int B, int TW, int NW>
int launch_fp8_stream(const Fp8Args& f, hipStream_t stream) {
  using C = StreamCfg<B, TW, NW, true>;
  StreamArgs sa{};
  TileArgs& a = sa.t;
  a.m0.row_ptr = f.row_ptr;
  a.m0.col_idx = f.col_idx;
  a.m0.vals8 = f.vals;
  a.row_order = f.row_order;
  a.X = reinterpret_cast<const uint16_t*>(f.X);
  a.Y = f.Y;
  a.syt = f.ldy;
  a.syi = 1;
  a.y_bf16 = f.y_bf16;
  a.y_fast = ((int64_t)256 * f.ldy * 4 + f.ldy * 4 < ((int64_t)1 << 31)) ? 1 : 0;
  a.y_pairs = (f.ldy % 2 == 0 && blast::aligned(f.Y, f.y_bf16 ? 4 : 8)) ? 1 : 0;
  a.T = f.T;
  a.nbr = f.n_units / (B / 64);
  a.act = -1;
  a.ntt = (f.T + C::TT - 1) / C::TT;
  if ((int64_t)a.ntt * a.nbr > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
  sa.x8_col = f.x_cg ? (B / 64) * f.x_cg : B;
  sa.x8_tok = (uint32_t)f.ldx;
  sa.x8_half = f.x_cg ? (uint32_t)f.x_cg : 64u;
  const int64_t slab = ((int64_t)a.ntt + 7) / 8 * C::TT * f.kdim;
  const int64_t grid = stream_grid<C, B>(sa, a.nbr, cu_count_fp8(), slab);
  auto launch = [&](auto pairs) -> int {
    constexpr auto kernel = &k_spmm_stream<B, false, TW, false, false, NW, false, true, pairs.value>;
    static blast::DeviceFlags lds_set;
    int dev = 0;
    BLAST_HIP_TRY(hipGetDevice(&dev));
    if (!lds_set.test(dev)) {
      BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)C::LDS_BYTES));
      lds_set.set(dev);
    }
    kernel<<<dim3((unsigned)grid), dim3(64 * NW), C::LDS_BYTES, stream>>>(sa);
    BLAST_LAUNCH_CHECK("k_spmm_stream (E5M2)");
    return BLAST_OK;
  };
  // An fp32 output of 64 to 256 MiB, between a quarter of the last-level cache and all of it, with few blocks per row, so that
  // the stores are what the launch does, is written through the L2.  Microseconds, non-temporal / through, the same buffers
  // again and again, then buffers that no cache holds: 4096 x 4096 at 90 %, 4096 tokens 22.0 / 18.2, 23.2 / 22.9; 8192 tokens
  // 40.2 / 32.1, 43.9 / 42.7; 14336 x 4096 at 90 %, 2048 tokens 34.3 / 30.8, 35.7 / 35.7; 4096 tokens 60.4 / 51.6, 62.8 / 63.8;
  // 53248 x 16384 at 95 % (6.4 blocks), 1000 tokens 84.2 / 81.1, 101.7 / 99.9.  Smaller: 14336 x 4096 at 90 %, 512 tokens 11.9 /
  // 11.1, 13.4 / 15.8; larger: 8192 tokens 113 / 126, 124 / 125; more blocks: at 70 % (9.6), 2048 tokens 53.9 / 53.2, 57.0 / 63.9.
  const int64_t y_bytes = (int64_t)f.T * a.nbr * B * 4;
  a.y_keep = B == 128 && !f.y_bf16 && a.y_pairs && y_bytes >= ((int64_t)64 << 20) && y_bytes <= ((int64_t)256 << 20) &&
             f.nnz < 8 * (int64_t)a.nbr;
  if constexpr (C::PAIR) {
    // With 64-wide blocks, rows two apart at 64 bytes of pitch put eight neighbouring lanes of a fragment read on four 16-byte
    // positions instead of eight.  Fewer, wider stores are worth it in bf16 (8192 x 3072 at 90 %, 2048 tokens, neighbouring
    // rows / pairs 14.4 / 13.3 us; 14336 x 4096 at 70 %, 4096 tokens 100 / 96), not in fp32 (17.4 / 17.7; 107 / 112).
    if (!a.y_fast || !a.y_pairs || (B == 64 && !a.y_bf16)) return launch(std::false_type{});
  }
  return launch(std::true_type{});
}

template <int B>
int launch_fp8_b(const Fp8Args& a, const blast_bsr_view* W, hipStream_t stream) {
  // up to two token tiles the stages of a row are dealt to the four waves (every wave streams weights);
  // beyond that the streaming kernel
  if (a.T <= 128) {
    // A row of n blocks is n * (B / 64) / 4 stages deep per wave.  When the fullest row is deeper than four
    // chunks' worth, take the packer's chunk plan (fp32 output only: chunks of a row add atomically).
    if (W->aux && !a.y_bf16 && W->max_row_blocks > 4 * blast::kChunkBlocks) {
      const int64_t nbr = W->rows / B, nbc = W->cols / B;
      const blast::AuxLayout L = blast::aux_layout(nbr, nbc, W->nnz);
      const char* ab = static_cast<const char*>(W->aux);
      Fp8Args c = a;
      c.hdr = reinterpret_cast<const int*>(ab + L.hdr_off);
      c.chunk_row = reinterpret_cast<const int*>(ab + L.chunk_row_off);
      c.chunk_kb = reinterpret_cast<const int*>(ab + L.chunk_kb_off);
      c.chunk_ke = reinterpret_cast<const int*>(ab + L.chunk_ke_off);
      const int64_t max_chunks = nbr + W->nnz / blast::kChunkBlocks;
      if (max_chunks * (B / 64) > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
      c.n_units = (int)(max_chunks * (B / 64));
      return launch_fp8<B, true, true>(c, stream);
    }
    return launch_fp8<B, true>(a, stream);
  }
  const int64_t rows = a.n_units / (B / 64), cus = cu_count_fp8();
  const int64_t tiles = (a.T + 255) / 256, half_tiles = (a.T + 127) / 128;
  const bool wide = tiles * rows >= 2 * cus;
  if constexpr (B == 128) {
    // (the streaming kernel holds a lane's offset into both column groups of a block in 32 bits: 2^25 tokens)
    if (a.x_cg > UINT32_MAX / 2) return launch_fp8<B, false>(a, stream);
    // A second 128-token tile that is hardly begun costs as much as the first; a wave without tokens costs nothing.
    // It shows where the tiles do not fit the CUs at once (two workgroups each): 53248 x 16384, 129 tokens, 90 % sparse
    // 35.0 against 37.1 us, 95 % 22.6 against 23.6; 160 tokens 95 % 24.1 against 23.6.
    if (a.T <= 128 + 16 && half_tiles * rows > 2 * cus) return launch_fp8<B, false>(a, stream);
    if (wide) return launch_fp8_stream<128, 4, 8>(a, stream);
    return launch_fp8_stream<128, 2, 4>(a, stream);
  } else {
    // A wave that owns its token tile starts copying two trips to the memory earlier than the streaming kernel with its
    // table of items, which shows while a workgroup slot (two per CU) has only a few blocks: 8192 x 3072, 1000 tokens, 614 blocks
    // (4.8 per slot) 11.7 against 13.5 us; 1843 blocks, 300 tokens (7.2) 12.6 against 13.0; 2048 tokens (29) 30.9
    // against 27.5.
    if (W->nnz * tiles < 6 * 2 * cus) return launch_fp8<B, false>(a, stream);
    // Its workgroups (256 tokens of a row) all fit at once and the streaming kernel's 128-token tiles do not: the fuller
    // the rows, the more the second, partly empty round costs.  14336 x 4096, 512 tokens (448 against 896 workgroups for
    // 512 places): half the blocks stored 26.6 against 31.8 us, 30 % 20.5 against 21.9; 8192 x 3072, 700 tokens: half 20.6
    // against 24.1, 30 % 16.7 against 17.5, 20 % 14.8 against 14.4; 4096 x 14336, 1500 tokens, 10 %: 25.5 against 22.7.
    if (tiles * rows <= 2 * cus && half_tiles * rows > 2 * cus && 4 * W->nnz >= rows * (W->cols / B))
      return launch_fp8<B, false>(a, stream);
    if (wide) return launch_fp8_stream<64, 4, 4>(a, stream);
    return launch_fp8_stream<64, 2, 4>(a, stream);
  }
}

}  // namespace

extern "C" int blast_quantize_e5m2(const uint16_t* in_bf16, int64_t n, uint8_t* out, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (n < 0) return BLAST_ERR_INVALID_ARG;
  if (n == 0) return BLAST_OK;
  if (!in_bf16 || !out) return BLAST_ERR_INVALID_ARG;
  const int64_t blocks = ((n + 7) / 8 + 255) / 256;
  if (blocks > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  k_quantize_e5m2<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(in_bf16, n, out);
  BLAST_LAUNCH_CHECK("k_quantize_e5m2");
  return BLAST_OK;
}

extern "C" int blast_quantize_e5m2_groups(const uint16_t* X_bf16, int64_t ldx, int64_t T, int64_t K, uint8_t* out,
                                          void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (T < 0 || K < 0 || K % 64 != 0) return BLAST_ERR_INVALID_ARG;
  if (T == 0 || K == 0) return BLAST_OK;
  if (!X_bf16 || !out || ldx < K || !blast::aligned(out, 16)) return BLAST_ERR_INVALID_ARG;
  const int64_t blocks = (T + kQuantTokens - 1) / kQuantTokens;
  if (blocks > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  const int wide = ldx % 8 == 0 && blast::aligned(X_bf16, 16);
  for (int64_t c = 0; c < K / 64; c += 65535) {  // (gridDim.y holds 65535 column groups)
    const int64_t n = K / 64 - c < 65535 ? K / 64 - c : 65535;
    k_quantize_e5m2_groups<<<dim3((unsigned)blocks, (unsigned)n), dim3(256), 0, stream>>>(X_bf16 + c * 64, ldx, T, wide,
                                                                                          out + c * 64 * T);
  }
  BLAST_LAUNCH_CHECK("k_quantize_e5m2_groups");
  return BLAST_OK;
}

extern "C" int blast_bsr_spmm_e5m2(const blast_bsr_view* W, const uint8_t* vals8, const uint8_t* X8, int64_t ldx,
                                   int32_t x_layout, int64_t T, void* Y, int64_t ldy, int32_t y_dtype,
                                   void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!W || !W->row_ptr) return BLAST_ERR_INVALID_ARG;
  if (W->rows < 0 || W->cols < 0 || W->nnz < 0 || W->nnz > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  if (!blast::supported_block(W->b)) return BLAST_ERR_UNSUPPORTED_BLOCK;
  if (W->rows % W->b || W->cols % W->b) return BLAST_ERR_SHAPE;
  if (W->rows / W->b > INT32_MAX / 4 || W->cols / W->b > INT32_MAX / 4) return BLAST_ERR_INVALID_ARG;
  if (x_layout != BLAST_TOKEN_MAJOR && x_layout != BLAST_FEATURE_MAJOR && x_layout != BLAST_COLUMN_GROUPS_64)
    return BLAST_ERR_INVALID_ARG;
  if (y_dtype != BLAST_F32 && y_dtype != BLAST_BF16) return BLAST_ERR_INVALID_ARG;
  if (T < 0 || T > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
  if (T == 0 || W->rows == 0) return BLAST_OK;
  const bool cg = x_layout == BLAST_COLUMN_GROUPS_64;  // activations in column groups; the output is token-major
  const bool tm = x_layout == BLAST_TOKEN_MAJOR || cg;
  if (!Y || ldy < (tm ? W->rows : T)) return BLAST_ERR_INVALID_ARG;
  if (W->cols > 0 && (!X8 || (!cg && ldx < (tm ? W->cols : T)))) return BLAST_ERR_INVALID_ARG;
  if (W->nnz > 0 && (!W->col_idx || !vals8)) return BLAST_ERR_INVALID_ARG;
  const int b = W->b;
  if (cg) {
    // only the tiled kernel reads this layout: 64-wide groups need b >= 64, offsets inside a group 32 bits
    if (b < 64 || !blast::aligned(X8, 16) || !blast::aligned(vals8, 16) || T * 64 >= ((int64_t)1 << 32))
      return BLAST_ERR_INVALID_ARG;
  }
  const bool fast = cg || (tm && b >= 64 && ldx % 16 == 0 && blast::aligned(X8, 16) && blast::aligned(vals8, 16) &&
                           T * ldx < ((int64_t)1 << 32));
  if (fast) {
    Fp8Args a{};
    a.row_ptr = W->row_ptr;
    a.col_idx = W->col_idx;
    a.row_order = W->row_order;
    a.vals = vals8;
    a.X = X8;
    a.ldx = cg ? 64 : ldx;
    a.x_cg = cg ? T * 64 : 0;
    a.kdim = W->cols;
    a.nnz = W->nnz;
    a.Y = Y;
    a.ldy = ldy;
    a.y_bf16 = y_dtype == BLAST_BF16 ? 1 : 0;
    a.y_fast = ((int64_t)64 * ldy * 4 + ldy * 4 < ((int64_t)1 << 31)) ? 1 : 0;
    a.T = (int)T;
    a.n_units = (int)(W->rows / b) * (b / 64);
    return b == 64 ? launch_fp8_b<64>(a, W, stream) : launch_fp8_b<128>(a, W, stream);
  }
  Fp8GenericArgs g{};
  g.row_ptr = W->row_ptr;
  g.col_idx = W->col_idx;
  g.vals = vals8;
  g.X = X8;
  g.sxk = tm ? 1 : ldx;
  g.sxt = tm ? ldx : 1;
  g.Y = Y;
  g.syt = tm ? ldy : 1;
  g.syi = tm ? 1 : ldy;
  g.y_bf16 = y_dtype == BLAST_BF16 ? 1 : 0;
  g.T = (int)T;
  g.b = b;
  const int64_t nbr = W->rows / b, tiles = (T + 63) / 64;
  if (tiles > 65535) return BLAST_ERR_INVALID_ARG;
  k_spmm_fp8_generic<<<dim3((unsigned)nbr, (unsigned)tiles), dim3(256), 0, stream>>>(g);
  BLAST_LAUNCH_CHECK("k_spmm_fp8_generic");
  return BLAST_OK;
}
