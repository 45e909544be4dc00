// Backward-pass products on the packed weight (BLaST Sec. 3.2: the pruned matrix serves forward and
// backward propagation alike).
//
//   dX = W~^T dY   runs as the forward product on the packed transpose that blast_bsr_transpose builds
//                  (the BCSC view of the same blocks, Sec. 3.4.1), so it has no kernel of its own;
//   dW~            the gradient of the stored blocks, a block-sampled dense-dense product: kern_sddmm.h.
#include "blast_common.h"

#include "kern_common.h"
#include "kern_sddmm.h"

using namespace blast_dev;

namespace {

int cu_count_bwd() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

template <int B, int KW, int UPW>
int launch_sddmm(SddmmArgs a, hipStream_t stream) {
  using C = SdCfg<B, KW, UPW>;
  static blast::DeviceFlags lds_set;
  int dev = 0;
  BLAST_HIP_TRY(hipGetDevice(&dev));
  if (!lds_set.test(dev)) {
    BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sddmm<B, KW, UPW>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES));
    lds_set.set(dev);
  }
  const int64_t sub_units = (int64_t)a.nnz * C::SUB * C::SUB;
  // Token chunks across workgroups (on top of the waves that share a unit): only when there are fewer
  // units than CUs, and never below 512 tokens per chunk - the atomics on the output cost more than
  // idle workgroup slots otherwise.
  const int64_t want = (int64_t)cu_count_bwd();
  int64_t tsplit = (want + sub_units - 1) / sub_units;
  const int64_t max_split = (a.T + 511) / 512;
  if (tsplit > max_split) tsplit = max_split;
  if (tsplit < 1) tsplit = 1;
  int64_t chunk = ((a.T + tsplit - 1) / tsplit + C::KT - 1) / C::KT * C::KT;
  tsplit = (a.T + chunk - 1) / chunk;
  const int64_t units = sub_units * tsplit;
  if (units > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
  a.tsplit = (int)tsplit;
  a.chunk_tokens = (int)chunk;
  a.n_units = (int)units;
  if (tsplit > 1) {
    const int64_t n = (int64_t)a.nnz * B * B;
    k_zero_f32<<<dim3((unsigned)((n / 4 + 255) / 256 + 1)), dim3(256), 0, stream>>>(a.dvals, n);
    BLAST_LAUNCH_CHECK("k_zero_f32");
  }
  k_sddmm<B, KW, UPW><<<dim3((unsigned)((units + 8 * UPW - 1) / (8 * UPW) * 8)), dim3(64 * C::NW), C::LDS_BYTES, stream>>>(a);
  BLAST_LAUNCH_CHECK("k_sddmm");
  return BLAST_OK;
}

// Which form, by the units (64-wide sub-blocks of the stored blocks) per CU and the activations' bytes (`features` = rows
// + columns of the matrix).
//   up to 2: four waves per unit, or most SIMDs would idle (1.6 units, 700 tokens: 11.1 us against 13.1 with one wave;
//     exactly 2, the most that are resident at once, 2048 x 2048, 300 tokens: 8.6 against 10.7, 2000: 21.6 against 26.2).
//     Up to half a unit more per CU while a second round brings the activations in again cheaply (2.5 units, 128-wide
//     blocks, 4096 x 4096, 2000 tokens: 25.6 against 27.7; 16384 x 16384, 4096 tokens: 55.2 against 47.1), and up to a
//     unit more (two more of the small 32-wide ones) while the token walk is short: a lone wave's start and its last sums
//     weigh on few stages (64-wide, 2.5 units, 700 tokens: 14.8 against 16.4; 32-wide, 3 units, 200 tokens: 5.9 against
//     6.4, 1000 tokens 12.9 against 13.5; 64-wide, 3 units, 1000 tokens 22.3 against 19.8).
//   up to what is resident at once with a wave per workgroup (rings in 128 of a CU's 160 KiB): a wave per unit, dealt
//     to the CUs one by one; every XCD then streams X once (4.8 units, 2000 tokens: 40 us; four waves per unit 48, four
//     units per workgroup 51, whose 308 workgroups load some CUs twice).  Not 32-wide units on a short walk, of which a
//     workgroup starts four at once (8 units, 512 tokens: 12.9 us against 14.9, four waves per unit 14.1).
//   more: four neighbouring units, blocks of one row or quarters of one block, in a workgroup, so that the tiles they
//     share are still in the L1 or L2 (11.2 units, 128-wide blocks, 4096 tokens: 144 us; a wave per workgroup 184, four
//     waves per unit 172).  From 6 units on for 128-wide blocks, whose quarters share both tiles (6.5 units, 14336 x 4096,
//     4096 tokens: 104 us, a wave per workgroup 112; 7.8 units 105 and 130; 5.6 units 103 and 102, 2000 tokens 52 and 48).
template <int B>
int sddmm_form(const SddmmArgs& a, int64_t features, hipStream_t stream) {
  using One = SdCfg<B, 1, 1>;
  const int64_t units = (int64_t)a.nnz * One::SUB * One::SUB, cus = cu_count_bwd();
  const bool short_walk = a.T > (B == 32 ? 64 : 300) && a.T <= (B == 32 ? 1200 : 800);
  const int64_t per_unit = a.T * features * 2 / (One::SUB * One::SUB);  // activations, of which a block's units share a tile
  const bool cheap_round = (units == 2 * cus && per_unit <= (50 << 20)) ||
                           (B > 32 && a.T > 300 && 2 * units <= 5 * cus && per_unit <= (20 << 20));
  if (units < 2 * cus || cheap_round || (short_walk && units < (B == 32 ? 4 : 3) * cus))
    return launch_sddmm<B, 4, 1>(a, stream);
  const bool resident = units * (int64_t)One::LDS_BYTES <= cus * ((B == 128 ? 96 : 128) << 10);
  if (resident && !(B == 32 && short_walk && a.T <= 800)) return launch_sddmm<B, 1, 1>(a, stream);
  return launch_sddmm<B, 1, 4>(a, stream);
}

}  // namespace

extern "C" int blast_bsr_sddmm(const blast_bsr_view* W, const uint16_t* dY, int64_t ldy, const uint16_t* X,
                               int64_t ldx, int32_t layout, int64_t T, float* dvals, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!W || !W->row_ptr) return BLAST_ERR_INVALID_ARG;
  if (W->rows < 0 || W->cols < 0 || W->nnz < 0 || W->nnz > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  if (!blast::supported_block(W->b)) return BLAST_ERR_UNSUPPORTED_BLOCK;
  if (W->rows % W->b || W->cols % W->b) return BLAST_ERR_SHAPE;
  if (W->rows / W->b > INT32_MAX / 2 || W->cols / W->b > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
  if (layout != BLAST_TOKEN_MAJOR && layout != BLAST_FEATURE_MAJOR) return BLAST_ERR_INVALID_ARG;
  if (T < 0 || T > INT32_MAX / 2) return BLAST_ERR_INVALID_ARG;
  if (W->nnz == 0) return BLAST_OK;
  if (!W->col_idx || !dvals || !blast::aligned(dvals, 16)) return BLAST_ERR_INVALID_ARG;
  const int b = W->b;
  const int64_t n_out = W->nnz * b * b;
  if (T == 0) {  // an empty sum
    k_zero_f32<<<dim3((unsigned)((n_out / 4 + 255) / 256 + 1)), dim3(256), 0, stream>>>(dvals, n_out);
    BLAST_LAUNCH_CHECK("k_zero_f32");
    return BLAST_OK;
  }
  if (!dY || !X) return BLAST_ERR_INVALID_ARG;
  if (ldy < (layout == BLAST_TOKEN_MAJOR ? W->rows : T) || ldx < (layout == BLAST_TOKEN_MAJOR ? W->cols : T))
    return BLAST_ERR_INVALID_ARG;

  const bool fast = layout == BLAST_TOKEN_MAJOR && b >= 32 && ldy % 8 == 0 && ldx % 8 == 0 &&
                    blast::aligned(dY, 16) && blast::aligned(X, 16);
  if (fast) {
    SddmmArgs a{};
    a.row_ptr = W->row_ptr;
    a.col_idx = W->col_idx;
    a.dY = dY;
    a.X = X;
    a.ldy = ldy;
    a.ldx = ldx;
    a.dvals = dvals;
    a.T = (int)T;
    a.nbr = (int)(W->rows / b);
    a.nnz = (int)W->nnz;
    switch (b) {
      case 32: return sddmm_form<32>(a, W->rows + W->cols, stream);
      case 64: return sddmm_form<64>(a, W->rows + W->cols, stream);
      default: return sddmm_form<128>(a, W->rows + W->cols, stream);
    }
  }
  SddmmGenericArgs g{};
  g.row_ptr = W->row_ptr;
  g.col_idx = W->col_idx;
  g.dY = dY;
  g.X = X;
  if (layout == BLAST_TOKEN_MAJOR) {
    g.syt = ldy; g.syi = 1; g.sxt = ldx; g.sxk = 1;
  } else {
    g.syt = 1; g.syi = ldy; g.sxt = 1; g.sxk = ldx;
  }
  g.dvals = dvals;
  g.T = (int)T;
  g.nbr = (int)(W->rows / b);
  g.b = b;
  k_sddmm_generic<<<dim3((unsigned)W->nnz), dim3(256), 0, stream>>>(g);
  BLAST_LAUNCH_CHECK("k_sddmm_generic");
  return BLAST_OK;
}
