// Block-norm pruning and packing of a dense bf16 weight into the block-compressed
// format (BLaST Sec. 3.2: score each b x b block by its Frobenius norm, drop the
// lowest until the target sparsity is reached; Sec. 3.4.1: compressed block
// storage from which the product kernel derives its work).
//
// Everything runs on the device, on the caller's stream:
//   score  -> one wave per block, 16-byte loads, fp64 sum of squares
//   select -> exact radix select on the fp64 bit patterns + index-ordered tie-break
//   count  -> per block-row / block-column populations, exclusive scans
//   fill   -> ordered compaction of column indices, gather of block values
//   order  -> rank block rows by population (schedule for load balance)
//   csc    -> column-grouped index of the same blocks (used by the fused MLP)
// Up to 65536 blocks a selection is one workgroup, and up to 49152 (1024 block rows and columns) all that follows it one launch.
#include "blast_common.h"

#include <type_traits>

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Workgroup barrier.  LDS_ONLY: only the workgroup's LDS traffic is ordered - global stores still in flight are
// not waited for (the plain barrier waits for their acknowledgement, a trip to the memory side every time).
template <bool LDS_ONLY>
__device__ __forceinline__ void wg_barrier() {
  if (LDS_ONLY)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else
    __syncthreads();
}

// Exclusive scan of one int per thread over the whole workgroup (blockDim.x a
// multiple of 64, at most 1024).  `wave_tot` is LDS scratch of >= 16 ints.
// Returns the exclusive prefix; `total` receives the workgroup sum.  A chain of instructions and two barriers: shifts between
// lanes by the vector unit instead of through LDS, the waves' sums read in one go and scanned by every wave.
template <bool LDS_ONLY = false>
__device__ __forceinline__ int block_exscan(int v, int* wave_tot, int& total) {
  const int lane = lane_id(), nw = blockDim.x / kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int inc = blast::lanes_scan(v);
  wg_barrier<LDS_ONLY>();  // protect wave_tot from the previous use
  if (lane == kWave - 1) wave_tot[wave] = inc;
  wg_barrier<LDS_ONLY>();
  const int waves = blast::lanes_scan(lane < nw ? wave_tot[lane] : 0);
  total = __builtin_amdgcn_readlane(waves, 15);
  const int base = wave > 0 ? __builtin_amdgcn_readlane(waves, wave - 1) : 0;
  return base + inc - v;
}

__device__ __forceinline__ double sq_bf16_pair(uint32_t w) {
  // two bf16 packed in a dword; each widened exactly to fp32, squared in fp64
  double lo = (double)__uint_as_float(w << 16);
  double hi = (double)__uint_as_float(w & 0xFFFF0000u);
  return lo * lo + hi * hi;
}

// One wave per block: squared Frobenius norm in fp64.  The summation tree depends only on b, so equal blocks get equal
// scores wherever they sit: 256 partial sums of every 256th 16-byte piece, four to a lane (lane, lane + 64, ...), halved
// eight times - the first two times inside a lane.
// blockIdx.y == 1: a second matrix of the same shape (the gradient of the mask update) into a second score array.
// What bounds it: how much of the HBM read is in flight.  A workgroup per block waited for two loads a thread and then
// for eight barriers; a wave has eight loads a lane under way and no barrier.  8192 x 2048, b = 64: 9.6 -> 8.2 us
// (33.5 MB, 4.1 TB/s), prune-and-grow step of a 1B-shaped layer 149.0 -> 144.8 us.
template <int B>
__global__ __launch_bounds__(256) void k_block_scores(const uint16_t* __restrict__ W, int64_t ldw, int nbc, int64_t n,
                                                      double* __restrict__ score, const uint16_t* __restrict__ W1,
                                                      int64_t ldw1, double* __restrict__ score1) {
  constexpr int CPR = B / 8, CHUNKS = B * CPR, SLOTS = CHUNKS < 256 ? (CHUNKS + kWave - 1) / kWave : 4;
  constexpr int ROUNDS = (CHUNKS + 255) / 256;
  if (blockIdx.y == 1) {
    W = W1;
    ldw = ldw1;
    score = score1;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (blk >= n) return;
  const int64_t br = blk / nbc, bc = blk % nbc;
  const uint16_t* base = W + br * B * ldw + bc * B;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int q = 0; q < ROUNDS; ++q) {
    uint4 v[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
      const int c = q * 256 + u * kWave + lane;
      v[u] = uint4{0u, 0u, 0u, 0u};
      if (CHUNKS >= kWave || c < CHUNKS) v[u] = *reinterpret_cast<const uint4*>(base + (int64_t)(c / CPR) * ldw + c % CPR * 8);
    }
#pragma unroll
    for (int u = 0; u < SLOTS; ++u)
      s[u] += (sq_bf16_pair(v[u].x) + sq_bf16_pair(v[u].y)) + (sq_bf16_pair(v[u].z) + sq_bf16_pair(v[u].w));
  }
  double r = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) r += __shfl_down(r, d, kWave);
  if (lane == 0) score[blk] = r;
}

// One workgroup per block: mean of an fp32 sensitivity matrix over the block (2D average pooling,
// BLaST Sec. 3.3), accumulated in fp64 with the same tree as the Frobenius scores.
__global__ __launch_bounds__(256) void k_pooled_scores(const float* __restrict__ S, int64_t lds, int nbc, int b,
                                                       double* __restrict__ score) {
  __shared__ double red[256];
  const int64_t blk = blockIdx.x;
  const int64_t br = blk / nbc, bc = blk % nbc;
  const float* base = S + br * b * lds + bc * b;
  const int cpr = b / 4, nchunks = b * cpr;
  double s = 0.0;
  for (int c = threadIdx.x; c < nchunks; c += 256) {
    const int i = c / cpr, j4 = c % cpr;
    const float4 v = *reinterpret_cast<const float4*>(base + (int64_t)i * lds + j4 * 4);
    s += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) {
    if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) score[blk] = red[0] / ((double)b * (double)b) + 0.0;  // + 0.0: no negative zero
}

__global__ void k_fill_u8(uint8_t* p, int64_t n, uint8_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_i32(int* p, int64_t n, int v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Bit pattern of a double mapped to an unsigned integer with the same order (any finite sign; -0.0 is
// canonicalised to +0.0 by the scoring kernels, so equal scores have equal keys).
__device__ __forceinline__ unsigned long long order_key(unsigned long long bits) {
  return (bits >> 63) ? ~bits : (bits | 0x8000000000000000ull);
}

// Exact selection of the n_keep highest scores (0 < n_keep < n), compared through
// order-preserving integer keys.
// An 8-pass most-significant-digit radix select finds the n_keep-th largest
// pattern; everything above it is kept, and of the entries equal to it the
// first ones in index order fill the remaining quota.
// The passes read the keys from global memory only until the keys that still share the selected prefix
// fit in LDS (kSelectCand of them); those are then collected once and the remaining passes run on LDS.
constexpr int kSelectCand = 4096;

// Workgroup 1 of a two-workgroup launch selects from a second score array into a second mask (the mask update
// of prune-and-grow ranks the weight and the gradient at the same sparsity: the two selections run side by side).
__global__ __launch_bounds__(1024) void k_select_topk(const double* __restrict__ score0, int64_t n, int64_t n_keep,
                                                      uint8_t* __restrict__ mask0,
                                                      const double* __restrict__ score1 = nullptr,
                                                      uint8_t* __restrict__ mask1 = nullptr) {
  const double* __restrict__ score = blockIdx.x == 0 ? score0 : score1;
  uint8_t* __restrict__ mask = blockIdx.x == 0 ? mask0 : mask1;
  __shared__ unsigned long long cand[kSelectCand];
  __shared__ unsigned hist[256];
  __shared__ unsigned long long s_prefix;
  __shared__ long long s_remaining;
  __shared__ int wave_tot[16];
  __shared__ long long s_running;
  __shared__ long long s_eq_total;
  __shared__ int s_ncand;  // < 0: the candidates are still the whole array
  __shared__ int s_fill;
  __shared__ unsigned s_h;
  const unsigned long long* key = reinterpret_cast<const unsigned long long*>(score);
  const int lane = lane_id();
  const bool pairs_ok = (reinterpret_cast<uintptr_t>(score) & 15u) == 0;
  if (threadIdx.x == 0) {
    s_prefix = 0ull;
    s_remaining = n_keep;
    s_running = 0;
    s_eq_total = 0;
    s_ncand = n <= kSelectCand ? (int)n : -1;
    s_fill = 0;
    s_h = 0u;
  }
  if (n <= kSelectCand)
    for (int i = threadIdx.x; i < (int)n; i += blockDim.x) cand[i] = order_key(key[i]);
  for (int pass = 7; pass >= 0; --pass) {
    if (threadIdx.x < 256) hist[threadIdx.x] = 0u;
    __syncthreads();
    const unsigned long long prefix = s_prefix;
    const unsigned long long himask = (pass == 7) ? 0ull : (~0ull << (8 * (pass + 1)));
    const int ncand = s_ncand;
    if (ncand >= 0) {
      for (int i = threadIdx.x; i < ncand; i += blockDim.x) {
        const unsigned long long k = cand[i];
        if ((k & himask) == prefix) atomicAdd(&hist[(unsigned)(k >> (8 * pass)) & 255u], 1u);
      }
    } else {
      // A thread adds a run of equal digits with one atomic: in the leading passes, where scores of similar
      // magnitude all carry the same digit, every key would otherwise hit the same LDS word.
      unsigned run_bin = 0u, run_len = 0u;
      auto count = [&](unsigned long long raw) {
        const unsigned long long k = order_key(raw);
        if ((k & himask) == prefix) {
          const unsigned bin = (unsigned)(k >> (8 * pass)) & 255u;
          if (run_len != 0u && bin != run_bin) {
            atomicAdd(&hist[run_bin], run_len);
            run_len = 0u;
          }
          run_bin = bin;
          ++run_len;
        }
      };
      // two keys per load, eight loads in flight: one workgroup walks the whole array, so the walk is
      // bound by how many bytes it keeps in flight
      const int64_t npair = pairs_ok ? n / 2 : 0;
      const ulonglong2* key2 = reinterpret_cast<const ulonglong2*>(key);
#pragma unroll 8
      for (int64_t p = threadIdx.x; p < npair; p += blockDim.x) {
        const ulonglong2 kk = key2[p];
        count(kk.x);
        count(kk.y);
      }
      for (int64_t i = 2 * npair + threadIdx.x; i < n; i += blockDim.x) count(key[i]);
      if (run_len != 0u) atomicAdd(&hist[run_bin], run_len);
    }
    __syncthreads();
    // Digit d of this pass: the bin where the count of larger digits, S(d), first satisfies
    // S(d) < remaining <= S(d) + hist[d].  One thread per bin; the suffix sums come from a scan of the
    // bins in descending order.
    {
      const long long rem = s_remaining;
      const int d = 255 - (int)threadIdx.x;  // thread t looks at bin 255 - t
      const int h = (threadIdx.x < 256) ? (int)hist[d & 255] : 0;
      int total;
      const int larger = block_exscan(h, wave_tot, total);  // sum of hist over digits > d
      __syncthreads();
      if (threadIdx.x < 256 && (long long)larger < rem && rem <= (long long)larger + h) {
        s_remaining = rem - larger;
        s_prefix = prefix | ((unsigned long long)d << (8 * pass));
        s_h = (unsigned)h;              // keys that share the prefix including this digit
        if (pass == 0) s_eq_total = h;  // entries equal to the n_keep-th largest
      }
    }
    __syncthreads();
    if (ncand < 0 && pass > 0 && s_h <= (unsigned)kSelectCand) {
      // collect the keys that carry the new prefix (exactly s_h of them); their order does not matter
      const unsigned long long newmask = ~0ull << (8 * pass), newprefix = s_prefix;
      for (int64_t base = 0; base < n; base += 4 * (int64_t)blockDim.x) {
        unsigned long long k[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t i = base + u * (int64_t)blockDim.x + threadIdx.x;
          in[u] = i < n;
          k[u] = in[u] ? order_key(key[i]) : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool take = in[u] && (k[u] & newmask) == newprefix;
          const unsigned long long bal = __ballot(take);
          int wbase = 0;
          if (lane == 0 && bal != 0ull) wbase = atomicAdd(&s_fill, __popcll(bal));
          wbase = __shfl(wbase, 0, kWave);
          if (take) cand[wbase + __popcll(bal & ((1ull << lane) - 1ull))] = k[u];
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) s_ncand = s_fill;
      __syncthreads();
    }
  }
  const unsigned long long kth = s_prefix;
  const long long need_eq = s_remaining;
  if (need_eq == s_eq_total) {
    // every entry equal to the threshold is kept (always so when the scores are distinct): no ordering needed
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) mask[i] = order_key(key[i]) >= kth ? 1 : 0;
    return;
  }
  for (int64_t base = 0; base < n; base += blockDim.x) {
    const int64_t i = base + threadIdx.x;
    const unsigned long long k = (i < n) ? order_key(key[i]) : 0ull;
    const int eq = (i < n && k == kth) ? 1 : 0;
    int total;
    const long long pos = s_running + block_exscan(eq, wave_tot, total);
    if (i < n) mask[i] = (k > kth || (eq && pos < need_eq)) ? 1 : 0;
    __syncthreads();
    if (threadIdx.x == 0) s_running += total;
    __syncthreads();
  }
}

// One wave per line: population of mask along a row (stride 1) or a column (stride nbc).
__global__ __launch_bounds__(256) void k_line_counts(const uint8_t* __restrict__ mask, int n_lines, int line_len,
                                                     int64_t line_stride, int64_t elem_stride, int* __restrict__ cnt) {
  const int line = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (line >= n_lines) return;
  int c = 0;
  for (int j = lane_id(); j < line_len; j += kWave) c += mask[line * line_stride + j * elem_stride] ? 1 : 0;
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) c += __shfl_xor(c, d, kWave);
  if (lane_id() == 0) cnt[line] = c;
}

// Single workgroup: ptr[0..n] = exclusive scan of cnt[0..n).  total_out (may be null) gets ptr[n].
__global__ __launch_bounds__(1024) void k_exscan(const int* __restrict__ cnt, int n, int* __restrict__ ptr,
                                                 int* __restrict__ total_out) {
  __shared__ int wave_tot[16];
  __shared__ int s_running;
  if (threadIdx.x == 0) s_running = 0;
  __syncthreads();
  for (int base = 0; base < n; base += blockDim.x) {
    const int i = base + threadIdx.x;
    const int v = (i < n) ? cnt[i] : 0;
    int total;
    const int ex = s_running + block_exscan(v, wave_tot, total);
    if (i < n) ptr[i] = ex;
    __syncthreads();
    if (threadIdx.x == 0) s_running += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    ptr[n] = s_running;
    if (total_out) *total_out = s_running;
  }
}

// One workgroup per block row: kept block columns, ascending, into col_idx; the
// owning block row of every stored block into blk_row (for the gather).
__global__ __launch_bounds__(256) void k_fill_cols(const uint8_t* __restrict__ mask, int nbc,
                                                   const int* __restrict__ row_ptr, int* __restrict__ col_idx,
                                                   int* __restrict__ blk_row, int64_t nnz_cap) {
  __shared__ int wave_tot[16];
  const int br = blockIdx.x;
  const int start = row_ptr[br];
  int running = 0;
  for (int base = 0; base < nbc; base += blockDim.x) {
    const int c = base + threadIdx.x;
    const int f = (c < nbc && mask[(int64_t)br * nbc + c]) ? 1 : 0;
    int total;
    const int pos = running + block_exscan(f, wave_tot, total);
    if (f) {
      const int64_t k = (int64_t)start + pos;
      if (k < nnz_cap) {
        col_idx[k] = c;
        blk_row[k] = br;
      }
    }
    running += total;
  }
}

// One workgroup per stored block: copy its b x b values, row-major, 16 bytes per lane.  A block whose mask
// code is 2 (regrown, BLaST Sec. 3.2) is stored as zeros: it joins the structure without changing the product.
// (The grid is sized by the capacity: workgroups past the number of stored blocks leave.)
__global__ __launch_bounds__(256) void k_gather_blocks(const uint16_t* __restrict__ W, int64_t ldw, int b,
                                                       const int* __restrict__ col_idx, const int* __restrict__ blk_row,
                                                       const uint8_t* __restrict__ mask, int nbc,
                                                       uint16_t* __restrict__ vals, const int* __restrict__ nnz_dev) {
  const int64_t k = blockIdx.x;
  if (k >= *nnz_dev) return;
  const int64_t br = blk_row[k], bc = col_idx[k];
  const uint16_t* src = W + br * b * ldw + bc * b;
  uint16_t* dst = vals + k * b * b;
  const int cpr = b / 8, nchunks = b * cpr;
  const bool zero = mask[br * nbc + bc] == 2;
  for (int c = threadIdx.x; c < nchunks; c += 256) {
    const int i = c / cpr, j8 = c % cpr;
    *reinterpret_cast<uint4*>(dst + (int64_t)c * 8) =
        zero ? uint4{0u, 0u, 0u, 0u} : *reinterpret_cast<const uint4*>(src + (int64_t)i * ldw + j8 * 8);
  }
}

// out = 1 where the weight's own selection keeps the block, 2 where only the gradient's does, else 0
__global__ __launch_bounds__(256) void k_merge_masks(const uint8_t* __restrict__ mw, const uint8_t* __restrict__ mg,
                                                     int64_t n, uint8_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = mw[i] ? 1 : (mg[i] ? 2 : 0);
}

// row_order[rank] = r with rank = number of rows that sort before r under
// (population descending, row index ascending) -- a stable sort by counting.
// row_ptr2 (may be null) adds the populations of a second matrix with the same block rows.
__global__ __launch_bounds__(256) void k_row_order(const int* __restrict__ row_ptr, const int* __restrict__ row_ptr2,
                                                   int nbr, int* __restrict__ row_order) {
  // the populations pass through LDS in slabs: every thread compares its row with all of them
  constexpr int kSlab = 2048;
  __shared__ __attribute__((aligned(16))) int cnt[kSlab];
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  int cr = 0;
  if (r < nbr) {
    cr = row_ptr[r + 1] - row_ptr[r];
    if (row_ptr2) cr += row_ptr2[r + 1] - row_ptr2[r];
  }
  int rank = 0;
  for (int base = 0; base < nbr; base += kSlab) {
    const int m = nbr - base < kSlab ? nbr - base : kSlab;
    __syncthreads();
    for (int q = threadIdx.x; q < m; q += blockDim.x) {
      int cq = row_ptr[base + q + 1] - row_ptr[base + q];
      if (row_ptr2) cq += row_ptr2[base + q + 1] - row_ptr2[base + q];
      cnt[q] = cq;
    }
    __syncthreads();
    if (r < nbr) {
      // four populations per LDS read, several reads in flight: a serial chain of single reads would cost
      // one LDS round trip per row
      int q = 0;
#pragma unroll 4
      for (; q + 4 <= m; q += 4) {
        const int4 c4 = *reinterpret_cast<const int4*>(&cnt[q]);
        rank += (c4.x > cr || (c4.x == cr && base + q < r)) ? 1 : 0;
        rank += (c4.y > cr || (c4.y == cr && base + q + 1 < r)) ? 1 : 0;
        rank += (c4.z > cr || (c4.z == cr && base + q + 2 < r)) ? 1 : 0;
        rank += (c4.w > cr || (c4.w == cr && base + q + 3 < r)) ? 1 : 0;
      }
      for (; q < m; ++q) {
        const int cq = cnt[q];
        rank += (cq > cr || (cq == cr && base + q < r)) ? 1 : 0;
      }
    }
  }
  if (r < nbr) row_order[rank] = r;
}

// One workgroup per block column: its stored blocks by ascending block row; for
// each, the block row and the position k of the block in vals / col_idx.
// csc_blk null: it follows csc_row at the next 16-byte boundary after nnz entries, nnz read from nnz_dev (the
// layout of the aux buffer; nothing is written when nnz exceeds the capacity).
__global__ __launch_bounds__(256) void k_fill_csc(const uint8_t* __restrict__ mask, int nbr, int nbc,
                                                  const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
                                                  const int* __restrict__ col_ptr, int* __restrict__ csc_row,
                                                  int* __restrict__ csc_blk, int64_t nnz_cap,
                                                  const int* __restrict__ nnz_dev) {
  __shared__ int wave_tot[16];
  if (!csc_blk) {
    const int64_t nnz = *nnz_dev;
    if (nnz > nnz_cap) return;
    csc_blk = csc_row + (nnz + 3) / 4 * 4;
  }
  const int c = blockIdx.x;
  const int start = col_ptr[c];
  int running = 0;
  for (int base = 0; base < nbr; base += blockDim.x) {
    const int r = base + threadIdx.x;
    const int f = (r < nbr && mask[(int64_t)r * nbc + c]) ? 1 : 0;
    int total;
    const int pos = running + block_exscan(f, wave_tot, total);
    if (f) {
      int lo = row_ptr[r], hi = row_ptr[r + 1] - 1;  // col_idx ascending in the row: find c
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col_idx[mid] < c) lo = mid + 1; else hi = mid;
      }
      const int64_t e = (int64_t)start + pos;
      if (e < nnz_cap) {
        csc_row[e] = r;
        csc_blk[e] = lo;
      }
    }
    running += total;
  }
}

// Where one chunk plan goes.
struct PlanOut {
  int chunk;        // blocks per chunk, at most
  int* hdr;         // {n_chunks, max_row_blocks, chunk, chunks of the rows that have several}
  int* chunk_row;
  int* chunk_kb;
  int* chunk_ke;
  int64_t cap;
  int* row_slot;    // may be null: per row, its rank if it has several chunks, else -1
  int* row_chunk0;  // may be null: per row, the index of its first chunk if it has several, else -1
};

// Cuts the block rows, in schedule order, into chunks of at most `chunk` blocks, once per requested plan; run by
// every thread of one workgroup.  An empty row still gets one (empty) chunk: its output has to be written.
// `sh` is LDS scratch of 3 ints.
__device__ __forceinline__ void chunk_plans(const int* row_ptr, const int* row_order, int nbr, const PlanOut& narrow,
                                            const PlanOut& wide, int* __restrict__ max_row_out, int* wave_tot,
                                            int* sh) {
  int& s_running = sh[0];
  int& s_heavy = sh[1];
  int& s_split = sh[2];
  for (int which = 0; which < 2; ++which) {
    const PlanOut o = which ? wide : narrow;
    const int chunk = o.chunk;
    __syncthreads();
    if (threadIdx.x == 0) {
      s_running = 0;
      s_heavy = 0;
      s_split = 0;
    }
    __syncthreads();
    for (int base = 0; base < nbr; base += blockDim.x) {
      const int rank = base + threadIdx.x;
      int r = 0, kb = 0, ke = 0, nch = 0;
      if (rank < nbr) {
        r = row_order[rank];
        kb = row_ptr[r];
        ke = row_ptr[r + 1];
        nch = (ke - kb + chunk - 1) / chunk;
        if (nch < 1) nch = 1;
        atomicMax(&s_heavy, ke - kb);
        if (nch > 1) atomicAdd(&s_split, nch);
        if (o.row_slot) o.row_slot[r] = nch > 1 ? rank : -1;
      }
      int total;
      const int first = s_running + block_exscan(nch, wave_tot, total);
      if (rank < nbr && o.row_chunk0) o.row_chunk0[r] = nch > 1 ? first : -1;
      for (int j = 0; j < nch; ++j) {
        const int64_t e = (int64_t)first + j;
        if (e < o.cap) {
          o.chunk_row[e] = r | (nch > 1 ? (int)0x80000000u : 0);
          const int b0 = kb + j * chunk;
          o.chunk_kb[e] = b0;
          o.chunk_ke[e] = (b0 + chunk < ke) ? b0 + chunk : ke;
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) s_running += total;
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      o.hdr[0] = s_running;
      o.hdr[1] = s_heavy;
      if (which == 0) *max_row_out = s_heavy;  // next to nnz, so that one copy brings both to the host
      o.hdr[2] = chunk;
      o.hdr[3] = s_split;
    }
  }
}

// Single workgroup: both chunk plans of a matrix.
__global__ __launch_bounds__(1024) void k_chunk_plan(const int* __restrict__ row_ptr, const int* __restrict__ row_order,
                                                     int nbr, PlanOut narrow, PlanOut wide,
                                                     int* __restrict__ max_row_out) {
  __shared__ int wave_tot[16];
  __shared__ int sh[3];
  chunk_plans(row_ptr, row_order, nbr, narrow, wide, max_row_out, wave_tot, sh);
}

// Both plans of a matrix, placed in its aux buffer.
inline void plan_outputs(char* ab, const blast::AuxLayout& A, PlanOut& narrow, PlanOut& wide) {
  narrow = PlanOut{blast::kChunkBlocks, reinterpret_cast<int*>(ab + A.hdr_off), reinterpret_cast<int*>(ab + A.chunk_row_off),
                   reinterpret_cast<int*>(ab + A.chunk_kb_off), reinterpret_cast<int*>(ab + A.chunk_ke_off), A.chunk_cap,
                   reinterpret_cast<int*>(ab + A.row_slot_off), reinterpret_cast<int*>(ab + A.row_chunk0_off)};
  wide = PlanOut{blast::kWideChunkBlocks, reinterpret_cast<int*>(ab + A.whdr_off), reinterpret_cast<int*>(ab + A.wchunk_row_off),
                 reinterpret_cast<int*>(ab + A.wchunk_kb_off), reinterpret_cast<int*>(ab + A.wchunk_ke_off), A.wchunk_cap,
                 nullptr, nullptr};
}

// ---- small matrices: a workgroup per job ----
//
// A layer-sized matrix has a few thousand to a few ten thousand blocks; scored, the rest of the packing is as many integer
// operations, and as a dozen dependent launches it costs a dozen launch latencies.  So a selection is one workgroup (up to
// kOneWorkgroupN blocks; both of a mask update in one up to kSmallN) and the rest one launch (up to kSmallN blocks with what a
// thread owns in registers, up to kBigN in two walks; at most 1024 block rows and block columns), in which a workgroup makes the
// row arrays and another the column arrays: a thread owns `per` consecutive blocks in row-major
// order; the selection's keys, the positions and the per-line populations live in LDS.  The workgroup's 16 waves
// share one compute unit, so what such a job costs is instructions per thread: no integer division per block, both
// chunk plans' scans in one (two 16-bit counts in one word: a plan has at most a chunk per 16 blocks and one per row, kBigN / 16 +
// 1024), barriers that do not wait for global stores.
constexpr int kSmallPer = 8;
constexpr int kSmallN = 1024 * kSmallPer;
static_assert((blast::kChunkBlocks & (blast::kChunkBlocks - 1)) == 0 &&
              (blast::kWideChunkBlocks & (blast::kWideChunkBlocks - 1)) == 0, "chunk sizes are powers of two");

constexpr int kRanked = 16;  // candidates that a wave ranks by comparing each with all
constexpr int kWideBits = 11, kWideBins = 1 << kWideBits;  // a digit where every pass reads the scores again

// LDS scratch of select_small, one per group (an array of them: the bins are read four at a time, so the size keeps the
// alignment too).
struct alignas(16) SelectShared {
  unsigned hist[256];
  uint4 wave_keys[16];  // of a wave: the smallest and the largest upper word, differing bits of the lower words
  uint2 wave_zeros[16];  // of a wave: the smallest upper word of a key that is no zero's, its zeros
  int wave_tot[16];
  unsigned long long kth;        // the n_keep-th key ...
  int kth_at;                    // ... and its index: what is kept sorts before it, or is it
  int rem, eq, digit, fill, open;
  int cand[kRanked];
};
static_assert(sizeof(SelectShared) % 16 == 0 && offsetof(SelectShared, hist) % 16 == 0, "16-byte reads of hist");

// Over a row of 16 lanes, and over a wave: every lane has the result.
template <int CTRL>
__device__ __forceinline__ unsigned from_lane(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <typename F>
__device__ __forceinline__ unsigned reduce_row(unsigned v, F f) {
  v = f(v, from_lane<0x121>(v));  // rotations of the row by 1, 2, 4, 8
  v = f(v, from_lane<0x122>(v));
  v = f(v, from_lane<0x124>(v));
  return f(v, from_lane<0x128>(v));
}
template <typename F>
__device__ __forceinline__ unsigned reduce_wave(unsigned v, F f) {
  v = reduce_row(v, f);
  auto row = [&](int lane) { return (unsigned)__builtin_amdgcn_readlane((int)v, lane); };
  return f(f(row(0), row(16)), f(row(32), row(48)));
}

// The n_keep-th of n scores (0 < n_keep < n) under (score descending, index ascending), into sh.kth and
// sh.kth_at, by a group of NT threads of a workgroup of GROUPS * NT: the caller's groups select side by side (every
// barrier is the workgroup's; a selection that is through waits for the others).  STAGED: keys, LDS of n entries, receives the
// keys of the scores.
//
// Most-significant-digit radix select on the keys' distances from the smallest one (its upper word: reducing 64 bits takes
// twice the instructions): scores of one matrix share their leading bits, or differ in all of the exponent's where they lie on
// both sides of a power of two, and a digit that most keys carry sends their counts to one LDS word.  The passes start at the
// largest distance's leading bit, eight bits at a time; as soon as at most 16 keys carry the selected prefix, a wave ranks
// those by comparing each with all (40 ns each, a pass a microsecond: mask update with its wait, with up to 64 ranked that way 11.9 us
// on 64 blocks of 64 x 64 and 23.5 on 4096, with 16 8.2 and 20.9).
// Kernel of the mask update, 4096 blocks of 64 x 64, normal: from the leading bit in which keys differ, the exponent's there, the
// first pass took 5.6 us, every key adding to one of two words, 12.9 us in all; from the distance 6.5.  (Blocks of 32 x 32, whose
// scores lie between two powers of two: 6.7 and 6.7.)
// A few scores far from the others still leave those one bin: a wave a quarter of whose first keys share a digit counts the
// lanes that carry its first lane's with one addition (16384 blocks, mask update with its wait: 44 us, one score 100 times the
// others 51; counting so in every wave costs 0.7 us of 4096 normal ones).
// Where every pass reads the scores again (not STAGED) a pass that tells nothing is dear, so there digits have eleven bits, which still
// part the others where one score is a million times theirs, and zeros stay out of the passes, see below; both where
// select_small<..., false> is launched, with times.
// What bounds it is not the work but its dependent steps and, in a workgroup that runs every instruction once or
// twice with caches full of weights, the fetching of instructions: loops are left rolled.  4096 blocks, weight and gradient
// (timestamps): keys unrolled over registers and passes down to one key, the two selections in turn: 16 us; keys in LDS,
// side by side: 12.8 us; and by the distance, bounds in 32 bits: 6.5.
template <int NT, int GROUPS, bool STAGED = true>
__device__ __forceinline__ void select_small(const double* __restrict__ score, int n, int n_keep, unsigned long long* keys,
                                             SelectShared* shared) {
  const int lane = lane_id(), group = GROUPS == 1 ? 0 : threadIdx.x / NT, tid = threadIdx.x - group * NT;
  SelectShared& sh = shared[group];
  const unsigned long long* bits = reinterpret_cast<const unsigned long long*>(score);
  auto key_of = [&](int i) { return STAGED ? keys[i] : order_key(bits[i]); };
  auto lesser = [](unsigned x, unsigned y) { return x < y ? x : y; };
  auto greater = [](unsigned x, unsigned y) { return x > y ? x : y; };
  auto either = [](unsigned x, unsigned y) { return x | y; };
  auto plus = [](unsigned x, unsigned y) { return x + y; };
  constexpr unsigned long long kZero = 1ull << 63;  // the key of a zero
  const unsigned long long key0 = order_key(bits[0]);
  unsigned least = ~0u, most = 0u, diff = 0u;  // of the keys' upper words; bits in which their lower words differ
#pragma unroll 4
  for (int i = tid; i < n; i += NT) {
    const unsigned long long k = order_key(bits[i]);
    if (STAGED) keys[i] = k;
    least = min(least, (unsigned)(k >> 32));
    most = max(most, (unsigned)(k >> 32));
    diff |= (unsigned)k ^ (unsigned)key0;
  }
  least = reduce_wave(least, lesser);
  most = reduce_wave(most, greater);
  diff = reduce_wave(diff, either);
  if (lane == 0) sh.wave_keys[tid / kWave] = make_uint4(least, most, diff, 0u);
  wg_barrier<true>();
  const uint4 of_wave = sh.wave_keys[lane % (NT / kWave)];  // (every row of 16 lanes reads the 8 or 16 waves')
  least = reduce_row(of_wave.x, lesser);
  most = reduce_row(of_wave.y, greater);
  diff = reduce_row(of_wave.z, either);
  // No score below zero, some zero, each pass another walk over the scores: the zeros sort after all others and stay out of the
  // passes, whose first would do no more than tell them from the rest - a key less than `low` carries no prefix (its distance wraps
  // to 2^63 or more, those of the others stay below).
  int apart = 0;
  if constexpr (!STAGED) {
    static_assert(STAGED || GROUPS == 1, "a barrier that is the group's decision");
    if (least == (unsigned)(kZero >> 32) && most != least) {
      unsigned other = ~0u, zeros = 0u;
#pragma unroll 4
      for (int i = tid; i < n; i += NT) {
        const unsigned long long k = key_of(i);
        other = min(other, k == kZero ? ~0u : (unsigned)(k >> 32));
        zeros += k == kZero ? 1u : 0u;
      }
      other = reduce_wave(other, lesser);
      zeros = reduce_wave(zeros, plus);
      if (lane == 0) sh.wave_zeros[tid / kWave] = make_uint2(other, zeros);
      wg_barrier<true>();
      const uint2 zeros_of = sh.wave_zeros[lane % (NT / kWave)];
      other = reduce_row(zeros_of.x, lesser);
      zeros = reduce_row(lane % 16 < NT / kWave ? zeros_of.y : 0u, plus);
      if (other > least) {  // (a score whose upper word is zero's stays among them)
        least = other;
        apart = (int)zeros;
      }
    }
  }
  // bits at and above `fixed` are decided, in the keys' distance from `low`; the rem-th of the eq keys that carry the decided bits
  // is the one
  int fixed, rem = n_keep, eq = n - apart;
  unsigned long long low, prefix = 0ull;
  if (n_keep > n - apart) {
    fixed = 0;
    low = kZero;
    rem -= n - apart;
    eq = apart;
  } else if (most != least) {
    fixed = 64 - __builtin_clz(most - least);
    low = (unsigned long long)least << 32;
  } else {
    fixed = diff != 0u ? 32 - __builtin_clz(diff) : 0;
    low = ((unsigned long long)least << 32 | (unsigned)key0) >> fixed << fixed;
  }
  auto carries = [&](unsigned long long k) { return fixed == 64 || ((k - low) >> fixed) == (prefix >> fixed); };
  constexpr int BITS = STAGED ? 8 : kWideBits, BINS = 1 << BITS;
  unsigned* const hist = STAGED ? sh.hist : reinterpret_cast<unsigned*>(keys);
#pragma unroll 1
  for (;;) {
    const bool active = fixed > 0 && eq > kRanked;
    if (tid == 0) {
      sh.open = active ? 1 : 0;
      sh.fill = 0;
    }
    if (STAGED) {
      if (tid < BINS) hist[tid] = 0u;
    } else {
      for (int j = tid; j < BINS; j += NT) hist[j] = 0u;
    }
    wg_barrier<true>();
    int open = 0;
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) open |= shared[q].open;
    if (open == 0) break;
    const int sft = fixed > BITS ? fixed - BITS : 0, width = fixed - sft;
    if (active) {
      auto digit_of = [&](unsigned long long k) { return (unsigned)((k - low) >> sft) & ((1u << width) - 1u); };
      const unsigned long long k0 = key_of(tid < n ? tid : n - 1);
      const unsigned sample = carries(k0) ? digit_of(k0) : (unsigned)BINS + lane;
      if (__popcll(__ballot(sample == (unsigned)__builtin_amdgcn_readfirstlane((int)sample))) <= kWave / 4) {
#pragma unroll 2
        for (int i = tid; i < n; i += NT) {
          const unsigned long long k = key_of(i);
          if (carries(k)) atomicAdd(&hist[digit_of(k)], 1u);
        }
      } else {
        for (int i = tid; i < n; i += NT) {
          const unsigned long long k = key_of(i);
          if (carries(k)) {
            const unsigned digit = digit_of(k);
            const unsigned long long same = __ballot(digit == (unsigned)__builtin_amdgcn_readfirstlane((int)digit));
            if (!(same >> lane & 1ull))
              atomicAdd(&hist[digit], 1u);
            else if (lane == __builtin_ctzll(same))
              atomicAdd(&hist[digit], (unsigned)__popcll(same));
          }
        }
      }
    }
    wg_barrier<true>();
    auto look = [&](int bin, int h, int larger) {  // `larger` = keys in bins above this one
      if (larger < rem && rem <= larger + h) {
        sh.rem = rem - larger;
        sh.eq = h;
        sh.digit = bin;
      }
    };
    if constexpr (!STAGED) {  // (one group: every thread is here, with an active selection)
      static_assert(BINS == 2 * NT, "two bins a thread");
      const uint2 h = *reinterpret_cast<const uint2*>(&hist[BINS - 2 - 2 * tid]);
      int total;
      const int larger = block_exscan<true>((int)(h.x + h.y), sh.wave_tot, total);
      look(BINS - 1 - 2 * tid, (int)h.y, larger);
      look(BINS - 2 - 2 * tid, (int)h.x, larger + (int)h.y);
    } else if (active && tid < kWave) {
      // lane l looks at bins 255 - 4l ... 252 - 4l
      const uint4 h = *reinterpret_cast<const uint4*>(&hist[252 - 4 * lane]);
      const int h4[4] = {(int)h.w, (int)h.z, (int)h.y, (int)h.x};
      const int sum = (h4[0] + h4[1]) + (h4[2] + h4[3]);
      int inc = sum;
#pragma unroll 1
      for (int d = 1; d < kWave; d <<= 1) {
        const int v = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += v;
      }
      int larger = inc - sum;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        look(255 - 4 * lane - u, h4[u], larger);
        larger += h4[u];
      }
    }
    wg_barrier<true>();
    if (active) {
      rem = sh.rem;
      eq = sh.eq;
      prefix |= (unsigned long long)(unsigned)sh.digit << sft;
      fixed = sft;
    }
  }
  int eq_mine = 0, eq_before = 0;
  if (eq <= kRanked) {
#pragma unroll 2
    for (int i = tid; i < n; i += NT)
      if (carries(key_of(i))) sh.cand[atomicAdd(&sh.fill, 1)] = i;
  } else {
    // more equal keys than that: a thread counts those in its stretch of the indices
    const int per = (n + NT - 1) / NT, e0 = tid * per;
    int mine = 0;
    for (int i = e0; i < e0 + per && i < n; ++i) mine += key_of(i) - low == prefix ? 1 : 0;
    int inc = mine;
    for (int d = 1; d < kWave; d <<= 1) {
      const int v = __shfl_up(inc, d, kWave);
      if (lane >= d) inc += v;
    }
    if (lane == kWave - 1) sh.wave_tot[tid / kWave] = inc;
    eq_mine = mine;
    eq_before = inc - mine;
  }
  wg_barrier<true>();
  if (eq <= kRanked) {
    if (tid < kWave) {
      const int at = lane < eq ? sh.cand[lane] : 0;
      const unsigned long long k = lane < eq ? key_of(at) : 0ull;
      int before = 0;
#pragma unroll 1
      for (int c = 0; c < eq; ++c) {
        const unsigned long long kc = __shfl(k, c, kWave);
        const int ac = __shfl(at, c, kWave);
        before += (kc > k || (kc == k && ac < at)) ? 1 : 0;
      }
      if (lane < eq && before == rem - 1) {
        sh.kth = k;
        sh.kth_at = at;
      }
    }
  } else {
    for (int w = 0; w < tid / kWave; ++w) eq_before += sh.wave_tot[w];
    if (eq_before < rem && rem <= eq_before + eq_mine) {
      const int per = (n + NT - 1) / NT;
      int i = tid * per;
      for (int c = rem - eq_before;; ++i)
        if (key_of(i) - low == prefix && --c == 0) break;
      sh.kth = prefix + low;
      sh.kth_at = i;
    }
  }
  wg_barrier<true>();
}

__device__ __forceinline__ bool select_keeps(const SelectShared& sh, unsigned long long k, int i) {
  return k > sh.kth || (k == sh.kth && i <= sh.kth_at);
}

// One workgroup: mask[i] = 1 for the n_keep highest of n scores, else 0; workgroup 1 of a launch of two: of a second array
// (the mask update ranks the weight and the gradient at the same sparsity).  STAGED: the keys in dynamic LDS, n <= kStagedN.
// Otherwise every pass reads the scores again, which the L2 holds: two or three passes, where k_select_topk has eight over what it
// has not collected yet.  Mask update with its wait, k_select_topk / this, us: 24576 blocks of 32 x 32, normal 74 / 60, half of the
// gradient zero 74 / 63, half of both 74 / 63, equal scores 112 / 89, a few far above the others 74 / 60; 43008 blocks 104 / 85, 104 /
// 90, 105 / 90, 170 / 134, 104 / 85, and weights that are zero outside a fifth of the blocks 170 / 88; 65536 of 16 x 16 121 / 99, 121 /
// 106, 125 / 107, 226 / 192, 121 / 99, 226 / 101.  (With the zeros in the passes and digits of eight bits, 43008 blocks: 85, 107, 116,
// 159, 105, 187; 128000 blocks 205 / 168, with half of the gradient zero 204 / 222, so the line is at 65536.)
constexpr int kStagedN = 20000, kOneWorkgroupN = 1 << 16;
template <bool STAGED>
__global__ __launch_bounds__(1024) void k_select_small(const double* __restrict__ score0, int n, int n_keep,
                                                       uint8_t* __restrict__ mask0, const double* __restrict__ score1,
                                                       uint8_t* __restrict__ mask1) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long keys[];
  __shared__ SelectShared ssh[1];
  static_assert(kStagedN * 8 + sizeof(ssh) <= 160 * 1024, "the keys fit the LDS of a CU");
  const double* __restrict__ score = blockIdx.x == 0 ? score0 : score1;
  uint8_t* __restrict__ mask = blockIdx.x == 0 ? mask0 : mask1;
  select_small<1024, 1, STAGED>(score, n, n_keep, keys, ssh);
  const unsigned long long* bits = reinterpret_cast<const unsigned long long*>(score);
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) mask[i] = select_keeps(ssh[0], STAGED ? keys[i] : order_key(bits[i]), i) ? 1 : 0;
}

// One workgroup: the mask update of prune-and-grow on n <= kSmallN blocks - both selections, side by side, and their
// merge (1 where the weight's selection keeps the block, 2 where only the gradient's does, else 0).  Dynamic LDS: 2 n keys.
__global__ __launch_bounds__(1024) void k_masks_small(const double* __restrict__ score_w,
                                                      const double* __restrict__ score_g, int n, int n_keep,
                                                      uint8_t* __restrict__ mask) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long keys[];
  __shared__ SelectShared ssh[2];
  const bool grad = threadIdx.x >= 512;
  select_small<512, 2>(grad ? score_g : score_w, n, n_keep, grad ? keys + n : keys, ssh);
  for (int i = threadIdx.x; i < n; i += 1024)
    mask[i] = select_keeps(ssh[0], keys[i], i) ? 1 : (select_keeps(ssh[1], keys[n + i], i) ? 2 : 0);
}

// Rows by population, descending, stable: rord (LDS) and row_order get the schedule of nbr <= 1024 rows; run by a
// workgroup of 1024 threads.  rcnt: 1024 populations in LDS, zero beyond nbr (which never counts).  P threads share
// a row, each comparing it with a contiguous part of the rows (four populations per LDS read).
__device__ __forceinline__ void schedule_small(const int* rcnt, int nbr, int* rord, int* __restrict__ row_order) {
  const int tid = threadIdx.x;
  const int pl = 31 - __clz(1024 / nbr);         // log2 P, P = largest power of two <= 1024 / nbr ...
  const int lp = pl > 6 ? 6 : pl, P = 1 << lp;   // ... and <= 64, so that the P threads sit in one wave
  const int r = tid >> lp, part = tid & (P - 1);
  const int len = (((nbr + P - 1) >> lp) + 3) & ~3;
  const int cr = r < nbr ? rcnt[r] : 0;
  int rank = 0;
  const int q0 = part * len;
#pragma unroll 4
  for (int q = q0; q < q0 + len; q += 4) {
    const int4 c4 = *reinterpret_cast<const int4*>(&rcnt[q]);
    rank += (c4.x > cr || (c4.x == cr && q < r)) ? 1 : 0;
    rank += (c4.y > cr || (c4.y == cr && q + 1 < r)) ? 1 : 0;
    rank += (c4.z > cr || (c4.z == cr && q + 2 < r)) ? 1 : 0;
    rank += (c4.w > cr || (c4.w == cr && q + 3 < r)) ? 1 : 0;
  }
  for (int d = P >> 1; d > 0; d >>= 1) rank += __shfl_xor(rank, d, kWave);
  if (r < nbr && part == 0) {
    rord[rank] = r;
    row_order[rank] = r;
  }
}

// Both chunk plans of nbr <= 1024 rows in schedule order, cut into chunks of at most 16 / 64 blocks (an empty row
// still gets one chunk: its output has to be written); run by a workgroup of 1024 threads.  rptr, rord: row pointers
// and schedule in LDS.  Populations fall along the schedule: the first row is the fullest, the rows that a plan cuts come before
// the others.  Thread 0 returns with the fullest row's population.
__device__ __forceinline__ int chunk_plans_small(const int* rptr, const int* rord, int nbr, const PlanOut& narrow,
                                                 const PlanOut& wide, int* wave_tot) {
  const int tid = threadIdx.x;
  constexpr int ls0 = __builtin_ctz(blast::kChunkBlocks), ls1 = __builtin_ctz(blast::kWideChunkBlocks);
  int r = 0, kb = 0, ke = 0, n0 = 0, n1 = 0, next = 0;  // next: the population of the next row in the schedule
  if (tid < nbr) {
    r = rord[tid];
    kb = rptr[r];
    ke = rptr[r + 1];
    const int rn = tid + 1 < nbr ? rord[tid + 1] : r;
    next = tid + 1 < nbr ? rptr[rn + 1] - rptr[rn] : 0;
    n0 = (ke - kb + (1 << ls0) - 1) >> ls0;
    n1 = (ke - kb + (1 << ls1) - 1) >> ls1;
    n0 = n0 < 1 ? 1 : n0;
    n1 = n1 < 1 ? 1 : n1;
    narrow.row_slot[r] = n0 > 1 ? tid : -1;
  }
  int total;
  const int first = block_exscan<true>(n0 | (n1 << 16), wave_tot, total);
  if (tid < nbr) {
    const int f0 = first & 0xFFFF, f1 = first >> 16;
    narrow.row_chunk0[r] = n0 > 1 ? f0 : -1;
    for (int j = 0; j < n0; ++j) {
      const int e = f0 + j, b0 = kb + (j << ls0);
      if (e < narrow.cap) {
        narrow.chunk_row[e] = r | (n0 > 1 ? (int)0x80000000u : 0);
        narrow.chunk_kb[e] = b0;
        narrow.chunk_ke[e] = (b0 + (1 << ls0) < ke) ? b0 + (1 << ls0) : ke;
      }
    }
    for (int j = 0; j < n1; ++j) {
      const int e = f1 + j, b0 = kb + (j << ls1);
      if (e < wide.cap) {
        wide.chunk_row[e] = r | (n1 > 1 ? (int)0x80000000u : 0);
        wide.chunk_kb[e] = b0;
        wide.chunk_ke[e] = (b0 + (1 << ls1) < ke) ? b0 + (1 << ls1) : ke;
      }
    }
  }
  // chunks of the rows that a plan cuts: these rows are the first, the last of them knows
  if (n0 > 1 && next <= 1 << ls0) narrow.hdr[3] = (first & 0xFFFF) + n0;
  if (n1 > 1 && next <= 1 << ls1) wide.hdr[3] = (first >> 16) + n1;
  if (tid == 0) {
    narrow.hdr[0] = total & 0xFFFF;
    narrow.hdr[1] = ke - kb;
    narrow.hdr[2] = 1 << ls0;
    if (n0 <= 1) narrow.hdr[3] = 0;
    wide.hdr[0] = total >> 16;
    wide.hdr[1] = ke - kb;
    wide.hdr[2] = 1 << ls1;
    if (n1 <= 1) wide.hdr[3] = 0;
  }
  return ke - kb;
}

struct SmallOut {
  int* row_ptr;
  int* col_idx;
  int* row_order;
  int* col_ptr;       // null without aux
  int* csc_row;       // csc_blk follows at the next 16-byte boundary after nnz entries
  int* scalars;       // {nnz, max_row_blocks}
  int64_t nnz_cap;
};

struct GatherArgs {
  const uint16_t* W;
  int64_t ldw;
  int b;
  uint16_t* vals;
  int span;  // candidate blocks of a workgroup, at most 32
  int code;  // mask code of every block where there is no mask
};

// More blocks than kSmallN, the index arrays still made by a workgroup each: a thread owns up to kBigPer blocks (a multiple
// of four), flags in 64 bits, positions in 16.
constexpr int kBigPer = 48, kBigN = 1024 * kBigPer;
static_assert(kBigN < 65536 && kBigN / blast::kChunkBlocks + 1024 < 32768, "positions in 16 bits, two counts in a 32-bit word");

// Flags of the blocks a thread owns (bit j: block tid * per + j is kept).
__device__ __forceinline__ unsigned small_flags(const uint8_t* __restrict__ mask, int code, int n, int per) {
  const int e0 = threadIdx.x * per;
  unsigned keep = 0u;
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j)
    keep |= (j < per && e0 + j < n && (mask ? mask[e0 + j] : code) != 0) ? 1u << j : 0u;
  return keep;
}
__device__ __forceinline__ unsigned long long big_flags(const uint8_t* __restrict__ mask, int code, int n, int per) {
  const int e0 = threadIdx.x * per;
  const bool words = mask && (reinterpret_cast<uintptr_t>(mask) & 3u) == 0;
  unsigned long long keep = 0ull;
#pragma unroll 4
  for (int j = 0; j < per; j += 4) {
    unsigned four = 0u;
    if (words && e0 + j + 3 < n) {
      const unsigned v = *reinterpret_cast<const unsigned*>(mask + e0 + j);
      const unsigned any = ((((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) >> 7) & 0x01010101u;  // a bit per byte that is not 0
      four = (any * 0x01020408u) >> 24;
    } else {
      for (int u = 0; u < 4; ++u) four |= (e0 + j + u < n && (mask ? mask[e0 + j + u] : code) != 0) ? 1u << u : 0u;
    }
    keep |= (unsigned long long)four << j;
  }
  return keep;
}

// This thread's share of the blocks that are kept among the first c0, a multiple of four, of a workgroup of 1024.
__device__ __forceinline__ int count_before(const uint8_t* __restrict__ mask, int code, int c0) {
  int before = 0;
  if (!mask) return threadIdx.x == 0 && code != 0 ? c0 : 0;
  if ((reinterpret_cast<uintptr_t>(mask) & 3u) == 0) {
#pragma unroll 4
    for (int i = 4 * threadIdx.x; i < c0; i += 4096) {
      const unsigned v = *reinterpret_cast<const unsigned*>(mask + i);
      before += __popc((((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) & 0x80808080u);
    }
  } else {
#pragma unroll 4
    for (int i = threadIdx.x; i < c0; i += 1024) before += mask[i] != 0 ? 1 : 0;
  }
  return before;
}

// Everything that follows the mask, in one launch.  Workgroup 0: row pointers, schedule, chunk plans; workgroup 1 (with
// aux): the column-grouped index; the others: ga.span candidate blocks each, whose places among the stored blocks
// they count for themselves - column indices and values.  A block whose mask code is 2 (regrown, BLaST Sec. 3.2) is
// stored as zeros: it joins the structure without changing the product.  No mask: every block has the code ga.code.
// What bounds it: the index jobs, a chain of scans and barriers in a workgroup each.  Three 8192 x 2048 matrices, b = 64,
// 80 % sparse, after a mask update: as one workgroup for all index arrays and a launch for the values 12 + 4.6 us per
// matrix and 187 us for the update and re-packing together, as two and the rest 9 us and 163; the launch takes 6.6 us (4096
// blocks of 32 x 32; 8.8 before) since the scans shift by the vector unit and the chunk plans add nothing up with atomics, 3.4
// us of whose 7.7 in the row job these were.
// BIG: more than kSmallN blocks, at most kBigN, which took nine launches.  A thread's blocks in two walks, as they do not fit
// registers; a workgroup of values that has any counts the flags before its blocks itself, whole lines from the L2.  Packing with its
// wait, nine launches / this, 80 % sparse: 8704 blocks of 32 x 32 62 / 35 us, 16384 70 / 38, 43008 89 / 51, 14336 of 64 x 64
// 72 / 37, of 128 x 128 101 / 58; none left out, 43008 blocks: 115 / 88, 1024 x 48 blocks of 16 x 16 143 / 108 (150 where the
// column job counted the columns before it knew their first blocks' places).  48841 blocks of 128 x 128, 98 % and 80 % sparse:
// 85 / 50, 198 / 160 (162 and 230 where workgroups without a value counted too, and each thread its own stretch of the flags, so
// that a load touched dozens of lines).  Three 8192 x 2048 matrices, b = 32, mask update and packing: 320 us before, then 208,
// 198 with the scans above.
template <bool BIG>
__global__ __launch_bounds__(1024) void k_pack_small(const uint8_t* __restrict__ mask, int nbr, int nbc, SmallOut o,
                                                     PlanOut narrow, PlanOut wide, GatherArgs ga) {
  __shared__ __attribute__((aligned(16))) int cnt[1024];  // populations of the rows, or of the columns
  using Flags = std::conditional_t<BIG, unsigned long long, unsigned>;
  using Place = std::conditional_t<BIG, uint16_t, int>;
  struct RowArrays {
    int rptr[1025], rord[1024];
  };
  // rows: these; columns: position of a stored block in col_idx / vals by row-major block index, [n], and flags, [n]
  __shared__ __attribute__((aligned(16))) char arrays[BIG ? 16 : kSmallN * 5];
  extern __shared__ __attribute__((aligned(16))) char big_arrays[];
  char* const scratch = BIG ? big_arrays : arrays;
  static_assert(sizeof(RowArrays) <= kSmallN * 5, "one or the other");
  RowArrays& row = *reinterpret_cast<RowArrays*>(scratch);
  __shared__ int wave_tot[16];
  const int tid = threadIdx.x;
  const int n = nbr * nbc;
  // blocks per thread (uniform); without BIG the loops below are unrolled to kSmallPer
  const int per = BIG ? (((n + 1023) >> 10) + 3) & ~3 : (n + 1023) >> 10, most = BIG ? per : kSmallPer;
  const int e0 = tid * per;
  auto population = [](Flags f) { return BIG ? __popcll(f) : __popc((unsigned)f); };
  const int jobs = o.col_ptr ? 2 : 1;
  const bool values = (int)blockIdx.x >= jobs;
  Flags keep = 0;
  if constexpr (BIG) {
    if (!values) keep = big_flags(mask, ga.code, n, per);
  } else {
    keep = small_flags(mask, ga.code, n, per);
  }

  if (values) {
    // ---- the values of the candidates [c0, c0 + ga.span) -----------------------------------------------------------
    const int c0 = ((int)blockIdx.x - jobs) * ga.span;
    const int cand = c0 + lane_id();
    const int code = lane_id() < ga.span && cand < n ? (mask ? mask[cand] : ga.code) : 0;
    const unsigned kept = (unsigned)__ballot(code != 0), zero = (unsigned)__ballot(code == 2);
    if (BIG && kept == 0u) return;  // (all waves have the same)
    int before = 0;  // stored blocks before c0
    if constexpr (BIG) {
      before = count_before(mask, ga.code, c0);
#pragma unroll
      for (int d = kWave / 2; d > 0; d >>= 1) before += __shfl_xor(before, d, kWave);
    } else {
#pragma unroll
      for (int j = 0; j < kSmallPer; ++j) before += __popcll(__ballot(((keep >> j) & 1u) && e0 + j < c0));
    }
    if (lane_id() == 0) wave_tot[tid / kWave] = before;
    __syncthreads();
    int first = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) first += wave_tot[w];
    const int nk = __popc(kept);
    if (tid < ga.span && (kept >> tid & 1u)) {
      const int k = first + __popc(kept & ((1u << tid) - 1u));
      if (k < o.nnz_cap) o.col_idx[k] = (c0 + tid) % nbc;
    }
    const int cpr = ga.b / 8, lcpr = __builtin_ctz(cpr), lcpb = __builtin_ctz(ga.b * cpr);  // 16-byte pieces per row, per block
    const int total = nk << lcpb;
    constexpr int kAhead = 4;
    for (int p0 = tid; p0 < total; p0 += kAhead * 1024) {
      uint4 v[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int p = p0 + u * 1024;
        v[u] = uint4{0u, 0u, 0u, 0u};
        if (p < total) {
          // the (p >> lcpb)-th kept candidate
          unsigned left = kept;
          for (int q = p >> lcpb; q > 0; --q) left &= left - 1u;
          const int c = __builtin_ctz(left);
          if (!(zero >> c & 1u)) {
            const int piece = p & ((1 << lcpb) - 1), i = piece >> lcpr, j8 = piece & (cpr - 1);
            const int br = (c0 + c) / nbc, bc = (c0 + c) - br * nbc;
            v[u] = *reinterpret_cast<const uint4*>(ga.W + ((int64_t)br * ga.b + i) * ga.ldw + (int64_t)bc * ga.b + j8 * 8);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int p = p0 + u * 1024;
        if (p < total && first + (p >> lcpb) < o.nnz_cap)
          *reinterpret_cast<uint4*>(ga.vals + (((int64_t)first << lcpb) + p) * 8) = v[u];
      }
    }
    return;
  }

  if (blockIdx.x == 0) {
    cnt[tid] = 0;
    // ---- rows: pointers, schedule, chunk plans -----------------------------------------------------------------------
    wg_barrier<true>();
    {
      int r = e0 / nbc, c = e0 - r * nbc, run = 0;  // a thread adds its blocks of a row at once
#pragma unroll
      for (int j = 0; j < most; ++j) {
        if (j < per && e0 + j < n) {
          run += (int)((keep >> j) & 1u);
          if (++c == nbc || j == per - 1 || e0 + j == n - 1) {
            if (run) atomicAdd(&cnt[r], run);
            run = 0;
            if (c == nbc) {
              c = 0;
              ++r;
            }
          }
        }
      }
    }
    wg_barrier<true>();
    int nnz;
    const int ex = block_exscan<true>(tid < nbr ? cnt[tid] : 0, wave_tot, nnz);
    if (tid < nbr) {
      row.rptr[tid] = ex;
      o.row_ptr[tid] = ex;
    }
    if (tid == 0) {
      row.rptr[nbr] = nnz;
      o.row_ptr[nbr] = nnz;
      o.scalars[0] = nnz;
      if (!o.col_ptr) o.scalars[1] = 0;
    }
    schedule_small(cnt, nbr, row.rord, o.row_order);
    wg_barrier<true>();
    if (!o.col_ptr) return;
    const int heavy = chunk_plans_small(row.rptr, row.rord, nbr, narrow, wide, wave_tot);
    if (tid == 0) o.scalars[1] = heavy;
    return;
  }

  Place* const kpos = reinterpret_cast<Place*>(scratch);
  uint8_t* const flag = reinterpret_cast<uint8_t*>(kpos + n);
  // ---- columns: the position of a stored block is the number of kept blocks before it, in row-major order for
  // col_idx / vals and in column-major order for the column-grouped index --------------------------------------------
  int nnz;
  int k = block_exscan<true>(population(keep), wave_tot, nnz);
#pragma unroll
  for (int j = 0; j < most; ++j) {
    if (j < per && e0 + j < n) {
      const bool kp = (int)((keep >> j) & 1u);
      flag[e0 + j] = kp ? 1 : 0;
      if (kp) kpos[e0 + j] = (Place)k++;
    }
  }
  wg_barrier<true>();
  {
    const bool fits = nnz <= o.nnz_cap;
    int* csc_blk = o.csc_row + (nnz + 3) / 4 * 4;
    Flags keep_c = 0;
    const int c0 = e0 / nbr, r0 = e0 - c0 * nbr;
    {
      int r = r0, at = r0 * nbc + c0;
#pragma unroll
      for (int j = 0; j < most; ++j) {
        if (j < per && e0 + j < n) {
          keep_c |= flag[at] ? (Flags)1 << j : (Flags)0;
          at += nbc;
          if (++r == nbr) {
            r = 0;
            at = at - n + 1;  // top of the next column
          }
        }
      }
    }
    int total;
    int e = block_exscan<true>(population(keep_c), wave_tot, total);
    int r = r0, c = c0, at = r0 * nbc + c0;
#pragma unroll
    for (int j = 0; j < most; ++j) {
      if (j < per && e0 + j < n) {
        if (r == 0) o.col_ptr[c] = e;  // (the kept blocks of the columns before it)
        if ((keep_c >> j) & 1u) {
          if (fits) {
            o.csc_row[e] = r;
            csc_blk[e] = kpos[at];
          }
          ++e;
        }
        at += nbc;
        if (++r == nbr) {
          r = 0;
          ++c;
          at = at - n + 1;
        }
      }
    }
    if (tid == 0) o.col_ptr[nbc] = nnz;
  }
}

struct TransposeArgs {
  // the matrix: its column-grouped index (BCSC), row pointers and column indices
  const int* col_ptr;
  const int* csc_row;
  const int* csc_blk;
  const int* row_ptr;
  const int* col_idx;
  const uint16_t* vals;
  int64_t nbr, nbc, nnz;
  // its transpose: BSR arrays, and in aux (null pointers without) the column-grouped index
  int* row_ptr_t;
  int* col_idx_t;
  uint16_t* vals_t;
  int* row_order_t;
  int* col_ptr_t;
  int* csc_row_t;
  int* csc_blk_t;
  PlanOut narrow, wide;  // aux only
  int* max_row_out;      // aux only: the fullest row of the transpose
  int index_job;         // workgroup 0 makes schedule and chunk plans (up to 1024 rows, fewer than 65536 chunks)
};

// The whole packed transpose in one launch.  Workgroup 0 writes the pointer arrays and, for up to 1024 block rows of
// the transpose, its schedule and chunk plans; the others turn the blocks, kTransposeElems values each (one block of
// 128 x 128, four of 64 x 64, ...), and write their entries of the index arrays.  A block of the transpose is read
// and written in 16-byte pieces, whole lines; the turn happens in LDS (row pitch b + 2 elements, so that a column
// walk does not stay on one bank).
// What bounds it: the latency of the index job beside a copy of the blocks.  In a training step of an 8192 x 3072
// matrix (b = 64, 1229 blocks, 2000 tokens: forward, transpose, dX, dW) the ten launches before it (copies of the
// four index arrays, schedule, chunk plans, inverse permutation, blocks two bytes at a time, a copy back of one
// number) were 45 us of kernels and their gaps; the step took 199 us with them and takes 147 us with this one.
constexpr int kTransposeElems = 16384;
template <int B>
__global__ __launch_bounds__(1024) void k_transpose(const TransposeArgs a) {
  constexpr int NB = kTransposeElems / (B * B);  // blocks per workgroup
  constexpr int CPR = B / 8, PITCH = B + 2;      // 16-byte pieces per block row; LDS row pitch
  constexpr int kTile = B * PITCH;
  __shared__ __attribute__((aligned(16))) uint16_t tile[NB * kTile];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    for (int64_t i = tid; i <= a.nbc; i += 1024) a.row_ptr_t[i] = a.col_ptr[i];
    if (a.col_ptr_t)
      for (int64_t i = tid; i <= a.nbr; i += 1024) a.col_ptr_t[i] = a.row_ptr[i];
    if (!a.index_job) return;
    // the index job's LDS lies over the tile
    struct Sched {
      int rcnt[1024], rptr[1025], rord[1024], wave_tot[16];
    };
    static_assert(sizeof(Sched) <= sizeof(tile), "the schedule fits the tile");
    Sched& s = *reinterpret_cast<Sched*>(tile);
    const int n = (int)a.nbc;
    s.rcnt[tid] = tid < n ? a.col_ptr[tid + 1] - a.col_ptr[tid] : 0;
    if (tid < n) s.rptr[tid] = a.col_ptr[tid];
    if (tid == 0) s.rptr[n] = a.col_ptr[n];
    wg_barrier<true>();
    schedule_small(s.rcnt, n, s.rord, a.row_order_t);
    wg_barrier<true>();
    if (!a.max_row_out) return;
    const int heavy = chunk_plans_small(s.rptr, s.rord, n, a.narrow, a.wide, s.wave_tot);
    if (tid == 0) *a.max_row_out = heavy;
    return;
  }
  const int64_t e0 = (int64_t)(blockIdx.x - 1) * NB;
  if (tid < NB && e0 + tid < a.nnz) {
    const int64_t e = e0 + tid;
    a.col_idx_t[e] = a.csc_row[e];
    if (a.csc_row_t) {
      a.csc_row_t[e] = a.col_idx[e];
      a.csc_blk_t[a.csc_blk[e]] = (int)e;
    }
  }
#pragma unroll
  for (int q = 0; q < kTransposeElems / 8 / 1024; ++q) {
    const int p = q * 1024 + tid, blk = p / (B * CPR), i = p / CPR % B, c = p % CPR;
    if (e0 + blk < a.nnz) {
      const uint4 v = *reinterpret_cast<const uint4*>(a.vals + (int64_t)a.csc_blk[e0 + blk] * (B * B) + i * B + c * 8);
      uint32_t* dst = reinterpret_cast<uint32_t*>(tile + blk * kTile + i * PITCH + c * 8);
      dst[0] = v.x;
      dst[1] = v.y;
      dst[2] = v.z;
      dst[3] = v.w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kTransposeElems / 8 / 1024; ++q) {
    const int p = q * 1024 + tid, blk = p / (B * CPR), j = p / CPR % B, c = p % CPR;
    if (e0 + blk < a.nnz) {
      const uint16_t* src = tile + blk * kTile + c * 8 * PITCH + j;
      uint32_t w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = (uint32_t)src[2 * u * PITCH] | ((uint32_t)src[(2 * u + 1) * PITCH] << 16);
      *reinterpret_cast<uint4*>(a.vals_t + (e0 + blk) * (B * B) + j * B + c * 8) = uint4{w[0], w[1], w[2], w[3]};
    }
  }
}

// One workgroup per block of the dense matrix: copies the stored block there, or writes zeros where the
// block row's column list (ascending) has no entry for it.
__global__ __launch_bounds__(256) void k_unpack_blocks(const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
                                                       const uint16_t* __restrict__ vals, int nbc, int b,
                                                       uint16_t* __restrict__ W, int64_t ldw) {
  const int64_t blk = blockIdx.x;
  const int br = (int)(blk / nbc), bc = (int)(blk % nbc);
  int lo = row_ptr[br], hi = row_ptr[br + 1];
  int k = -1;
  while (lo < hi) {  // binary search for bc in [lo, hi)
    const int mid = (lo + hi) >> 1;
    const int c = col_idx[mid];
    if (c == bc) {
      k = mid;
      break;
    }
    if (c < bc) lo = mid + 1; else hi = mid;
  }
  uint16_t* dst = W + (int64_t)br * b * ldw + (int64_t)bc * b;
  const uint16_t* src = k >= 0 ? vals + (int64_t)k * b * b : nullptr;
  const int cpr = b / 8, nchunks = b * cpr;
  for (int c = threadIdx.x; c < nchunks; c += 256) {
    const int i = c / cpr, j8 = c % cpr;
    *reinterpret_cast<uint4*>(dst + (int64_t)i * ldw + j8 * 8) =
        src ? *reinterpret_cast<const uint4*>(src + (int64_t)c * 8) : uint4{0u, 0u, 0u, 0u};
  }
}

// Scores of the n blocks of W, and of a second matrix of its shape where there is one.
int launch_block_scores(int b, const uint16_t* W, int64_t ldw, int64_t nbc, int64_t n, double* score, const uint16_t* W1,
                        int64_t ldw1, double* score1, hipStream_t stream) {
  const dim3 grid((unsigned)((n + 3) / 4), W1 ? 2 : 1);
  const int c = (int)nbc;
  switch (b) {
    case 16: k_block_scores<16><<<grid, dim3(256), 0, stream>>>(W, ldw, c, n, score, W1, ldw1, score1); break;
    case 32: k_block_scores<32><<<grid, dim3(256), 0, stream>>>(W, ldw, c, n, score, W1, ldw1, score1); break;
    case 64: k_block_scores<64><<<grid, dim3(256), 0, stream>>>(W, ldw, c, n, score, W1, ldw1, score1); break;
    default: k_block_scores<128><<<grid, dim3(256), 0, stream>>>(W, ldw, c, n, score, W1, ldw1, score1); break;
  }
  BLAST_LAUNCH_CHECK("k_block_scores");
  return BLAST_OK;
}

struct PackWs {
  size_t scores_off, mask_off, rcnt_off, ccnt_off, blk_row_off, scalars_off, bytes;
};

PackWs pack_ws_layout(int64_t nbr, int64_t nbc, int32_t mode, int64_t nnz_cap) {
  using blast::align_up;
  const size_t n = (size_t)nbr * (size_t)nbc;
  PackWs L;
  size_t off = 0;
  L.scores_off = off;
  if (mode == BLAST_PACK_TOPK_FROBENIUS) off += align_up(8 * n, 256);
  L.mask_off = off;
  if (mode == BLAST_PACK_TOPK_FROBENIUS) off += align_up(n, 256);
  L.rcnt_off = off;
  off += align_up(4 * (size_t)nbr, 256);
  L.ccnt_off = off;
  off += align_up(4 * (size_t)nbc, 256);
  L.blk_row_off = off;
  off += align_up(4 * (size_t)(nnz_cap > 0 ? nnz_cap : 1), 256);
  L.scalars_off = off;
  off += 256;
  L.bytes = off;
  return L;
}

int check_shape(int64_t rows, int64_t cols, int32_t b) {
  if (rows < 0 || cols < 0) return BLAST_ERR_INVALID_ARG;
  if (!blast::supported_block(b)) return BLAST_ERR_UNSUPPORTED_BLOCK;
  if (rows % b || cols % b) return BLAST_ERR_SHAPE;
  if (rows / b > INT32_MAX / 2 || cols / b > INT32_MAX / 2 || (rows / b) * (cols / b) > (int64_t)INT32_MAX)
    return BLAST_ERR_INVALID_ARG;
  return BLAST_OK;
}

// mask = the n_keep highest of n <= kSmallN scores (0 < n_keep < n), merged with the n_keep highest of scores1.
int launch_masks_small(const double* scores, const double* scores1, int64_t n, int64_t n_keep, uint8_t* mask, hipStream_t stream) {
  static blast::DeviceFlags lds_set;
  int dev = 0;
  BLAST_HIP_TRY(hipGetDevice(&dev));
  if (!lds_set.test(dev)) {
    BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_masks_small),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kSmallN * 8));
    lds_set.set(dev);
  }
  k_masks_small<<<dim3(1), dim3(1024), (size_t)n * 16, stream>>>(scores, scores1, (int)n, (int)n_keep, mask);
  BLAST_LAUNCH_CHECK("k_masks_small");
  return BLAST_OK;
}

// mask = the n_keep highest of n scores (0 < n_keep < n), and mask1 those of scores1 where there is one.
int launch_select(const double* scores, const double* scores1, int64_t n, int64_t n_keep, uint8_t* mask, uint8_t* mask1,
                  hipStream_t stream) {
  static blast::DeviceFlags lds_set;
  int dev = 0;
  BLAST_HIP_TRY(hipGetDevice(&dev));
  if (!lds_set.test(dev)) {
    BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_select_small<true>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, kStagedN * 8));
    lds_set.set(dev);
  }
  const dim3 grid(scores1 ? 2 : 1);
  if (n > kOneWorkgroupN) {
    k_select_topk<<<grid, dim3(1024), 0, stream>>>(scores, n, n_keep, mask, scores1, mask1);
    BLAST_LAUNCH_CHECK("k_select_topk");
  } else if (n <= kStagedN) {
    k_select_small<true><<<grid, dim3(1024), (size_t)n * 8, stream>>>(scores, (int)n, (int)n_keep, mask, scores1, mask1);
    BLAST_LAUNCH_CHECK("k_select_small");
  } else {
    k_select_small<false><<<grid, dim3(1024), kWideBins * sizeof(unsigned), stream>>>(scores, (int)n, (int)n_keep, mask, scores1,
                                                                                      mask1);
    BLAST_LAUNCH_CHECK("k_select_small");
  }
  return BLAST_OK;
}

// A small pinned buffer per host thread (allocated on first use and kept) through which numbers come back from the
// device: a copy into pageable memory costs a call tens of microseconds more.  Kernels can store to it themselves, those
// of every GPU the thread uses.
// Null when it cannot be had.
int* pinned_ints() {
  static thread_local int* pinned = nullptr;
  if (!pinned) {
    void* p = nullptr;
    if (hipHostMalloc(&p, 64, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) {
      pinned = static_cast<int*>(p);
    } else {
      (void)hipGetLastError();
    }
  }
  return pinned;
}

template <int B>
int launch_transpose(const TransposeArgs& a, hipStream_t stream) {
  constexpr int NB = kTransposeElems / (B * B);
  k_transpose<B><<<dim3((unsigned)(1 + (a.nnz + NB - 1) / NB)), dim3(1024), 0, stream>>>(a);
  BLAST_LAUNCH_CHECK("k_transpose");
  return BLAST_OK;
}

}  // namespace

extern "C" int64_t blast_n_keep(int64_t n_blocks, double sparsity) {
  if (n_blocks < 0 || !(sparsity >= 0.0 && sparsity <= 1.0)) return -1;
  const int64_t s_bp = (int64_t)(sparsity * 10000.0 + 0.5);
  const int64_t n_zero = (int64_t)(((__int128)s_bp * n_blocks + 9999) / 10000);
  return n_blocks - (n_zero > n_blocks ? n_blocks : n_zero);
}

extern "C" size_t blast_bsr_aux_bytes(int64_t rows, int64_t cols, int32_t b, int64_t nnz_cap) {
  if (check_shape(rows, cols, b) != BLAST_OK || nnz_cap < 0) return 0;
  return blast::aux_layout(rows / b, cols / b, nnz_cap).bytes;
}

extern "C" int blast_bsr_pack_bound(int64_t rows, int64_t cols, int32_t b, int32_t mode, double sparsity,
                                    int64_t* nnz_cap, size_t* aux_bytes, size_t* ws_bytes) {
  if (mode != BLAST_PACK_MASK && mode != BLAST_PACK_TOPK_FROBENIUS) return BLAST_ERR_INVALID_ARG;
  if (int rc = check_shape(rows, cols, b)) return rc;
  const int64_t nbr = rows / b, nbc = cols / b, n = nbr * nbc;
  int64_t cap = n;
  if (mode == BLAST_PACK_TOPK_FROBENIUS) {
    cap = blast_n_keep(n, sparsity);
    if (cap < 0) return BLAST_ERR_INVALID_ARG;
  }
  if (nnz_cap) *nnz_cap = cap;
  if (aux_bytes) *aux_bytes = blast::aux_layout(nbr, nbc, cap).bytes;
  if (ws_bytes) *ws_bytes = pack_ws_layout(nbr, nbc, mode, cap).bytes;
  return BLAST_OK;
}

namespace {

// Validates the arguments of a packing call and enqueues all of its work.  The two result scalars {number of
// stored blocks, stored blocks of the fullest row} are left at *scalars_out (device memory: `result` when the
// caller gave one, else a slot of the workspace); n_keep_out gets the number of blocks the scoring mode keeps
// (-1 in mask mode).
int pack_enqueue(const uint16_t* W, int64_t ldw, int64_t rows, int64_t cols, int32_t b, int32_t mode,
                 const uint8_t* block_mask, double sparsity, int32_t* row_ptr, int32_t* col_idx, uint16_t* vals,
                 int32_t* row_order, void* aux, size_t aux_bytes, int64_t nnz_cap, int32_t* result, void* ws,
                 size_t ws_bytes, hipStream_t stream, int** scalars_out) {
  if (mode != BLAST_PACK_MASK && mode != BLAST_PACK_TOPK_FROBENIUS) return BLAST_ERR_INVALID_ARG;
  if (int rc = check_shape(rows, cols, b)) return rc;
  if (!row_ptr || nnz_cap < 0) return BLAST_ERR_INVALID_ARG;
  const int64_t nbr = rows / b, nbc = cols / b, n = nbr * nbc;
  if (n > 0 && (!W || ldw < cols || ldw % 8 || !blast::aligned(W, 16))) return BLAST_ERR_INVALID_ARG;
  if (mode == BLAST_PACK_MASK && n > 0 && !block_mask) return BLAST_ERR_INVALID_ARG;
  int64_t n_keep = -1;
  if (mode == BLAST_PACK_TOPK_FROBENIUS) {
    n_keep = blast_n_keep(n, sparsity);
    if (n_keep < 0) return BLAST_ERR_INVALID_ARG;
  }
  if (nnz_cap > 0 && (!col_idx || !vals || !blast::aligned(vals, 16))) return BLAST_ERR_INVALID_ARG;
  if (nbr > 0 && !row_order) return BLAST_ERR_INVALID_ARG;
  const PackWs L = pack_ws_layout(nbr, nbc, mode, nnz_cap);
  if (!ws || ws_bytes < L.bytes || !blast::aligned(ws, 16)) return BLAST_ERR_WORKSPACE;
  const blast::AuxLayout A = blast::aux_layout(nbr, nbc, nnz_cap);
  if (aux && (aux_bytes < A.bytes || !blast::aligned(aux, 16))) return BLAST_ERR_WORKSPACE;
  const int64_t gather_grid = (mode == BLAST_PACK_TOPK_FROBENIUS && n_keep < nnz_cap) ? n_keep : nnz_cap;
  if (gather_grid > INT32_MAX) return BLAST_ERR_INVALID_ARG;

  char* wsb = static_cast<char*>(ws);
  double* scores = reinterpret_cast<double*>(wsb + L.scores_off);
  int* rcnt = reinterpret_cast<int*>(wsb + L.rcnt_off);
  int* ccnt = reinterpret_cast<int*>(wsb + L.ccnt_off);
  int* blk_row = reinterpret_cast<int*>(wsb + L.blk_row_off);
  int* nnz_dev = result ? result : reinterpret_cast<int*>(wsb + L.scalars_off);
  *scalars_out = nnz_dev;
  const uint8_t* mask = block_mask;
  uint8_t* m = mode == BLAST_PACK_TOPK_FROBENIUS ? reinterpret_cast<uint8_t*>(wsb + L.mask_off) : nullptr;
  if (m) mask = m;
  char* ab = static_cast<char*>(aux);
  PlanOut narrow{}, wide{};
  if (aux) plan_outputs(ab, A, narrow, wide);
  int* col_ptr = aux ? reinterpret_cast<int*>(ab + A.col_ptr_off) : nullptr;  // (this offset does not depend on nnz)
  int* csc_row = aux ? reinterpret_cast<int*>(ab + A.csc_row_off) : nullptr;
  const bool scored = mode == BLAST_PACK_TOPK_FROBENIUS && n > 0 && n_keep > 0 && n_keep < n;
  if (scored) {
    if (int rc = launch_block_scores(b, W, ldw, nbc, n, scores, nullptr, 0, nullptr, stream)) return rc;
  }

  const bool small = n > 0 && n <= kBigN && nbr <= 1024 && nbc <= 1024, big = small && n > kSmallN;
  if (m && small && !scored) mask = nullptr;  // every block has the same code: no launch that writes it n times
  if (m && n > 0 && mask) {
    if (!scored) {
      k_fill_u8<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(m, n, n_keep == n ? 1 : 0);
      BLAST_LAUNCH_CHECK("k_fill_u8");
    } else {
      if (int rc = launch_select(scores, nullptr, n, n_keep, m, nullptr, stream)) return rc;
    }
  }
  if (small) {
    // every index array and the values: one launch
    const SmallOut o{row_ptr, col_idx, row_order, col_ptr, csc_row, nnz_dev, nnz_cap};
    // Sixteen candidates are up to 128 KiB of values; of 128-wide blocks four are, and eight still fill the chip when there
    // are many.  (Sixteen of those, every block kept, eight matrices: 2048 x 2048 255 us, with four 138; 4096 x 14336 388,
    // with four 375 and with eight 366, at 90 % sparsity 145, 161 and 138.)
    const int span = b < 64 && big ? 32 : b < 128 ? 16 : n < 2048 ? 4 : 8;
    const unsigned spans = nnz_cap > 0 ? (unsigned)((n + span - 1) / span) : 0u;
    const dim3 grid((aux ? 2u : 1u) + spans);
    const GatherArgs ga{W, ldw, b, vals, span, n_keep == n ? 1 : 0};
    if (big) {
      static blast::DeviceFlags lds_set;
      int dev = 0;
      BLAST_HIP_TRY(hipGetDevice(&dev));
      if (!lds_set.test(dev)) {
        BLAST_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pack_small<true>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, kBigN * 3));
        lds_set.set(dev);
      }
      k_pack_small<true><<<grid, dim3(1024), (size_t)n * 3, stream>>>(mask, (int)nbr, (int)nbc, o, narrow, wide, ga);
    } else {
      k_pack_small<false><<<grid, dim3(1024), 0, stream>>>(mask, (int)nbr, (int)nbc, o, narrow, wide, ga);
    }
    BLAST_LAUNCH_CHECK("k_pack_small");
    return BLAST_OK;
  } else {
    if (nbr > 0) {
      k_line_counts<<<dim3((unsigned)((nbr + 3) / 4)), dim3(256), 0, stream>>>(mask, (int)nbr, (int)nbc, nbc, 1, rcnt);
      BLAST_LAUNCH_CHECK("k_line_counts(rows)");
    }
    k_exscan<<<dim3(1), dim3(1024), 0, stream>>>(rcnt, (int)nbr, row_ptr, nnz_dev);
    BLAST_LAUNCH_CHECK("k_exscan(rows)");
    if (nbr > 0) {
      k_row_order<<<dim3((unsigned)((nbr + 255) / 256)), dim3(256), 0, stream>>>(row_ptr, nullptr, (int)nbr, row_order);
      BLAST_LAUNCH_CHECK("k_row_order");
    }
    if (aux) {
      k_chunk_plan<<<dim3(1), dim3(1024), 0, stream>>>(row_ptr, row_order, (int)nbr, narrow, wide, nnz_dev + 1);
      BLAST_LAUNCH_CHECK("k_chunk_plan");
    } else {
      k_fill_i32<<<dim3(1), dim3(64), 0, stream>>>(nnz_dev + 1, 1, 0);
      BLAST_LAUNCH_CHECK("k_fill_i32");
    }
    if (nbr > 0) {
      k_fill_cols<<<dim3((unsigned)nbr), dim3(256), 0, stream>>>(mask, (int)nbc, row_ptr, col_idx, blk_row, nnz_cap);
      BLAST_LAUNCH_CHECK("k_fill_cols");
    }
    if (aux) {
      if (nbc > 0 && nbr > 0) {
        k_line_counts<<<dim3((unsigned)((nbc + 3) / 4)), dim3(256), 0, stream>>>(mask, (int)nbc, (int)nbr, 1, nbc, ccnt);
        BLAST_LAUNCH_CHECK("k_line_counts(cols)");
      } else if (nbc > 0) {
        k_fill_i32<<<dim3((unsigned)((nbc + 255) / 256)), dim3(256), 0, stream>>>(ccnt, nbc, 0);
        BLAST_LAUNCH_CHECK("k_fill_i32(cols)");
      }
      k_exscan<<<dim3(1), dim3(1024), 0, stream>>>(ccnt, (int)nbc, col_ptr, nullptr);
      BLAST_LAUNCH_CHECK("k_exscan(cols)");
      if (nbc > 0 && nbr > 0 && nnz_cap > 0) {
        k_fill_csc<<<dim3((unsigned)nbc), dim3(256), 0, stream>>>(mask, (int)nbr, (int)nbc, row_ptr, col_idx, col_ptr,
                                                                  csc_row, nullptr, nnz_cap, nnz_dev);
        BLAST_LAUNCH_CHECK("k_fill_csc");
      }
    }
  }
  // Nothing needs the number of stored blocks on the host: the gather's grid is the capacity (workgroups past
  // the device's count leave), and the column-grouped index is placed by the device's count.
  if (gather_grid > 0) {
    k_gather_blocks<<<dim3((unsigned)gather_grid), dim3(256), 0, stream>>>(W, ldw, b, col_idx, blk_row, mask, (int)nbc,
                                                                         vals, nnz_dev);
    BLAST_LAUNCH_CHECK("k_gather_blocks");
  }
  return BLAST_OK;
}

}  // namespace

extern "C" int blast_bsr_pack_enqueue(const uint16_t* W, int64_t ldw, int64_t rows, int64_t cols, int32_t b,
                                      int32_t mode, const uint8_t* block_mask, double sparsity, int32_t* row_ptr,
                                      int32_t* col_idx, uint16_t* vals, int32_t* row_order, void* aux, size_t aux_bytes,
                                      int64_t nnz_cap, int32_t* result, void* ws, size_t ws_bytes, void* stream_) {
  if (!result || !blast::aligned(result, 8)) return BLAST_ERR_INVALID_ARG;
  int* scalars = nullptr;
  return pack_enqueue(W, ldw, rows, cols, b, mode, block_mask, sparsity, row_ptr, col_idx, vals, row_order, aux,
                      aux_bytes, nnz_cap, result, ws, ws_bytes, static_cast<hipStream_t>(stream_), &scalars);
}

extern "C" int blast_bsr_pack(const uint16_t* W, int64_t ldw, int64_t rows, int64_t cols, int32_t b, int32_t mode,
                              const uint8_t* block_mask, double sparsity, int32_t* row_ptr, int32_t* col_idx,
                              uint16_t* vals, int32_t* row_order, void* aux, size_t aux_bytes, int64_t nnz_cap,
                              int64_t* nnz_out, int32_t* max_row_blocks_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!nnz_out) return BLAST_ERR_INVALID_ARG;
  int* scalars = nullptr;
  if (int rc = pack_enqueue(W, ldw, rows, cols, b, mode, block_mask, sparsity, row_ptr, col_idx, vals, row_order, aux,
                            aux_bytes, nnz_cap, nullptr, ws, ws_bytes, stream, &scalars))
    return rc;
  int host_vals[2] = {0, 0};
  int* pinned = pinned_ints();
  int* landing = pinned ? pinned : host_vals;
  BLAST_HIP_TRY(hipMemcpyAsync(landing, scalars, 2 * sizeof(int), hipMemcpyDeviceToHost, stream));
  BLAST_HIP_TRY(hipStreamSynchronize(stream));
  host_vals[0] = landing[0];
  host_vals[1] = landing[1];
  *nnz_out = host_vals[0];
  if (max_row_blocks_out) *max_row_blocks_out = aux ? host_vals[1] : 0;
  if (host_vals[0] > nnz_cap) return BLAST_ERR_CAPACITY;
  return BLAST_OK;
}

extern "C" int blast_bsr_joint_row_order(const blast_bsr_view* A, const blast_bsr_view* Bm, int32_t* row_order,
                                         void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!A || !Bm || !A->row_ptr || !Bm->row_ptr) return BLAST_ERR_INVALID_ARG;
  if (int rc = check_shape(A->rows, A->cols, A->b)) return rc;
  if (A->rows != Bm->rows || A->b != Bm->b) return BLAST_ERR_SHAPE;
  const int64_t nbr = A->rows / A->b;
  if (nbr == 0) return BLAST_OK;
  if (!row_order) return BLAST_ERR_INVALID_ARG;
  k_row_order<<<dim3((unsigned)((nbr + 255) / 256)), dim3(256), 0, stream>>>(A->row_ptr, Bm->row_ptr, (int)nbr,
                                                                              row_order);
  BLAST_LAUNCH_CHECK("k_row_order(joint)");
  return BLAST_OK;
}

extern "C" int blast_bsr_transpose(const blast_bsr_view* W, int32_t* row_ptr_t, int32_t* col_idx_t, uint16_t* vals_t,
                                   int32_t* row_order_t, void* aux_t, size_t aux_t_bytes,
                                   int32_t* max_row_blocks_t_out, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!W || !W->row_ptr || W->nnz < 0 || W->nnz > INT32_MAX) return BLAST_ERR_INVALID_ARG;
  if (int rc = check_shape(W->rows, W->cols, W->b)) return rc;
  const int64_t nbr = W->rows / W->b, nbc = W->cols / W->b, nnz = W->nnz;
  const int b = W->b;
  if (!W->aux) return BLAST_ERR_WORKSPACE;  // the column-grouped index of the packer is the input here
  if (!row_ptr_t || (nbc > 0 && !row_order_t)) return BLAST_ERR_INVALID_ARG;
  if (nnz > 0 && (!W->col_idx || !W->vals || !col_idx_t || !vals_t || !blast::aligned(vals_t, 16) ||
                  !blast::aligned(W->vals, 16)))
    return BLAST_ERR_INVALID_ARG;
  const blast::AuxLayout A = blast::aux_layout(nbr, nbc, nnz);   // of the input
  const blast::AuxLayout At = blast::aux_layout(nbc, nbr, nnz);  // of the output
  if (aux_t && (aux_t_bytes < At.bytes || !blast::aligned(aux_t, 16))) return BLAST_ERR_WORKSPACE;
  const char* ab = static_cast<const char*>(W->aux);
  const int* col_ptr = reinterpret_cast<const int*>(ab + A.col_ptr_off);
  const int* csc_row = reinterpret_cast<const int*>(ab + A.csc_row_off);
  const int* csc_blk = reinterpret_cast<const int*>(ab + A.csc_blk_off);
  // BSR of the transpose = the column-grouped (BCSC) view of the input, with every block turned; the column-grouped
  // index of the transpose is the row-grouped one of the input
  TransposeArgs ta{};
  ta.col_ptr = col_ptr;
  ta.csc_row = csc_row;
  ta.csc_blk = csc_blk;
  ta.row_ptr = W->row_ptr;
  ta.col_idx = W->col_idx;
  ta.vals = W->vals;
  ta.nbr = nbr;
  ta.nbc = nbc;
  ta.nnz = nnz;
  ta.row_ptr_t = row_ptr_t;
  ta.col_idx_t = col_idx_t;
  ta.vals_t = vals_t;
  ta.row_order_t = row_order_t;
  // (the plans' scan holds two counts in one word: fewer than 65536 chunks)
  ta.index_job = nbc > 0 && nbc <= 1024 && nbc + nnz / blast::kChunkBlocks < 65536;
  int* landing = nullptr;
  if (aux_t) {
    char* at = static_cast<char*>(aux_t);
    plan_outputs(at, At, ta.narrow, ta.wide);
    ta.col_ptr_t = reinterpret_cast<int*>(at + At.col_ptr_off);
    ta.csc_row_t = reinterpret_cast<int*>(at + At.csc_row_off);
    ta.csc_blk_t = reinterpret_cast<int*>(at + At.csc_blk_off);
    if (max_row_blocks_t_out) landing = pinned_ints();
    if (landing) *landing = 0;
    ta.max_row_out = landing ? landing : ta.narrow.hdr + 1;
  }
  int rc;
  switch (b) {
    case 16: rc = launch_transpose<16>(ta, stream); break;
    case 32: rc = launch_transpose<32>(ta, stream); break;
    case 64: rc = launch_transpose<64>(ta, stream); break;
    default: rc = launch_transpose<128>(ta, stream); break;
  }
  if (rc) return rc;
  if (!ta.index_job) {  // more rows than one workgroup's schedule holds (or none)
    if (nbc > 0) {
      k_row_order<<<dim3((unsigned)((nbc + 255) / 256)), dim3(256), 0, stream>>>(row_ptr_t, nullptr, (int)nbc, row_order_t);
      BLAST_LAUNCH_CHECK("k_row_order(transpose)");
    }
    if (aux_t) {
      k_chunk_plan<<<dim3(1), dim3(1024), 0, stream>>>(row_ptr_t, row_order_t, (int)nbc, ta.narrow, ta.wide,
                                                       ta.max_row_out);
      BLAST_LAUNCH_CHECK("k_chunk_plan(transpose)");
    }
  }
  int heavy = 0;
  if (aux_t && max_row_blocks_t_out) {
    if (!landing)
      BLAST_HIP_TRY(hipMemcpyAsync(&heavy, ta.narrow.hdr + 1, sizeof(int), hipMemcpyDeviceToHost, stream));
    BLAST_HIP_TRY(hipStreamSynchronize(stream));
    if (landing) heavy = *static_cast<volatile int*>(landing);
  }
  if (max_row_blocks_t_out) *max_row_blocks_t_out = heavy;
  return BLAST_OK;
}

// ---- one mask update of blocked prune-and-grow (BLaST Sec. 3.2, generate_masks()) ----

extern "C" size_t blast_generate_masks_workspace(int64_t rows, int64_t cols, int32_t b) {
  if (check_shape(rows, cols, b) != BLAST_OK) return 0;
  const size_t n = (size_t)(rows / b) * (size_t)(cols / b);
  return 2 * blast::align_up(8 * (n > 0 ? n : 1), 256) + 2 * blast::align_up(n > 0 ? n : 1, 256);
}

extern "C" int blast_generate_masks(const uint16_t* W, int64_t ldw, const uint16_t* G, int64_t ldg, int64_t rows,
                                    int64_t cols, int32_t b, double sparsity, uint8_t* mask_out, void* ws,
                                    size_t ws_bytes, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (int rc = check_shape(rows, cols, b)) return rc;
  const int64_t nbc = cols / b, n = (rows / b) * nbc;
  const int64_t n_keep = blast_n_keep(n, sparsity);
  if (n_keep < 0) return BLAST_ERR_INVALID_ARG;
  if (n == 0) return BLAST_OK;
  if (!W || !G || !mask_out || ldw < cols || ldg < cols || ldw % 8 || ldg % 8 || !blast::aligned(W, 16) ||
      !blast::aligned(G, 16))
    return BLAST_ERR_INVALID_ARG;
  if (!ws || ws_bytes < blast_generate_masks_workspace(rows, cols, b) || !blast::aligned(ws, 16))
    return BLAST_ERR_WORKSPACE;
  char* wsb = static_cast<char*>(ws);
  double* scores = reinterpret_cast<double*>(wsb);
  double* scores_g = reinterpret_cast<double*>(wsb + blast::align_up(8 * (size_t)n, 256));
  uint8_t* mw = reinterpret_cast<uint8_t*>(wsb + 2 * blast::align_up(8 * (size_t)n, 256));
  uint8_t* mg = mw + blast::align_up((size_t)n, 256);
  const dim3 per_elem((unsigned)((n + 255) / 256));
  if (n_keep == 0 || n_keep == n) {  // nothing survives and nothing regrows, or everything is kept by W itself
    k_fill_u8<<<per_elem, dim3(256), 0, stream>>>(mask_out, n, n_keep == n ? 1 : 0);
    BLAST_LAUNCH_CHECK("k_fill_u8");
    return BLAST_OK;
  }
  if (int rc = launch_block_scores(b, W, ldw, nbc, n, scores, G, ldg, scores_g, stream)) return rc;
  if (n <= kSmallN) {  // both selections and the merge in one workgroup
    return launch_masks_small(scores, scores_g, n, n_keep, mask_out, stream);
  }
  if (int rc = launch_select(scores, scores_g, n, n_keep, mw, mg, stream)) return rc;
  k_merge_masks<<<per_elem, dim3(256), 0, stream>>>(mw, mg, n, mask_out);
  BLAST_LAUNCH_CHECK("k_merge_masks");
  return BLAST_OK;
}

// Eq. (2).  Past i = m - d the cube would turn negative and push s above s_max; the iteration is held
// inside [0, m - d].
extern "C" double blast_sparsity_schedule(int64_t i, int64_t m, int64_t d, double s_init, double s_max) {
  const int64_t span = m - d;
  if (span <= 0) return s_max;
  if (i < 0) i = 0;
  if (i > span) i = span;
  const double f = 1.0 - (double)i / (double)span;
  return s_max + (s_init - s_max) * f * f * f;
}

// ---- block selection from a sensitivity matrix (BLaST Sec. 3.3) ----

extern "C" size_t blast_pooled_topk_mask_workspace(int64_t rows, int64_t cols, int32_t b) {
  if (check_shape(rows, cols, b) != BLAST_OK) return 0;
  const size_t n = (size_t)(rows / b) * (size_t)(cols / b);
  return blast::align_up(8 * (n > 0 ? n : 1), 256);
}

extern "C" int blast_pooled_topk_mask(const float* S, int64_t lds, int64_t rows, int64_t cols, int32_t b,
                                      double sparsity, uint8_t* mask_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (int rc = check_shape(rows, cols, b)) return rc;
  const int64_t nbc = cols / b, n = (rows / b) * nbc;
  const int64_t n_keep = blast_n_keep(n, sparsity);
  if (n_keep < 0) return BLAST_ERR_INVALID_ARG;
  if (n == 0) return BLAST_OK;
  if (!S || !mask_out || lds < cols || lds % 4 || !blast::aligned(S, 16)) return BLAST_ERR_INVALID_ARG;
  if (!ws || ws_bytes < blast_pooled_topk_mask_workspace(rows, cols, b) || !blast::aligned(ws, 16))
    return BLAST_ERR_WORKSPACE;
  if (n_keep == 0 || n_keep == n) {
    k_fill_u8<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(mask_out, n, n_keep == n ? 1 : 0);
    BLAST_LAUNCH_CHECK("k_fill_u8");
    return BLAST_OK;
  }
  double* scores = static_cast<double*>(ws);
  k_pooled_scores<<<dim3((unsigned)n), dim3(256), 0, stream>>>(S, lds, (int)nbc, b, scores);
  BLAST_LAUNCH_CHECK("k_pooled_scores");
  return launch_select(scores, nullptr, n, n_keep, mask_out, nullptr, stream);
}

// The dense form of a packed matrix: W_new of prune_weights() (BLaST Sec. 3.2), zeros outside the stored blocks.
extern "C" int blast_bsr_unpack(const blast_bsr_view* Wp, uint16_t* W, int64_t ldw, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!Wp || !Wp->row_ptr || Wp->nnz < 0) return BLAST_ERR_INVALID_ARG;
  if (int rc = check_shape(Wp->rows, Wp->cols, Wp->b)) return rc;
  const int64_t nbr = Wp->rows / Wp->b, nbc = Wp->cols / Wp->b, n = nbr * nbc;
  if (n == 0) return BLAST_OK;
  if (!W || ldw < Wp->cols || ldw % 8 || !blast::aligned(W, 16)) return BLAST_ERR_INVALID_ARG;
  if (Wp->nnz > 0 && (!Wp->col_idx || !Wp->vals || !blast::aligned(Wp->vals, 16))) return BLAST_ERR_INVALID_ARG;
  k_unpack_blocks<<<dim3((unsigned)n), dim3(256), 0, stream>>>(Wp->row_ptr, Wp->col_idx, Wp->vals, (int)nbc, Wp->b, W, ldw);
  BLAST_LAUNCH_CHECK("k_unpack_blocks");
  return BLAST_OK;
}
