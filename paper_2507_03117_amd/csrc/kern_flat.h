// Decode kernel for large layers with one-byte (E5M2) weights: the stored blocks of many short rows as one stream.
//
// k_decode gives every (block row, 16-row slice) a workgroup of its own.  On a large, unevenly filled layer that is
// thousands of workgroups most of which hold one to three blocks for four waves: each pays the chain of index loads,
// one trip to the memory, a reduction and a store, hardly a wave ever has a second block in flight, and the fullest
// row is a quarter of its length in sequence.  Here one workgroup of sixteen waves per CU takes a list of block rows
// (one 16-row slice of them) and treats their blocks as one stream:
//  - the rows are dealt to the workgroups by work: ranks of the schedule to the 8 XCDs in octets, every other octet
//    mirrored, the slices of a row all on one XCD (its L2 then serves the activation tile of a block to all of them);
//    inside an XCD the longest rows one by one to the group with the least work, the short rest in one cut of its
//    prefix sum that levels the groups;
//  - the stream is cut into sixteen equal pieces, one per wave, wherever the cuts fall; a wave copies the slices and
//    activation tiles of its piece global -> LDS through a ring of its own, across rows and matrices, and no wave
//    waits for another until the end;
//  - the sums of a row (of one matrix) that a wave starts are left in an LDS entry of that row, the first sums of a
//    piece that begins inside a row in an entry of the wave; after one barrier the entries of a row are added in the
//    order of the stream, activated and stored: the sums of a row do not depend on timing.  (With CHUNK a row is what the
//    chunk plan made of one, and the chunks of a cut row meet through fp32 atomics.)
// What bounds it (one-byte weights, 16384 x 53248 layer with Zipf rows, 5 tokens, timestamps of every workgroup): the
// stream runs at 4.3 TB/s of weights, 13 us of the gate/up launch; 6 us pass before it starts (two trips for the rows,
// the deal, a trip for the columns), and the workgroup that holds the fullest row (256 blocks of 163 on average) ends
// 6 us after the others.  Layer: 58 -> 43 us (another mask: 67 -> 45), of which the rows of the chunked down product
// being cleared by the gate/up launch is 5.  Eight waves with four-slot rings instead of sixteen with two: 54 us (the
// fullest row is an eighth of its length in sequence); every wave dealing the rows for itself: 50 (the waves of a SIMD
// share its scalar unit).
#pragma once
#include "kern_decode.h"

namespace blast_dev {

// XI: copy instructions per activation tile, i.e. XI * 512 / B token rows.
template <int B, bool DUAL, int XI>
struct FlatCfg {
  using D = DecCfg<B, DUAL, 1, XI, false, true>;
  static constexpr int NW = 16;
  static constexpr int SLICES = B / 16;
  static constexpr int MAX_SLOTS = 32 / SLICES;  // row groups per XCD of 32 CUs
  static constexpr int XR = D::XR;
  static constexpr int NM = DUAL ? 2 : 1;
  static constexpr int PM = 512;                 // stored blocks of the rows taken at a time, at most
  static constexpr int ACC_LDS = 52 * XR * 64;   // entries of 16 rows x T tokens: 18 rows and 16 waves at T = 8 (DUAL)
  static constexpr int TAB_LDS = (6 * 64 + 2 * PM + NW + 8) * 4;  // the group's rows, the blocks of a batch, head_seg
  static constexpr int FIT = (160 * 1024 - ACC_LDS - TAB_LDS) / (NW * D::SLOT);
  static constexpr int NSLOT = FIT > 4 ? 4 : FIT;
  static constexpr int OPS = D::NI + D::NIX;
  static constexpr int WAVE_LDS = NSLOT * D::SLOT;
  static constexpr size_t LDS_BYTES = (size_t)NW * WAVE_LDS + ACC_LDS + TAB_LDS;
  static_assert(NSLOT >= 2 && (NSLOT - 1) * OPS < 64, "a block in flight beside the one being multiplied");
};

template <int B, bool DUAL, bool CHUNK, int XI>
__global__ __launch_bounds__(1024) void k_decode_flat(const DecArgs a) {
  static_assert(!(DUAL && CHUNK), "the activation needs complete sums: the gated product is never split");
  using C = FlatCfg<B, DUAL, XI>;
  using D = typename C::D;
  constexpr int KST = D::KST, NI = D::NI, NIX = D::NIX, NSLOT = C::NSLOT, NM = C::NM, NW = C::NW;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int G = gridDim.x, w = blockIdx.x;
  const int x = w & 7, j = w >> 3, q = j % C::SLICES, slot = j / C::SLICES, nslot = (G >> 3) / C::SLICES;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  unsigned char* ring = smem + wave * C::WAVE_LDS;
  // fp32 sums, [T tokens][16 rows] each: first sums of the waves [NW], then the sums of the rows taken at a time [NM * RM]
  float* const heads = reinterpret_cast<float*>(smem + NW * C::WAVE_LDS);
  const int entry = a.T * 16;
  float* const entries = heads + NW * entry;
  const int room = (C::ACC_LDS / 4 / entry - NW) / NM, RM = room < 64 ? room : 64;
  int* const head_seg = reinterpret_cast<int*>(smem + NW * C::WAVE_LDS + C::ACC_LDS);  // [NW] which (row, matrix) the latter belong to
  int* const n_rows_at = head_seg + NW;
  int* const t_row = n_rows_at + 8;  // the group's rows: block row, first block and number of blocks per matrix,
  int* const t_k0 = t_row + 64;      // position of the first block in the stream
  int* const t_n0 = t_k0 + 64;
  int* const t_k1 = t_n0 + 64;
  int* const t_n1 = t_k1 + 64;
  int* const t_pos = t_n1 + 64;
  int* const b_blk = t_pos + 64;     // [PM] the stream of a batch: block,
  int* const b_col = b_blk + C::PM;  // [PM] its column and, from bit 24 on, which (row of the batch, matrix) it is

  // ---- the first wave deals the rows of this XCD: every workgroup of the XCD arrives at the same answer ----------
  // (one wave, not all of them at once: they would share the four scalar units)
  if (wave == 0) {
    const int n_items = CHUNK ? ld_idx(a.hdr, 0) : a.n_units;
    const int rank = (lane << 3) + ((lane & 1) ? 7 - x : x);
    const bool have = rank < n_items;  // one row per lane (the host takes this kernel for at most 512 rows)
    int row = 0, k0 = 0, n0 = 0, k1 = 0, n1 = 0;
    if (have) {
      if (CHUNK) {
        row = a.chunk_row[rank];
        k0 = a.chunk_kb[rank];
        n0 = a.chunk_ke[rank] - k0;
      } else {
        row = a.row_order ? a.row_order[rank] : rank;
        k0 = a.m0.row_ptr[row];
        n0 = a.m0.row_ptr[row + 1] - k0;
        if (DUAL) {
          k1 = a.m1.row_ptr[row];
          n1 = a.m1.row_ptr[row + 1] - k1;
        }
      }
    }
    constexpr int kGreedy = 16;  // rows dealt one by one; the later ones are short
    unsigned long long mine = 0ull;
    const int len = have ? n0 + n1 + 1 : 0;
    const int nrx = __builtin_popcountll(__ballot(have));
    int load[C::MAX_SLOTS];
#pragma unroll
    for (int s = 0; s < C::MAX_SLOTS; ++s) load[s] = s < nslot ? 0 : 0x3FFFFFFF;
    const int ng = nrx < kGreedy ? nrx : kGreedy;
    for (int k = 0; k < ng; ++k) {
      const int l = BLAST_LANE(len, k);
      int best = 0, bl = load[0];
#pragma unroll
      for (int s = 1; s < C::MAX_SLOTS; ++s) {
        const bool less = load[s] < bl;
        best = less ? s : best;
        bl = less ? load[s] : bl;
      }
#pragma unroll
      for (int s = 0; s < C::MAX_SLOTS; ++s) load[s] += s == best ? l : 0;
      if (best == slot) mine |= 1ull << k;
    }
    const int rest = lane >= ng ? len : 0;
    const int incl = blast::lanes_scan(rest);
    const int total = BLAST_LANE(incl, 63);
    if (total > 0) {
      // the rest, of `total` work, is cut where it levels the groups: group s is given what it lacks to `level`
      int level = total;
#pragma unroll
      for (int s = 0; s < C::MAX_SLOTS; ++s) level += s < nslot ? load[s] : 0;
      level = (level + nslot - 1) / nslot;
      int lack_sum = 0, from = 0, to = 0;
#pragma unroll
      for (int s = 0; s < C::MAX_SLOTS; ++s) {
        const int lack = s < nslot && load[s] < level ? level - load[s] : 0;
        if (s == slot) from = lack_sum;
        lack_sum += lack;
        if (s == slot) to = lack_sum;
      }
      // (groups above the level make the lacks add up to more than there is: scaled down to it)
      const float f = (float)total / (float)lack_sum;
      const int lo = (int)((float)from * f + 0.5f);
      const int hi = slot == nslot - 1 ? total : (int)((float)to * f + 0.5f);
      const int begin = incl - rest;  // a row belongs to the group its beginning falls to
      mine |= __ballot(rest > 0 && begin >= lo && begin < hi);
    }
    const bool own = (mine >> lane) & 1ull;
    const int blocks = own ? n0 + n1 : 0;
    const int pos = blast::lanes_scan(blocks) - blocks;
    if (own) {
      const int i = __builtin_popcountll(mine & ((1ull << lane) - 1ull));
      t_row[i] = row;
      t_k0[i] = k0;
      t_n0[i] = n0;
      t_k1[i] = k1;
      t_n1[i] = n1;
      t_pos[i] = pos;
    }
    if (lane == 0) *n_rows_at = __builtin_popcountll(mine);
  } else if (DUAL && wave == NW - 1 && a.z_blocks > 0) {
    // the side job (see DecArgs), dealt to the last waves while the first ones deal rows; a workgroup that is dealt no
    // row has its share of it all the same
    for (int ci = w; ci < a.z_blocks; ci += G) decode_zero_job<B, 64>(a, ci);
  }

  // ---- per-lane constants of the copies and fragments, as in decode_unit --------------------------------------
  uint32_t woff[NI], xoff[NIX], foff[KST], fxoff[KST];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const int p = ni * 64 + lane;
    const int r = p / D::CPRW8, s = p % D::CPRW8;
    woff[ni] = (uint32_t)(q * D::SLW + r * B + ((s ^ D::key8(r)) << 4));
  }
#pragma unroll
  for (int xi = 0; xi < NIX; ++xi) {
    const int p = xi * 64 + lane, r = p / D::CPRW, s = p % D::CPRW;
    const int t = r < a.T ? r : a.T - 1;
    xoff[xi] = (uint32_t)t * (uint32_t)a.sxt * 2u + (uint32_t)((s ^ D::key(r)) << 4);
  }
  const int xrow = l16 % C::XR;
#pragma unroll
  for (int s = 0; s < KST; ++s) {
    foff[s] = (uint32_t)(l16 * B + (((2 * s + (g >> 1)) ^ D::key8(l16)) << 4) + ((g & 1) << 3));
    fxoff[s] = (uint32_t)(xrow * (B * 2) + (((4 * s + g) ^ D::key(xrow)) << 4));
  }

  __syncthreads();  // the table is there
  const int n_rows = __builtin_amdgcn_readfirstlane(*n_rows_at);

  // ---- a batch of rows at a time (almost always there is one batch) ------------------------------------------------
  int nr;
#pragma unroll 1
  for (int r0 = 0; r0 < n_rows; r0 += nr) {
    nr = n_rows - r0 < RM ? n_rows - r0 : RM;
    const int base = __builtin_amdgcn_readfirstlane(t_pos[r0]);
    int n;  // blocks of the batch
    for (;; --nr) {  // (the host takes this kernel only where a row has at most PM blocks)
      const int last = r0 + nr - 1;
      n = __builtin_amdgcn_readfirstlane(t_pos[last] + t_n0[last] + t_n1[last]) - base;
      if (n <= C::PM || nr == 1) break;
    }
    // clear the entries (a matrix without blocks in a row leaves its entry alone)
    for (int e = threadIdx.x; e < NM * nr * entry; e += 64 * NW) entries[e] = 0.0f;
    if (threadIdx.x < NW) head_seg[threadIdx.x] = -1;
    // the stream of the batch: a wave writes the blocks of its rows, the columns of 256 of them in one trip
    for (int i = wave; i < nr; i += NW) {
      const int k0 = t_k0[r0 + i], n0 = t_n0[r0 + i], k1 = t_k1[r0 + i], n01 = n0 + t_n1[r0 + i], at = t_pos[r0 + i] - base;
      for (int o0 = lane; o0 < n01; o0 += 256) {
        int k[4], c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int o = o0 + 64 * u;
          k[u] = DUAL && o >= n0 ? k1 + o - n0 : k0 + o;
          c[u] = 0;
          if (o < n01) c[u] = (DUAL && o >= n0 ? a.m1 : a.m0).col_idx[k[u]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int o = o0 + 64 * u;
          if (o < n01) {
            b_blk[at + o] = k[u];
            b_col[at + o] = c[u] | (i * NM + (DUAL && o >= n0 ? 1 : 0)) << 24;
          }
        }
      }
    }
    __syncthreads();
    // this wave's piece, a block per lane
    const int p_lo = n * wave / NW, cnt = n * (wave + 1) / NW - p_lo;
    int vk = 0, vc = 0, vs = -1;
    if (lane < cnt) {
      vk = b_blk[p_lo + lane];
      vc = b_col[p_lo + lane];
      vs = vc >> 24;
      vc &= 0xFFFFFF;
    }
    auto issue = [&](int b) {
      const int k = BLAST_LANE(vk, b), c = BLAST_LANE(vc, b);
      const MatDev& m = (DUAL && (BLAST_LANE(vs, b) & 1)) ? a.m1 : a.m0;
      const unsigned char* wblk = m.vals8 + (int64_t)k * (B * B);
      const unsigned char* xcol = reinterpret_cast<const unsigned char*>(a.X) + (int64_t)c * (B * 2);
      unsigned char* dst = ring + (b % NSLOT) * D::SLOT;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) BLAST_GLDS16(wblk + woff[ni], dst + ni * 1024);
#pragma unroll
      for (int xi = 0; xi < NIX; ++xi) BLAST_GLDS16(xcol + xoff[xi], dst + D::SLW + xi * 1024);
    };
#pragma unroll 1
    for (int b = 0; b < NSLOT - 1; ++b)
      if (b < cnt) issue(b);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // (row, matrix) of the block being multiplied; the first one of the piece may have begun in an earlier piece
    int seg = cnt > 0 ? BLAST_LANE(vs, 0) : -1;
    bool head = false;
    if (cnt > 0 && p_lo > 0) head = __builtin_amdgcn_readfirstlane(b_col[p_lo - 1] >> 24) == seg;
#pragma unroll 1
    for (int b = 0; b < cnt; ++b) {
      const int next_seg = b + 1 < cnt ? BLAST_LANE(vs, b + 1) : -1;
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the fragments of the slot that is refilled have been read
      asm volatile("" ::: "memory");
      if (b + NSLOT - 1 < cnt) issue(b + NSLOT - 1);
      const int later = (cnt - 1 - b) < (NSLOT - 1) ? (cnt - 1 - b) : (NSLOT - 1);
      if (later >= 3)
        __builtin_amdgcn_s_waitcnt(BLAST_VMCNT(3 * C::OPS));
      else if (later == 2)
        __builtin_amdgcn_s_waitcnt(BLAST_VMCNT(2 * C::OPS));
      else if (later == 1)
        __builtin_amdgcn_s_waitcnt(BLAST_VMCNT(C::OPS));
      else
        __builtin_amdgcn_s_waitcnt(BLAST_VMCNT(0));
      asm volatile("" ::: "memory");
      const unsigned char* st = ring + (b % NSLOT) * D::SLOT;
      // every fragment of the block is on its way before the first is widened
      uint2 wc[KST];
      bf16x8 xf[KST];
#pragma unroll
      for (int s = 0; s < KST; ++s) {
        wc[s] = *reinterpret_cast<const uint2*>(st + foff[s]);
        xf[s] = *reinterpret_cast<const bf16x8*>(st + D::SLW + fxoff[s]);
      }
#pragma unroll
      for (int s = 0; s < KST; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[s], e5m2x8_to_bf16x8(wc[s]), acc, 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * KST, 0);
      asm volatile("" ::: "memory");
      if (next_seg != seg) {
        float* const e = head ? heads + wave * entry : entries + seg * entry;
        if (head && lane == 0) head_seg[wave] = seg;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (4 * g + t < a.T) e[(4 * g + t) * 16 + l16] = acc[t];
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
        seg = next_seg;
        head = false;
      }
    }
    __syncthreads();

    // ---- a row's sums in the order of the stream; result layout: lane -> row l16, register t -> token 4 * g + t ----
    const int hs = lane < NW ? head_seg[lane] : -1;
#pragma unroll 1
    for (int i = wave; i < nr; i += NW) {
      const int rr = __builtin_amdgcn_readfirstlane(t_row[r0 + i]);
      // the waves whose first sums belong to this row, per matrix
      unsigned long long more[NM];
#pragma unroll
      for (int m = 0; m < NM; ++m) more[m] = __ballot(hs == i * NM + m);
      const int64_t orow = (int64_t)(CHUNK ? rr & 0x7FFFFFFF : rr) * B + q * 16 + l16;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int tok = 4 * g + t;
        if (tok < a.T) {
          float v[NM];
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            v[m] = entries[(i * NM + m) * entry + tok * 16 + l16];
            for (unsigned long long hb = more[m]; hb; hb &= hb - 1)
              v[m] += heads[__builtin_ctzll(hb) * entry + tok * 16 + l16];
          }
          float y = v[0];
          if (DUAL) y = apply_act(a.act, y) * v[NM - 1];
          const int64_t off = (int64_t)tok * a.syt + orow * a.syi;
          if (CHUNK && rr < 0)
            atomicAdd(reinterpret_cast<float*>(a.Y) + off, y);  // fp32 output, zeroed before the launch
          else if (a.y_bf16)
            reinterpret_cast<uint16_t*>(a.Y)[off] = f32_to_bf16_rne(y);
          else
            reinterpret_cast<float*>(a.Y)[off] = y;
        }
      }
    }
    if (r0 + nr < n_rows) __syncthreads();  // the entries are cleared for the next batch
  }
}

}  // namespace blast_dev
