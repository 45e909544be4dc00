// Device-side helpers shared by the product kernels.
#pragma once
#include <type_traits>

#include "blast_common.h"

namespace blast_dev {


typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct MatDev {
  const int* row_ptr;
  const int* col_idx;
  const uint16_t* vals;
  const uint8_t* vals8 = nullptr;  // E5M2 codes of the same blocks (kernels instantiated for one-byte weights)
};

struct TileArgs {
  MatDev m0, m1;         // m1 only for the dual (gate/up) kernel
  const int* row_order;  // may be null
  const uint16_t* X;
  int64_t sxt, sxk;      // element strides of X along tokens / features
  void* Y;
  int64_t syt, syi;      // element strides of Y along tokens / rows
  int y_bf16;
  int T;
  int nbr;               // block rows of the output
  int64_t kdim;          // features contracted over (columns of the matrix); host-side scheduling only
  int ntt;               // token tiles
  int act;               // gated product: the activation of the gate; single matrix: < 0 none, else applied to the output
  int x_vec;             // 1: 16-byte loads of X are legal (sxk == 1, aligned)
  int y_fast;            // 1: syi == 1 and every byte offset inside a 256-token slab of Y fits 31 bits
  int y_keep;            // E5M2 product with 128-wide blocks: 1: the output is written through the L2, else past the caches
  int y_pairs;           // 1: two neighbouring rows of a token may be stored as one value (Y and syt aligned to two values)
  int x_grp16;           // 16-wide blocks only: X is stored in column groups of 16 features, [kdim/16][T][16]
  int y_grp16;           // ... and so is Y, [rows/16][T][16]
};

// Index arrays are read-only for the lifetime of a launch: reading them through the
// constant address space lets uniform loads go through the scalar unit, so they never
// sit in the vector-memory counter that the DMA pipeline is tracked with.
__device__ __forceinline__ int ld_idx(const int* p, int i) {
  return reinterpret_cast<const __attribute__((address_space(4))) int*>(reinterpret_cast<uintptr_t>(p))[i];
}

// fp32 -> bf16, round to nearest even (the hardware conversion of gfx950).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  const __bf16 h = static_cast<__bf16>(f);
  return __builtin_bit_cast(uint16_t, h);
}

// Stores a value of 2, 4 or 8 bytes (naturally aligned) through the L2 of this XCD to the memory side.  An output that no
// later instruction of the launch reads gains nothing from staying in the L2, and what is dirty there when the launch
// ends is written back before the next one may start: the output of a short launch then leaves while it still computes.
template <class T>
__device__ __forceinline__ void store_through(T* p, T v) {
  using U = std::conditional_t<sizeof(T) == 2, uint16_t, std::conditional_t<sizeof(T) == 4, uint32_t, unsigned long long>>;
  static_assert(sizeof(T) == sizeof(U), "two, four or eight bytes");
  __hip_atomic_store(reinterpret_cast<U*>(p), __builtin_bit_cast(U, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// g * Phi(g), Phi the normal distribution function, from its tail: Phi(-t) = 2^(t R(t)) / 2 for t = |g|, R a polynomial
// fitted to (log2 Phi(-t) + 1) / t on [0, 6] so that t times the tail's error is below 2e-9 (least squares, reweighted to
// equal ripple); its leading coefficient is negative, so the tail goes on falling beyond 6 and is 0 at infinity.  More
// accurate than 0.5 g (1 + erf(g / sqrt 2)), which rounds a sum in between (root mean square error against 64 bits over
// normal g, that with erff / this: standard deviation 0.25 5.3e-9 / 4.2e-9, 1: 2.51e-8 / 1.75e-8, 5: 6.4e-8 / 4.8e-8), in 18
// instructions without a branch, where erff has 60 in two arms, the second beyond 1.4, 64 values a lane
// (two-matrix MLP of 1600 and 6400 features at 80 %, 333 tokens: 21.1 -> 20.2 us; over 32 calls of 1024 to 4096 features and 300
// to 4096 tokens on the streaming kernel 1 % less time on average.  Rows of one or two blocks under thousands of tokens, whose
// values hardly ever need the second arm and which multiply little, take up to 4 % more: 1024 and 4096 features at 90 %, 64-wide,
// 4096 tokens 28.9 / 30.0 us).
__device__ __forceinline__ float gelu(float g) {
  const float t = __builtin_fabsf(g);
  float r = -5.96657159e-8f;
  r = __builtin_fmaf(r, t, 1.44687544e-6f);
  r = __builtin_fmaf(r, t, -1.56093192e-5f);
  r = __builtin_fmaf(r, t, 9.60514999e-5f);
  r = __builtin_fmaf(r, t, -3.27383575e-4f);
  r = __builtin_fmaf(r, t, 6.75653209e-5f);
  r = __builtin_fmaf(r, t, 6.89349836e-3f);
  r = __builtin_fmaf(r, t, -5.24200164e-2f);
  r = __builtin_fmaf(r, t, -4.59224194e-1f);
  r = __builtin_fmaf(r, t, -1.15110409f);
  const float tail = 0.5f * __builtin_amdgcn_exp2f(t * r);
  // max(g, 0) - |g| tail, rounded once; infinity has no tail (a finite factor), minus infinity has no value (0 g)
  return __builtin_fmaf(-__builtin_fminf(t, 3.402823466e38f), tail, g > 0.0f ? g : 0.0f * g);
}

// Activation of the output of a single product in the kernels that end with many values a lane (streaming, shared tiles).
__device__ __forceinline__ float post_act(int act, float g) {
  if (act == BLAST_ACT_SILU) return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
  if (act == BLAST_ACT_GELU) return gelu(g);
  return g > 0.0f ? g : 0.0f;
}

// Activation of a gated product, and of a single one in the other kernels.  It has its GELU from erff: with the shorter one beside
// the SiLU of their usual calls the kernels are laid out otherwise, and these calls are slower (16384 x 53248 at 95 % Zipf,
// 128-wide, 2048 tokens: 720 / 724 us; 4096 x 14336, 128-wide, eight layers, at 90 % 27 tokens 179 / 183 us, at 95 % 13 tokens 96
// / 100; two-matrix MLP of 2048 and 8192 features at 70 %, 32-wide, SiLU, 1 token 13.7 / 14.4, 48 tokens 18.0 / 18.8; of 1024 and
// 4096 at 90 %, 16-wide, GELU, 4096 tokens 37.6 / 38.8).
__device__ __forceinline__ float apply_act(int act, float g) {
  if (act == BLAST_ACT_SILU) return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
  if (act == BLAST_ACT_GELU) return 0.5f * g * (1.0f + erff(g * 0.70710678118654752440f));
  return g > 0.0f ? g : 0.0f;
}

}  // namespace blast_dev
