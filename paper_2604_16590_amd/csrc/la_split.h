// la_split.h -- fp32 contractions on the bf16 matrix cores (internal).
//
// An fp32 value is the sum of three bf16 values, x = h + m + l (h = x rounded
// to bf16, m = x - h rounded, l = the rest, which is exact: 24 bits in all),
// so a product of two fp32 values is nine bf16 products; the three smallest
// (m l, l m, l l: at most 2^-26 of the whole) are left out and the other six
// are summed in FP32.  The bf16 matrix cores run at 16 times the fp32 ones'
// rate, so six products take 3/8 of the time, and 32 tokens or features are
// summed per accumulation instead of 4.
//
// The matrix cores align an instruction's products and its accumulator
// before they add, and drop the bits below the alignment towards minus
// infinity, so small products beside a large accumulator lose their low
// bits, all to one side (all six accumulated onto a running sum of 4,096
// tokens: S off by 2.7e-6).  The five small products are therefore summed
// from zero, smallest first, and join the running sum on the vector ALUs;
// the h h products are accumulated onto it.
//
// The split is exact for |x| in [2^-100, 2^127): below, l (and m) leave the
// bf16 range, above, h rounds to infinity, and an infinity's rest is NaN.
// Two values within it may still have a product h h = inf beside h m = -inf,
// so operands are held below 2^63: then no product and no sum of small
// products overflows.  Kernels test their operands (`SplitRange`) and take
// the fp32 matrix instructions for a step whose operands leave the range, so
// infinities and extreme scales give what they gave there.
#pragma once
#include "la_device.h"

namespace la {

// The three bf16 parts of a pair of fp32 values, packed.
struct Split2 {
  uint32_t h, m, l;
};
__device__ __forceinline__ Split2 split2(float a, float b) {
  Split2 s;
  s.h = pack_bf16(a, b);
  const float a1 = a - bf16lo(s.h), b1 = b - bf16hi(s.h);
  s.m = pack_bf16(a1, b1);
  s.l = pack_bf16(a1 - bf16lo(s.m), b1 - bf16hi(s.m));
  return s;
}

// Largest magnitudes of the values a lane has seen, in C classes; `bad` when
// some value is too large, or all of a class (not all zero) are too small for
// the split.  A small value beside a larger one of its class is split to less
// than 2^-27 of the larger, so a class holds only values that are summed into
// the same results: a column of a contraction's operand (its rows are what is
// summed over), or one token's run.  NaN passes: its parts are NaN.
template <int C = 1>
struct SplitRange {
  float mx[C] = {};
  __device__ __forceinline__ void see(int c, float a) { mx[c] = fmaxf(mx[c], fabsf(a)); }
  __device__ __forceinline__ void see(int c, float a, float b) {
    mx[c] = fmaxf(fmaxf(mx[c], fabsf(a)), fabsf(b));
  }
  __device__ __forceinline__ bool bad() const {
    float hi = mx[0], lo = mx[0];
#pragma unroll
    for (int c = 1; c < C; ++c) {
      hi = fmaxf(hi, mx[c]);
      lo = fminf(lo, mx[c]);
    }
    bool b = !(hi < 0x1p63f);
    if (lo < 0x1p-90f)  // a class of zeros, or a bad one
#pragma unroll
      for (int c = 0; c < C; ++c) b |= mx[c] > 0.f && mx[c] < 0x1p-90f;
    return b;
  }
};

// An operand in three bf16 parts; acc += A B over one 32-deep step.  One
// chain at a time: an accumulator passes from one product to the next
// without a stall (four chains in turn took 1.25 ms where one after the
// other took 0.97, on 8 heads of 524,288 tokens at d = 128).
struct Bf16x3 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ void mfma_split(const Bf16x3& a, const Bf16x3& b, f32x4& acc) {
  f32x4 t = mfma_bf16(a.h, b.l, f32x4{0.f, 0.f, 0.f, 0.f});
  t = mfma_bf16(a.l, b.h, t);
  t = mfma_bf16(a.m, b.m, t);
  t = mfma_bf16(a.h, b.m, t);
  t = mfma_bf16(a.m, b.h, t);
  acc = mfma_bf16(a.h, b.h, acc + t);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

// gfx950 transposing LDS read of 16-bit elements: within each 16-lane
// block, lane i receives as element k (k = 0..3) element i & 3 of the
// 8-byte chunk addressed by lane (i >> 2) + 4k of the block.  When lane L
// of a block addresses token row t0 + (L >> 2), features f0 + 4 (L & 3)
// .. + 3 of a row-major bf16 tile, lane i receives tokens t0 .. t0 + 3 of
// feature f0 + i: a token-major matrix-core operand straight from LDS.
__device__ __forceinline__ u32x2 lds_read_tr16(const void* p) {
  const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
  return __builtin_bit_cast(u32x2, r);
}

}  // namespace la
