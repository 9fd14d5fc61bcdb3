// fp32 products on the bf16 matrix unit.  An fp32 number of magnitude 2^-100 to 2^127 is the sum of three
// bf16 numbers, exactly: h its rounding, m the rounding of what is left, l the rest (24 significant bits in
// 8 + 8 + 8, each part within half a unit of the one before).  Of the nine products of two such sums six are
// formed (h h, h m, m h, m m, h l, l h); each of the three left out is at most about 2^-25 of the product,
// their sum 2^-24, and they change sign with the roundings.  One 32-deep step of six products takes the
// matrix unit 96 clocks where fp32 operands take 256, and unlike fp32 products they leave the vector ALU to
// a SIMD's other waves.
//
// Infinities have no such sum (their m is inf - inf), and a number within 2^-9 of the largest has an
// infinite h: both end as a NaN or an infinity in a product.  Below 2^-102 l may be a bf16 subnormal, below
// 2^-110 it may be none at all: up to 2^-126 of the number is lost.  That shows where the number is a value
// (of V, Y, or K and Q, whose averages alpha_L and alpha_R / c_R are), and in a logit where it meets a huge
// one: an operand of the first products need not be looked at if the other one is neither small nor huge.
// Every user looks at these (`Watch`) and, if it meets one, does the work again with fp32 operands.
#pragma once
#include "mrt_bf16_tiles.hpp"

namespace mrt {
namespace {

struct Split8 {
  bf16x8 h, m, l;
};
// two numbers' parts, packed (eleven instructions; left to the compiler, the conversions of a vector's
// elements and of their parts are not paired: twice as many)
struct Split2 {
  unsigned h, m, l;
};
__device__ inline unsigned pack2(float x, float y) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{x, y}, bf16x2));
}
__device__ inline Split2 split2(float x, float y) {
  Split2 s;
  s.h = pack2(x, y);
  x -= __uint_as_float(s.h << 16);
  y -= __uint_as_float(s.h & 0xffff0000u);
  s.m = pack2(x, y);
  x -= __uint_as_float(s.m << 16);
  y -= __uint_as_float(s.m & 0xffff0000u);
  s.l = pack2(x, y);
  return s;
}
__device__ inline Split8 split8(f32x4 a, f32x4 b) {
  const Split2 s[4] = {split2(a[0], a[1]), split2(a[2], a[3]), split2(b[0], b[1]), split2(b[2], b[3])};
  return Split8{as_bf16x8(uint4{s[0].h, s[1].h, s[2].h, s[3].h}), as_bf16x8(uint4{s[0].m, s[1].m, s[2].m, s[3].m}),
                as_bf16x8(uint4{s[0].l, s[1].l, s[2].l, s[3].l})};
}

// What makes a workgroup do its work again.  Was one of the numbers seen an infinity or a NaN?  Times zero,
// either is a NaN, which a sum keeps.  (The zero and the sum's bits are opaque: the library is built without
// honouring NaNs.)  Was an operand too small to be split?  The magnitudes' minimum costs half an instruction a
// number; only a wave that finds a zero or less than 2^-100 tells the two apart.  Was one huge?  (4680
// tokens, 12 heads, T = 2: 139 us without a look at the operands, 146 with one at every operand, 163 telling
// zeros apart at once, without a branch; as it is 142.)
enum { kSeeNone = 0, kSeeSmall = 1, kSeeHuge = 2 };
struct Watch {
  float zero = 0.f, sum = 0.f;
  float huge;                       // where what a small operand may have lost, 2^-126, is more than 2^-66 of a scaled logit
  bool odd = false;                 // a small or huge operand; the same in all lanes
  __device__ inline explicit Watch(float scale) : huge(0x1p60f / fmaxf(fabsf(scale), 1.f)) { asm("" : "+s"(zero)); }
  __device__ inline void see(f32x4 x) {
#pragma unroll
    for (int r = 0; r < 4; ++r) sum = fmaf(x[r], zero, sum);
  }
  // operands; called once they are split, so that the first do not wait for the last
  template <int SEE, int N>
  __device__ inline void see_split(const f32x4 (&v)[N]) {
    if constexpr (SEE != kSeeNone) {
      const float small = 0x1p-100f;
      float least = 1.f, most = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float x = fabsf(v[i][e]), y = fabsf(v[i][e + 1]);
          if constexpr ((SEE & kSeeSmall) != 0) least = fminf(fminf(x, y), least);
          if constexpr ((SEE & kSeeHuge) != 0) most = fmaxf(fmaxf(x, y), most);
        }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < small || most > huge) == 0, 1)) return;
      unsigned nonzero = ~0u;       // twice the least magnitude's bits, less one: zeros wrap to the largest
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned twice = (__float_as_uint(v[i][e]) << 1) - 1u;
          nonzero = twice < nonzero ? twice : nonzero;
        }
      if (__builtin_amdgcn_ballot_w64(((SEE & kSeeSmall) != 0 && nonzero < (__float_as_uint(small) << 1) - 1u) || most > huge) != 0)
        odd = true;
    }
  }
  __device__ inline bool unusual() const {
    unsigned bits = __float_as_uint(sum);
    asm("" : "+v"(bits));
    return odd || (bits & 0x7fffffffu) >= 0x7f800000u;
  }
};

// Softmax weights carry a factor 2^24 in products of split operands, from their exponentials to the division by
// their sum: down to the smallest fp32 number they then have all their parts (a weight's loss is below 2^-158 of
// the largest one's, where fp32 itself rounds it at 2^-150).
constexpr float kWeight = 0x1p24f;

// 2^24 e^x for x <= 0 or little above, to the last place or so: the hardware's 2^y, whose result is never subnormal, of
// x log2(e) rounded to multiples of 2^-14, and the part that the rounding left out.  0 where e^x rounds to 0.
__device__ inline float exp_near(float x) {
  const float L = 1.44269502f, tail = 1.92596299e-8f;        // log2(e) = L + tail
  const float at = fmaxf(x, -200.f);
  const float y = fmaf(at, L, 768.f);                        // 512 and above: multiples of 2^-14
  const float rest = fmaf(at, tail, fmaf(at, L, 768.f - y));
  const float e = exp2_fast(y - 744.f);
  return fmaf(e, rest * kLn2, e);
}

// LDS tile of ROWS rows as three planes: unpadded and swizzled at 128 features, padded at 64 (both
// operand reads conflict-free, see tile_off).
template <int D> constexpr bool kSwz32 = D == 128;
template <int D> constexpr int kLdS = D == 128 ? D : D + kPad;      // bf16 elements
template <int D> constexpr int kRowFloats = 3 * kLdS<D> / 2;        // LDS floats per row, all planes

// features 4 quad .. 4 quad + 3 of a row
template <int D, int ROWS>
__device__ inline void store_split(u16* tile, int row, int quad, f32x4 v) {
  const Split2 a = split2(v[0], v[1]), b = split2(v[2], v[3]);
  u16* at = tile + tile_off<kLdS<D>, kSwz32<D>>(row, quad >> 1) + 4 * (quad & 1);
  *(uint2*)at = uint2{a.h, b.h};
  *(uint2*)(at + ROWS * kLdS<D>) = uint2{a.m, b.m};
  *(uint2*)(at + 2 * ROWS * kLdS<D>) = uint2{a.l, b.l};
}

// first product, 16 rows of the tile from `row0` (a multiple of 16) on the accumulator rows against
// the wave's operand q; NT such tiles at once.  The small products have sums of their own.
template <int D, int ROWS, int NT>
__device__ inline void logits_split(const u16* tile, const Split8 (&q)[D / 32], f32x4* s, int g, int c) {
  f32x4 hi[NT], lo[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) hi[t] = lo[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    bf16x8 a[NT][3];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int plane = 0; plane < 3; ++plane)
        a[t][plane] = ld_lds_16B(tile + plane * ROWS * kLdS<D> + tile_off<kLdS<D>, kSwz32<D>>(16 * t + c, 4 * ks + g));
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      lo[t] = mfma(a[t][2], q[ks].h, lo[t]);
      hi[t] = mfma(a[t][0], q[ks].h, hi[t]);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) lo[t] = mfma(a[t][0], q[ks].l, lo[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) lo[t] = mfma(a[t][1], q[ks].m, lo[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) lo[t] = mfma(a[t][1], q[ks].h, lo[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) lo[t] = mfma(a[t][0], q[ks].m, lo[t]);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) s[t] = hi[t] + lo[t];
}

// second product, one step of 32 rows: o[vt] += Val^T p; features as in pv_step
template <int D, int ROWS>
__device__ inline void pv_split(const u16* rows, const Split8& p, f32x4 (&o)[D / 16], int lane) {
  const int g = lane >> 4, s = lane & 15, e = s >> 2, q = s & 3;
#pragma unroll
  for (int vt = 0; vt < D / 16; vt += 2) {
    bf16x8 a[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const u16* p0 = rows + tile_off<kLdS<D>, kSwz32<D>>(4 * g + e, q + 2 * vt) + 4 * i;
#pragma unroll
      for (int plane = 0; plane < 3; ++plane) {
        const u16* at = p0 + plane * ROWS * kLdS<D>;
        a[i][plane] = __builtin_bit_cast(
            bf16x8, __builtin_shufflevector(ld_lds_tr(at), ld_lds_tr(at + 16 * kLdS<D>), 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][2], p.h, o[vt + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][0], p.l, o[vt + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][1], p.m, o[vt + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][1], p.h, o[vt + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][0], p.m, o[vt + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) o[vt + i] = mfma(a[i][0], p.h, o[vt + i]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace
}  // namespace mrt
