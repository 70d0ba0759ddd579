// The base field of BLS12-381 G1, F_q (381-bit q), for the MSM kernels, on
// fourteen signed limbs of 28 bits.
//
// In 32-bit limbs every partial product of a Montgomery product is two
// instructions: the multiply-add and the add of its carry into the column's
// counter (300 and 288 of them at twelve limbs).  With 28-bit limbs the 28
// products of a column fit a signed 64-bit accumulator with room for operands
// a few bits above 28, so there are no carry counts, sums and differences
// are fourteen independent 32-bit adds with no reduction, and two products
// can share one reduction.  A product is 392 multiply-adds (301 for a square)
// and about 80 shifts and masks.
//
// A value is sum_i v_i 2^(28 i), congruent to the element it stands for times
// 2^392 (Montgomery form).  Products are (a b - m q) / 2^392 with
// 0 <= m < 2^392, so for |a b| < 2^9 q^2 they lie in (-1.2 q, 0.2 q)
// (q = 2^380.7), and come out normalised: limbs 0 .. 12 in [0, 2^28), the
// sign in limb 13.  Operand limbs may reach 2^28 + 2^30 in one factor with the
// other normalised, or 2^29 in both: columns then stay below 2^62.8.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace zk {
namespace fq {

constexpr int kN = 14;       // limbs
constexpr int kBits = 28;
constexpr uint32_t kMask = (1u << kBits) - 1;
constexpr int kWords = 12;   // 32-bit words of a packed element

// q = (x0 - 1)^2 (x0^4 - x0^2 + 1) / 3 + x0, x0 = -0xd201000000010000.
struct Words {
  uint32_t v[kWords];
};
constexpr Words kQ = {{0xffffaaabu, 0xb9feffffu, 0xb153ffffu, 0x1eabfffeu, 0xf6b0f624u, 0x6730d2a0u, 0xf38512bfu,
                       0x64774b84u, 0x434bacd7u, 0x4b1ba7b6u, 0x397fe69au, 0x1a0111eau}};

constexpr Words pow2_mod_q(int e) {  // 2^e mod q
  Words x{};
  x.v[0] = 1;
  for (int s = 0; s < e; ++s) {
    uint32_t c = 0;
    for (int i = 0; i < kWords; ++i) {
      const uint32_t hi = x.v[i] >> 31;
      x.v[i] = (x.v[i] << 1) | c;
      c = hi;
    }
    bool ge = true;
    for (int i = kWords - 1; i >= 0; --i)
      if (x.v[i] != kQ.v[i]) {
        ge = x.v[i] > kQ.v[i];
        break;
      }
    if (!ge) continue;
    uint64_t br = 0;
    for (int i = 0; i < kWords; ++i) {
      const uint64_t d = (uint64_t)x.v[i] - kQ.v[i] - br;
      x.v[i] = (uint32_t)d;
      br = (d >> 32) & 1u;
    }
  }
  return x;
}

constexpr int32_t limb(const Words& w, int i) {
  uint32_t r = 0;
  for (int b = 0; b < kBits; ++b) {
    const int bit = kBits * i + b;
    if (bit < 32 * kWords) r |= ((w.v[bit / 32] >> (bit % 32)) & 1u) << b;
  }
  return (int32_t)r;
}

struct Limbs {
  int32_t v[kN];
};
constexpr Limbs limbs_of(const Words& w) {
  Limbs r{};
  for (int i = 0; i < kN; ++i) r.v[i] = limb(w, i);
  return r;
}

constexpr Limbs kQ28 = limbs_of(kQ);
constexpr uint32_t inv_mod_2_28(uint32_t a) {  // a^-1 mod 2^28, Newton
  uint32_t x = a;
  for (int i = 0; i < 5; ++i) x *= 2u - a * x;
  return x & kMask;
}
constexpr uint32_t kInv = inv_mod_2_28(kQ.v[0]);
constexpr Limbs kOne = limbs_of(pow2_mod_q(392));    // Montgomery form of 1
constexpr Limbs kTo392 = limbs_of(pow2_mod_q(400));  // times this: form 2^384 -> form 2^392
constexpr Limbs kTo384 = limbs_of(pow2_mod_q(384));  // times this: form 2^392 -> form 2^384

struct Fq {
  int32_t v[kN];
};

__device__ __forceinline__ Fq constant(const Limbs& c) {
  Fq r;
#pragma unroll
  for (int i = 0; i < kN; ++i) r.v[i] = c.v[i];
  return r;
}
__device__ __forceinline__ Fq zero() { return constant(Limbs{}); }
__device__ __forceinline__ Fq one() { return constant(kOne); }

// Hides how a's limbs were computed.  A limb whose sign extension or negation
// the compiler has already formed, in another block or as a 64-bit value,
// enters a product as a 64-bit operand: four instructions instead of one.
__device__ __forceinline__ Fq opaque(Fq a) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < kN; ++i) asm("" : "+v"(a.v[i]));
#endif
  return a;
}

// Limb by limb, no carries.
__device__ __forceinline__ Fq add(const Fq& a, const Fq& b) {
  Fq r;
#pragma unroll
  for (int i = 0; i < kN; ++i) r.v[i] = a.v[i] + b.v[i];
  return r;
}
__device__ __forceinline__ Fq sub(const Fq& a, const Fq& b) {
  Fq r;
#pragma unroll
  for (int i = 0; i < kN; ++i) r.v[i] = a.v[i] - b.v[i];
  return r;
}
__device__ __forceinline__ Fq neg(const Fq& a) {
  Fq r;
#pragma unroll
  for (int i = 0; i < kN; ++i) r.v[i] = -a.v[i];
  return opaque(r);
}
__device__ __forceinline__ Fq dbl(const Fq& a) { return add(a, a); }

// Limbs 0 .. 12 back to [0, 2^28).
__device__ __forceinline__ Fq normalise(const Fq& a) {
  Fq r;
  int32_t c = 0;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const int32_t x = a.v[i] + c;
    r.v[i] = i + 1 < kN ? (int32_t)((uint32_t)x & kMask) : x;
    c = x >> kBits;
  }
  return r;
}

// All limbs zero (the representation of 0 that infinity's ZZ keeps).
__device__ __forceinline__ bool all_zero(const Fq& a) {
  int32_t o = 0;
#pragma unroll
  for (int i = 0; i < kN; ++i) o |= a.v[i];
  return o == 0;
}

// a = 0 mod q, for |a| < 8 q.  The multiple k of q that a would be follows
// from its lowest 28 bits; anything but a k within 8 of 0 (all but one in
// 2^24 values) is ruled out by it, the rest is compared in full.
__device__ __forceinline__ bool is_zero(const Fq& a) {
  const uint32_t k = ((uint32_t)a.v[0] * kInv) & kMask;
  if (((k + 8u) & kMask) > 16u) return false;
  const int32_t ks = (int32_t)(k << (32 - kBits)) >> (32 - kBits);
  int64_t c = 0;
  int32_t o = 0;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    c += (int64_t)a.v[i] - (int64_t)ks * kQ28.v[i];
    o |= i + 1 < kN ? (int32_t)((uint32_t)c & kMask) : (int32_t)c;
    c >>= kBits;
  }
  return o == 0;
}

__device__ __forceinline__ int64_t mad(int32_t a, int32_t b, int64_t acc) { return acc + (int64_t)a * b; }

// (sum of products - m q) / 2^392, column by column; col(i, acc) adds column
// i of the products to the accumulator.
template <class Col>
__device__ __forceinline__ Fq reduce(Col col) {
  int32_t m[kN];
  Fq r;
  int64_t acc = 0;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    acc = col(i, acc);
#pragma unroll
    for (int j = 0; j < i; ++j) acc = mad(m[j], -kQ28.v[i - j], acc);
    m[i] = (int32_t)(((uint32_t)acc * kInv) & kMask);
    acc = mad(m[i], -kQ28.v[0], acc);
    acc >>= kBits;
  }
#pragma unroll
  for (int i = kN; i < 2 * kN - 1; ++i) {
    acc = col(i, acc);
#pragma unroll
    for (int j = i - (kN - 1); j < kN; ++j) acc = mad(m[j], -kQ28.v[i - j], acc);
    r.v[i - kN] = (int32_t)((uint32_t)acc & kMask);
    acc >>= kBits;
  }
  r.v[kN - 1] = (int32_t)acc;
  return r;
}

__device__ __forceinline__ int64_t column(const Fq& a, const Fq& b, int i, int64_t acc) {
#pragma unroll
  for (int j = 0; j < kN; ++j)
    if (j <= i && i - j < kN) acc = mad(a.v[j], b.v[i - j], acc);
  return acc;
}

__device__ __forceinline__ Fq mul(const Fq& a, const Fq& b) {
  return reduce([&](int i, int64_t acc) { return column(a, b, i, acc); });
}

// a b + c d with one reduction.
__device__ __forceinline__ Fq mul_add(const Fq& a, const Fq& b, const Fq& c, const Fq& d) {
  return reduce([&](int i, int64_t acc) { return column(c, d, i, column(a, b, i, acc)); });
}

__device__ __forceinline__ Fq sqr(const Fq& a) {
  const Fq t = opaque(dbl(a));
  return reduce([&](int i, int64_t acc) {
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      if (2 * j < i && i - j < kN) acc = mad(t.v[j], a.v[i - j], acc);
      if (2 * j == i) acc = mad(a.v[j], a.v[j], acc);
    }
    return acc;
  });
}

// a^-1 = a^(q-2) (Fermat), left-to-right square-and-multiply; a != 0.
__device__ __forceinline__ Fq inverse(const Fq& a) {
  // q - 2 differs from q only in the lowest word (q mod 2^32 >= 2)
  Fq r = one();
#pragma unroll 1
  for (int i = 32 * kWords - 1; i >= 0; --i) {
    r = sqr(r);
    const uint32_t e = (i < 32) ? kQ.v[0] - 2u : kQ.v[i / 32];
    if ((e >> (i % 32)) & 1u) r = mul(r, a);
  }
  return r;
}

// Twelve 32-bit words (a value in [0, 2^384)) to limbs and back.
__device__ __forceinline__ Fq unpack(const uint32_t (&w)[kWords]) {
  Fq r;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const int k = kBits * i / 32, s = kBits * i % 32;
    uint32_t x = w[k];
    if (s) x = k + 1 < kWords ? (uint32_t)((((uint64_t)w[k + 1] << 32) | x) >> s) : x >> s;
    r.v[i] = (int32_t)(x & kMask);
  }
  return r;
}
// The canonical value in [0, q) of a product's result.
__device__ __forceinline__ void pack_canonical(uint32_t (&w)[kWords], const Fq& a) {
  Fq x;  // a + 2 q, in (0.8 q, 2.2 q)
#pragma unroll
  for (int i = 0; i < kN; ++i) x.v[i] = a.v[i] + 2 * kQ28.v[i];
  x = normalise(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    Fq d;
#pragma unroll
    for (int i = 0; i < kN; ++i) d.v[i] = x.v[i] - kQ28.v[i];
    d = normalise(d);
    const bool ge = d.v[kN - 1] >= 0;
#pragma unroll
    for (int i = 0; i < kN; ++i) x.v[i] = ge ? d.v[i] : x.v[i];
  }
#pragma unroll
  for (int k = 0; k < kWords; ++k) {
    const int i = 32 * k / kBits, s = 32 * k % kBits;
    uint64_t t = (uint64_t)(uint32_t)x.v[i] >> s;
    t |= (uint64_t)(uint32_t)x.v[i + 1] << (kBits - s);
    if (i + 2 < kN) t |= (uint64_t)(uint32_t)x.v[i + 2] << (2 * kBits - s);
    w[k] = (uint32_t)t;
  }
}

}  // namespace fq
}  // namespace zk
