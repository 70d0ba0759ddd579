// Compile-time constants of the matrix-core DFT rounds (ntt_mfma_impl.hpp),
// derived from a field's modulus and generator.
//
// A radix-16 round multiplies a column of sixteen elements by the matrix
// w_16^(i j).  An element x is 32 digits of 8 bits, and multiplication by
// w_16^k is linear in them: digit b contributes x_b (w_16^k 2^(8 b) mod p),
// whose own 32 digits, taken in [-128, 127], are one column of a 32 x 32
// matrix of signed bytes.  Sixteen such matrices (k = 0 .. 15) serve every
// entry of the radix-16 DFT, and those with even k (multiples of four) the
// radix-8 (radix-4) ones.
#pragma once
#include <cstdint>

#include "field.hpp"

namespace zk {
namespace mfma {

struct U256 {
  uint32_t v[8];
};

constexpr bool geq(const U256& a, const uint32_t (&p)[kLimbs]) {
  for (int i = 7; i >= 0; --i)
    if (a.v[i] != p[i]) return a.v[i] > p[i];
  return true;
}

// 2 a mod p for a < p < 2^255.
template <class F>
constexpr U256 dbl_mod(const U256& a) {
  U256 r{};
  for (int i = 0; i < 8; ++i) r.v[i] = (a.v[i] << 1) | (i ? a.v[i - 1] >> 31 : 0u);
  if (geq(r, F::P)) {
    uint64_t br = 0;
    for (int i = 0; i < 8; ++i) {
      const uint64_t d = (uint64_t)r.v[i] - F::P[i] - br;
      r.v[i] = (uint32_t)d;
      br = (d >> 32) & 1u;
    }
  }
  return r;
}

template <class F>
constexpr U256 add_mod(const U256& a, const U256& b) {
  U256 r{};
  uint64_t c = 0;
  for (int i = 0; i < 8; ++i) {
    c += (uint64_t)a.v[i] + b.v[i];
    r.v[i] = (uint32_t)c;
    c >>= 32;
  }
  if (geq(r, F::P)) {
    uint64_t br = 0;
    for (int i = 0; i < 8; ++i) {
      const uint64_t d = (uint64_t)r.v[i] - F::P[i] - br;
      r.v[i] = (uint32_t)d;
      br = (d >> 32) & 1u;
    }
  }
  return r;
}

// a b 2^-256 mod p (CIOS), for the constants only.
template <class F>
constexpr U256 mont_mul(const U256& a, const U256& b) {
  uint32_t t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = 0; i < 8; ++i) {
    uint64_t x = (uint64_t)a.v[0] * b.v[i] + t[0];
    uint64_t A = x >> 32;
    const uint32_t m = (uint32_t)x * F::INV;
    uint64_t y = (uint64_t)m * F::P[0] + (uint32_t)x;
    uint64_t C = y >> 32;
    for (int j = 1; j < 8; ++j) {
      x = (uint64_t)a.v[j] * b.v[i] + t[j] + A;
      A = x >> 32;
      y = (uint64_t)m * F::P[j] + (uint32_t)x + C;
      C = y >> 32;
      t[j - 1] = (uint32_t)y;
    }
    t[7] = (uint32_t)(A + C);
  }
  U256 r{};
  for (int i = 0; i < 8; ++i) r.v[i] = t[i];
  if (geq(r, F::P)) {
    uint64_t br = 0;
    for (int i = 0; i < 8; ++i) {
      const uint64_t d = (uint64_t)r.v[i] - F::P[i] - br;
      r.v[i] = (uint32_t)d;
      br = (d >> 32) & 1u;
    }
  }
  return r;
}

constexpr U256 from_u32(uint32_t x) { return U256{{x, 0, 0, 0, 0, 0, 0, 0}}; }

template <class F>
constexpr U256 pow2_mod(int e) {  // 2^e mod p
  U256 r = from_u32(1);
  for (int i = 0; i < e; ++i) r = dbl_mod<F>(r);
  return r;
}

// w_16 = g^((p - 1) / 16), Montgomery form: equals w_n^(n / 16) for every n.
template <class F>
constexpr U256 root16_mont() {
  const U256 g = mont_mul<F>(from_u32(F::GENERATOR), pow2_mod<F>(512));
  U256 r = pow2_mod<F>(256);
  for (int bit = 255; bit >= 4; --bit) {  // (p - 1) >> 4 (p - 1 only clears bit 0)
    r = mont_mul<F>(r, r);
    if ((F::P[bit / 32] >> (bit % 32)) & 1u) r = mont_mul<F>(r, g);
  }
  return r;
}

// The 32 digits in [-128, 127] of a value below p, as bytes packed into words.
// No modulus here exceeds 0x7f7f...7f, so no carry leaves the last digit.
constexpr U256 balanced_digits(const U256& a) {
  U256 r{};
  uint32_t carry = 0;
  for (int i = 0; i < 32; ++i) {
    uint32_t d = ((a.v[i / 4] >> (8 * (i % 4))) & 255u) + carry;
    carry = d >= 128u ? 1u : 0u;
    r.v[i / 4] |= (d & 255u) << (8 * (i % 4));
  }
  return r;
}

// The matrices' A-operand fragments: frag[k][lane] holds, for the 32x32x32
// product, matrix row m = lane mod 32, digits b = 16 (lane / 32) + 0 .. 15 of
// the input.  The rows are ordered so that the four accumulators a lane gets
// for rows 8 g + 4 h + 0 .. 3 (h = lane / 32) are the byte columns of output
// limb g + 4 h: row 8 g + 4 h + q is output digit 4 (g + 4 h) + q.
struct DigitTable {
  uint32_t frag[16][64][4];
};

template <class F>
constexpr DigitTable make_digit_table() {
  DigitTable T{};
  const U256 w = root16_mont<F>();
  U256 wk = pow2_mod<F>(256);
  for (int k = 0; k < 16; ++k) {
    U256 x = mont_mul<F>(wk, from_u32(1));  // w_16^k, plain
    for (int b = 0; b < 32; ++b) {
      const U256 d = balanced_digits(x);
      for (int m = 0; m < 32; ++m) {
        const int c = 4 * (m / 8 + 4 * ((m / 4) & 1)) + (m & 3);
        const uint32_t byte = (d.v[c / 4] >> (8 * (c % 4))) & 255u;
        T.frag[k][m + 32 * (b / 16)][(b % 16) / 4] |= byte << (8 * (b % 4));
      }
      for (int s = 0; s < 8; ++s) x = dbl_mod<F>(x);
    }
    wk = mont_mul<F>(wk, w);
  }
  return T;
}

// The modulus in signed 32-bit digits: p = sum_l pb_l 2^(32 l).
struct Signed256 {
  int32_t v[8];
};
template <class F>
constexpr Signed256 signed_modulus() {
  Signed256 r{};
  uint32_t carry = 0;
  for (int l = 0; l < 8; ++l) {
    const uint64_t d = (uint64_t)F::P[l] + carry;
    r.v[l] = (int32_t)(uint32_t)d;
    carry = (d >> 31) ? 1u : 0u;  // digits of 2^31 and above become negative
  }
  return r;
}

// Data digits enter the product as byte - 128.  Over a radix-rho DFT the 128s
// add rho 128 sum_b 2^(8 b) to output 0 and nothing mod p to the others.
template <class F>
constexpr U256 bias_correction(int rho) {
  U256 ones{};
  for (int i = 0; i < 8; ++i) ones.v[i] = 0x01010101u;
  // 0x0101...01 < p for every field here
  U256 r = ones;
  for (int s = 1; s < 128 * rho; s *= 2) r = dbl_mod<F>(r);
  return r;
}

// 2^224 / p, to single precision.
template <class F>
constexpr float inv_top() {
  double t = 0.0;
  for (int i = 0; i < 8; ++i) {
    double x = (double)F::P[i];
    for (int k = i; k < 7; ++k) x *= 1.0 / 4294967296.0;
    t += x;
  }
  return (float)(1.0 / t);
}

}  // namespace mfma
}  // namespace zk
