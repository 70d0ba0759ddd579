// NTT pass kernels whose DFT rounds run on the matrix cores (gfx950).
//
// A pass (PassArgs, ntt_kernels.hpp) is one radix-R Stockham pass over tiles
// of J columns x R points, as in ntt_pass_impl.hpp.  Here the R-point DFT is
// two or three rounds of radix 16, 8 or 4, each one product with a constant
// matrix: with the data in 8-bit digits and w_16^k as 32 x 32 matrices of
// signed bytes (mfma_tables.hpp), output i of a column is
//   sum_j M_(ij mod 16) x_j,
// 32 byte columns of at most 23 bits, accumulated in 32-bit integers by
// v_mfma_i32_32x32x32_i8.  What is left for the vector units per element and
// round is to add up the byte columns to a 256-bit integer (carries and one
// small multiple of p, combine()), and one Montgomery product by the twiddle
// between rounds, where radix-4 butterflies in 32-bit limbs need a product
// and a half per element and round more.
//
// Phases of a tile (one workgroup), all through LDS:
//   load     global -> product by the inter-pass twiddle -> digits
//   round q  digits -> MFMA -> combine -> limbs, in place
//   twiddle  limbs -> product by w_R^(i low) -> digits   (between rounds)
//   store    limbs -> last pass's factors -> global
// Digits are bytes offset by 128 (one XOR), see bias_correction.
#pragma once
#include "mfma_tables.hpp"
#include "ntt_pass_impl.hpp"

namespace zk {
namespace mfma {

// Compile-time loop, as detail::sfor; the body is inlined at any size.  Left
// to its estimate, the compiler keeps the larger bodies of kernels that share
// them as functions, and the arrays they capture go to scratch (336 bytes per
// lane at radix 2^8; quotient chain 2^24 16.7 ms against 11.8).
template <class Fn, int... I>
__device__ __forceinline__ void sfor_impl(Fn& fn, std::integer_sequence<int, I...>) {
  [[clang::always_inline]] (fn(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void sfor(Fn&& fn) {
  sfor_impl(fn, std::make_integer_sequence<int, N>{});
}


typedef int V4i __attribute__((ext_vector_type(4)));
typedef int V16i __attribute__((ext_vector_type(16)));
using detail::load_fe;
using detail::mul_many;
using detail::store_fe;
using detail::U32x4;

// The rounds of a radix-2^LOG_R pass, most significant digit first.  A round
// of radix rho takes its columns 32 at a time, so a tile of 2^LOG_TILE
// elements needs 2^LOG_TILE / rho >= 32.
template <int LOG_R, int LOG_TILE>
struct Rounds {
  static constexpr int N = LOG_R <= 4 ? 1 : LOG_R <= 8 && LOG_TILE > 8 ? 2 : LOG_R <= 6 ? 2 : 3;
  static constexpr int log(int q) {
    if (N == 1) return LOG_R;
    if (N == 2) return q == 0 ? (LOG_R + 1) / 2 : LOG_R / 2;
    return q == 0 ? (LOG_R + 2) / 3 : q == 1 ? (LOG_R + 1) / 3 : LOG_R / 3;
  }
  static constexpr int low(int q) {  // log2 stride of digit q: the later radices
    int s = 0;
    for (int k = q + 1; k < N; ++k) s += log(k);
    return s;
  }
  static constexpr int high(int q) {  // log2 product of the earlier radices
    int s = 0;
    for (int k = 0; k < q; ++k) s += log(k);
    return s;
  }
};

template <int LOG_R, int LOG_TILE, int LOG_THREADS>
struct Shape {
  using Rd = Rounds<LOG_R, LOG_TILE>;
  static constexpr int R = 1 << LOG_R;
  static constexpr int LOG_J = LOG_TILE - LOG_R;
  static constexpr int J = 1 << LOG_J;
  static constexpr int E = 1 << LOG_TILE;
  static constexpr int THREADS = 1 << LOG_THREADS;
  static constexpr int WAVES = THREADS / 64;
  static constexpr int U = E / THREADS;  // elements per lane
  // Threads holding two or more elements take the first radix-2 stage of each
  // round as they form the digits: half the matrix products for a 16-limb
  // addition and subtraction per pair.  Threads holding one element (small
  // transforms, where latency counts) leave the whole round to the matrices.
  static constexpr bool HALF = U >= 2;
  static constexpr int LDS_DATA = 2 * E;   // 16-byte halves
  static constexpr int LDS_A = 16 * 64;    // the matrices
  static constexpr int LDS_WGS = 163840 / (16 * (LDS_DATA + LDS_A));
  static constexpr int WAVES_SIMD = LDS_WGS * THREADS / 256;
  static constexpr int MIN_WAVES = WAVES_SIMD < 1 ? 1 : WAVES_SIMD > 4 ? 4 : WAVES_SIMD;
};

// 16-byte slot of half h of element e: within each 256-byte row the halves
// are permuted by the row, so that 16 lanes reading one half of elements in
// the same column of different rows (a round's operands, or a transposed
// store) touch different banks.
__device__ __forceinline__ uint32_t slot16(uint32_t e, uint32_t h) {
  const uint32_t row = e >> 3;
  return (row << 4) | ((((e & 7u) << 1) | h) ^ ((row ^ (row >> 4)) & 15u));
}

// The slot of element e0 + (d << S) from that of e0, where e0 has zeros in
// d's bits: one XOR and an offset, constants when d is one.
template <int S>
constexpr __host__ __device__ uint32_t slot_xor(uint32_t d) {
  const uint32_t x = d << S, row = x >> 3;
  return (((x & 7u) << 1) ^ row ^ (row >> 4)) & 15u;
}
template <int S>
__device__ __forceinline__ uint32_t slot_at(uint32_t slot0, uint32_t d) {
  return (slot0 ^ slot_xor<S>(d)) + (((d << S) >> 3) << 4);
}

__device__ __forceinline__ Fe lds_load(const U32x4* lds, uint32_t s) {
  const U32x4 lo = lds[s], hi = lds[s ^ 1u];
  Fe r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r.v[k] = lo[k];
    r.v[4 + k] = hi[k];
  }
  return r;
}

__device__ __forceinline__ void lds_store(U32x4* lds, uint32_t s, const Fe& x, uint32_t flip) {
  U32x4 lo, hi;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    lo[k] = x.v[k] ^ flip;
    hi[k] = x.v[4 + k] ^ flip;
  }
  lds[s] = lo;
  lds[s ^ 1u] = hi;
}

constexpr uint32_t kFlip = 0x80808080u;  // byte -> digit byte - 128

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ int64_t mad_i64(int32_t a, int32_t b, int64_t c) {
  int64_t r;
  uint64_t unused;
  asm("v_mad_i64_i32 %0, %1, %2, %3, %4" : "=v"(r), "=s"(unused) : "v"(a), "s"(b), "v"(c));
  return r;
}
__device__ __forceinline__ V16i mfma(V4i a, V4i b, V16i c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ void swap_halves(int& x, int& y) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  x = (int)r[0];
  y = (int)r[1];
}
#else
inline __device__ int64_t mad_i64(int32_t a, int32_t b, int64_t c) { return (int64_t)a * b + c; }
inline __device__ V16i mfma(V4i, V4i, V16i c) { return c; }
inline __device__ void swap_halves(int&, int&) {}
#endif

// The element with byte-pair columns u_l + 2^16 v_l at limb l (each below
// 2^30.1 in magnitude: a radix-16 column is at most 2^7 times the digit sum of
// a matrix row, below 2^22.01, and 2^22.01 (1 + 2^8) < 2^30.1; checked against
// the tables by the tests), reduced to [0, 1.3 p) below 2^256.  The multiple
// of p comes from the top limb's columns in single precision: they carry the
// quotient (at most 2^18.1 in magnitude) to within 2^-5, and rounding down
// after subtracting 1/8 leaves between 0.09 p and 1.16 p.
template <class F>
__device__ __forceinline__ Fe combine(const int (&u)[8], const int (&v)[8]) {
  constexpr Signed256 pb = signed_modulus<F>();
  const float t = __builtin_fmaf((float)v[7], 65536.0f, (float)u[7]);
  const int nq = -(int)__builtin_floorf(__builtin_fmaf(t, inv_top<F>(), -0.125f));
  Fe r;
  int32_t carry = 0;  // below 2^18.2 in magnitude, so u_l + carry fits 32 bits
  sfor<8>([&](auto l_) {
    constexpr int l = decltype(l_)::value;
    const int64_t acc = mad_i64(nq, pb.v[l], mad_i64(v[l], 65536, (int64_t)(u[l] + carry)));
    r.v[l] = (uint32_t)acc;
    carry = (int32_t)(acc >> 32);
  });
  return r;
}

// Digit value at which output i of a radix-2^LOG_RHO round is stored, and back.
template <bool HALF, int LOG_RHO>
__device__ __forceinline__ uint32_t out_digit(uint32_t i) {
  return HALF ? (i >> 1) | ((i & 1u) << (LOG_RHO - 1)) : i;
}
template <bool HALF, int LOG_RHO>
__device__ __forceinline__ uint32_t digit_out(uint32_t d) {
  return HALF ? ((d << 1) & ((1u << LOG_RHO) - 1)) | (d >> (LOG_RHO - 1)) : d;
}

// One pair of accumulator tiles (outputs i0 and i1 of 32 columns): lane
// (n, h) gets output i_h of column n.  `first`: i0 is output 0, whose digit
// offsets (bias_correction over `terms` terms) are added.
template <class F, int TERMS>
__device__ __forceinline__ Fe finish(const V16i& d0, const V16i& d1, bool first) {
  int u[8], v[8];
  sfor<4>([&](auto g_) {
    constexpr int g = decltype(g_)::value;
    u[g] = (d0[4 * g + 1] << 8) + d0[4 * g];
    v[g] = (d0[4 * g + 3] << 8) + d0[4 * g + 2];
    u[4 + g] = (d1[4 * g + 1] << 8) + d1[4 * g];
    v[4 + g] = (d1[4 * g + 3] << 8) + d1[4 * g + 2];
    swap_halves(u[g], u[4 + g]);
    swap_halves(v[g], v[4 + g]);
  });
  if (first) {
    constexpr U256 c0 = bias_correction<F>(TERMS);
    const bool zero = (threadIdx.x & 32u) == 0;
    sfor<8>([&](auto l_) {
      constexpr int l = decltype(l_)::value;
      u[l] += zero ? (int)(c0.v[l] & 0xffffu) : 0;
      v[l] += zero ? (int)(c0.v[l] >> 16) : 0;
    });
  }
  return combine<F>(u, v);
}

__device__ __forceinline__ V4i lds_half(const U32x4* lds, uint32_t slot) {
  const U32x4 x = lds[slot];
  return V4i{(int)x[0], (int)x[1], (int)x[2], (int)x[3]};
}

// Round q of the tile's R-point DFTs, in place: digit q of the point index
// becomes the output index of a radix-rho DFT over it.  Work is dealt in
// units of 32 columns x two outputs, one element per lane.
//
// HALF: digit values j < rho/2 hold x_j + x_(j + rho/2), the others
// x_j - x_(j + rho/2).  Even outputs sum over the former, odd ones over the
// latter, rho/2 terms each; a group is 32 columns and one parity.  Output i
// goes to digit value out_digit(i), among the group's own inputs, so that a
// wave that owns a group needs no other wave's agreement to write.
template <class F, int LOG_R, int LOG_TILE, int LOG_THREADS, int Q>
__device__ __forceinline__ void dft_round(U32x4* lds) {
  using S = Shape<LOG_R, LOG_TILE, LOG_THREADS>;
  using Rd = typename S::Rd;
  constexpr int LOG_RHO = Rd::log(Q), RHO = 1 << LOG_RHO;
  constexpr int LOG_LOW = Rd::low(Q), LOW = 1 << LOG_LOW;
  constexpr int SH = LOG_LOW + S::LOG_J;
  constexpr int STEP = 16 / RHO;  // w_rho = w_16^STEP
  constexpr int TERMS = S::HALF ? RHO / 2 : RHO;
  constexpr int PAIRS = S::HALF ? RHO / 4 : RHO / 2;  // per group
  const uint32_t lane = threadIdx.x & 63u, h = lane >> 5;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const V4i* amat = reinterpret_cast<const V4i*>(lds + S::LDS_DATA) + lane;
  // element with digit value 0 of this lane's column in column group nt
  auto base = [&](uint32_t nt) __attribute__((always_inline)) -> uint32_t {
    const uint32_t n = nt * 32u + (lane & 31u);
    const uint32_t c = n & (S::J - 1), m = n >> S::LOG_J;
    const uint32_t r = (m & (LOW - 1)) + ((m >> LOG_LOW) << (LOG_LOW + LOG_RHO));
    return (r << S::LOG_J) + c;
  };
  constexpr int PER = S::U < PAIRS ? S::U : PAIRS;  // pairs of a group taken by one wave
  constexpr int GROUPS = S::U / PER;                // groups per wave
  constexpr bool SHARED = PER < PAIRS;              // other waves read the slots this wave writes
  constexpr int G = PER >= 2 ? 2 : PER;             // pairs in flight
  Fe out[SHARED ? PER : G];
  sfor<GROUPS>([&](auto k_) {
    constexpr int k = decltype(k_)::value;
    const uint32_t unit = (wave * GROUPS + k) * PER;
    const uint32_t group = unit / PAIRS, pair0 = unit % PAIRS;
    const uint32_t parity = S::HALF ? group & 1u : 0u, nt = S::HALF ? group >> 1 : group;
    const uint32_t e0 = base(nt);
    const uint32_t in0 = slot_at<SH>(slot16(e0, h), parity * TERMS);
    // output i0 + h of pair p: digit value parity TERMS + 2 p + h
    const uint32_t out0 = slot_at<SH>(slot16(e0, 0), parity * TERMS + 2 * pair0 + h);
    V4i b[TERMS];
    sfor<TERMS>([&](auto j_) {
      constexpr int j = decltype(j_)::value;
      b[j] = lds_half(lds, slot_at<SH>(in0, j));
    });
    // Term 0's factor is w^0 = 1 for every output: its digits start the
    // accumulators (rows 8 g + 4 h + q are byte q of limb g + 4 h, which is
    // word g of this lane's half).
    V16i first_term;
    sfor<16>([&](auto r_) {
      constexpr int r = decltype(r_)::value;
      first_term[r] = (int)((unsigned)b[0][r / 4] << (24 - 8 * (r % 4))) >> 24;
    });
    sfor<PER / G>([&](auto g_) {
      constexpr int g = decltype(g_)::value;
      V16i acc[2 * G];
      sfor<2 * G>([&](auto t_) { acc[decltype(t_)::value] = first_term; });
      sfor<TERMS - 1>([&](auto j_) {
        constexpr int j = decltype(j_)::value + 1;
        sfor<2 * G>([&](auto t_) {
          constexpr int t = decltype(t_)::value;
          const uint32_t m = 2 * (pair0 + G * g + t / 2) + t % 2;
          const uint32_t i = S::HALF ? 2 * m + parity : m;
          acc[t] = mfma(amat[((i * j * STEP) & 15u) * 64u], b[j], acc[t]);
        });
      });
      sfor<G>([&](auto p_) {
        constexpr int p = decltype(p_)::value;
        const Fe x = finish<F, TERMS>(acc[2 * p], acc[2 * p + 1], parity == 0 && pair0 + G * g + p == 0);
        if constexpr (SHARED) out[G * g + p] = x;
        else lds_store(lds, slot_at<SH>(out0, 2 * (G * g + p)), x, 0u);
      });
    });
    if constexpr (SHARED) {
      static_assert(GROUPS == 1, "a shared group is a wave's only one");
      __syncthreads();  // every wave has read its inputs
      sfor<PER>([&](auto u_) {
        constexpr int u = decltype(u_)::value;
        lds_store(lds, slot_at<SH>(out0, 2 * u), out[u], 0u);
      });
    }
  });
}

// Element index of a thread's k-th element (k < U) in the load and twiddle
// phases: elements 2 m and 2 m + 1 differ in bit P only, the top bit of the
// next round's digit.
template <int P, int THREADS>
__device__ __forceinline__ uint32_t elem_at(uint32_t k) {
  const uint32_t x = (k >> 1) * THREADS + threadIdx.x;
  return ((x >> P) << (P + 1)) | ((k & 1u) << P) | (x & ((1u << P) - 1u));
}

// A product of a value below 2p and a canonical one is below 2p.  Sums and
// differences of a pair then have to fit eight limbs (the sum, unsigned) and
// 32 signed byte digits (the difference, in magnitude below 0.498 2^256).
// For p below 2^254 they do; for BLS12-381 Fr (p = 0.453 2^256) the pair is
// made canonical first.
template <class F>
constexpr bool kTight = F::P[7] >= 0x3f000000u;

// x_j + x_(j + rho/2) and x_j - x_(j + rho/2) as digits: the sum's bytes
// offset by 128 (see bias_correction), the difference plus 0x8080...80, whose
// bytes offset by 128 are its signed digits exactly.
__device__ __forceinline__ void pair_digits(Fe& x, Fe& y) {
  Fe s, d;
  unsigned int c = 0, br = 0, c2 = 0;
#pragma unroll
  for (int l = 0; l < kLimbs; ++l) s.v[l] = __builtin_addc(x.v[l], y.v[l], c, &c);
#pragma unroll
  for (int l = 0; l < kLimbs; ++l) d.v[l] = __builtin_subc(x.v[l], y.v[l], br, &br);
#pragma unroll
  for (int l = 0; l < kLimbs; ++l) d.v[l] = __builtin_addc(d.v[l], kFlip, c2, &c2);
  x = s;
  y = d;
}

// Digits of a thread's elements to LDS: element k at slot[k].
template <class F, bool HALF, int K>
__device__ __forceinline__ void store_digits(U32x4* lds, const uint32_t (&slot)[K], Fe (&x)[K], bool reduce) {
  if constexpr (HALF) {
    if (kTight<F> && reduce) {
      sfor<K>([&](auto k_) { x[decltype(k_)::value] = canon<F>(x[decltype(k_)::value]); });
    }
    sfor<K / 2>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      pair_digits(x[2 * k], x[2 * k + 1]);
    });
  }
  sfor<K>([&](auto k_) { lds_store(lds, slot[decltype(k_)::value], x[decltype(k_)::value], kFlip); });
}

// Products taken together (interleaved) in the load, twiddle and store loops.
template <int U>
constexpr int group() {
  return U >= 4 ? 4 : U;
}

// Rounds Q .. N - 1, with the twiddles w_R^(P_q i_q low) after all but the
// last (P_q the product of the earlier radices, low the digits after q).
template <class F, int LOG_R, int LOG_TILE, int LOG_THREADS, int Q>
__device__ __forceinline__ void rounds(U32x4* lds, const Fe* __restrict__ tw_r) {
  using S = Shape<LOG_R, LOG_TILE, LOG_THREADS>;
  using Rd = typename S::Rd;
  dft_round<F, LOG_R, LOG_TILE, LOG_THREADS, Q>(lds);
  __syncthreads();
  if constexpr (Q + 1 < Rd::N) {
    constexpr int K = group<S::U>();
    constexpr int LOG_LOW = Rd::low(Q), RHO = 1 << Rd::log(Q);
    constexpr int P = S::LOG_J + LOG_LOW - 1;  // top bit of digit Q + 1
#pragma unroll 1
    for (int it = 0; it < S::U; it += K) {
      Fe x[K], w[K];
      uint32_t slot[K];
      sfor<K>([&](auto k_) {
        constexpr int k = decltype(k_)::value;
        const uint32_t e = S::HALF ? elem_at<P, S::THREADS>(it + k) : threadIdx.x;
        const uint32_t r = e >> S::LOG_J;
        const uint32_t low = r & ((1u << LOG_LOW) - 1);
        const uint32_t i = digit_out<S::HALF, Rd::log(Q)>((r >> LOG_LOW) & (RHO - 1));
        slot[k] = slot16(e, 0);
        w[k] = load_fe(tw_r, (i * low) << Rd::high(Q));
        x[k] = lds_load(lds, slot[k]);
      });
      mul_many<F, K, K>(x, w);
      store_digits<F, S::HALF, K>(lds, slot, x, true);
    }
    __syncthreads();
    rounds<F, LOG_R, LOG_TILE, LOG_THREADS, Q + 1>(lds, tw_r);
  }
}

template <class F>
__device__ const DigitTable digit_table = make_digit_table<F>();

// BRIDGE: kPassBridge.  As much arithmetic as the two passes it replaces,
// without the vector's trip to memory and the launch between them (quotient
// chain 2^14 55.1 -> 50.0 us, 2^19 356 -> 336, 2^24 12.02 -> 11.62 ms).  Small
// chains gain by the launch; large ones less than the bytes saved would give,
// since their passes are held by the power that products and matrices draw.
template <class F, int LOG_R, int LOG_TILE, int LOG_THREADS, bool BRIDGE>
__global__ void __launch_bounds__((Shape<LOG_R, LOG_TILE, LOG_THREADS>::THREADS),
                                  (Shape<LOG_R, LOG_TILE, LOG_THREADS>::MIN_WAVES))
    mfma_pass_kernel(PassLaunch a) {
  using S = Shape<LOG_R, LOG_TILE, LOG_THREADS>;
  using Rd = typename S::Rd;
  __shared__ U32x4 lds[S::LDS_DATA + S::LDS_A];
  constexpr int K = group<S::U>();
  const uint32_t tile = pass_tile_index(a, blockIdx.x);
  // the matrices are fetched beside the first data and reach LDS after them
  constexpr int FRAGS = 16 * 64 / S::THREADS;
  U32x4 frag[FRAGS];
  sfor<FRAGS>([&](auto k_) {
    constexpr int k = decltype(k_)::value;
    frag[k] = reinterpret_cast<const U32x4*>(&digit_table<F>)[k * S::THREADS + threadIdx.x];
  });

  const uint64_t n = 1ull << a.log_n, ns = 1ull << a.log_ns;
  const uint64_t j0 = (uint64_t)tile << S::LOG_J;
  const uint32_t log_stride = a.log_n - LOG_R;
  const bool rev = a.flags & kPassReverseIn;
  const bool rev_load = !BRIDGE && rev;

  // load: element e = r J + c is point r of column j0 + c
#pragma unroll 1
  for (int it = 0; it < S::U; it += K) {
    Fe x[K], w[K];
    uint32_t elem[K], slot[K];
    bool reduce = false;  // the input is canonical, products are below 2p
    sfor<K>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      elem[k] = S::HALF ? elem_at<LOG_TILE - 1, S::THREADS>(it + k) : threadIdx.x;
      slot[k] = slot16(elem[k], 0);
    });
    sfor<K>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const uint32_t e = elem[k];
      const uint64_t idx = j0 + (e & (S::J - 1)) + ((uint64_t)(e >> S::LOG_J) << log_stride);
      x[k] = load_fe(a.in, rev_load ? ((n - idx) & (n - 1)) : idx);
    });
    if (!BRIDGE && (a.flags & kPassPreTable)) {
      sfor<K>([&](auto k_) {
        constexpr int k = decltype(k_)::value;
        const uint32_t e = elem[k];
        w[k] = load_fe(a.pre_table, j0 + (e & (S::J - 1)) + ((uint64_t)(e >> S::LOG_J) << log_stride));
      });
      mul_many<F, K, K>(x, w);
      reduce = true;
    }
    if (a.tw_pass) {  // inter-pass twiddle w_{Ns R}^(r (j mod Ns)), table [r][j mod Ns]
      sfor<K>([&](auto k_) {
        constexpr int k = decltype(k_)::value;
        const uint32_t e = elem[k];
        w[k] = load_fe(a.tw_pass, ((uint64_t)(e >> S::LOG_J) << a.log_ns) + ((j0 + (e & (S::J - 1))) & (ns - 1)));
      });
      mul_many<F, K, K>(x, w);
      reduce = true;
    } else if (a.tw_hi) {  // the same twiddle from the two-level tables
      const uint32_t log_mult = a.log_n - a.log_ns - LOG_R;
      Fe lo[K];
      sfor<K>([&](auto k_) {
        constexpr int k = decltype(k_)::value;
        const uint32_t e = elem[k];
        const uint64_t ex = ((uint64_t)(e >> S::LOG_J) * ((j0 + (e & (S::J - 1))) & (ns - 1))) << log_mult;
        w[k] = load_fe(a.tw_hi, ex >> a.log_lo);
        lo[k] = load_fe(a.tw_lo, ex & ((1ull << a.log_lo) - 1));
      });
      mul_many<F, K, K, true>(w, lo);  // canonical: the factor of the next product
      mul_many<F, K, K>(x, w);
      reduce = true;
    }
    store_digits<F, S::HALF, K>(lds, slot, x, reduce);
  }
  sfor<FRAGS>([&](auto k_) {
    constexpr int k = decltype(k_)::value;
    lds[S::LDS_DATA + k * S::THREADS + threadIdx.x] = frag[k];
  });
  __syncthreads();

  rounds<F, LOG_R, LOG_TILE, LOG_THREADS, 0>(lds, a.tw_r);

  // output k of column c sits at the slot with the digits of (i_1, i_2, ...)
  // in place of (r_1, r_2, ...)
  auto out_slot = [&](uint32_t k, uint32_t c) __attribute__((always_inline)) -> uint32_t {
    uint32_t r = 0;
    sfor<Rd::N>([&](auto d_) {
      constexpr int d = decltype(d_)::value;
      r |= out_digit<S::HALF, Rd::log(d)>((k >> Rd::high(d)) & ((1u << Rd::log(d)) - 1)) << Rd::low(d);
    });
    return slot16((r << S::LOG_J) + c, 0);
  };
  // the quotient's pointwise step: (A B - C) / (g^n - 1), C this output
  auto pointwise = [&](const Fe& x, uint64_t idx) __attribute__((always_inline)) -> Fe {
    const Fe ab = mul<F>(load_fe(a.pw_a, idx), load_fe(a.pw_b, idx));
    return mul<F, false>(sub_lazy<F>(ab, x), a.post_const);
  };

  if constexpr (BRIDGE) {
    static_assert(K == S::U, "every output is taken before any is overwritten");
    Fe x[K], w[K];
    uint32_t slot[K];
    uint64_t idx[K];
    sfor<K>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const uint32_t e = S::HALF ? elem_at<LOG_TILE - 1, S::THREADS>(k) : threadIdx.x;
      const uint32_t c = e & (S::J - 1), r = e >> S::LOG_J;
      // point r of column -j is element n - (j + i n/R): i = R - 1 - r, or -r if j = 0
      const uint32_t i = rev ? (S::R - (j0 + c ? 1u : 0u) - r) & (S::R - 1) : r;
      slot[k] = slot16(e, 0);
      idx[k] = j0 + c + ((uint64_t)i << log_stride);
      x[k] = lds_load(lds, out_slot(i, c));
    });
    if (a.flags & kPassPreTable) {
      sfor<K>([&](auto k_) { w[decltype(k_)::value] = load_fe(a.pre_table, idx[decltype(k_)::value]); });
      mul_many<F, K, K>(x, w);
    }
    if (a.flags & kPassPostPointwise) {
      sfor<K>([&](auto k_) {
        constexpr int k = decltype(k_)::value;
        x[k] = pointwise(x[k], idx[k]);
      });
    }
    __syncthreads();
    store_digits<F, S::HALF, K>(lds, slot, x, true);
    __syncthreads();
    rounds<F, LOG_R, LOG_TILE, LOG_THREADS, 0>(lds, a.tw_r);
  }

  // store: the first pass writes J R consecutive elements, output index
  // fastest; later passes write runs of J columns.
  const bool k_fast = BRIDGE || a.log_ns == 0;
#pragma unroll 1
  for (int it = 0; it < S::U; it += K) {
    Fe x[K], w[K];
    uint64_t idx[K];
    sfor<K>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      const uint32_t e = (it + q) * S::THREADS + threadIdx.x;
      const uint32_t c = k_fast ? e >> LOG_R : e & (S::J - 1);
      const uint32_t k = k_fast ? e & (S::R - 1) : e >> S::LOG_J;
      x[q] = lds_load(lds, out_slot(k, c));
      const uint64_t j = j0 + c;
      if constexpr (BRIDGE)
        idx[q] = ((rev ? ((1ull << log_stride) - j) & ((1ull << log_stride) - 1) : j) << LOG_R) + k;
      else
        idx[q] = ((j >> a.log_ns) << (a.log_ns + LOG_R)) + (j & (ns - 1)) + ((uint64_t)k << a.log_ns);
    });
    if constexpr (!BRIDGE) {
      if (a.flags & kPassPostTable) {
        sfor<K>([&](auto q_) { w[decltype(q_)::value] = load_fe(a.post_table, idx[decltype(q_)::value]); });
        mul_many<F, K, K>(x, w);
      }
      if (a.flags & kPassPostConst) {
        sfor<K>([&](auto q_) { w[decltype(q_)::value] = a.post_const; });
        mul_many<F, K, K>(x, w);
      }
      if (a.flags & kPassPostPointwise) {
        sfor<K>([&](auto q_) {
          constexpr int q = decltype(q_)::value;
          x[q] = pointwise(x[q], idx[q]);
        });
      }
      if (a.log_ns + LOG_R == a.log_n) {  // the last pass's outputs are canonical
        sfor<K>([&](auto q_) { x[decltype(q_)::value] = canon<F>(x[decltype(q_)::value]); });
      }
    }
    sfor<K>([&](auto q_) { store_fe(a.out, idx[decltype(q_)::value], x[decltype(q_)::value]); });
  }
}

template <class F, bool BRIDGE, int LOG_R, int LOG_TILE, int LOG_THREADS>
hipError_t launch_one(const PassLaunch& a0, hipStream_t s) {
  using S = Shape<LOG_R, LOG_TILE, LOG_THREADS>;
  PassLaunch a = a0;
  a.log_grp_tiles = a.log_n - LOG_TILE;
  const uint64_t tiles = ((1ull << a.log_n) >> LOG_TILE) * (a.grp_jobs ? a.grp_jobs : 1u);
  hipLaunchKernelGGL((mfma_pass_kernel<F, LOG_R, LOG_TILE, LOG_THREADS, BRIDGE>), dim3((uint32_t)tiles),
                     dim3(S::THREADS), 0, s, a);
  return hipGetLastError();
}

// Elements per lane by the number of elements in the launch (all jobs of a
// grouped one).  One while the launch does not fill the chip: each of a lane's
// elements adds to the pass's latency (radix 2^8 at 2^16, 7.0 / 8.3 us for the
// first / last pass with one, 7.4 / 9.2 with two).  Then two or four, whichever
// needs the shorter rounds of resident workgroups: 256 CUs hold about 1,280
// workgroups of 2^9 elements or 768 of 2^10, and a round of the latter takes
// about 1.13 times as long (radix 2^7 at 2^20: 1.6 rounds against 1.3, 27.7 /
// 36.3 us against 32.8 / 40.8; at 2^19 16.0 / 21.6 against 17.2 / 24.3).  From
// 2^21 always four: their tiles read and write runs twice as long (radix 2^8
// at 2^24: 0.442 / 0.589 ms against 0.493 / 0.751).
constexpr uint32_t kTwoLog = 18, kFourLog = 21;
inline bool four_per_lane(uint64_t elements) {
  if (elements >> kFourLog) return true;
  const uint64_t rounds4 = ((elements >> 10) + 767) / 768, rounds2 = ((elements >> 9) + 1279) / 1280;
  return 113 * rounds4 < 100 * rounds2;
}

// Passes of multi-pass transforms (radix 2^3 .. 2^9; bridges 2^6 .. 2^9).  A
// bridge's launch holds one or three vectors of a plan whose first and last
// radix agree: of radix 2^8 these are 3 x 2^16 elements or fewer (8 + 8), or
// 2^23 and more, of radix 2^9 2^18 and more (9 + 9).
template <class F, bool BRIDGE>
hipError_t dispatch_multi(int log_r, const PassLaunch& a, hipStream_t s) {
  const uint64_t total = (a.grp_jobs ? a.grp_jobs : 1ull) << a.log_n;
  if (total >> kTwoLog && a.log_n >= 10 && four_per_lane(total)) {
    if constexpr (!BRIDGE) {
      switch (log_r) {
        case 3: return launch_one<F, BRIDGE, 3, 10, 8>(a, s);
        case 4: return launch_one<F, BRIDGE, 4, 10, 8>(a, s);
        case 5: return launch_one<F, BRIDGE, 5, 10, 8>(a, s);
      }
    }
    switch (log_r) {
      case 6: return launch_one<F, BRIDGE, 6, 10, 8>(a, s);
      case 7: return launch_one<F, BRIDGE, 7, 10, 8>(a, s);
      case 8: return launch_one<F, BRIDGE, 8, 10, 8>(a, s);
      case 9: return launch_one<F, BRIDGE, 9, 10, 8>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (total >> kTwoLog && a.log_n >= 9) {
    if constexpr (!BRIDGE) {
      switch (log_r) {
        case 3: return launch_one<F, BRIDGE, 3, 9, 8>(a, s);
        case 4: return launch_one<F, BRIDGE, 4, 9, 8>(a, s);
        case 5: return launch_one<F, BRIDGE, 5, 9, 8>(a, s);
        case 8: return launch_one<F, BRIDGE, 8, 9, 8>(a, s);
      }
    }
    switch (log_r) {
      case 6: return launch_one<F, BRIDGE, 6, 9, 8>(a, s);
      case 7: return launch_one<F, BRIDGE, 7, 9, 8>(a, s);
      case 9: return launch_one<F, BRIDGE, 9, 10, 9>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  if constexpr (!BRIDGE) {
    switch (log_r) {
      case 3: return launch_one<F, BRIDGE, 3, 8, 8>(a, s);
      case 4: return launch_one<F, BRIDGE, 4, 9, 9>(a, s);
      case 5: return launch_one<F, BRIDGE, 5, 8, 8>(a, s);
      case 9: return launch_one<F, BRIDGE, 9, 10, 10>(a, s);
    }
  }
  switch (log_r) {
    case 6: return launch_one<F, BRIDGE, 6, 8, 8>(a, s);
    case 7: return launch_one<F, BRIDGE, 7, 9, 9>(a, s);
    case 8: return launch_one<F, BRIDGE, 8, 9, 9>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// A pass of a multi-pass transform, or a transform of 2^8 to 2^11 points in
// one tile.  Keep in step with mfma_supported() and bridge_supported().
template <class F>
hipError_t dispatch(int log_r, const PassLaunch& a, hipStream_t s) {
  if ((uint32_t)log_r == a.log_n) {
    switch (log_r) {
      case 8: return launch_one<F, false, 8, 8, 8>(a, s);
      case 9: return launch_one<F, false, 9, 9, 9>(a, s);
      case 10: return launch_one<F, false, 10, 10, 10>(a, s);
      case 11: return launch_one<F, false, 11, 11, 10>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  return a.flags & kPassBridge ? dispatch_multi<F, true>(log_r, a, s) : dispatch_multi<F, false>(log_r, a, s);
}

}  // namespace mfma
}  // namespace zk
