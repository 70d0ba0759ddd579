// Multi-scalar multiplication on BLS12-381 G1: Q = sum_i s_i P_i.
//
// MSM is the paper's other dominant proving kernel (Section II-A, Fig. 4(a));
// the libraries it measures compute it with Pippenger's bucket method and
// their cost is counted in point additions and doublings (Table V).  This is
// the bucket method laid out for MI355X:
//
// * Fixed bases with per-window multiples.  The points of a Groth16 MSM are
//   the proving key's, fixed across proofs, so msm_bases_create stores, for
//   c-bit windows w = 0 .. W-1, the affine multiples 2^(c w) P_i (W n points:
//   1.5 GiB at n = 2^20, c = 16, small next to 288 GB of HBM).  A scalar's
//   window digits then all index one set of 2^c - 1 buckets, and the
//   window-by-window Horner combination, a chain of W c point doublings that
//   no amount of parallelism shortens, disappears from every MSM.
// * Counting sort of (digit, point) pairs: per-workgroup histograms in LDS
//   (each entry keeps its rank within its group and bucket), a prefix over
//   the groups per bucket, one scan over the buckets, and a scatter put the
//   points of each bucket next to each other, with no global atomics.
// * Bucket accumulation: the sorted entries are cut into equal runs, one per
//   lane, across bucket boundaries; a lane adds its run's points into XYZZ
//   accumulators with mixed (XYZZ + affine) additions, 8 multiplications
//   and 2 squarings each, and the segments at the runs' ends then combine
//   per bucket.  XYZZ coordinates (x = X / ZZ, y = Y / ZZZ) keep additions
//   free of inversions.
// * Bucket reduction by bits: sum_k k B_k = sum_b 2^b G_b with
//   G_b = sum of the buckets whose index has bit b set, formed by a tree over
//   the buckets that sums the odd nodes of every level beside the nodes
//   themselves; the c terms 2^b G_b are doubled in parallel and summed by a
//   tree: a critical path of a few dozen point operations, where the
//   running-sum method is a serial chain of 2^(c+1) additions.
// * Everything after the accumulation is bound by the latency of point
//   operations in few waves: there four lanes share a point, one coordinate
//   each, and an addition is four products in sequence instead of fourteen.
//
// Field arithmetic: fq.hpp (14 x 28-bit limbs).
// Scalars arrive as the NTT library's Montgomery limbs over BLS12-381 Fr and
// are converted with one product by 1.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "field.hpp"
#include "fq.hpp"
#include "msm.hpp"

namespace zk {
namespace msm {
namespace {

using fq::Fq;

struct Affine {
  Fq x, y;
};
struct Xyzz {
  Fq X, Y, ZZ, ZZZ;
};

// Coordinates are products' results or normalised, so limbs 0 .. 12 are in
// [0, 2^28) and values within (-2 q, 4 q).  Infinity has ZZ = ZZZ = 0 with all
// limbs zero; no other point has.
__device__ __forceinline__ Xyzz infinity() {
  Xyzz r;
  r.X = fq::one();
  r.Y = fq::one();
  r.ZZ = fq::zero();
  r.ZZZ = fq::zero();
  return r;
}

__device__ __forceinline__ Xyzz from_affine(const Affine& a) {
  Xyzz r;
  r.X = a.x;
  r.Y = a.y;
  r.ZZ = fq::one();
  r.ZZZ = fq::one();
  return r;
}

// 2 P in XYZZ (y^2 = x^3 + b, a = 0): U = 2Y, V = U^2, W = U V, S = X V,
// M = 3 X^2; X3 = M^2 - 2S, Y3 = M (S - X3) - W Y, ZZ3 = V ZZ, ZZZ3 = W ZZZ.
__device__ __forceinline__ Xyzz dbl(const Xyzz& p) {
  const Fq U = fq::dbl(p.Y);
  const Fq V = fq::sqr(U), XX = fq::sqr(p.X);
  const Fq W = fq::mul(U, V), S = fq::mul(p.X, V);
  const Fq M = fq::normalise(fq::add(fq::dbl(XX), XX));
  Xyzz r;
  r.X = fq::normalise(fq::sub(fq::sqr(M), fq::dbl(S)));
  r.Y = fq::mul_add(M, fq::sub(S, r.X), fq::neg(W), p.Y);
  r.ZZ = fq::mul(V, p.ZZ);
  r.ZZZ = fq::mul(W, p.ZZZ);
  return r;
}

// 2 A for an affine point (ZZ = ZZZ = 1).
__device__ __forceinline__ Xyzz dbl_affine(const Affine& a) {
  const Fq U = fq::dbl(a.y);
  const Fq V = fq::sqr(U), XX = fq::sqr(a.x);
  const Fq W = fq::mul(U, V), S = fq::mul(a.x, V);
  const Fq M = fq::normalise(fq::add(fq::dbl(XX), XX));
  Xyzz r;
  r.X = fq::normalise(fq::sub(fq::sqr(M), fq::dbl(S)));
  r.Y = fq::mul_add(M, fq::sub(S, r.X), fq::neg(W), a.y);
  r.ZZ = V;
  r.ZZZ = W;
  return r;
}

// P + A with A affine, P not infinity: U2 = x2 ZZ1, S2 = y2 ZZZ1,
// P = U2 - X1, R = S2 - Y1, PP = P^2, PPP = P PP, Q = X1 PP;
// X3 = R^2 - PPP - 2Q, Y3 = R (Q - X3) - Y1 PPP, ZZ3 = ZZ1 PP,
// ZZZ3 = ZZZ1 PPP.  P = 0 means x-coordinates agree: the points are equal
// (double A) or opposite (`cancelled`: infinity).
__device__ __forceinline__ Xyzz add_mixed(const Xyzz& p, const Affine& a, bool& cancelled) {
  Fq P = fq::sub(fq::mul(a.x, p.ZZ), p.X);
  const Fq R = fq::sub(fq::mul(a.y, p.ZZZ), p.Y);
  if (fq::is_zero(P)) {
    cancelled = !fq::is_zero(R);
    return cancelled ? infinity() : dbl_affine(a);
  }
  P = fq::opaque(P);  // is_zero has its limbs' 64-bit extensions
  const Fq PP = fq::sqr(P);
  const Fq PPP = fq::mul(P, PP), Q = fq::mul(p.X, PP);
  Xyzz r;
  r.X = fq::normalise(fq::sub(fq::sub(fq::sqr(R), PPP), fq::dbl(Q)));
  r.Y = fq::mul_add(R, fq::sub(Q, r.X), fq::neg(p.Y), PPP);
  r.ZZ = fq::mul(p.ZZ, PP);
  r.ZZZ = fq::mul(p.ZZZ, PPP);
  return r;
}

// A packed affine point: x then y, twelve 32-bit words each, as three 16-byte
// loads.
struct Packed {
  uint4 v[6];
};
__device__ __forceinline__ Packed load_packed(const uint32_t* __restrict__ pts, uint64_t i) {
  const uint4* q = reinterpret_cast<const uint4*>(pts + kPointWords * i);
  Packed r;
#pragma unroll
  for (int k = 0; k < 6; ++k) r.v[k] = q[k];
  return r;
}
__device__ __forceinline__ Affine unpack(const Packed& p) {
  uint32_t x[fq::kWords], y[fq::kWords];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint4 u = p.v[k], w = p.v[3 + k];
    x[4 * k] = u.x, x[4 * k + 1] = u.y, x[4 * k + 2] = u.z, x[4 * k + 3] = u.w;
    y[4 * k] = w.x, y[4 * k + 1] = w.y, y[4 * k + 2] = w.z, y[4 * k + 3] = w.w;
  }
  return Affine{fq::unpack(x), fq::unpack(y)};
}
__device__ __forceinline__ void store_affine(uint32_t* __restrict__ pts, uint64_t i, const Fq& x, const Fq& y) {
  uint32_t wx[fq::kWords], wy[fq::kWords];
  fq::pack_canonical(wx, x);
  fq::pack_canonical(wy, y);
#pragma unroll
  for (int k = 0; k < fq::kWords; ++k) {
    pts[kPointWords * i + k] = wx[k];
    pts[kPointWords * i + fq::kWords + k] = wy[k];
  }
}

// Working points in memory: four coordinates of fourteen limbs.
__device__ __forceinline__ void store_xyzz(uint32_t* __restrict__ p, uint64_t i, const Xyzz& a) {
  int2* q = reinterpret_cast<int2*>(p + kAccWords * i);
#pragma unroll
  for (int k = 0; k < fq::kN / 2; ++k) {
    q[k] = make_int2(a.X.v[2 * k], a.X.v[2 * k + 1]);
    q[7 + k] = make_int2(a.Y.v[2 * k], a.Y.v[2 * k + 1]);
    q[14 + k] = make_int2(a.ZZ.v[2 * k], a.ZZ.v[2 * k + 1]);
    q[21 + k] = make_int2(a.ZZZ.v[2 * k], a.ZZZ.v[2 * k + 1]);
  }
}
__device__ __forceinline__ Xyzz load_xyzz(const uint32_t* __restrict__ p, uint64_t i) {
  const int2* q = reinterpret_cast<const int2*>(p + kAccWords * i);
  Xyzz r;
#pragma unroll
  for (int k = 0; k < fq::kN / 2; ++k) {
    const int2 x = q[k], y = q[7 + k], z = q[14 + k], t = q[21 + k];
    r.X.v[2 * k] = x.x, r.X.v[2 * k + 1] = x.y;
    r.Y.v[2 * k] = y.x, r.Y.v[2 * k + 1] = y.y;
    r.ZZ.v[2 * k] = z.x, r.ZZ.v[2 * k + 1] = z.y;
    r.ZZZ.v[2 * k] = t.x, r.ZZZ.v[2 * k + 1] = t.y;
  }
  return r;
}

// ---------------------------------------------------------------------------
// Points shared by four lanes: lane 0 of a quad holds X, lane 1 Y, lane 2 ZZ
// and lane 3 ZZZ.  All four lanes are active in every operation, so that
// limbs can move between them by DPP.  A lone wave issues one multiply-add in
// eight cycles, whatever its parallelism, so an addition's fourteen products
// cost it fourteen times one product's latency in one lane and four times in
// four (addition 16 -> 6 us, doubling 15 -> 5 us, one wave per SIMD).

template <int A, int B, int C, int D>
__device__ __forceinline__ int quad_perm(int x) {
  return __builtin_amdgcn_update_dpp(0, x, A | (B << 2) | (C << 4) | (D << 6), 0xf, 0xf, true);
}
template <int A, int B, int C, int D>
__device__ __forceinline__ Fq quad_perm(const Fq& a) {
  Fq r;
#pragma unroll
  for (int i = 0; i < fq::kN; ++i) r.v[i] = quad_perm<A, B, C, D>(a.v[i]);
  return r;
}
template <int L>
__device__ __forceinline__ Fq bcast(const Fq& a) {
  return quad_perm<L, L, L, L>(a);
}
__device__ __forceinline__ Fq sel(bool c, const Fq& a, const Fq& b) {
  Fq r;
#pragma unroll
  for (int i = 0; i < fq::kN; ++i) r.v[i] = c ? a.v[i] : b.v[i];
  return r;
}
__device__ __forceinline__ uint32_t quad_lane() { return threadIdx.x & 3u; }

// Infinity's coordinate of this lane.
__device__ __forceinline__ Fq q_infinity() { return sel(quad_lane() < 2, fq::one(), fq::zero()); }

__device__ __forceinline__ Fq q_dbl(const Fq& a) {
  const uint32_t q = quad_lane();
  const Fq u = fq::dbl(a);  // lane 1: U
  const Fq r1 = fq::sqr(sel(q == 1, u, a));  // lane 0: X^2, lane 1: V
  const Fq V = bcast<1>(r1);
  const Fq M = fq::normalise(fq::add(fq::dbl(r1), r1));  // lane 0
  // lane 0: M^2, lane 1: W = U V, lane 2: ZZ V, lane 3: S = X V
  const Fq x2 = sel(q == 0, M, sel(q == 1, u, sel(q == 2, a, bcast<0>(a))));
  const Fq r2 = fq::mul(x2, sel(q == 0, M, V));
  const Fq S = bcast<3>(r2), W = bcast<1>(r2);
  const Fq X3 = fq::normalise(fq::sub(r2, fq::dbl(S)));  // lane 0
  // lane 0: M (S - X3), lane 1: W Y, lane 3: W ZZZ
  const Fq r3 = fq::mul(sel(q == 0, M, a), sel(q == 0, fq::sub(S, X3), W));
  const Fq Y3 = fq::normalise(fq::sub(bcast<0>(r3), r3));
  return sel(q == 0, X3, sel(q == 1, Y3, sel(q == 2, r2, r3)));
}

// P1 + P2: U1 = X1 ZZ2, U2 = X2 ZZ1, S1 = Y1 ZZZ2, S2 = Y2 ZZZ1,
// P = U2 - U1, R = S2 - S1, PP = P^2, PPP = P PP, Q = U1 PP;
// X3 = R^2 - PPP - 2Q, Y3 = R (Q - X3) - S1 PPP, ZZ3 = ZZ1 ZZ2 PP,
// ZZZ3 = ZZZ1 ZZZ2 PPP.
__device__ __forceinline__ Fq q_add(const Fq& a, const Fq& b) {
  const uint32_t q = quad_lane();
  const Fq r1 = fq::mul(a, quad_perm<2, 3, 0, 1>(b));  // U1, S1, U2, S2
  const Fq o = quad_perm<2, 3, 0, 1>(r1);
  const Fq d = sel(q < 2, fq::sub(o, r1), fq::sub(r1, o));  // P, R, P, R
  const Fq r2 = fq::mul(sel(q < 2, d, a), sel(q < 2, d, b));  // PP, R^2, ZZ1 ZZ2, ZZZ1 ZZZ2
  // PPP, Q, ZZ3, PPP
  const Fq x3 = sel(q == 1, bcast<0>(r1), sel(q == 2, r2, bcast<2>(d)));
  const Fq r3 = fq::mul(x3, bcast<0>(r2));
  const Fq X3 = fq::normalise(fq::sub(fq::sub(r2, bcast<0>(r3)), fq::dbl(r3)));  // lane 1
  // S1 PPP, R (Q - X3), -, ZZZ3
  const Fq x4 = sel(q == 0, bcast<1>(r1), sel(q == 1, d, r2));
  const Fq r4 = fq::mul(x4, sel(q == 1, fq::sub(r3, X3), r3));
  const Fq Y3 = fq::normalise(fq::sub(r4, bcast<0>(r4)));  // lane 1
  Fq r = sel(q == 0, bcast<1>(X3), sel(q == 1, Y3, sel(q == 2, r3, r4)));
  const bool ainf = quad_perm<2, 2, 2, 2>((int)fq::all_zero(a)) != 0;
  const bool binf = quad_perm<2, 2, 2, 2>((int)fq::all_zero(b)) != 0;
  const int dz = (int)fq::is_zero(d);
  const bool same_x = quad_perm<0, 0, 0, 0>(dz) != 0, same_y = quad_perm<1, 1, 1, 1>(dz) != 0;
  if (__any(same_x && !ainf && !binf)) {  // equal or opposite points
    const Fq two = q_dbl(a);
    r = same_x ? sel(same_y, two, q_infinity()) : r;
  }
  return sel(ainf, b, sel(binf, a, r));
}

__device__ __forceinline__ Fq q_load(const uint32_t* p, uint64_t i) {
  const int2* s = reinterpret_cast<const int2*>(p + kAccWords * i + fq::kN * quad_lane());
  Fq r;
#pragma unroll
  for (int k = 0; k < fq::kN / 2; ++k) {
    const int2 x = s[k];
    r.v[2 * k] = x.x, r.v[2 * k + 1] = x.y;
  }
  return r;
}
__device__ __forceinline__ void q_store(uint32_t* p, uint64_t i, const Fq& a) {
  int2* s = reinterpret_cast<int2*>(p + kAccWords * i + fq::kN * quad_lane());
#pragma unroll
  for (int k = 0; k < fq::kN / 2; ++k) s[k] = make_int2(a.v[2 * k], a.v[2 * k + 1]);
}

// ---------------------------------------------------------------------------
// Precomputation: table[w n + i] = 2^(c w) P_i, affine, Montgomery form 2^392.
// One lane per point walks the windows with c doublings each, keeping the
// XYZZ multiples in `scratch`, then turns all W of them affine with one
// inversion (prefix products of the ZZZ, Fermat inversion, back-substitution;
// 1/ZZ = (ZZ/ZZZ)^2).

// Points first .. first + count of n; scratch holds `count` points' rows.
__global__ void __launch_bounds__(128) precompute_kernel(const uint32_t* __restrict__ pts, uint64_t n,
                                                         uint64_t first, uint64_t count, int c, int windows,
                                                         uint32_t* __restrict__ table,
                                                         uint32_t* __restrict__ scratch) {
  const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  const uint64_t i = first + k;
  Affine a = unpack(load_packed(pts, i));
  a.x = fq::mul(a.x, fq::constant(fq::kTo392));
  a.y = fq::mul(a.y, fq::constant(fq::kTo392));
  store_affine(table, i, a.x, a.y);
  if (windows == 1) return;
  // scratch rows of this point: windows x XYZZ, then the prefix products of ZZZ
  uint32_t* my = scratch + k * windows * kScratchWords;
  uint32_t* prefix = my + kAccWords * windows;
  Xyzz p = from_affine(a);
  Fq pre = fq::one();
#pragma unroll 1
  for (int w = 1; w < windows; ++w) {
#pragma unroll 1
    for (int d = 0; d < c; ++d) p = dbl(p);
    store_xyzz(my, w, p);
    pre = fq::mul(pre, p.ZZZ);
#pragma unroll
    for (int l = 0; l < fq::kN; ++l) prefix[fq::kN * w + l] = (uint32_t)pre.v[l];
  }
  Fq inv = fq::inverse(pre);  // 1 / prod_w ZZZ_w
#pragma unroll 1
  for (int w = windows - 1; w >= 1; --w) {
    const Xyzz q = load_xyzz(my, w);
    Fq prev = fq::one();
    if (w > 1) {
#pragma unroll
      for (int l = 0; l < fq::kN; ++l) prev.v[l] = (int32_t)prefix[fq::kN * (w - 1) + l];
    }
    const Fq t = fq::mul(inv, prev);   // 1 / ZZZ_w
    inv = fq::mul(inv, q.ZZZ);         // 1 / prod_{v<w} ZZZ_v
    const Fq izz = fq::sqr(fq::mul(q.ZZ, t));  // (1 / Z)^2
    store_affine(table, (uint64_t)w * n + i, fq::mul(q.X, izz), fq::mul(q.Y, t));
  }
}

// ---------------------------------------------------------------------------
// Digits and counting sort.

// Scalar k of n from the Montgomery form: s = S 2^-256 (a product by 1).
__device__ __forceinline__ Fe scalar_plain(const uint32_t* __restrict__ sc, uint64_t i) {
  Fe s, one;
#pragma unroll
  for (int j = 0; j < kLimbs; ++j) {
    s.v[j] = sc[8 * i + j];
    one.v[j] = j == 0 ? 1u : 0u;
  }
  return mul<Bls12_381Fr>(s, one);
}

// Bits [c w, c w + c) of s.  The limbs are picked by unrolled selects, not
// by a run-time index, so s stays in registers.
__device__ __forceinline__ uint32_t digit(const Fe& s, int c, int w) {
  const int lo = c * w;
  const int word = lo >> 5, sh = lo & 31;
  uint32_t w0 = 0u, w1 = 0u;
#pragma unroll
  for (int k = 0; k < kLimbs; ++k) {
    w0 = k == word ? s.v[k] : w0;
    w1 = k == word + 1 ? s.v[k] : w1;
  }
  const uint64_t bits = ((uint64_t)w1 << 32) | w0;
  return (uint32_t)(bits >> sh) & ((1u << c) - 1u);
}

// Counting sort without global atomics.  Workgroup g takes scalars
// [g B, g B + B) with B windows <= 65535, so that each bucket's count in the
// group fits 16 bits: the group's histogram lives in LDS as 16-bit halves of
// 32-bit words (2^c x 2 bytes, at most 128 KiB), and each digit's LDS
// increment returns its rank among the group's digits of that bucket.
// hist[g 2^c + d] = the group's count of digit d.
constexpr int kHistThreads = 1024;
constexpr uint32_t kHistWords = 1u << 15;  // 2^16 16-bit counters

__global__ void __launch_bounds__(kHistThreads) hist_kernel(const uint32_t* __restrict__ sc, uint64_t n, int c,
                                                            int windows, uint32_t per_group,
                                                            uint16_t* __restrict__ digits, uint16_t* __restrict__ ranks,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kHistWords];
  const uint32_t nb = 1u << c, words = (nb + 1) / 2;
  const uint32_t t = threadIdx.x;
  for (uint32_t k = t; k < words; k += kHistThreads) h[k] = 0u;
  __syncthreads();
  const uint64_t first = (uint64_t)blockIdx.x * per_group;
  for (uint32_t k = t; k < per_group; k += kHistThreads) {
    const uint64_t i = first + k;
    if (i >= n) break;
    const Fe s = scalar_plain(sc, i);
    for (int w = 0; w < windows; ++w) {
      const uint32_t d = digit(s, c, w);
      const uint64_t e = (uint64_t)w * n + i;
      digits[e] = (uint16_t)d;
      if (d) {
        const uint32_t sh = (d & 1u) * 16u;
        ranks[e] = (uint16_t)(atomicAdd(&h[d >> 1], 1u << sh) >> sh);
      }
    }
  }
  __syncthreads();
  uint32_t* row = hist + (uint64_t)blockIdx.x * nb;
  for (uint32_t d = t; d < nb; d += kHistThreads) row[d] = (h[d >> 1] >> ((d & 1u) * 16u)) & 0xFFFFu;
}

// Per bucket d: hist[g 2^c + d] <- the counts of d in groups before g, and
// counts[d] = the total.
__global__ void __launch_bounds__(256) column_scan_kernel(uint32_t* __restrict__ hist, uint32_t nb, uint32_t groups,
                                                          uint32_t* __restrict__ counts) {
  const uint32_t d = blockIdx.x * blockDim.x + threadIdx.x;
  if (d >= nb) return;
  uint32_t run = 0;
  for (uint32_t g = 0; g < groups; ++g) {
    const uint64_t k = (uint64_t)g * nb + d;
    const uint32_t v = hist[k];
    hist[k] = run;
    run += v;
  }
  counts[d] = run;
}

// Exclusive scan of counts[0 .. nb) into offsets[0 .. nb] (offsets[nb] =
// total), nb = 2^c <= 2^16.  One workgroup of 1024 threads; thread t keeps
// the run [t per, t per + per) of counts in registers (per <= 64; 16-byte
// loads and stores when per is a multiple of 4), and a tree over the runs'
// sums in LDS gives each run its start.
constexpr uint32_t kScanThreads = 1024, kScanPer = 64;

__global__ void __launch_bounds__(kScanThreads) scan_kernel(const uint32_t* __restrict__ counts, uint32_t nb,
                                                            uint32_t* __restrict__ offsets,
                                                            uint32_t* __restrict__ big_count) {
  __shared__ uint32_t part[kScanThreads];
  const uint32_t t = threadIdx.x;
  const uint32_t per = (nb + kScanThreads - 1) / kScanThreads;
  const uint32_t lo = t * per;
  const bool vec = (per & 3u) == 0;
  uint32_t v[kScanPer];
#pragma unroll
  for (uint32_t q = 0; q < kScanPer / 4; ++q) {
    if (vec && 4 * q < per) {
      const uint4 u = reinterpret_cast<const uint4*>(counts + lo)[q];
      v[4 * q] = u.x, v[4 * q + 1] = u.y, v[4 * q + 2] = u.z, v[4 * q + 3] = u.w;
    } else {
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t j = 4 * q + r;
        v[j] = !vec && j < per && lo + j < nb ? counts[lo + j] : 0u;
      }
    }
  }
  uint32_t s = 0;
#pragma unroll
  for (uint32_t j = 0; j < kScanPer; ++j) s += j < per ? v[j] : 0u;
  part[t] = s;
  __syncthreads();
  for (uint32_t off = 1; off < kScanThreads; off <<= 1) {
    const uint32_t x = t >= off ? part[t - off] : 0u;
    __syncthreads();
    part[t] += x;
    __syncthreads();
  }
  uint32_t run = part[t] - s;  // exclusive prefix of this run
#pragma unroll
  for (uint32_t j = 0; j < kScanPer; ++j) {
    const uint32_t x = v[j];
    v[j] = run;
    run += j < per ? x : 0u;
  }
#pragma unroll
  for (uint32_t q = 0; q < kScanPer / 4; ++q) {
    if (vec && 4 * q < per) {
      reinterpret_cast<uint4*>(offsets + lo)[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t j = 4 * q + r;
        if (!vec && j < per && lo + j < nb) offsets[lo + j] = v[j];
      }
    }
  }
  if (t == kScanThreads - 1) offsets[nb] = part[kScanThreads - 1];
  if (t < 2) big_count[t] = 0u;  // the combine step's lists of large buckets start empty
}

// entries[offsets[d] + (earlier groups' count of d) + rank] = w n + i for
// every nonzero digit d: one thread per entry, no atomics.  Workgroup L takes
// window L mod W of scalar block L / W, so that the workgroups in flight at
// once read the histogram rows of a few groups, which stay in L2.
__global__ void __launch_bounds__(256) scatter_kernel(const uint16_t* __restrict__ digits,
                                                      const uint16_t* __restrict__ ranks, uint64_t n, int windows,
                                                      uint32_t per_group, uint32_t nb,
                                                      const uint32_t* __restrict__ hist,
                                                      const uint32_t* __restrict__ offsets,
                                                      uint32_t* __restrict__ entries) {
  const uint32_t w = blockIdx.x % (uint32_t)windows, blk = blockIdx.x / (uint32_t)windows;
  const uint64_t i = (uint64_t)blk * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t e = (uint64_t)w * n + i;
  const uint32_t d = digits[e];
  if (d) entries[offsets[d] + hist[(i / per_group) * nb + d] + ranks[e]] = (uint32_t)e;
}

// ---------------------------------------------------------------------------
// Bucket accumulation, balanced over lanes.  The E sorted entries are cut
// into runs of K = max(kmin, ceil(E / lanes)) consecutive positions, one run
// per lane, whatever the bucket sizes: every lane does the same number of
// mixed additions, and the grid is sized to the device's resident waves, so
// that the accumulation is one round of equal lanes.  A run crosses bucket
// boundaries: lane j keeps one accumulator per bucket segment of its run and
// stores the segment containing the run's first position in head[j], the one
// containing its last position (when it is another) in tail[j], and every
// segment between them, a whole bucket, straight into buckets[d].

__device__ __forceinline__ uint32_t lane_span(uint32_t E, uint32_t lanes, uint32_t kmin) {
  return max(kmin, (uint32_t)(((uint64_t)E + lanes - 1) / lanes));
}

constexpr uint32_t kAccumulateThreads = 128;

__global__ void __launch_bounds__(kAccumulateThreads, 2) accumulate_kernel(const uint32_t* __restrict__ table,
                                                         const uint32_t* __restrict__ entries,
                                                         const uint32_t* __restrict__ offsets, uint32_t nb,
                                                         uint32_t lanes, uint32_t kmin, uint32_t* __restrict__ head,
                                                         uint32_t* __restrict__ tail,
                                                         uint32_t* __restrict__ buckets) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= lanes) return;
  const uint32_t E = offsets[nb];
  const uint32_t K = lane_span(E, lanes, kmin);
  const uint64_t start = (uint64_t)j * K;
  if (start >= E) return;
  const uint32_t lo_pos = (uint32_t)start;
  const uint32_t end = (uint32_t)min<uint64_t>(start + K, E);
  // the bucket holding position lo_pos: offsets[cur] <= lo_pos < offsets[cur + 1]
  uint32_t lo = 0, hi = nb;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (offsets[mid] <= lo_pos) lo = mid; else hi = mid;
  }
  uint32_t cur = lo, next = offsets[cur + 1];
  bool first = true, empty = true;  // empty: the accumulator is infinity
  Xyzz acc = infinity();
  Packed next_pt = load_packed(table, entries[lo_pos]);
#pragma unroll 1
  for (uint32_t k = lo_pos; k < end; ++k) {
    const Packed pt = next_pt;  // loaded one addition ahead
    if (k + 1 < end) next_pt = load_packed(table, entries[k + 1]);
    if (k == next) {  // bucket cur ends before position k
      if (first) store_xyzz(head, j, acc); else store_xyzz(buckets, cur, acc);
      first = false;
      empty = true;
      do {
        ++cur;
        next = offsets[cur + 1];
      } while (next <= k);  // skip empty buckets
    }
    const Affine a = unpack(pt);
    if (empty) {
      acc = from_affine(a);
      empty = false;
    } else {
      acc = add_mixed(acc, a, empty);
    }
  }
  if (first) store_xyzz(head, j, acc); else store_xyzz(tail, j, acc);
}

// Bucket d from the lanes' segments: the segment in the lane holding its
// first position (that lane's head or tail), plus the heads of the lanes
// that start inside it, by one quad.  A bucket that begins and ends strictly
// inside one lane's run was stored by that lane; an empty bucket is infinity.
// A bucket spanning more than kCombineSerial runs (skewed scalars: many equal
// digits) is listed for the big-bucket kernels, kBigRuns runs an item.

__global__ void __launch_bounds__(256) combine_kernel(const uint32_t* __restrict__ offsets, uint32_t nb,
                                                      uint32_t lanes, uint32_t kmin,
                                                      const uint32_t* __restrict__ head,
                                                      const uint32_t* __restrict__ tail,
                                                      uint32_t* __restrict__ buckets, BigLists big) {
  const uint32_t d = (blockIdx.x * blockDim.x + threadIdx.x) / 4;
  const uint32_t lo = d < nb ? offsets[d] : 0u, hi = d < nb ? offsets[d + 1] : 0u;
  const uint32_t E = offsets[nb];
  const uint32_t K = lane_span(E, lanes, kmin);
  uint32_t j = 1, jh = 0;  // runs j .. jh are still to be added
  bool store = d < nb;
  Fq acc = q_infinity();
  if (lo < hi) {
    const uint32_t jl = lo / K;
    jh = (hi - 1) / K;
    j = jl + 1;
    const uint64_t run_end = min<uint64_t>((uint64_t)(jl + 1) * K, E);
    if (jh - jl > kCombineSerial) {
      if (quad_lane() == 0) {
        const uint32_t items = (jh - jl + kBigRuns - 1) / kBigRuns;
        const uint32_t at = atomicAdd(&big.count[1], items);
        const uint32_t b = atomicAdd(&big.count[0], 1u);
        big.bucket[b] = make_uint4(d, at, items, 0u);
        for (uint32_t k = 0; k < items; ++k) big.item[at + k] = b;
      }
      store = false;
      jh = 0;
    } else if (lo == jl * K) {
      acc = q_load(head, jl);
    } else if (hi >= run_end) {
      acc = q_load(tail, jl);
    } else {
      store = false;  // stored by its lane
    }
  }
  while (__any(j <= jh)) {
    const Fq x = j <= jh ? q_load(head, j) : q_infinity();
    acc = q_add(acc, x);
    ++j;
  }
  if (store) q_store(buckets, d, acc);
}

// Sum of the workgroup's points, one per quad, in quad 0 (a power of two of
// quads; sh: one point per quad).
__device__ __forceinline__ Fq quads_sum(Fq p, uint32_t* sh) {
  const uint32_t g = threadIdx.x / 4;
  q_store(sh, g, p);
  __syncthreads();
  for (uint32_t half = blockDim.x / 8; half > 0; half >>= 1) {
    const bool mine = g < half;
    if (__any(mine)) {
      p = q_add(p, mine ? q_load(sh, g + half) : q_infinity());
    }
    __syncthreads();
    if (mine) q_store(sh, g, p);
    __syncthreads();
  }
  return p;
}

constexpr int kBigThreads = 256;

// One item of a listed bucket: the heads of kBigRuns of the runs that start
// inside it, and with the first item the segment of the run it starts in (it
// spans more than one run, so that is the head or the tail of that lane).
__global__ void __launch_bounds__(kBigThreads) big_item_kernel(const uint32_t* __restrict__ offsets, uint32_t nb,
                                                               uint32_t lanes, uint32_t kmin,
                                                               const uint32_t* __restrict__ head,
                                                               const uint32_t* __restrict__ tail, BigLists big) {
  __shared__ alignas(16) uint32_t sh[kBigThreads / 4 * kAccWords];
  const uint32_t items = big.count[1], g = threadIdx.x / 4;
  const uint32_t E = offsets[nb];
  const uint32_t K = lane_span(E, lanes, kmin);
  for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {  // the same for every thread of the workgroup
    const uint4 b = big.bucket[big.item[it]];
    const uint32_t d = b.x, part = it - b.y;
    const uint32_t lo = offsets[d], hi = offsets[d + 1];
    const uint32_t jl = lo / K, jh = (hi - 1) / K;
    Fq acc = q_infinity();
    if (part == 0 && g == 0) acc = lo == jl * K ? q_load(head, jl) : q_load(tail, jl);
    const uint32_t first = jl + 1 + part * kBigRuns;
    for (uint32_t k = 0; k < kBigRuns; k += kBigThreads / 4) {
      const uint32_t j = first + k + g;
      const bool have = j <= jh;
      if (__any(have)) acc = q_add(acc, have ? q_load(head, j) : q_infinity());
    }
    acc = quads_sum(acc, sh);
    if (g == 0) q_store(big.part, it, acc);
  }
}

// The listed buckets from their items' sums.
__global__ void __launch_bounds__(kBigThreads) big_bucket_kernel(BigLists big, uint32_t* __restrict__ buckets) {
  __shared__ alignas(16) uint32_t sh[kBigThreads / 4 * kAccWords];
  const uint32_t n = big.count[0], g = threadIdx.x / 4;
  for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
    const uint4 b = big.bucket[k];
    Fq acc = q_infinity();
    for (uint32_t i = 0; i < b.z; i += kBigThreads / 4) {
      const bool have = i + g < b.z;
      if (__any(have)) acc = q_add(acc, have ? q_load(big.part, b.y + i + g) : q_infinity());
    }
    acc = quads_sum(acc, sh);
    if (g == 0) q_store(buckets, b.x, acc);
  }
}

// ---------------------------------------------------------------------------
// Reduction by bits.  A binary tree over the buckets: node i of level l is the
// sum of buckets i 2^l .. (i + 1) 2^l - 1, and G_l is the sum of the odd nodes
// of level l.  A workgroup holds 2^levels points (its S list) and, level by
// level, adds neighbours in every list it has (S, and the odd nodes of the
// levels below) and starts a list with the odd nodes of this one, so that
// each level is at most 2^(levels - 1) additions at the same time, one per
// quad.  It ends with one point per list: S, G_0, .., G_(levels-1).
constexpr int kTreeThreads = 512;

// in: 2^levels points; lists: true for the whole scheme, false for S alone.
// Returns list t in quad t.
__device__ __forceinline__ Fq tree_lists(const uint32_t* __restrict__ in, int levels, bool lists, uint32_t* sh) {
  const uint32_t g = threadIdx.x / 4;
  if (levels == 0) return g == 0 ? q_load(in, 0) : q_infinity();
  for (int l = 0; l < levels; ++l) {
    const uint32_t half = 1u << (levels - l - 1);       // points of a list after this level
    const uint32_t nlists = lists ? (uint32_t)l + 1u : 1u;
    const bool mine = g < nlists * half;
    const uint32_t* src = l == 0 ? in : sh;
    Fq a = q_infinity(), b = a, s = a;
    if (mine) {
      a = q_load(src, 2 * g);  // list g / half, points 2 (g mod half) and the next
      b = q_load(src, 2 * g + 1);
    }
    if (__any(mine)) s = q_add(a, b);
    __syncthreads();
    if (mine) {
      q_store(sh, g, s);
      if (lists && g < half) q_store(sh, nlists * half + g, b);  // the odd nodes of this level
    }
    __syncthreads();
  }
  const uint32_t n = lists ? (uint32_t)levels + 1u : 1u;
  return g < n ? q_load(sh, g) : q_infinity();
}

// Workgroup k: 2^levels buckets from k 2^levels; list t's result to
// out[t nblk + k] (t = 0: S, 1 + b: G_b).
__global__ void __launch_bounds__(kTreeThreads) tree_kernel(const uint32_t* __restrict__ buckets, int levels,
                                                            uint32_t* __restrict__ out) {
  __shared__ alignas(16) uint32_t sh[2 * (kTreeThreads / 4) * kAccWords];
  const uint32_t g = threadIdx.x / 4;
  const Fq r = tree_lists(buckets + ((uint64_t)blockIdx.x << levels) * kAccWords, levels, true, sh);
  if (g <= (uint32_t)levels) q_store(out, (uint64_t)g * gridDim.x + blockIdx.x, r);
}

// The workgroups' results, 2^levels per list: workgroup t > 0 sums list t
// into G_(t-1); workgroup 0 runs the scheme on the S list, whose bits are
// those above the first kernel's `below`.
__global__ void __launch_bounds__(kTreeThreads) tree_top_kernel(const uint32_t* __restrict__ in, int levels, int below,
                                                                uint32_t* __restrict__ G) {
  __shared__ alignas(16) uint32_t sh[2 * (kTreeThreads / 4) * kAccWords];
  const uint32_t g = threadIdx.x / 4, t = blockIdx.x;
  const Fq r = tree_lists(in + ((uint64_t)t << levels) * kAccWords, levels, t == 0, sh);
  if (t > 0) {
    if (g == 0) q_store(G, t - 1, r);
  } else if (g >= 1 && g <= (uint32_t)levels) {
    q_store(G, (uint64_t)below + g - 1, r);
  }
}

// result = sum_b 2^b G_b (b < c <= 16): quad b doubles G_b b times, then a
// tree sums the c scaled points.
__global__ void __launch_bounds__(64) final_kernel(const uint32_t* __restrict__ G, int c, uint32_t* __restrict__ res) {
  __shared__ alignas(16) uint32_t sh[16 * kAccWords];
  const int b = (int)threadIdx.x / 4;
  Fq p = b < c ? q_load(G, (uint64_t)b) : q_infinity();
#pragma unroll 1
  for (int k = 0; k + 1 < c; ++k) {
    const Fq two = q_dbl(p);
    p = sel(k < b && b < c, two, p);
  }
  p = quads_sum(p, sh);
  if (b == 0) {
    // the result leaves the device canonical, in Montgomery form 2^384
    uint32_t w[fq::kWords];
    fq::pack_canonical(w, fq::mul(p, fq::constant(fq::kTo384)));
#pragma unroll
    for (int k = 0; k < fq::kWords; ++k) res[fq::kWords * quad_lane() + k] = w[k];
  }
}

inline uint32_t blocks(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

}  // namespace

hipError_t launch_precompute(const uint32_t* pts, uint64_t n, uint64_t first, uint64_t count, int c, int windows,
                             uint32_t* table, uint32_t* scratch, hipStream_t s) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(precompute_kernel, dim3(blocks(count, 128)), dim3(128), 0, s, pts, n, first, count, c, windows,
                     table, scratch);
  return hipGetLastError();
}

hipError_t accumulate_lanes(uint32_t* lanes) {
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(accumulate_kernel),
                                                     kAccumulateThreads, 0);
  if (e != hipSuccess) return e;
  *lanes = (uint32_t)std::max(1, cus * std::max(1, per_cu)) * kAccumulateThreads;
  return hipSuccess;
}

hipError_t launch_msm(const MsmLaunch& m, hipStream_t s) {
  const uint32_t nb = 1u << m.c;  // bucket 0 unused
  hipError_t e;
  // counting sort: group histograms, their column prefixes, bucket offsets,
  // then the scatter
  hipLaunchKernelGGL(hist_kernel, dim3(m.groups), dim3(kHistThreads), 0, s, m.scalars, m.n, m.c, m.windows,
                     m.per_group, m.digits, m.ranks, m.hist);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(column_scan_kernel, dim3(blocks(nb, 256)), dim3(256), 0, s, m.hist, nb, m.groups, m.counts);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanThreads), 0, s, m.counts, nb, m.offsets, m.big.count);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks(m.n, 256) * (uint32_t)m.windows), dim3(256), 0, s, m.digits,
                     m.ranks, m.n, m.windows, m.per_group, nb, m.hist, m.offsets, m.entries);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // bucket sums: equal runs of sorted entries per lane, then the runs'
  // boundary segments into their buckets
  hipLaunchKernelGGL(accumulate_kernel, dim3(blocks(m.lanes, kAccumulateThreads)), dim3(kAccumulateThreads), 0, s,
                     m.table, m.entries, m.offsets, nb, m.lanes, m.kmin, m.head, m.tail, m.buckets);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(combine_kernel, dim3(blocks((uint64_t)nb * 4, 256)), dim3(256), 0, s, m.offsets, nb, m.lanes,
                     m.kmin, m.head, m.tail, m.buckets, m.big);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const uint32_t item_blocks = std::min<uint32_t>(max_big_items(m.lanes), 512u);
  hipLaunchKernelGGL(big_item_kernel, dim3(item_blocks), dim3(kBigThreads), 0, s, m.offsets, nb, m.lanes, m.kmin,
                     m.head, m.tail, m.big);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(big_bucket_kernel, dim3(std::min<uint32_t>(max_big_buckets(m.lanes), 512u)), dim3(kBigThreads), 0,
                     s, m.big, m.buckets);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // reduction by bits
  const int low = std::min(m.c, kTreeLevels);
  hipLaunchKernelGGL(tree_kernel, dim3(1u << (m.c - low)), dim3(kTreeThreads), 0, s, m.buckets, low, m.level_a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(tree_top_kernel, dim3(1 + low), dim3(kTreeThreads), 0, s, m.level_a, m.c - low, low, m.level_b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(final_kernel, dim3(1), dim3(64), 0, s, m.level_b, m.c, m.result);
  return hipGetLastError();
}

}  // namespace msm
}  // namespace zk
