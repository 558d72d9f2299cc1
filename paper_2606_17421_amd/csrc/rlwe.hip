// Symmetric RLWE encryption, decryption and the decrypt-then-encrypt refresh
// (gfx950), batched over ciphertexts [count][2][limbs][N] in NTT form.
//
// Encryption (the ciphertext form of section 2.1, made by the trusted side in
// section 3.2): c0 = pt + NTT(e) - a (.) s, c1 = a, per limb, with the
// secret s and the fresh randomness a (uniform, NTT form) and e (small
// integer coefficients) supplied by the caller.  Decryption: the coefficient
// residues INTT(c0 + c1 (.) s) per limb.  Refresh (the DtE equation of
// section 3.2, ct' = Enc(Dec(ct))): the integer plaintext polynomial is
// recovered from limbs 0 and 1 by CRT to centred integers (exact while its
// coefficients lie within q0 q1 / 2 in magnitude) and encrypted afresh under
// limbs_out limbs.
//
// Encryption and decryption, up to N = 2^15, are one kernel each: the error's
// residues (or c0 + c1 (.) s) are formed as the transform loads its row and the
// combine (or the coefficients) leave with its stores.  At 2^16 (a row exceeds the LDS) the same
// work rides on the first and last passes of the staged transforms.  100
// features at 2^16 and 8 limbs, encoded, encrypted and decrypted: 1065 -> 815 us
// (separate error, transform and pointwise passes before; the encoding, 400 us,
// is the same in both); 500 of 2^14 and 4 limbs 478 -> 322 us.  These kernels and
// the refresh's run on the latency plan at every count: their loads and Barrett
// products beside the butterflies gain more from twice the waves a SIMD than
// the butterflies lose to a fourth group.  On the other plan : on this one, us, 4
// limbs, encrypt / decrypt / refresh: 16 of 2^13 9.5 : 9.1 / 8.8 : 8.1 / fused, 200
// of 2^13 27.2 : 24.9 / 27.0 : 25.2 / 51.7 : 49.0, 768 of 2^13 106 : 95 / 84 : 75 /
// 160 : 150, 16 of 2^14 15.1 : 14.4 / 15.1 : 13.2 / 36.2 : 32.8, 768 of 2^14 203 :
// 198 / 184 : 161 / 328 : 314 (the two plans are one at the other sizes).  The
// refresh, up to N = 2^15, is two transform kernels (decrypt + inverse, lift +
// forward + combine), or up to 2^13 for decode-size counts one fused kernel split
// by output limb; at 2^16 the staged passes of decryption and encryption around
// the lift.
#include <type_traits>

#include "ntt_core.hpp"

namespace ckks {
namespace {

constexpr int kThreads = 256;  // pointwise kernels

// Signed 64-bit x mod q, in [0, q).
__device__ __forceinline__ uint32_t reduce_i64(int64_t x, uint32_t q, double qr) {
  const uint64_t ax = static_cast<uint64_t>(x < 0 ? -x : x);
  const uint32_t r = reduce_u64(ax, q, qr);
  return (x < 0 && r != 0) ? q - r : r;
}

// 16-byte accesses use native vector types.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int32_t v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4u ld4(const uint32_t* p) { return *reinterpret_cast<const v4u*>(p); }
__device__ __forceinline__ v4s ld4(const int32_t* p) { return *reinterpret_cast<const v4s*>(p); }
__device__ __forceinline__ void st4(uint32_t* p, v4u v) { *reinterpret_cast<v4u*>(p) = v; }

// floor(w 2^32 / q) for w < q (the Shoup companion of w): the fp64 estimate is
// within one of it, and one remainder check fixes it.
__device__ __forceinline__ uint32_t shoup_const(uint32_t w, uint32_t q, double qr) {
  uint32_t ws = static_cast<uint32_t>(static_cast<double>(w) * 4294967296.0 * qr);
  const int64_t r = static_cast<int64_t>((static_cast<uint64_t>(w) << 32) - static_cast<uint64_t>(ws) * q);
  if (r < 0) --ws;
  else if (r >= static_cast<int64_t>(q)) ++ws;
  return ws;
}

// e mod q for |e| < q.
__device__ __forceinline__ uint32_t small_residue(int32_t e, uint32_t q) {
  return e < 0 ? static_cast<uint32_t>(e) + q : static_cast<uint32_t>(e);
}

// (x0 + q0 k - [neg] q0 q1 + e) mod q_l, the refreshed residue of one
// coefficient: x0 < q0 and k < q1 are the CRT digits, neg the centring flag,
// |e| < q_l the fresh error.  With ka = k + [neg](2 q - q1) (< 2^32; 2 q >
// q1) the centring folds into the product q0 ka = q0 k - [neg] q0 q1 (mod q);
// the lazy Shoup product lies in [0, 2q), so x0 mod q + product + e mod q lies
// in [0, 4q) < 2^32 and two conditional subtractions finish.
struct LiftConst {
  uint32_t q, q0l, q0ls, d2;
};
__device__ __forceinline__ LiftConst lift_const(uint32_t q0, uint32_t q1, uint32_t q, double qr) {
  LiftConst c;
  c.q = q;
  c.q0l = q0 >= q ? q0 - q : q0;  // q0 < 2q
  c.q0ls = shoup_const(c.q0l, q, qr);
  c.d2 = 2 * q - q1;
  return c;
}
__device__ __forceinline__ uint32_t lift_residue(const LiftConst& c, uint32_t x0, uint32_t k, bool neg, int32_t e) {
  const uint32_t ka = neg ? k + c.d2 : k;
  const uint32_t p = mul_shoup_lazy(ka, c.q0l, c.q0ls, c.q);
  const uint32_t x0l = min(x0, x0 - c.q);
  uint32_t t = x0l + p + small_residue(e, c.q);
  t = min(t, t - 2 * c.q);
  return min(t, t - c.q);
}

// Buffer resource over one row of N words (row bases live in scalar
// registers; per-lane offsets and per-element constants index into it).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, uint32_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, n * 4, 0x00020000);
}

// Fused refresh for N <= 2^13 and at most one workgroup per CU (a decode-size
// group): one workgroup per ciphertext and output limb.  Limbs 0
// and 1 of c0 + c1 (.) s are read coalesced and inverse-transformed in LDS;
// the CRT value over q0 q1 is kept as its two digits x = x0 + q0 k (k with the
// centring flag in bit 31) in the group-0 layout that the forward transform
// starts from, rebuilt mod q_l with 32-bit Barrett products, the fresh error
// added, transformed, combined with a and s and written coalesced.  The two
// inverse transforms are repeated per output limb, so the chain per workgroup
// is three transforms on limbs_out times the workgroups.  16 residues per
// thread (1024 threads at 2^14) keeps the live state in registers.
template <int LOGN>
struct RefreshPlan {
  static_assert(LOGN <= 13, "the fused refresh serves N <= 2^13");
  static constexpr int LOGE = 4;
  using P = Plan<LOGN, LOGE>;
  static constexpr int kWavesPerSimd = 4;
};

template <int LOGN>
__global__ __launch_bounds__(RefreshPlan<LOGN>::P::T, RefreshPlan<LOGN>::kWavesPerSimd) void refresh_kernel(
    Tables tb, const uint32_t* __restrict__ ct_in, uint32_t limbs_in, const uint32_t* __restrict__ s_ntt,
    const uint32_t* __restrict__ a, const int32_t* __restrict__ e, uint32_t limbs_out,
    uint32_t* __restrict__ ct_out) {
  using P = typename RefreshPlan<LOGN>::P;
  constexpr int LOGE = RefreshPlan<LOGN>::LOGE;
  constexpr int N = P::B;
  __shared__ uint32_t lds[P::lds_words];
  const size_t c = blockIdx.x;
  const uint32_t t = threadIdx.x;
  const uint32_t vofs = pos_coalesced<LOGE>(t, 0) * 4;  // byte offset of element 0 in the coalesced layout

  uint32_t x0[P::E], v[P::E];
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    const uint32_t q = tb.q[l], mu = tb.barrett[l];
    const auto r_c0 = row_rsrc(ct_in + ((c * 2) * limbs_in + l) * N, N);
    const auto r_c1 = row_rsrc(ct_in + ((c * 2 + 1) * limbs_in + l) * N, N);
    const auto r_s = row_rsrc(s_ntt + static_cast<size_t>(l) * N, N);
    if (l == 1) __syncthreads();  // the last (workgroup-wide) exchange of limb 0 is read out
#pragma unroll
    for (int j = 0; j < P::E; ++j) {
      const uint32_t c0 = __builtin_amdgcn_raw_buffer_load_b32(r_c0, vofs, j << 8, 0);
      const uint32_t c1 = __builtin_amdgcn_raw_buffer_load_b32(r_c1, vofs, j << 8, 0);
      const uint32_t sv = __builtin_amdgcn_raw_buffer_load_b32(r_s, vofs, j << 8, 0);
      v[j] = add_mod(c0, mul_mod_barrett(c1, sv, q, mu), q);
    }
    wave_relayout<LOGN, LOGE, true>(v, t, lds);
    const size_t tl = static_cast<size_t>(l) << LOGN;
    inv_block<LOGN, LOGN, LOGE>(v, t, 0, tb.inv + tl, tb.inv_shoup + tl, q, lds);
    const uint32_t ni = tb.ninv[l], nis = tb.ninv_shoup[l];
#pragma unroll
    for (int j = 0; j < P::E; ++j) {
      v[j] = mul_shoup(v[j], ni, nis, q);
      if (l == 0) x0[j] = v[j];
    }
  }
  // CRT digits: x = x0 + q0 k in [0, q0 q1), k = (r1 - r0) q0^-1 mod q1;
  // bit 31 of kf marks x > q0 q1 / 2 (centred value x - q0 q1).
  const uint32_t q0 = tb.q[0], q1 = tb.q[1];
  const uint32_t w = tb.qinv[0 * tb.L + 1], ws = tb.qinv_shoup[0 * tb.L + 1];  // q0^-1 mod q1
  const uint64_t half = static_cast<uint64_t>(q0) * q1 / 2;
  uint32_t kf[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j) {
    const uint32_t r0m = x0[j] >= q1 ? x0[j] - q1 : x0[j];  // x0 < q0 < 2 q1
    const uint32_t k = mul_shoup(sub_mod(v[j], r0m, q1), w, ws, q1);
    const uint64_t x = static_cast<uint64_t>(x0[j]) + static_cast<uint64_t>(q0) * k;
    kf[j] = k | (x > half ? 0x80000000u : 0u);
  }
  // the error row through a buffer resource: the per-j offsets j T are scalar constants
  const auto er = row_rsrc(e + c * N, N);
  {
    const uint32_t l = blockIdx.y;
    const uint32_t q = tb.q[l], mu = tb.barrett[l];
    const LiftConst lc = lift_const(q0, q1, q, tb.q_recip[l]);
#pragma unroll
    for (int j = 0; j < P::E; ++j) {
      const int32_t ev = static_cast<int32_t>(
          __builtin_amdgcn_raw_buffer_load_b32(er, t * 4, P::template pos<0>(0, j) * 4, 0));
      v[j] = lift_residue(lc, x0[j], kf[j] & 0x7fffffffu, (kf[j] >> 31) != 0, ev);
    }
    const size_t tl = static_cast<size_t>(l) << LOGN;
    fwd_block<LOGN, LOGN, LOGE>(v, t, 0, tb.fwd + tl, tb.fwd_shoup + tl, q, lds);
    wave_relayout<LOGN, LOGE, false>(v, t, lds);
    const auto r_o0 = row_rsrc(ct_out + ((c * 2) * limbs_out + l) * N, N);
    const auto r_o1 = row_rsrc(ct_out + ((c * 2 + 1) * limbs_out + l) * N, N);
    const auto r_a = row_rsrc(a + (c * limbs_out + l) * N, N);
    const auto r_s = row_rsrc(s_ntt + static_cast<size_t>(l) * N, N);
#pragma unroll
    for (int j = 0; j < P::E; ++j) {
      const uint32_t av = __builtin_amdgcn_raw_buffer_load_b32(r_a, vofs, j << 8, 0);
      const uint32_t sv = __builtin_amdgcn_raw_buffer_load_b32(r_s, vofs, j << 8, 0);
      __builtin_amdgcn_raw_buffer_store_b32(sub_mod(v[j], mul_mod_barrett(av, sv, q, mu), q), r_o0, vofs, j << 8, 0);
      __builtin_amdgcn_raw_buffer_store_b32(av, r_o1, vofs, j << 8, 0);
    }
  }
}

// Two-kernel refresh for N <= 2^15: the same arithmetic as the fused kernel,
// with each transform in a workgroup of its own and the whole-row plan's
// occupancy (two workgroups per CU up to 2^14, one at 2^15).
// (1) per (ciphertext, limb 0 or 1): c0 + c1 (.) s read coalesced, inverse
//     transform, the coefficient residues written to c1 row 0 / 1 of ct_out
//     (scratch);
// (2) per (ciphertext, output limb): the CRT digits of the two scratch rows,
//     the value mod q_l plus the fresh error, the forward transform, and
//     c0 = . - a (.) s written coalesced;
// c1 = a: rows from 2 on by (2), rows 0 and 1 (the scratch) copied afterwards.
template <int LOGN>
__global__ __launch_bounds__((WholePlan<LOGN, true>::P::T), (WholePlan<LOGN, true>::kWavesPerSimd)) void dec_intt_kernel(
    Tables tb, const uint32_t* __restrict__ ct_in, uint32_t limbs_in, const uint32_t* __restrict__ s_ntt,
    uint32_t limbs_used, uint32_t* __restrict__ out, uint32_t out_gstride) {
  using P = typename WholePlan<LOGN, true>::P;
  constexpr int LOGE = WholePlan<LOGN, true>::LOGE;
  constexpr int N = P::B;
  __shared__ uint32_t lds[P::lds_words];
  const size_t c = blockIdx.x / limbs_used;
  const uint32_t l = blockIdx.x % limbs_used, t = threadIdx.x;
  const uint32_t q = tb.q[l], mu = tb.barrett[l];
  const uint32_t vofs = pos_coalesced<LOGE>(t, 0) * 4;
  const auto r_c0 = row_rsrc(ct_in + ((c * 2) * limbs_in + l) * N, N);
  const auto r_c1 = row_rsrc(ct_in + ((c * 2 + 1) * limbs_in + l) * N, N);
  const auto r_s = row_rsrc(s_ntt + static_cast<size_t>(l) * N, N);
  uint32_t v[P::E], xb[P::E], xs[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j) {
    v[j] = __builtin_amdgcn_raw_buffer_load_b32(r_c0, vofs, j << 8, 0);
    xb[j] = __builtin_amdgcn_raw_buffer_load_b32(r_c1, vofs, j << 8, 0);
    xs[j] = __builtin_amdgcn_raw_buffer_load_b32(r_s, vofs, j << 8, 0);
  }
#pragma unroll
  for (int j = 0; j < P::E; ++j) v[j] = add_mod(v[j], mul_mod_barrett(xb[j], xs[j], q, mu), q);
  wave_relayout<LOGN, LOGE, true>(v, t, lds);
  const size_t tl = static_cast<size_t>(l) << LOGN;
  inv_block<LOGN, LOGN, LOGE>(v, t, 0, tb.inv + tl, tb.inv_shoup + tl, q, lds);
  const uint32_t ni = tb.ninv[l], nis = tb.ninv_shoup[l];
  uint32_t* r = out + (c * out_gstride + l) * N;
#pragma unroll
  for (int j = 0; j < P::E; ++j) r[P::template pos<0>(t, j)] = mul_shoup(v[j], ni, nis, q);
}

template <int LOGN>
__global__ __launch_bounds__((WholePlan<LOGN, true>::P::T), (WholePlan<LOGN, true>::kWavesPerSimd)) void dte_lift_ntt_kernel(
    Tables tb, const int32_t* __restrict__ e, const uint32_t* __restrict__ s_ntt, const uint32_t* __restrict__ a,
    uint32_t limbs_out, uint32_t* __restrict__ ct_out) {
  using P = typename WholePlan<LOGN, true>::P;
  constexpr int LOGE = WholePlan<LOGN, true>::LOGE;
  constexpr int N = P::B;
  __shared__ uint32_t lds[P::lds_words];
  // logical id = c * limbs_out + l.  Consecutive workgroup ids alternate XCDs, so
  // each XCD is given a contiguous range of logical ids: the limbs of one
  // ciphertext then run together on one XCD and read its two scratch rows and
  // its error row from HBM once, the other limbs from that XCD's L2.
  const uint32_t G = gridDim.x;
  uint32_t lid = blockIdx.x;
  if ((G & 7u) == 0) lid = (lid & 7u) * (G >> 3) + (lid >> 3);
  const size_t c = lid / limbs_out;
  const uint32_t l = lid % limbs_out, t = threadIdx.x;
  // scratch rows: coefficient residues mod q0, q1; element j of thread t of the
  // group-0 layout sits at t + T j (buffer loads: the offset j T is a constant)
  const auto rr0 = row_rsrc(ct_out + ((c * 2 + 1) * limbs_out) * N, N);
  const auto rr1 = row_rsrc(ct_out + ((c * 2 + 1) * limbs_out + 1) * N, N);
  const auto rer = row_rsrc(e + c * N, N);
  const uint32_t q0 = tb.q[0], q1 = tb.q[1];
  const uint32_t w = tb.qinv[0 * tb.L + 1], ws = tb.qinv_shoup[0 * tb.L + 1];  // q0^-1 mod q1
  const uint64_t half = static_cast<uint64_t>(q0) * q1 / 2;
  const uint32_t q = tb.q[l], mu = tb.barrett[l];
  const LiftConst lc = lift_const(q0, q1, q, tb.q_recip[l]);
  uint32_t v[P::E];
  // keeps the element loads below the per-limb constants: scheduled above them,
  // the loads' live ranges spill registers
  __builtin_amdgcn_sched_barrier(0);
  // loads in batches of 8 elements, each batch issued before the previous one is
  // used (group 0: element j of thread t at t + T j)
  constexpr int kB = 8;
  uint32_t xa[2][kB], xb[2][kB];
  int32_t ea[2][kB];
  auto load = [&](int set, int j0) {
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const uint32_t jo = P::template pos<0>(0, j0 + i) * 4;
      xa[set][i] = __builtin_amdgcn_raw_buffer_load_b32(rr0, t * 4, jo, 0);
      xb[set][i] = __builtin_amdgcn_raw_buffer_load_b32(rr1, t * 4, jo, 0);
      ea[set][i] = static_cast<int32_t>(__builtin_amdgcn_raw_buffer_load_b32(rer, t * 4, jo, 0));
    }
  };
  load(0, 0);
#pragma unroll
  for (int j0 = 0; j0 < P::E; j0 += kB) {
    const int cur = (j0 / kB) & 1;
    if (j0 + kB < P::E) load(cur ^ 1, j0 + kB);
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const uint32_t x0 = xa[cur][i];
      const uint32_t r0m = x0 >= q1 ? x0 - q1 : x0;                          // x0 < q0 < 2 q1
      const uint32_t k = mul_shoup(sub_mod(xb[cur][i], r0m, q1), w, ws, q1);
      const bool neg = static_cast<uint64_t>(x0) + static_cast<uint64_t>(q0) * k > half;
      v[j0 + i] = lift_residue(lc, x0, k, neg, ea[cur][i]);
    }
  }
  const size_t tl = static_cast<size_t>(l) << LOGN;
  fwd_block<LOGN, LOGN, LOGE>(v, t, 0, tb.fwd + tl, tb.fwd_shoup + tl, q, lds);
  wave_relayout<LOGN, LOGE, false>(v, t, lds);
  __builtin_amdgcn_sched_barrier(0);  // the combine's loads stay after the transform
  const uint32_t vofs = pos_coalesced<LOGE>(t, 0) * 4;
  const auto ra = row_rsrc(a + (c * limbs_out + l) * N, N);
  const auto rs = row_rsrc(s_ntt + static_cast<size_t>(l) * N, N);
  const auto ro = row_rsrc(ct_out + ((c * 2) * limbs_out + l) * N, N);
  const auto ro1 = row_rsrc(ct_out + ((c * 2 + 1) * limbs_out + l) * N, N);  // c1 row l (rows 0, 1 are the scratch)
  uint32_t ya[2][kB], ys[2][kB];
  auto load_as = [&](int set, int j0) {
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      ya[set][i] = __builtin_amdgcn_raw_buffer_load_b32(ra, vofs, (j0 + i) << 8, 0);
      ys[set][i] = __builtin_amdgcn_raw_buffer_load_b32(rs, vofs, (j0 + i) << 8, 0);
    }
  };
  load_as(0, 0);
#pragma unroll
  for (int j0 = 0; j0 < P::E; j0 += kB) {
    const int cur = (j0 / kB) & 1;
    if (j0 + kB < P::E) load_as(cur ^ 1, j0 + kB);
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const uint32_t ax = ya[cur][i];
      __builtin_amdgcn_raw_buffer_store_b32(sub_mod(v[j0 + i], mul_mod_barrett(ax, ys[cur][i], q, mu), q), ro, vofs,
                                            (j0 + i) << 8, 0);
      if (l >= 2) __builtin_amdgcn_raw_buffer_store_b32(ax, ro1, vofs, (j0 + i) << 8, 0);
    }
  }
}

// Elements of one row in the coalesced layout, as buffer loads in batches of kB,
// each batch issued before the previous one is used (x[0], x[1] alternate).
constexpr int kB = 8;
struct RowAt {
  __amdgpu_buffer_rsrc_t r;
  uint32_t ofs;
  __device__ __forceinline__ uint32_t load(int j) const { return __builtin_amdgcn_raw_buffer_load_b32(r, ofs, j << 8, 0); }
  __device__ __forceinline__ void store(uint32_t x, int j) const { __builtin_amdgcn_raw_buffer_store_b32(x, r, ofs, j << 8, 0); }
};

// c0 = v + pt - a (.) s and c1 = a for the elements j < E of one row (pt absent
// without kPt); every position 64 j + ofs / 4 of the row.
template <int E, bool kPt>
__device__ __forceinline__ void combine_row(const uint32_t (&v)[E], const RowAt& pt, const RowAt& a, const RowAt& s,
                                            const RowAt& c0, const RowAt& c1, uint32_t q, uint32_t mu) {
  constexpr int B = kB < E ? kB : E;
  uint32_t ya[2][B], ys[2][B], yp[2][B];
  auto load = [&](int set, int j0) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      ya[set][i] = a.load(j0 + i);
      ys[set][i] = s.load(j0 + i);
      if constexpr (kPt) yp[set][i] = pt.load(j0 + i);
    }
  };
  load(0, 0);
#pragma unroll
  for (int j0 = 0; j0 < E; j0 += B) {
    const int cur = (j0 / B) & 1;
    if (j0 + B < E) load(cur ^ 1, j0 + B);
#pragma unroll
    for (int i = 0; i < B; ++i) {
      uint32_t x = v[j0 + i];
      if constexpr (kPt) x = add_mod(x, yp[cur][i], q);
      c0.store(sub_mod(x, mul_mod_barrett(ya[cur][i], ys[cur][i], q, mu), q), j0 + i);
      c1.store(ya[cur][i], j0 + i);
    }
  }
}

// Encryption for N <= 2^15: one workgroup per (ciphertext, limb) row takes the
// error's residues through the forward transform and combines on the way out:
// 5 row transfers (e from L2 for all limbs but one) where error rows, a batched
// transform and a pointwise pass took 8.  The limbs of a ciphertext run
// together on one XCD and read its error row from HBM once.
template <int LOGN, bool kPt>
__global__ __launch_bounds__((WholePlan<LOGN, true>::P::T), (WholePlan<LOGN, true>::kWavesPerSimd)) void encrypt_kernel(
    Tables tb, const uint32_t* __restrict__ pt, const uint32_t* __restrict__ s_ntt, const uint32_t* __restrict__ a,
    const int32_t* __restrict__ e, uint32_t limbs, uint32_t* __restrict__ ct) {
  using P = typename WholePlan<LOGN, true>::P;
  constexpr int LOGE = WholePlan<LOGN, true>::LOGE;
  constexpr int N = P::B;
  __shared__ uint32_t lds[P::lds_words];
  const uint32_t G = gridDim.x;
  uint32_t lid = blockIdx.x;
  if ((G & 7u) == 0) lid = (lid & 7u) * (G >> 3) + (lid >> 3);
  const size_t c = lid / limbs;
  const uint32_t l = lid % limbs, t = threadIdx.x;
  const uint32_t q = tb.q[l], mu = tb.barrett[l];
  const auto er = row_rsrc(e + c * N, N);
  uint32_t v[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j)
    v[j] = small_residue(static_cast<int32_t>(__builtin_amdgcn_raw_buffer_load_b32(er, t * 4, P::template pos<0>(0, j) * 4, 0)), q);
  const size_t tl = static_cast<size_t>(l) << LOGN;
  fwd_block<LOGN, LOGN, LOGE>(v, t, 0, tb.fwd + tl, tb.fwd_shoup + tl, q, lds);
  wave_relayout<LOGN, LOGE, false>(v, t, lds);
  __builtin_amdgcn_sched_barrier(0);  // the combine's loads stay after the transform
  const uint32_t vofs = pos_coalesced<LOGE>(t, 0) * 4;
  const size_t row = (c * limbs + l) * N;
  combine_row<P::E, kPt>(v, {row_rsrc(kPt ? pt + row : nullptr, N), vofs}, {row_rsrc(a + row, N), vofs},
                         {row_rsrc(s_ntt + tl, N), vofs}, {row_rsrc(ct + ((c * 2) * limbs + l) * N, N), vofs},
                         {row_rsrc(ct + ((c * 2 + 1) * limbs + l) * N, N), vofs}, q, mu);
}

// ---- N = 2^16 (a row exceeds the LDS): the transforms' column and block passes
// of the batched kernels with the pointwise work folded into their first loads
// and last stores.  A column pass over the error forms each limb's residues as it
// loads; a block pass combines as it stores.
// Decryption's block pass forms c0 + c1 (.) s as it loads.  6 row transfers per
// limb for an encryption (10 with separate passes), 5 for a decryption (7).
constexpr int kColLogE = 6;
constexpr int kColThreads = 256;
constexpr int kColBlocks = (1 << (16 - kColLogE)) / kColThreads;
constexpr int kBlkLogB = 10;
constexpr int kBlkLogE = 4;
constexpr int kBlocksPerRow = 1 << (16 - kBlkLogB);

// Column pass of the c0 row (c, l) of ct [count][2][limbs][N], from the error, left
// in the lazy range.  The limbs of one ciphertext are numbered together on one
// XCD and share the error row.
__global__ __launch_bounds__(kColThreads, 2) void enc16_cols_kernel(Tables tb, const int32_t* __restrict__ e,
                                                                    uint32_t limbs, uint32_t* __restrict__ ct) {
  using P = Plan<16, kColLogE>;
  const uint32_t G = gridDim.x;
  uint32_t lid = blockIdx.x;
  if ((G & 7u) == 0) lid = (lid & 7u) * (G >> 3) + (lid >> 3);
  const uint32_t l = lid % limbs, cb = (lid / limbs) % kColBlocks;
  const size_t c = lid / limbs / kColBlocks;
  const uint32_t col = cb * kColThreads + threadIdx.x;
  const uint32_t q = tb.q[l];
  const int32_t* ec = e + (c << 16) + col;
  uint32_t v[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j) v[j] = small_residue(ec[P::template pos<0>(0, j)], q);
  const size_t tl = static_cast<size_t>(l) << 16;
  fwd_group<16, 16, kColLogE, 0>(v, col, 0, tb.fwd + tl, tb.fwd_shoup + tl, q);  // [0, 4q)
  uint32_t* o = ct + (((c * 2) * limbs + l) << 16) + col;
#pragma unroll
  for (int j = 0; j < P::E; ++j) __builtin_nontemporal_store(v[j], &o[P::template pos<0>(0, j)]);
}

// Thread -> (ciphertext c, coefficient quad k4) over count * N/4 quads.
struct Quad {
  size_t c;
  uint32_t k;
  bool ok;
};
__device__ __forceinline__ Quad quad_of(uint32_t n, uint32_t count) {
  const size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  const uint32_t per = n >> 2;
  Quad r;
  r.c = i / per;
  r.k = static_cast<uint32_t>(i % per) * 4;
  r.ok = r.c < count;
  return r;
}

// Refresh lift.  dec rows (c * 2 limbs_out + limbs_out + {0, 1}) hold the
// decrypted coefficient residues mod q0, q1.  x = r0 + q0 ((r1 - r0) q0^-1
// mod q1) is the CRT value in [0, q0 q1); centred, plus the fresh error, it
// is written mod q_l into the c0 rows of ct_out for l < limbs_out.
__global__ __launch_bounds__(kThreads) void dte_lift_kernel(Tables tb, const int32_t* __restrict__ e,
                                                            uint32_t count, uint32_t limbs_out,
                                                            uint32_t* __restrict__ ct_out) {
  const uint32_t n = tb.n;
  const Quad p = quad_of(n, count);
  if (!p.ok) return;
  const uint32_t q0 = tb.q[0], q1 = tb.q[1];
  const uint32_t w = tb.qinv[0 * tb.L + 1], ws = tb.qinv_shoup[0 * tb.L + 1];  // q0^-1 mod q1
  const uint64_t Q2 = static_cast<uint64_t>(q0) * q1;
  const uint32_t* d0 = ct_out + ((p.c * 2) * limbs_out + limbs_out) * n + p.k;
  const v4u r0v = ld4(d0);
  const v4u r1v = ld4(d0 + n);
  const v4s ev = ld4(e + p.c * n + p.k);
  int64_t m[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t r0 = r0v[j];
    const uint32_t r0m = r0 >= q1 ? r0 - q1 : r0;  // r0 < q0 < 2 q1
    const uint32_t t = mul_shoup(sub_mod(r1v[j], r0m, q1), w, ws, q1);
    const uint64_t x = static_cast<uint64_t>(r0) + static_cast<uint64_t>(q0) * t;  // [0, q0 q1)
    const int64_t xc = x > Q2 / 2 ? static_cast<int64_t>(x) - static_cast<int64_t>(Q2) : static_cast<int64_t>(x);
    m[j] = xc + ev[j];
  }
  for (uint32_t l = 0; l < limbs_out; ++l) {
    const uint32_t q = tb.q[l];
    const double qr = tb.q_recip[l];
    v4u o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = reduce_i64(m[j], q, qr);
    st4(ct_out + ((p.c * 2) * limbs_out + l) * n + p.k, o);
  }
}

// Block pass of the c0 rows of ct [count][2][limbs][N], in place, with the combine.
template <bool kPt>
__global__ __launch_bounds__(1 << (kBlkLogB - kBlkLogE)) void rlwe16_blocks_combine_kernel(
    Tables tb, const uint32_t* __restrict__ pt, const uint32_t* __restrict__ s_ntt, const uint32_t* __restrict__ a,
    uint32_t limbs, uint32_t* ct) {
  using P = Plan<kBlkLogB, kBlkLogE>;
  __shared__ uint32_t lds[P::lds_words];
  const size_t r = blockIdx.x / kBlocksPerRow;
  const uint32_t blk = blockIdx.x % kBlocksPerRow, t = threadIdx.x;
  const size_t c = r / limbs;
  const uint32_t l = static_cast<uint32_t>(r % limbs);
  const uint32_t q = tb.q[l], mu = tb.barrett[l];
  const size_t boff = static_cast<size_t>(blk) << kBlkLogB;
  uint32_t* c0 = ct + (((c * 2) * limbs + l) << 16) + boff;
  uint32_t v[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j) v[j] = __builtin_nontemporal_load(&c0[P::template pos<0>(t, j)]);
  const size_t tl = static_cast<size_t>(l) << 16;
  fwd_block<16, kBlkLogB, kBlkLogE>(v, t, blk, tb.fwd + tl, tb.fwd_shoup + tl, q, lds);
  wave_relayout<kBlkLogB, kBlkLogE, false>(v, t, lds);
  const size_t row = (r << 16) + boff;
  const uint32_t n = P::B;
  combine_row<P::E, kPt>(v, {row_rsrc(kPt ? pt + row : nullptr, n), t * 4}, {row_rsrc(a + row, n), t * 4},
                         {row_rsrc(s_ntt + tl + boff, n), t * 4}, {row_rsrc(c0, n), t * 4},
                         {row_rsrc(c0 + (static_cast<size_t>(limbs) << 16), n), t * 4}, q, mu);
}

// Inverse block pass of c0 + c1 (.) s, limbs l < limbs_used of ct [count][2][ct_limbs][N],
// into row c * out_gstride + l of `out` (the column pass follows).
__global__ __launch_bounds__(1 << (kBlkLogB - kBlkLogE)) void dec16_blocks_kernel(
    Tables tb, const uint32_t* __restrict__ ct, uint32_t ct_limbs, const uint32_t* __restrict__ s_ntt,
    uint32_t limbs_used, uint32_t* __restrict__ out, uint32_t out_gstride) {
  using P = Plan<kBlkLogB, kBlkLogE>;
  __shared__ uint32_t lds[P::lds_words];
  const size_t r = blockIdx.x / kBlocksPerRow;
  const uint32_t blk = blockIdx.x % kBlocksPerRow, t = threadIdx.x;
  const size_t c = r / limbs_used;
  const uint32_t l = static_cast<uint32_t>(r % limbs_used);
  const uint32_t q = tb.q[l], mu = tb.barrett[l];
  const size_t boff = static_cast<size_t>(blk) << kBlkLogB, tl = static_cast<size_t>(l) << 16;
  const uint32_t* c0 = ct + (((c * 2) * ct_limbs + l) << 16) + boff + t;
  const uint32_t* c1 = c0 + (static_cast<size_t>(ct_limbs) << 16);
  const uint32_t* sp = s_ntt + tl + boff + t;
  uint32_t v[P::E], x1[P::E], xs[P::E];
#pragma unroll
  for (int j = 0; j < P::E; ++j) {
    v[j] = __builtin_nontemporal_load(&c0[64 * j]);
    x1[j] = __builtin_nontemporal_load(&c1[64 * j]);
    xs[j] = sp[64 * j];
  }
#pragma unroll
  for (int j = 0; j < P::E; ++j) v[j] = add_mod(v[j], mul_mod_barrett(x1[j], xs[j], q, mu), q);
  wave_relayout<kBlkLogB, kBlkLogE, true>(v, t, lds);
  inv_block<16, kBlkLogB, kBlkLogE>(v, t, blk, tb.inv + tl, tb.inv_shoup + tl, q, lds);
  uint32_t* o = out + ((c * out_gstride + l) << 16) + boff;
#pragma unroll
  for (int j = 0; j < P::E; ++j) __builtin_nontemporal_store(v[j], &o[P::template pos<0>(t, j)]);
}

template <int LOGN>
hipError_t launch_encrypt_whole(const Tables& t, const uint32_t* pt, const uint32_t* s_ntt, const uint32_t* a,
                                const int32_t* e, uint32_t count, uint32_t limbs, uint32_t* ct, hipStream_t s) {
  const auto k = pt ? encrypt_kernel<LOGN, true> : encrypt_kernel<LOGN, false>;
  k<<<count * limbs, WholePlan<LOGN, true>::P::T, 0, s>>>(t, pt, s_ntt, a, e, limbs, ct);
  return hipGetLastError();
}

template <int LOGN>
hipError_t launch_decrypt_whole(const Tables& t, const uint32_t* ct, const uint32_t* s_ntt, uint32_t count,
                                uint32_t limbs, uint32_t* m, hipStream_t s) {
  dec_intt_kernel<LOGN><<<count * limbs, WholePlan<LOGN, true>::P::T, 0, s>>>(t, ct, limbs, s_ntt, limbs, m, limbs);
  return hipGetLastError();
}

template <int LOGN>
hipError_t launch_refresh_two(const Tables& t, const uint32_t* ct_in, uint32_t limbs_in, const uint32_t* s_ntt,
                              const uint32_t* a, const int32_t* e, uint32_t count, uint32_t limbs_out,
                              uint32_t* ct_out, hipStream_t s) {
  constexpr uint32_t T = WholePlan<LOGN, true>::P::T;
  dec_intt_kernel<LOGN><<<dim3(2 * count), T, 0, s>>>(
      t, ct_in, limbs_in, s_ntt, 2, ct_out + static_cast<size_t>(limbs_out) * t.n, 2 * limbs_out);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  dte_lift_ntt_kernel<LOGN><<<dim3(count * limbs_out), T, 0, s>>>(t, e, s_ntt, a, limbs_out, ct_out);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  // c1 rows 0 and 1 (the scratch) = a rows 0 and 1; the kernel wrote the others
  const size_t ct_bytes = static_cast<size_t>(2) * limbs_out * t.n * 4, a_bytes = ct_bytes / 2;
  return hipMemcpy2DAsync(ct_out + static_cast<size_t>(limbs_out) * t.n, ct_bytes, a, a_bytes, 2 * t.n * 4, count,
                          hipMemcpyDeviceToDevice, s);
}

template <int LOGN>
hipError_t launch_refresh_fused(const Tables& t, const uint32_t* ct_in, uint32_t limbs_in, const uint32_t* s_ntt,
                                const uint32_t* a, const int32_t* e, uint32_t count, uint32_t limbs_out,
                                uint32_t* ct_out, hipStream_t s) {
  refresh_kernel<LOGN><<<dim3(count, limbs_out), RefreshPlan<LOGN>::P::T, 0, s>>>(t, ct_in, limbs_in, s_ntt, a, e,
                                                                                 limbs_out, ct_out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_encrypt(const Tables& t, const uint32_t* pt, const uint32_t* s_ntt, const uint32_t* a,
                          const int32_t* e, uint32_t count, uint32_t limbs, uint32_t* ct, hipStream_t s) {
  switch (t.log_n) {
    case 10: return launch_encrypt_whole<10>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    case 11: return launch_encrypt_whole<11>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    case 12: return launch_encrypt_whole<12>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    case 13: return launch_encrypt_whole<13>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    case 14: return launch_encrypt_whole<14>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    case 15: return launch_encrypt_whole<15>(t, pt, s_ntt, a, e, count, limbs, ct, s);
    default: break;
  }
  const uint32_t rows = count * limbs;
  enc16_cols_kernel<<<rows * kColBlocks, kColThreads, 0, s>>>(t, e, limbs, ct);
  const auto blocks = pt ? rlwe16_blocks_combine_kernel<true> : rlwe16_blocks_combine_kernel<false>;
  blocks<<<rows * kBlocksPerRow, 1 << (kBlkLogB - kBlkLogE), 0, s>>>(t, pt, s_ntt, a, limbs, ct);
  return hipGetLastError();
}

hipError_t launch_decrypt(const Tables& t, const uint32_t* ct, const uint32_t* s_ntt, uint32_t count,
                          uint32_t limbs, uint32_t* m, hipStream_t s) {
  switch (t.log_n) {
    case 10: return launch_decrypt_whole<10>(t, ct, s_ntt, count, limbs, m, s);
    case 11: return launch_decrypt_whole<11>(t, ct, s_ntt, count, limbs, m, s);
    case 12: return launch_decrypt_whole<12>(t, ct, s_ntt, count, limbs, m, s);
    case 13: return launch_decrypt_whole<13>(t, ct, s_ntt, count, limbs, m, s);
    case 14: return launch_decrypt_whole<14>(t, ct, s_ntt, count, limbs, m, s);
    case 15: return launch_decrypt_whole<15>(t, ct, s_ntt, count, limbs, m, s);
    default: break;
  }
  dec16_blocks_kernel<<<count * limbs * kBlocksPerRow, 1 << (kBlkLogB - kBlkLogE), 0, s>>>(t, ct, limbs, s_ntt, limbs, m,
                                                                                          limbs);
  return launch_ntt16_cols(t, m, static_cast<size_t>(count) * limbs, limbs, true, s, limbs);
}

hipError_t launch_refresh(const Tables& t, const uint32_t* ct_in, uint32_t limbs_in, const uint32_t* s_ntt,
                          const uint32_t* a, const int32_t* e, uint32_t count, uint32_t limbs_out,
                          uint32_t* ct_out, hipStream_t s) {
  // Up to 2^13, launches of at most one fused workgroup (ciphertext x output
  // limb) per CU take the fused kernel split by output limb, whose chain is
  // three transforms (64 ciphertexts x 4 limbs at 2^13: 26.7 against 30.7 us);
  // larger ones, and every count at 2^14 (its fused workgroup is 1024
  // threads), the two-kernel route (32 ciphertexts at 2^14: 40.9 against
  // 41.8 us; 128: 62.5 against 89.5 us; 768: 0.36 against 0.52 ms).  At 2^15
  // it replaces the pointwise passes (768 ciphertexts x 4 limbs: 0.79 against
  // 1.01 ms; 32: 66 against 72 us).
  if (t.log_n >= 14 || static_cast<size_t>(count) * limbs_out > t.num_cus) {
    switch (t.log_n) {
      case 10: return launch_refresh_two<10>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      case 11: return launch_refresh_two<11>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      case 12: return launch_refresh_two<12>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      case 13: return launch_refresh_two<13>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      case 14: return launch_refresh_two<14>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      case 15: return launch_refresh_two<15>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
      default: break;
    }
  }
  switch (t.log_n) {
    case 10: return launch_refresh_fused<10>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
    case 11: return launch_refresh_fused<11>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
    case 12: return launch_refresh_fused<12>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
    case 13: return launch_refresh_fused<13>(t, ct_in, limbs_in, s_ntt, a, e, count, limbs_out, ct_out, s);
    default: break;
  }
  // N = 2^16: limbs 0 and 1 of c0 + c1 (.) s, inverse-transformed, in the c1 rows
  // 0 and 1 of ct_out (scratch); the lift into the c0 rows (a pass of its own:
  // in the column pass's loads every limb repeats it, 157 -> 216 us for 50
  // ciphertexts of 4 limbs); the column pass; the block pass with the combine,
  // which writes every c1 row.
  const uint32_t gs = 2 * limbs_out;
  uint32_t* dec = ct_out + static_cast<size_t>(limbs_out) * t.n;
  dec16_blocks_kernel<<<count * 2 * kBlocksPerRow, 1 << (kBlkLogB - kBlkLogE), 0, s>>>(t, ct_in, limbs_in, s_ntt, 2, dec,
                                                                                      gs);
  hipError_t err = launch_ntt16_cols(t, dec, static_cast<size_t>(count) * 2, 2, true, s, gs);
  if (err != hipSuccess) return err;
  const size_t quads = static_cast<size_t>(count) * (t.n / 4);
  dte_lift_kernel<<<static_cast<uint32_t>((quads + kThreads - 1) / kThreads), kThreads, 0, s>>>(t, e, count, limbs_out,
                                                                                               ct_out);
  const uint32_t rows = count * limbs_out;
  err = launch_ntt16_cols(t, ct_out, rows, limbs_out, false, s, gs);
  if (err != hipSuccess) return err;
  rlwe16_blocks_combine_kernel<false><<<rows * kBlocksPerRow, 1 << (kBlkLogB - kBlkLogE), 0, s>>>(t, nullptr, s_ntt, a,
                                                                                                 limbs_out, ct_out);
  return hipGetLastError();
}

}  // namespace ckks
