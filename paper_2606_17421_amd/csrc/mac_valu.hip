// Vector-ALU modular MAC kernels (gfx950).
//
// Scalar weights: per limb a modular GEMM (d_out x d_in) . (d_in x 2N); each
// thread owns one (component, NTT slot) column and kRows output rows, keeps
// u64 accumulators fed by v_mad_u64_u32, and reduces every 15 products
// (15 * 2^60 + 2^30 < 2^64).  Weights are wave-uniform (scalar loads).
// Full-polynomial weights: slot-wise products, the plaintexts streamed once
// from HBM; each thread owns one (limb, slot), both ciphertext components and
// a group of output rows.
#include "ckks_internal.hpp"

namespace ckks {
namespace {

constexpr int kThreads = 256;
constexpr int kRows = 8;
constexpr int kLazy = 15;

__global__ __launch_bounds__(kThreads) void mac_scalar_valu_kernel(
    Tables tb, const uint32_t* __restrict__ w_enc, const uint32_t* __restrict__ ct_in,
    uint32_t* __restrict__ ct_out, uint32_t d_out, uint32_t d_in, uint32_t limbs) {
  const uint32_t n = tb.n;
  const uint32_t col = blockIdx.x * kThreads + threadIdx.x;  // < 2N
  const uint32_t c = col >> tb.log_n;
  const uint32_t k = col & (n - 1);
  const uint32_t l = blockIdx.z;
  const uint32_t j0 = blockIdx.y * kRows;
  const uint32_t q = tb.q[l];
  const double qr = tb.q_recip[l];
  const size_t in_stride = 2ull * limbs * n;
  const uint32_t* x_ptr = ct_in + (static_cast<size_t>(c) * limbs + l) * n + k;
  size_t w_row[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const uint32_t j = min(j0 + r, d_out - 1);  // clamp: rows past d_out are computed, not stored
    w_row[r] = static_cast<size_t>(j) * d_in * limbs + l;
  }
  uint64_t acc[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) acc[r] = 0;
  uint32_t i = 0;
  while (i < d_in) {
    const uint32_t stop = min(d_in, i + kLazy);
    for (; i < stop; ++i) {
      const uint64_t x = x_ptr[i * in_stride];
#pragma unroll
      for (int r = 0; r < kRows; ++r) acc[r] += x * w_enc[w_row[r] + static_cast<size_t>(i) * limbs];
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = reduce_u64(acc[r], q, qr);
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const uint32_t j = j0 + r;
    if (j < d_out)
      ct_out[((static_cast<size_t>(j) * 2 + c) * limbs + l) * n + k] = static_cast<uint32_t>(acc[r]);
  }
}

// Full-polynomial weights: thread = (limb l, slots k .. k+3) for kPolyRows
// outputs j0 .. j0 + kPolyRows - 1, with 16-byte loads.  Each ciphertext
// residue quad is loaded once per kPolyRows outputs; every plaintext residue
// is read exactly once.  Workgroups with the same (l, slot block) and
// consecutive row groups are adjacent in logical order, and each XCD runs a
// contiguous range of logical ids, so the shared ciphertext columns are
// fetched once into that XCD's L2.  Per input the row loads are all issued before
// the first product (a ragged last group re-reads row 0 for its missing rows and
// discards those sums), so a wave waits on memory once per input instead of once
// per row: 31.1 -> 24.9 us at 32 x 32, 2^13, 4 limbs (the next input's loads issued
// ahead of the products as well gave nothing).  Outputs are stored
// non-temporally (written once): 621 -> 600 us at 64 x 64, 2^15, 6 limbs; 53 ->
// 49.5 us at 32 x 32, 2^14, 4 limbs.  launch_mac_poly chooses the rows per thread
// and whether the plaintexts, each read once, pass the caches by.
constexpr int kPolySlots = 4;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <bool kNonTemporal>
__device__ __forceinline__ uint4 load_pt(const uint4* p) {
  if constexpr (kNonTemporal) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
  } else {
    return *p;
  }
}

template <int kPolyRows, bool kNonTemporal>
__global__ __launch_bounds__(kThreads) void mac_poly_kernel(
    Tables tb, const uint32_t* __restrict__ pt, const uint32_t* __restrict__ ct_in,
    uint32_t* __restrict__ ct_out, uint32_t d_out, uint32_t d_in, uint32_t limbs) {
  const uint32_t n = tb.n;
  const uint32_t groups = (d_out + kPolyRows - 1) / kPolyRows;
  const uint32_t blocks_per_row = n / (kThreads * kPolySlots);
  // blockIdx.x = (l * blocks_per_row + kb) * groups + g
  // Consecutive workgroup ids alternate XCDs: each XCD takes a contiguous
  // range of logical ids, so the row groups sharing a column block meet in one L2.
  const uint32_t G = gridDim.x;
  uint32_t lid = blockIdx.x;
  if ((G & 7u) == 0) lid = (lid & 7u) * (G >> 3) + (lid >> 3);
  const uint32_t g = lid % groups;
  const uint32_t lk = lid / groups;
  const uint32_t l = lk / blocks_per_row;
  const uint32_t k = ((lk % blocks_per_row) * kThreads + threadIdx.x) * kPolySlots;
  const uint32_t j0 = g * kPolyRows;
  const uint32_t rows = d_out - j0 < kPolyRows ? d_out - j0 : kPolyRows;  // workgroup-uniform
  const uint32_t q = tb.q[l];
  const double qr = tb.q_recip[l];
  const size_t ln = static_cast<size_t>(limbs) * n;
  const uint4* p_ptr = reinterpret_cast<const uint4*>(pt + (static_cast<size_t>(j0) * d_in * limbs + l) * n + k);
  const size_t p_row = static_cast<size_t>(d_in) * ln / 4;  // one output's plaintexts, in uint4
  const size_t ln4 = ln / 4;
  const uint4* x_ptr = reinterpret_cast<const uint4*>(ct_in + static_cast<size_t>(l) * n + k);
  uint64_t a0[kPolyRows][kPolySlots], a1[kPolyRows][kPolySlots];
#pragma unroll
  for (int r = 0; r < kPolyRows; ++r)
#pragma unroll
    for (int e = 0; e < kPolySlots; ++e) a0[r][e] = a1[r][e] = 0;
  uint32_t i = 0;
  while (i < d_in) {
    const uint32_t stop = min(d_in, i + kLazy);
    for (; i < stop; ++i) {
      const uint4 x0 = x_ptr[(2ull * i) * ln4], x1 = x_ptr[(2ull * i + 1) * ln4];
      uint4 pv[kPolyRows];
#pragma unroll
      for (int r = 0; r < kPolyRows; ++r) {
        const uint32_t rr = r < rows ? r : 0;  // rows >= 1; sums of rows past d_out are not stored
        pv[r] = load_pt<kNonTemporal>(&p_ptr[rr * p_row + static_cast<size_t>(i) * ln4]);
      }
      const uint32_t xs0[4] = {x0.x, x0.y, x0.z, x0.w}, xs1[4] = {x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int r = 0; r < kPolyRows; ++r) {
        const uint32_t ps[4] = {pv[r].x, pv[r].y, pv[r].z, pv[r].w};
#pragma unroll
        for (int e = 0; e < kPolySlots; ++e) {
          a0[r][e] += static_cast<uint64_t>(ps[e]) * xs0[e];
          a1[r][e] += static_cast<uint64_t>(ps[e]) * xs1[e];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kPolyRows; ++r)
#pragma unroll
      for (int e = 0; e < kPolySlots; ++e) {
        a0[r][e] = reduce_u64(a0[r][e], q, qr);
        a1[r][e] = reduce_u64(a1[r][e], q, qr);
      }
  }
#pragma unroll
  for (int r = 0; r < kPolyRows; ++r) {
    if (r < rows) {
      u32x4* o = reinterpret_cast<u32x4*>(ct_out + ((static_cast<size_t>(j0 + r) * 2) * limbs + l) * n + k);
      __builtin_nontemporal_store(u32x4{static_cast<uint32_t>(a0[r][0]), static_cast<uint32_t>(a0[r][1]),
                                        static_cast<uint32_t>(a0[r][2]), static_cast<uint32_t>(a0[r][3])}, &o[0]);
      __builtin_nontemporal_store(u32x4{static_cast<uint32_t>(a1[r][0]), static_cast<uint32_t>(a1[r][1]),
                                        static_cast<uint32_t>(a1[r][2]), static_cast<uint32_t>(a1[r][3])}, &o[ln4]);
    }
  }
}

__global__ __launch_bounds__(kThreads) void zero_kernel(uint32_t* p, size_t words) {
  const size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  const size_t stride = static_cast<size_t>(gridDim.x) * kThreads;
  for (size_t k = i; k < words; k += stride) p[k] = 0;
}

}  // namespace

hipError_t launch_mac_scalar_valu(const Tables& t, const uint32_t* w_enc, const uint32_t* ct_in,
                                  uint32_t* ct_out, uint32_t d_out, uint32_t d_in, uint32_t limbs,
                                  hipStream_t s) {
  dim3 grid(2 * t.n / kThreads, (d_out + kRows - 1) / kRows, limbs);
  mac_scalar_valu_kernel<<<grid, kThreads, 0, s>>>(t, w_enc, ct_in, ct_out, d_out, d_in, limbs);
  return hipGetLastError();
}

// A call whose plaintexts fit the last-level cache (256 MiB) may find them there:
// a product that is called again on the same weights.  Loaded plainly they stay,
// non-temporally they do not, and a call over other weights each time, which
// never finds its own, gains the other way round.  Nothing here tells the two
// apart, so calls that fit load plainly, which costs neither of them against
// loads that were always plain.  In us, the same plaintexts / others every call
// (1.6 GB in turn):
//                                     plain, 2 rows   non-temporal, 2 / 4 rows
//   32 x 32, 2^13, 4 limbs (134 MB)   24.5 / 34.3     27.3 / 29.1   27.7 / 29.5
//   24 x 32, 2^14, 4 limbs (201 MB)   36.3 / 44.8     39.5 / 40.0   46.7 / 48.1
//   8 x 96, 2^12, 3 limbs (38 MB)     39.8 / 58.3     50.7 / 55.7   63.2 / 67.1
//   32 x 32, 2^14, 4 limbs (268 MB)   49.6 / 59.6     52.5 / 53.0   48.5 / 49.1
//   64 x 16, 2^14, 4 limbs (268 MB)   54.1 / 66.2     57.9 / 59.9   68.5 / 70.7
//   80 x 14, 2^14, 4 limbs (294 MB)   63.5 / 67.8     62.9 / 64.4   59.5 / 61.0
//   64 x 80, 2^12, 4 limbs (336 MB)   69.4 / 69.1     63.7 / 64.7   68.5 / 69.1
//   24 x 80, 2^15, 4 limbs (1 GB)     212 / 212       196 / 196     167 / 167
// From 8 workgroups a CU four rows are the faster whatever the size (256 x 16,
// 2^13, 4 limbs: 101.6 us against 111 with two, non-temporal both, and 117 plain).
// Three of the four-row kernel's workgroups fit a CU (130 registers): just past
// the cache, where part of the plaintexts may still be found, a grid of two or
// three a CU gains in both columns and a larger one need not; below two, two rows
// fill the chip better.
hipError_t launch_mac_poly(const Tables& t, const uint32_t* pt, const uint32_t* ct_in,
                           uint32_t* ct_out, uint32_t d_out, uint32_t d_in, uint32_t limbs,
                           hipStream_t s) {
  constexpr size_t kCache = size_t(256) << 20, kPast = size_t(288) << 20;
  const size_t bytes = static_cast<size_t>(d_out) * d_in * limbs * t.n * 4;
  const size_t blocks = static_cast<size_t>(limbs) * (t.n / (kThreads * kPolySlots)), cus = t.num_cus;
  const size_t grid4 = (static_cast<size_t>(d_out) + 3) / 4 * blocks, grid2 = (static_cast<size_t>(d_out) + 1) / 2 * blocks;
  const bool four = grid4 >= 8 * cus || (grid4 >= 2 * cus && (bytes >= kPast || (bytes >= kCache && grid4 <= 3 * cus)));
  const uint32_t grid = static_cast<uint32_t>(four ? grid4 : grid2);
  const auto mac = four ? mac_poly_kernel<4, true> : bytes >= kPast ? mac_poly_kernel<2, true> : mac_poly_kernel<2, false>;
  mac<<<grid, kThreads, 0, s>>>(t, pt, ct_in, ct_out, d_out, d_in, limbs);
  return hipGetLastError();
}

hipError_t launch_zero(uint32_t* p, size_t words, hipStream_t s) {
  if (words == 0) return hipSuccess;
  size_t grid = (words + kThreads - 1) / kThreads;
  if (grid > 65536) grid = 65536;
  zero_kernel<<<static_cast<uint32_t>(grid), kThreads, 0, s>>>(p, words);
  return hipGetLastError();
}

}  // namespace ckks
