// Scalar-weight ct x pt MAC on the gfx950 matrix cores, exact, through small
// coprime moduli (a residue number system of int8 channels).
//
// Per limb the MAC is C = V . X mod q with V the centred integer weights
// (d_out x d_in) and X the ciphertext residues (d_in x 2N).  Encoded scalar
// weights are one small integer per weight, the same in every limb, so the
// integer sums T = sum_i v_i (x_i - 2^29) are bounded by R 2^29, R the largest
// sum_i |v_i| of a row.  With coprime m_0 .. m_7 <= 256 and R 2^29 below 0.46 M,
// M = 2^63.3 their product (R < 2^33.2), T is determined by its residues mod the
// m_k, and each residue is one int8 contraction on v_mfma_i32_16x16x64_i8: 8
// products per modular MAC, where the base-256 digit split takes 12, or 16 when
// the weights need a fourth digit.
//
// With B operand bytes b_i = (x_i - 2^29) (M / m_k)^-1 mod m_k and A operand
// bytes v_i mod m_k, channel k's sum is congruent to r_k = T (M / m_k)^-1, and
//     T = sum_k r_k (M / m_k) - alpha M,   alpha = round(sum_k r_k / m_k),
// holds for any representatives r_k >= 0 (one m_k more in r_k is one more in
// alpha).  The epilogue takes the r_k as bytes: the products by
// (M / m_k mod q) go byte by byte through v_dot4_u32_u8, and alpha through
// fixed-point bytes 2^15 / m_k (error below 0.025 with |T| / M <= 0.46).
//
// Kernels of one call, on one stream:
//   rns_prep     weights -> A operand planes, per (16 rows, 64 k) partial sums
//                of v and |v|, and the checks that every limb holds the same
//                integer and whether it needs a fourth digit;
//   rns_decide   whether these kernels take the call, per-row constants 2^29 sum v;
//   rns_convert  a chunk of ciphertext columns -> B operand planes;
//   rns_gemm     the contraction and the epilogue over that chunk.
// The planes hold MFMA fragments (16 bytes a lane) in the order the
// contraction stages them, so its global-to-LDS copies are linear.  Everything
// lives in the space that the digit split needs for its fragments.
//
// 1024 -> 6144, N = 2^16, 8 limbs, weights of four digits: 53.6-57.9 ms a call
// against 65.6-71.6 ms for the digit split on the same boxes (52 ms the
// contraction, 2.5 ms the conversions).  The contraction issues at 49% of the
// matrix pipe's cycles and 2.0 GHz (the digit split: 80% of twice the products
// at 1.85 GHz); both run at the chip's power limit, which operand movement
// takes more of here (192 bytes L2 -> LDS and 512 bytes LDS -> registers per
// MFMA against 128 and 128).  Three-digit weights (12 products) are slower in
// this form at every size measured, 58.1 against 53.0 ms at this shape, and
// stay with the digit split.  Four-digit weights are slower in it too where the
// contraction is shallow or the space holds few rounds of workgroups (fit below).
#include <type_traits>
#include <utility>

#include "ckks_internal.hpp"

namespace ckks {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;

constexpr int kCh = kRnsChannels;  // 8
__constant__ const uint32_t kM[kCh] = {256, 247, 245, 243, 241, 239, 233, 229};

// Residue of an operand word: u in [0, 2^30) stands for u - 2^29.  y = sum of
// its bytes times (256^b w mod m) plus a constant is congruent to
// (u - 2^29) w + 128 and below 2^18, one multiply-high divides it exactly by m,
// and the byte (y mod m) - 128 is an int8 in the right class.
struct Conv {
  uint32_t bytes;  // 256^b w mod m in byte b
  uint32_t add;    // 128 + (-2^29 w mod m)
  uint32_t gceil;  // ceil(2^32 / m)
  uint32_t m;
};
constexpr uint32_t cm(int k) {
  constexpr uint32_t m[kCh] = {256, 247, 245, 243, 241, 239, 233, 229};
  return m[k];
}
constexpr uint32_t inv_mod(uint32_t a, uint32_t m) {
  for (uint32_t x = 1; x < m; ++x)
    if (a % m * x % m == 1) return x;
  return 0;
}
constexpr Conv make_conv(int k, bool weights) {  // w = 1 for the weights, (M / m)^-1 for the ciphertexts
  const uint32_t m = cm(k);
  uint32_t w = 1;
  if (!weights) {
    uint32_t p = 1;
    for (int i = 0; i < kCh; ++i)
      if (i != k) p = p * (cm(i) % m) % m;
    w = inv_mod(p, m);
  }
  Conv c{0, 0, 0, m};
  uint32_t pw = w % m;
  for (int b = 0; b < 4; ++b) {
    c.bytes |= pw << (8 * b);
    pw = pw * 256 % m;
  }
  const uint32_t off = static_cast<uint32_t>((static_cast<uint64_t>(1) << 29) % m) * w % m;
  c.add = 128 + (m - off) % m;
  c.gceil = static_cast<uint32_t>(((static_cast<uint64_t>(1) << 32) + m - 1) / m);
  return c;
}

// o byte e = r[e] byte 0, then -128 on every byte.
__device__ __forceinline__ uint32_t pack4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3) {
  const uint32_t a = __builtin_amdgcn_perm(r1, r0, 0x0c0c0400u);
  const uint32_t b = __builtin_amdgcn_perm(r3, r2, 0x04000c0cu);
  return (a | b) ^ 0x80808080u;
}

__device__ __forceinline__ uint32_t conv1(uint32_t u, const Conv& c) {
  const uint32_t y = __builtin_amdgcn_udot4(u, c.bytes, c.add, false);
  return y + __mul24(static_cast<int>(__umulhi(y, c.gceil)), -static_cast<int>(c.m));
}

__device__ __forceinline__ v4i conv16(const uint32_t (&u)[16], const Conv& c) {
  v4i f;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    f[g] = static_cast<int>(pack4(conv1(u[4 * g], c), conv1(u[4 * g + 1], c), conv1(u[4 * g + 2], c), conv1(u[4 * g + 3], c)));
  return f;
}

// f(channel) for every channel, the channel a compile-time constant.
template <typename F, int... K>
__device__ __forceinline__ void for_channels_of(F f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);
}
template <typename F>
__device__ __forceinline__ void for_channels(F f) {
  for_channels_of(f, std::make_integer_sequence<int, kCh>{});
}

// ---- geometry ---------------------------------------------------------------
constexpr int kTM = 256;      // weight rows of a workgroup tile
constexpr int kTN = 128;      // ciphertext columns of a workgroup tile (a strip)
constexpr int kStages = 4;    // LDS ring, one 64-deep k-step a stage
constexpr int kThreads = 512;
constexpr int kStepA = kTM / 16 * 64;          // 16-byte fragments of one k-step
constexpr int kStepB = kTN / 16 * 64;
constexpr int kStep = kStepA + kStepB;

struct Part {       // of one row and 64 k
  int64_t sum;
  uint64_t abs;     // bits 0-61: the sum of |v|
};
constexpr uint64_t kWide = uint64_t{1} << 62;    // some |v| needs a fourth base-256 digit
constexpr uint64_t kDiffer = uint64_t{1} << 63;  // some limb holds another integer

struct Layout {
  uint32_t rb, rows, ks;  // row blocks, padded rows, padded k-steps
  size_t part, rowc, planes, strips;  // byte offsets
  size_t strip_bytes;          // column planes of one strip
};

Layout layout_of(uint32_t d_out, uint32_t d_in, uint32_t limbs) {
  Layout s;
  s.rb = (d_out + kTM - 1) / kTM;
  s.rows = s.rb * kTM;
  s.ks = (d_in + 127) / 128 * 2;  // whole pairs of k-steps
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o = off;
    off += (b + 255) & ~size_t(255);
    return o;
  };
  s.part = take(static_cast<size_t>(s.ks) * s.rows * sizeof(Part));
  s.rowc = take(static_cast<size_t>(limbs) * s.rows * 4);
  s.planes = take(static_cast<size_t>(kCh) * s.rows * s.ks * 64);
  s.strips = off;
  s.strip_bytes = static_cast<size_t>(kCh) * s.ks * kStepB * 16;
  return s;
}

// ---- weights ----------------------------------------------------------------
// One workgroup per (16-row tile, 64 k): the limbs of its weights are adjacent
// in w_enc, so it reads whole lines.
constexpr int kPrepThreads = 256;
constexpr int kVPitch = 68;  // words per row of the LDS tile

__global__ __launch_bounds__(kPrepThreads) void rns_prep_kernel(
    const uint32_t* __restrict__ qtab, const uint32_t* __restrict__ w_enc, uint32_t d_out, uint32_t d_in,
    uint32_t limbs, uint32_t rows, uint32_t ks_total, v4i* __restrict__ planes, Part* __restrict__ part) {
  __shared__ uint32_t u[16 * kVPitch];  // v + 2^29
  const uint32_t mt = blockIdx.x, ks = blockIdx.y, tid = threadIdx.x;
  const uint32_t kn = ks * 64 < d_in ? (d_in - ks * 64 < 64 ? d_in - ks * 64 : 64) : 0;
  const uint32_t words = kn * limbs;
  const uint32_t q0 = qtab[0];
  constexpr uint32_t kOff = 1u << 29;
  for (uint32_t i = tid; i < 16 * kVPitch; i += kPrepThreads) u[i] = kOff;
  __syncthreads();
  for (uint32_t r = 0; r < 16; ++r) {
    const uint32_t row = mt * 16 + r;
    if (row >= d_out) break;
    const uint32_t* src = w_enc + (static_cast<size_t>(row) * d_in + ks * 64) * limbs;
    for (uint32_t i = tid; i < kn; i += kPrepThreads) {
      const uint32_t w = src[static_cast<size_t>(i) * limbs];
      u[r * kVPitch + i] = (w > (q0 >> 1) ? w - q0 : w) + kOff;
    }
  }
  __syncthreads();
  uint32_t bad = 0, wide = 0;
  for (uint32_t r = 0; r < 16; ++r) {
    const uint32_t row = mt * 16 + r;
    if (row >= d_out) break;
    const uint32_t* src = w_enc + (static_cast<size_t>(row) * d_in + ks * 64) * limbs;
    for (uint32_t i = tid; i < words; i += kPrepThreads) {
      const uint32_t k = i / limbs, l = i - k * limbs;
      const int32_t v = static_cast<int32_t>(u[r * kVPitch + k] - kOff);
      const uint32_t want = static_cast<uint32_t>(v) + (v < 0 ? qtab[l] : 0u);
      bad |= src[i] ^ want;
      wide |= static_cast<uint32_t>(v + 0x808080) > 0xffffffu;
    }
  }
  const uint64_t marks = (__syncthreads_or(bad != 0) ? kDiffer : 0) | (__syncthreads_or(wide != 0) ? kWide : 0);
  {  // partial sums: 16 threads a row, 4 k each
    const uint32_t r = tid >> 4, c = tid & 15;
    int64_t s = 0;
    uint64_t a = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int32_t v = static_cast<int32_t>(u[r * kVPitch + c * 4 + e] - kOff);
      s += v;
      a += static_cast<uint64_t>(v < 0 ? -static_cast<int64_t>(v) : v);
    }
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) {
      s += __shfl_down(s, d, 16);
      a += __shfl_down(a, d, 16);
    }
    if (c == 0) part[static_cast<size_t>(ks) * rows + mt * 16 + r] = Part{s, a | marks};
  }
  const uint32_t wave = tid >> 6, lane = tid & 63;
  uint32_t x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = u[(lane & 15) * kVPitch + (lane >> 4) * 16 + i];
  // plane k of row block rb, k-step ks: fragment (mt % 16, lane)
  const uint32_t rb = mt / (kTM / 16), m16 = mt % (kTM / 16);
  for_channels([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    constexpr Conv c = make_conv(k, true);
    if ((k & 3) == static_cast<int>(wave))
      planes[((static_cast<size_t>(rb) * kCh + k) * ks_total + ks) * kStepA + m16 * 64 + lane] = conv16(x, c);
  });
}

// One workgroup: whether these kernels take the call (kRnsTaken) and, for every
// limb and row, 2^29 sum v mod q.  They do when the weights are the same
// integers in every limb, every row sum is within the bound, and at least
// `wide_needed` of the 16-row tiles need a fourth weight digit: with three digits
// the digit split takes 12 products with less operand traffic and is the faster.
constexpr int kDecideThreads = 1024;
__global__ __launch_bounds__(kDecideThreads) void rns_decide_kernel(Tables tb, const Part* __restrict__ part,
                                                                    uint32_t rows, uint32_t ks_total, uint32_t limbs,
                                                                    uint64_t limit, uint32_t wide_needed,
                                                                    uint32_t* __restrict__ rowc,
                                                                    uint32_t* __restrict__ decision) {
  __shared__ uint32_t wide_tiles;
  if (threadIdx.x == 0) wide_tiles = 0;
  __syncthreads();
  uint32_t unfit = 0;
  for (uint32_t r = threadIdx.x; r < rows; r += kDecideThreads) {  // rows is a multiple of kTM
    int64_t s = 0;
    uint64_t a = 0, marks = 0;
#pragma unroll 8
    for (uint32_t ks = 0; ks < ks_total; ++ks) {
      const Part p = part[static_cast<size_t>(ks) * rows + r];
      s += p.sum;
      a += p.abs & (kWide - 1);
      marks |= p.abs & (kWide | kDiffer);
    }
    unfit |= (marks & kDiffer) != 0 || a > limit;
    if ((r & 15) == 0 && (marks & kWide)) atomicAdd(&wide_tiles, 1u);  // the marks are the tile's
    const uint64_t as = static_cast<uint64_t>(s < 0 ? -s : s);
    for (uint32_t l = 0; l < limbs; ++l) {
      const uint32_t q = tb.q[l];
      const double qr = tb.q_recip[l];
      const uint32_t m = reduce_u64(static_cast<uint64_t>(reduce_u64(as, q, qr)) << 29, q, qr);
      rowc[static_cast<size_t>(l) * rows + r] = s < 0 && m ? q - m : m;
    }
  }
  unfit = __syncthreads_or(unfit);
  if (threadIdx.x == 0) *decision = !unfit && wide_tiles >= wide_needed ? kRnsTaken : 0u;
}

// ---- ciphertext columns -------------------------------------------------------
// A thread converts 16 consecutive k of one column; a wave takes 64 adjacent
// columns (256-byte rows) and writes four 256-byte runs per plane.  Bound by
// memory: 4 bytes read and 8 written per residue, 4.9 TB/s.
constexpr int kConvThreads = 256;
__global__ __launch_bounds__(kConvThreads) void rns_convert_kernel(
    const uint32_t* __restrict__ decision, const uint32_t* __restrict__ ct_in, uint32_t log_n, uint32_t d_in,
    uint32_t limbs, uint32_t ks_total, uint32_t strip0, uint32_t strips, v4i* __restrict__ planes) {
  if (*decision != kRnsTaken) return;
  const uint32_t id = blockIdx.x * (kConvThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t kgroups = ks_total * 4, hs = id / kgroups, kg = id - hs * kgroups;  // k groups of a half strip adjacent
  if (hs >= strips * 2) return;
  const uint32_t n = 1u << log_n, per_limb = 2 * n / kTN;
  const uint32_t gs = strip0 + (hs >> 1), l = gs / per_limb;
  const uint32_t col0 = (gs - l * per_limb) * kTN + (hs & 1) * 64;  // column in [0, 2N)
  const uint32_t comp = col0 >> log_n, k0 = col0 & (n - 1);
  const size_t row_words = static_cast<size_t>(2) * limbs * n;
  const uint32_t* src = ct_in + (static_cast<size_t>(comp) * limbs + l) * n + k0 + lane + static_cast<size_t>(kg) * 16 * row_words;
  uint32_t x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    x[i] = kg * 16 + i < d_in ? __builtin_nontemporal_load(&src[static_cast<size_t>(i) * row_words]) : 1u << 29;
  v4i* dst = planes + (static_cast<size_t>(hs >> 1) * kCh * ks_total + (kg >> 2)) * kStepB +
             ((hs & 1) * 4 + (lane >> 4)) * 64 + (lane & 15) + 16 * (kg & 3);
  for_channels([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    constexpr Conv w = make_conv(k, false);
    dst[static_cast<size_t>(k) * ks_total * kStepB] = conv16(x, w);
  });
}

// ---- contraction ----------------------------------------------------------------
// A 512-thread workgroup computes 256 rows x 128 columns of one limb, channel
// after channel: each wave 64 rows x 64 columns (16 accumulator tiles).  The
// operands of one k-step (16 KiB of weight and 8 KiB of column fragments) are
// copied global -> LDS by buffer loads, three k-steps ahead, into a ring of four;
// one barrier per k-step, in the middle of its MFMAs, so that the first
// fragments of the next k-step are on their way to registers meanwhile.  After
// a channel's contraction the sums are reduced to bytes (a multiply-high, a
// multiply-add and a byte insertion each) kept in two registers per output; the
// channels are combined at the end.  The two byte registers and the accumulator
// of every output are what bounds the tile: 128 x 128 tiles, two workgroups a
// CU, measured 56.5 ms, converting a chunk's columns inside the previous
// chunk's contraction 56.2 ms (55.3 ms as it stands, same box).
//   * The column fragments are the first MFMA operand, so a lane holds four
//     consecutive columns of one weight row and stores 16 bytes.
//   * Accumulators start from a multiple of m_k that makes them non-negative
//     (below 2^27 + 2^8): the quotient estimate mulhi(s, floor(2^32 / m)) is at
//     most one low, and only when s mod m < m / 31, so the remainder is below
//     255 for m <= 247 (and exact for 256).
struct Channel {
  uint32_t bias, g;
  int32_t neg_m;
};
__device__ __forceinline__ Channel channel(uint32_t k) {
  const uint32_t m = kM[k];
  Channel c;
  const uint32_t up = (1u << 26) / m + 1;
  c.bias = up * m;
  c.g = k == 0 ? 1u << 24 : 0xFFFFFFFFu / m;  // floor(2^32 / m): only 256 divides 2^32
  c.neg_m = -static_cast<int32_t>(m);
  return c;
}

__global__ __launch_bounds__(kThreads) void rns_gemm_kernel(
    Tables tb, const uint32_t* __restrict__ decision, const v4i* __restrict__ aplanes, const v4i* __restrict__ bplanes,
    const uint32_t* __restrict__ rowc, uint32_t* __restrict__ ct_out, uint32_t d_out, uint32_t limbs, uint32_t rblocks,
    uint32_t ks_total, uint32_t strip0, uint32_t strips) {
  __shared__ v4i lds[kStages * kStep];
  if (*decision != kRnsTaken) return;
  // Consecutive workgroup ids alternate XCDs: each XCD takes a contiguous range
  // of tiles, ordered by groups of 8 strips, then row block, then strip, so its
  // 32 resident workgroups cover about 4 row blocks x 8 strips (2 MiB of
  // fragments per channel).
  const uint32_t G = gridDim.x;
  uint32_t lid = blockIdx.x;
  if ((G & 7u) == 0) lid = (lid & 7u) * (G >> 3) + (lid >> 3);
  const uint32_t sg = lid / (8 * rblocks);
  const uint32_t gsz = strips - sg * 8 < 8 ? strips - sg * 8 : 8;
  const uint32_t rem = lid - sg * 8 * rblocks;
  const uint32_t rb = rem / gsz, strip = sg * 8 + rem % gsz;

  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t wr = wave >> 1, wc = wave & 1;
  const uint32_t total = ks_total * kCh;    // stages
  const rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<v4i*>(aplanes + static_cast<size_t>(rb) * kCh * ks_total * kStepA), 0, total * kStepA * 16, kRsrcWord3);
  const rsrc_t rbf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<v4i*>(bplanes + static_cast<size_t>(strip) * kCh * ks_total * kStepB), 0, total * kStepB * 16, kRsrcWord3);
  constexpr int kWaves = kThreads / 64;
  constexpr int kCopiesA = kStepA / 64 / kWaves, kCopiesB = kStepB / 64 / kWaves;  // 1 KiB copies per wave and stage
  static_assert(kCopiesA == 2 && kCopiesB == 1 && kStages == 4, "the waits below count them");
  auto issue_a = [&](uint32_t g, uint32_t slot) {
    g = g < total ? g : total - 1;  // past the end: the last stage again, into a slot nobody reads
#pragma unroll
    for (int i = 0; i < kCopiesA; ++i) {
      const uint32_t o = (wave * kCopiesA + i) * 64;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(lds + slot * kStep + o), 16,
                                               lane * 16, (g * kStepA + o) * 16, 0, 0);
    }
  };
  auto issue_b = [&](uint32_t g, uint32_t slot) {
    g = g < total ? g : total - 1;
#pragma unroll
    for (int i = 0; i < kCopiesB; ++i) {
      const uint32_t o = (wave * kCopiesB + i) * 64;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rbf, (__attribute__((address_space(3))) void*)(lds + slot * kStep + kStepA + o),
                                               16, lane * 16, (g * kStepB + o) * 16, 0, 0);
    }
  };

  v4i acc[4][4];            // [column tile][row tile]
  uint32_t st[2][4][4][4] = {};  // residue bytes of channels 0-3, 4-7
  v4i a01[2][2], b01[2][2], a23[2], b23[2];
  // fragment i of a k-step in ring slot 0 or 1: columns (b) and rows (a) of this
  // wave; the pair of slots in use alternates between 0, 1 and 2, 3
  uint32_t bo = kStepA + wc * 4 * 64 + lane, ao = wr * 4 * 64 + lane;
  auto load01 = [&](int set, uint32_t slot) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      b01[set][i] = lds[bo + slot * kStep + i * 64];
      a01[set][i] = lds[ao + slot * kStep + i * 64];
    }
  };
#pragma unroll
  for (int i = 0; i < kStages; ++i) {
    issue_a(i, i);
    issue_b(i, i);
  }
  uint32_t g = 0;
  asm volatile("s_waitcnt vmcnt(9)\n\ts_barrier" ::: "memory");  // stage 0 has landed, in every wave
  load01(0, 0);
  // Stages g and g + 1 (g even).
  auto pair = [&]() {
    const uint32_t p = g & 2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      auto mma = [&](const v4i& b, const v4i& a, v4i& c) {
        c = __builtin_amdgcn_mfma_i32_16x16x64_i8(b, a, c, 0, 0, 0);
      };
      // the second halves of this k-step's fragments, then quadrant by quadrant
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a23[i] = lds[ao + h * kStep + (2 + i) * 64];
        b23[i] = lds[bo + h * kStep + (2 + i) * 64];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ci = 0; ci < 2; ++ci)
#pragma unroll
        for (int ri = 0; ri < 2; ++ri) mma(b01[h][ci], a01[h][ri], acc[ci][ri]);
#pragma unroll
      for (int ci = 0; ci < 2; ++ci)
#pragma unroll
        for (int ri = 0; ri < 2; ++ri) mma(b01[h][ci], a23[ri], acc[ci][2 + ri]);
      __builtin_amdgcn_sched_barrier(0);
      // every wave has read stage g + h; the next one has landed
      asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (h == 0) {
        load01(1, 1);
      } else {
        ao = ao < 2 * kStep ? ao + 2 * kStep : ao - 2 * kStep;
        bo = bo < 2 * kStep ? bo + 2 * kStep : bo - 2 * kStep;
        load01(0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ri = 0; ri < 2; ++ri)
#pragma unroll
        for (int ci = 0; ci < 2; ++ci) mma(b23[ci], a01[h][ri], acc[2 + ci][ri]);
      __builtin_amdgcn_sched_barrier(0);
      issue_a(g + h + kStages, p + h);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ri = 0; ri < 2; ++ri)
#pragma unroll
        for (int ci = 0; ci < 2; ++ci) mma(b23[ci], a23[ri], acc[2 + ci][2 + ri]);
      __builtin_amdgcn_sched_barrier(0);
      issue_b(g + h + kStages, p + h);
    }
    g += 2;
  };
  auto contract = [&](uint32_t k) {
    const int bias = static_cast<int>(channel(k).bias);
#pragma unroll
    for (int ci = 0; ci < 4; ++ci)
#pragma unroll
      for (int ri = 0; ri < 4; ++ri) acc[ci][ri] = v4i{bias, bias, bias, bias};
    for (uint32_t s = 0; s < ks_total; s += 2) pair();
  };
  auto reduce = [&](const Channel& c, int s) {
    const uint32_t u = static_cast<uint32_t>(s);
    return u + static_cast<uint32_t>(__mul24(static_cast<int>(__umulhi(u, c.g)), c.neg_m));
  };
#pragma unroll
  for (int w = 0; w < 2; ++w) {
#pragma unroll 1
    for (uint32_t b = 0; b < 4; ++b) {
      contract(w * 4 + b);
      const Channel c = channel(w * 4 + b);
#pragma unroll
      for (int ci = 0; ci < 4; ++ci)
#pragma unroll
        for (int ri = 0; ri < 4; ++ri)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            st[w][ci][ri][r] = __builtin_amdgcn_alignbit(reduce(c, acc[ci][ri][r]), st[w][ci][ri][r], 8);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy into this workgroup's LDS outlives it

  // ---- combine and store
  const uint32_t n = tb.n, log_n = tb.log_n;
  const uint32_t per_limb = 2 * n / kTN;
  const uint32_t gs = strip0 + strip, l = gs / per_limb;
  const uint32_t col0 = (gs - l * per_limb) * kTN + wc * 64;
  const uint32_t comp = col0 >> log_n, k0 = col0 & (n - 1);
  const uint32_t* cw = tb.rns + l * kRnsConstWords;
  const uint32_t q = tb.q[l];
  const uint32_t row_bytes = 2u * limbs * n * 4u;
  const uint32_t row0 = rb * kTM + wr * 64;
  const uint32_t rows = row0 < d_out ? (d_out - row0 < 64 ? d_out - row0 : 64) : 0;
  uint32_t* dst = ct_out + ((static_cast<size_t>(row0) * 2 + comp) * limbs + l) * n + k0;
  const rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(dst, 0, rows * row_bytes, kRsrcWord3);
  const uint32_t mneg = cw[10], mu = cw[11];
#pragma unroll
  for (int ri = 0; ri < 4; ++ri) {
    const uint32_t rc = rowc[static_cast<size_t>(l) * rblocks * kTM + row0 + ri * 16 + (lane & 15)];
#pragma unroll
    for (int ci = 0; ci < 4; ++ci) {
      v4u o;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t w0 = st[0][ci][ri][r], w1 = st[1][ci][ri][r];
        uint32_t s[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
          s[b] = __builtin_amdgcn_udot4(w0, cw[b], __builtin_amdgcn_udot4(w1, cw[4 + b], b == 0 ? rc : 0u, false), false);
        const uint32_t f = __builtin_amdgcn_udot4(w0, cw[8], __builtin_amdgcn_udot4(w1, cw[9], 1u << 14, false), false);
        uint64_t t = static_cast<uint64_t>(s[2] + (s[3] << 8)) * 65536u + (s[0] + (s[1] << 8));
        t += static_cast<uint64_t>(f >> 15) * mneg;
        // t < 2^45: the quotient estimate from its upper bits is at most one low
        const uint32_t qt = __umulhi(static_cast<uint32_t>(t >> 16), mu);
        const uint32_t y = static_cast<uint32_t>(t) - qt * q;
        o[r] = min(y, y - q);
      }
      __builtin_amdgcn_raw_buffer_store_b128(o, ro, (ri * 16 + (lane & 15)) * row_bytes + 16 * (lane >> 4), ci * 64, 0);
    }
  }
}

uint32_t gcd(uint32_t a, uint32_t b) { return b ? gcd(b, a % b) : a; }

// Strips per chunk for column planes of `room` bytes (0: less than two rounds of
// one workgroup a CU).  A chunk is whole rounds where it can be, and a multiple of
// 8 workgroups, without which the contraction's tiles are not dealt out by XCD
// (8193 x 1024, N = 2^14, 8 limbs: 23.7 ms with 191 strips, 19.7 with 184).
uint32_t chunk_strips(const Tables& t, const Layout& s, uint32_t total, size_t room) {
  const uint32_t round = t.num_cus / gcd(t.num_cus, s.rb);
  uint32_t strips = room / s.strip_bytes < total ? static_cast<uint32_t>(room / s.strip_bytes) : total;
  if (strips < total) strips -= strips % (strips >= round ? round : 8);
  while (strips * s.rb % 8) --strips;
  return static_cast<size_t>(strips) * s.rb < 2 * t.num_cus ? 0 : strips;
}

// Whether the channels are worth trying on a shape, and if so how many 16-row
// tiles of the weights have to need a fourth digit.
//
// Both forms' times in microseconds are fitted to 80 layers of four-digit weights
// (d_out 300-12000, d_in 64-1024, N = 2^13-2^16, 2-16 limbs, 0.1-6.6e12
// products; residuals mostly below 5%, at most 12%).  The channels take their time by rounds of
// one 256 x 128 tile a CU, with a part that does not shrink with d_in (eight byte
// reductions, the combine, the stores), the conversions, and two launches a
// chunk; the digit split by 256-row steps of its 32-column workgroups.
// Measured, digit split against channels, N = 2^16, 8 limbs: 6144 outputs of
// d_in 1024 68.9 : 57.6 ms, 640 45.3 : 40.2, 384 29.9 : 29.3, 256 22.2 : 24.1,
// 160 16.8 : 25.0; 2400 x 1000, whose chunks are 2.15 rounds, 26.6 : 31.4;
// 8200 x 64 at 16 limbs 28.7 : 51.5.  The rule wants 8% by the fit, above its usual residual.
//
// Weights that turn out not to qualify lose the preparation and two empty
// launches a chunk (3.7 us each) before the digit split: 53.2 -> 53.8 ms for
// three-digit weights at 1024 -> 6144, but 27.1 -> 28.1 for 1024 -> 3072, whose
// chunks are a quarter of that size.  Nothing on the host can tell, so the channels are
// tried only where their gain is at least nine times that loss, and from 2^40
// products up.
struct Choice {
  uint32_t chunk;        // strips per chunk, 0: the channels are not tried
  uint32_t wide_needed;
};
Choice choose(const Tables& t, const Layout& s, uint32_t d_out, uint32_t d_in, uint32_t limbs, size_t room) {
  const Choice no{0, 0};
  if (static_cast<uint64_t>(d_out) * d_in * 2 * limbs * t.n < uint64_t{1} << 40) return no;
  const uint32_t total = limbs * (2 * t.n / kTN);
  const uint32_t chunk = chunk_strips(t, s, total, room);
  if (chunk == 0) return no;
  auto ceil_div = [](uint32_t a, uint32_t b) { return (a + b - 1) / b; };
  const uint32_t full = total / chunk, last = total % chunk, chunks = full + (last != 0);
  const double rounds = static_cast<double>(full) * ceil_div(chunk * s.rb, t.num_cus) + ceil_div(last * s.rb, t.num_cus);
  const double rns = rounds * (3.28 * s.ks + 17.3) + 0.0094 * total * s.ks + 8.3 * chunks;
  const uint32_t ks = ceil_div(d_in, 64);                                  // k-steps of the digit split
  const double cols = ceil_div(limbs * (2 * t.n / 32), t.num_cus), steps = cols * ceil_div(d_out, 32) / 8.0;
  const double mma = 1.2 * steps * ks, digit = mma + 2.1 * steps + 0.71 * cols * ks;
  const double lost = 7.4 * chunks + 1.8e-4 * s.rows * s.ks * limbs + 30;  // launches, preparation and decision
  const double gain = digit - 1.08 * rns;
  if (gain < 0 || digit - rns < 9 * lost) return no;
  // a tile of three-digit weights takes 12 of the 16 products
  const uint32_t tiles = ceil_div(d_out, 16);
  const double part = 1 - gain / (0.25 * mma);
  return {chunk, static_cast<uint32_t>(ceil((part < 0.5 ? 0.5 : part) * tiles))};
}

uint64_t row_limit() {  // largest sum |v| of a row: 0.46 M / 2^29
  long double m = 1;
  for (int k = 0; k < kCh; ++k) m *= cm(k);
  return static_cast<uint64_t>(0.46L * m / 536870912.0L);
}

}  // namespace

void rns_consts(const uint32_t* q, uint32_t L, uint32_t* out) {
  for (uint32_t l = 0; l < L; ++l) {
    uint32_t* w = out + static_cast<size_t>(l) * kRnsConstWords;
    for (int i = 0; i < kRnsConstWords; ++i) w[i] = 0;
    uint64_t all = 1;
    for (int k = 0; k < kCh; ++k) all = all * cm(k) % q[l];
    for (int k = 0; k < kCh; ++k) {
      uint64_t c = 1;  // M / m_k mod q
      for (int i = 0; i < kCh; ++i)
        if (i != k) c = c * cm(i) % q[l];
      for (int b = 0; b < 4; ++b) w[(k >> 2) * 4 + b] |= static_cast<uint32_t>((c >> (8 * b)) & 255) << (8 * (k & 3));
      w[8 + (k >> 2)] |= ((1u << 16) / cm(k) + 1) / 2 << (8 * (k & 3));  // 2^15 / m rounded
    }
    w[10] = static_cast<uint32_t>((q[l] - all) % q[l]);
    w[11] = static_cast<uint32_t>((uint64_t(1) << 48) / q[l]);
  }
}

hipError_t launch_mac_scalar_rns(const Tables& t, const uint32_t* w_enc, const uint32_t* ct_in, uint32_t* ct_out,
                                 uint32_t d_out, uint32_t d_in, uint32_t limbs, void* workspace,
                                 size_t workspace_bytes, uint32_t* decision, hipStream_t st, bool* launched) {
  *launched = false;
  const Layout s = layout_of(d_out, d_in, limbs);
  if (workspace_bytes <= s.strips) return hipSuccess;
  const Choice how = choose(t, s, d_out, d_in, limbs, workspace_bytes - s.strips);
  const uint32_t chunk = how.chunk;
  if (chunk == 0) return hipSuccess;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  Part* part = reinterpret_cast<Part*>(ws + s.part);
  uint32_t* rowc = reinterpret_cast<uint32_t*>(ws + s.rowc);
  v4i* aplanes = reinterpret_cast<v4i*>(ws + s.planes);
  v4i* bplanes = reinterpret_cast<v4i*>(ws + s.strips);
  const uint32_t total = limbs * (2 * t.n / kTN);
  rns_prep_kernel<<<dim3(s.rows / 16, s.ks), kPrepThreads, 0, st>>>(t.q, w_enc, d_out, d_in, limbs, s.rows, s.ks,
                                                                   aplanes, part);
  rns_decide_kernel<<<1, kDecideThreads, 0, st>>>(t, part, s.rows, s.ks, limbs, row_limit(),
                                             how.wide_needed, rowc, decision);
  for (uint32_t s0 = 0; s0 < total; s0 += chunk) {
    const uint32_t strips = total - s0 < chunk ? total - s0 : chunk;
    const size_t waves = static_cast<size_t>(strips) * 2 * s.ks * 4;
    rns_convert_kernel<<<static_cast<uint32_t>((waves + kConvThreads / 64 - 1) / (kConvThreads / 64)), kConvThreads, 0, st>>>(
        decision, ct_in, t.log_n, d_in, limbs, s.ks, s0, strips, bplanes);
    rns_gemm_kernel<<<s.rb * strips, kThreads, 0, st>>>(t, decision, aplanes, bplanes, rowc, ct_out, d_out, limbs, s.rb,
                                                       s.ks, s0, strips);
  }
  *launched = true;
  return hipGetLastError();
}

}  // namespace ckks
