// Shared pieces of the compressed-space operations (pbz_ops.hip: 16-byte vectors that lie inside one block;
// pbz_ops_staged.hip: every other kept count and alignment): packed integer arithmetic, N in its three widths, the
// record of a reduction's partial sums and the evaluation of the statistics from them.
#pragma once

#include <type_traits>

#include "pbz_device.h"
#include "pbz_internal.h"

namespace pbz {
namespace ops {

constexpr int kThreads = 256;
constexpr int kReduceGroupsOneSegment = 1024;


inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int ilog2_exact(int64_t v) {  // log2(v) when v is a power of two, else -1
  if (v < 1 || (v & (v - 1))) return -1;
  int s = 0;
  while ((int64_t(1) << s) < v) ++s;
  return s;
}

inline int stream_groups(int64_t items, int per_thread) {
  int64_t g = (items + int64_t(kThreads) * per_thread - 1) / (int64_t(kThreads) * per_thread);
  if (g < 1) g = 1;
  if (g > kReduceMaxGroups) g = kReduceMaxGroups;
  return int(g);
}

// ---------------------------------------------------------------------------------------------
// packed integer helpers on one dword
// ---------------------------------------------------------------------------------------------
template <int kIType>
__device__ __forceinline__ uint32_t negate_packed(uint32_t x) {
  if (kIType == PBZ_I8) {
    uint32_t y = ~x;
    return ((y & 0x7f7f7f7fu) + 0x01010101u) ^ (y & 0x80808080u);
  } else if (kIType == PBZ_I16) {
    uint32_t y = ~x;
    return ((y & 0x7fff7fffu) + 0x00010001u) ^ (y & 0x80008000u);
  } else {
    return uint32_t(-int32_t(x));
  }
}

typedef short short2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ short2v as_short2(uint32_t u) {
  short2v s;
  s.x = short(u & 0xffffu);
  s.y = short(u >> 16);
  return s;
}

// sum over the elements of one dword of a*b, as a double (exact)
template <int kIType>
__device__ __forceinline__ double dot_dword(uint32_t a, uint32_t b) {
  if (kIType == PBZ_I8) {
    return double(__builtin_amdgcn_sdot4(int(a), int(b), 0, false));
  } else if (kIType == PBZ_I16) {
    return double(__builtin_amdgcn_sdot2(as_short2(a), as_short2(b), 0, false));
  } else {
    return double(int32_t(a)) * double(int32_t(b));
  }
}

// exact integer dot product of two 16-byte vectors for 8- and 16-bit indices
template <int kIType>
__device__ __forceinline__ double dot_vec(const uint4& a, const uint4& b) {
  if (kIType == PBZ_I8) {
    int acc = __builtin_amdgcn_sdot4(int(a.x), int(b.x), 0, false);
    acc = __builtin_amdgcn_sdot4(int(a.y), int(b.y), acc, false);
    acc = __builtin_amdgcn_sdot4(int(a.z), int(b.z), acc, false);
    acc = __builtin_amdgcn_sdot4(int(a.w), int(b.w), acc, false);
    return double(acc);
  } else if (kIType == PBZ_I16) {
    // one dword: at most 2 * 32767^2 < 2^31; four of them need 64 bits
    long long acc = (long long)__builtin_amdgcn_sdot2(as_short2(a.x), as_short2(b.x), 0, false);
    acc += (long long)__builtin_amdgcn_sdot2(as_short2(a.y), as_short2(b.y), 0, false);
    acc += (long long)__builtin_amdgcn_sdot2(as_short2(a.z), as_short2(b.z), 0, false);
    acc += (long long)__builtin_amdgcn_sdot2(as_short2(a.w), as_short2(b.w), 0, false);
    return double(acc);
  } else {
    return dot_dword<PBZ_I32>(a.x, b.x) + dot_dword<PBZ_I32>(a.y, b.y) + dot_dword<PBZ_I32>(a.z, b.z) +
           dot_dword<PBZ_I32>(a.w, b.w);
  }
}

template <int kIType>
__device__ __forceinline__ int first_element(uint32_t x) {
  if (kIType == PBZ_I8) return int(int8_t(x & 0xffu));
  if (kIType == PBZ_I16) return int(int16_t(x & 0xffffu));
  return int(x);
}

template <int kIType>
__device__ __forceinline__ void unpack_dword(uint32_t x, double* out) {  // 4 / 2 / 1 elements
  if (kIType == PBZ_I8) {
    out[0] = double(int(int8_t(x & 0xffu)));
    out[1] = double(int(int8_t((x >> 8) & 0xffu)));
    out[2] = double(int(int8_t((x >> 16) & 0xffu)));
    out[3] = double(int(int8_t(x >> 24)));
  } else if (kIType == PBZ_I16) {
    out[0] = double(int(int16_t(x & 0xffffu)));
    out[1] = double(int(int16_t(x >> 16)));
  } else {
    out[0] = double(int32_t(x));
  }
}

// the low bytes (int8) or halves (int16) of 4 / 2 integers gathered into one dword by byte permutes
template <int kIType>
__device__ __forceinline__ uint32_t pack_dword(const int* v) {
  if (kIType == PBZ_I8) {
    const uint32_t lo = __builtin_amdgcn_perm(uint32_t(v[1]), uint32_t(v[0]), 0x0c0c0400u);   // v0.b0, v1.b0
    const uint32_t hi = __builtin_amdgcn_perm(uint32_t(v[3]), uint32_t(v[2]), 0x0c0c0400u);   // v2.b0, v3.b0
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
  }
  if (kIType == PBZ_I16) return __builtin_amdgcn_perm(uint32_t(v[1]), uint32_t(v[0]), 0x05040100u);
  return uint32_t(v[0]);
}

// rint(t) as an integer for |t| < 2^31: adding 1.5 * 2^52 rounds t to an integer in the current (nearest-even)
// mode and leaves that integer, in two's complement, in the low word of the sum
__device__ __forceinline__ int rint_to_int(double t) {
  return int(uint32_t(__builtin_bit_cast(uint64_t, t + 6755399441055744.0)));
}

// F1 N1 + F2 N2 with both products and the sum rounded separately (Algorithm 2 as printed): a fused
// multiply-add would skip one rounding and break A + (-A) == 0 when N has more than 37 significant bits.
__device__ __forceinline__ double unfused_sum_of_products(double f1, double n1, double f2, double n2) {
#pragma clang fp contract(off)
  const double p1 = f1 * n1;
  const double p2 = f2 * n2;
  return p1 + p2;
}

template <int kIType>
struct PerDword {
  static constexpr int value = kIType == PBZ_I8 ? 4 : kIType == PBZ_I16 ? 2 : 1;
};

// N comes in three widths: kNType = PBZ_F64, PBZ_F32, or kN16 for the two 16-bit types, which share a kernel:
// the 16-bit load is the same, both decodings are computed and `f16` (uniform) selects one, so that no branch
// surrounds a load.
constexpr int kN16 = PBZ_BF16;
constexpr int n_kernel_type(int ftype) { return ftype == PBZ_F64 ? PBZ_F64 : (ftype == PBZ_F32 ? PBZ_F32 : kN16); }

template <int kNType>
__device__ __forceinline__ double load_N(const void* N, int64_t k, bool f16 = false) {
  if (kNType == PBZ_F64) return static_cast<const double*>(N)[k];
  if (kNType == PBZ_F32) return double(static_cast<const float*>(N)[k]);
  const uint16_t h = static_cast<const uint16_t*>(N)[k];
  const float as_bf16 = bf16_bits_to_float(h);
  const float as_f16 = float(__builtin_bit_cast(_Float16, h));
  return double(f16 ? as_f16 : as_bf16);
}

template <int kNType>
__device__ __forceinline__ void store_N(void* N, int64_t k, double v, bool f16 = false) {
  if (kNType == PBZ_F64) {
    static_cast<double*>(N)[k] = v;
  } else if (kNType == PBZ_F32) {
    static_cast<float*>(N)[k] = float(v);
  } else {
    const uint16_t as_bf16 = double_to_bf16_bits(v);
    const uint16_t as_f16 = __builtin_bit_cast(uint16_t, double_to_f16(v));
    static_cast<uint16_t*>(N)[k] = f16 ? as_f16 : as_bf16;
  }
}

// a / b rounded to nearest from a correctly rounded reciprocal: one multiply, the exact remainder by fused
// multiply-add, one correction.  Agrees with the hardware division sequence except in rare double-rounding
// corner cases, at a sixth of its cost.
__device__ __forceinline__ double div_by(double a, double b, double inv_b) {
  const double q = a * inv_b;
  const double rem = fma(-q, b, a);
  return fma(rem, inv_b, q);
}

// ---------------------------------------------------------------------------------------------
// Block-wise statistics and reductions
// ---------------------------------------------------------------------------------------------
enum BlockwiseMode { kBwVariance = 0, kBwStd = 1, kBwCovariance = 2 };

enum { kS12 = 0, kS11 = 1, kS22 = 2, kD1 = 3, kD2 = 4, kNumSums = 5 };

struct ReduceTail {
  double* partials;
  double* out;
  int op;
  double r, n_blocks, vol;
  double s_l, s_c, w_l, w_c, w_s;   // Algorithm 12's stabilisers and weights
  int n_f16;                        // N is FP16 (as opposed to bfloat16) when it is 16 bits wide
  // Shifted first coefficients.  Variance and covariance centre the first coefficients N_k F_k0 by their mean
  // (Algorithms 8, 9); summing them and their squares raw and subtracting afterwards would cancel against the
  // square of the mean.  The passes that need them therefore sum d_k = N_k F_k0 - K, with K the first
  // coefficient of the segment's first block (a pilot value: exact centring needs the mean, which is not known
  // yet, but any K near it removes the cancellation), and put d_k^2, d1_k d2_k into S11, S22, S12 in place of
  // the raw squares and product.  pilot_n1 == nullptr: nothing is shifted (K = 0).
  const void* pilot_n1;
  const void* pilot_f1;
  const void* pilot_n2;
  const void* pilot_f2;
  int64_t seg_n_bytes, seg_f_bytes;  // distance between the segments' first N and F
  int ntype, itype;
};

// K of operand (N, F) in segment `segment`: the same expression wherever it is evaluated
__device__ __forceinline__ double pilot_value(const void* N, const void* F, const ReduceTail& t, int64_t segment) {
  if (!N) return 0.0;
  const char* n = static_cast<const char*>(N) + segment * t.seg_n_bytes;
  const char* f = static_cast<const char*>(F) + segment * t.seg_f_bytes;
  return load_float<double>(n, t.ntype, 0) * double(load_index(f, t.itype, 0));
}

// s: the five sums, with the first coefficients shifted by K1 / K2 where the pass shifts them (else K = 0)
__device__ __forceinline__ double finish_statistic(const double* s, const ReduceTail& t, double K1, double K2) {
  const double n = t.n_blocks;
  // the raw sums back from the shifted ones: sum (d + K) = D + n K, sum (d1 + K1)(d2 + K2) = S12 + K2 D1 + K1 D2 + n K1 K2
  const double D1 = s[kD1] + n * K1, D2 = s[kD2] + n * K2;
  const double S11 = s[kS11] + 2.0 * K1 * s[kD1] + n * K1 * K1;
  const double S22 = s[kS22] + 2.0 * K2 * s[kD2] + n * K2 * K2;
  const double S12 = s[kS12] + K2 * s[kD1] + K1 * s[kD2] + n * K1 * K2;
  switch (t.op) {
    case kDot: return S12 / (t.r * t.r);
    case kNorm2: return sqrt(S11) / t.r;
    case kDiffNorm2: return sqrt(s[kS11]) / t.r;    // S11 then holds sum (N1 F1 - N2 F2)^2
    case kCosine: return S12 / (sqrt(S11) * sqrt(S22));
    case kMean: return (D1 / t.r) / (n * sqrt(t.vol));
    // centring the first coefficients by their mean removes (sum d1)(sum d2) / n_blocks from the sum of products,
    // whatever constant they were shifted by
    case kCovariance: return ((s[kS12] - s[kD1] * s[kD2] / n) / (t.r * t.r)) / (n * t.vol);
    case kVariance: return ((s[kS11] - s[kD1] * s[kD1] / n) / (t.r * t.r)) / (n * t.vol);
    case kSsim: {   // Algorithm 12 from the means, variances and covariance of Algorithms 7-9
      const double scale = 1.0 / (t.r * n * sqrt(t.vol));
      const double mu_a = D1 * scale, mu_b = D2 * scale;
      const double per = 1.0 / (t.r * t.r * n * t.vol);
      // a difference inside the rounding of its two terms is the variance of a constant array: zero (its root
      // would turn 1e-16 into 1e-8)
      const double noise = 8.0 * 2.220446049250313e-16;
      double ca = s[kS11] - s[kD1] * s[kD1] / n, cb = s[kS22] - s[kD2] * s[kD2] / n;
      if (ca <= noise * s[kS11]) ca = 0.0;
      if (cb <= noise * s[kS22]) cb = 0.0;
      const double var_a = ca * per, var_b = cb * per;
      const double cov = (s[kS12] - s[kD1] * s[kD2] / n) * per;
      const double sd = sqrt(var_a) * sqrt(var_b);
      const double lum = (2.0 * mu_a * mu_b + t.s_l) / (mu_a * mu_a + mu_b * mu_b + t.s_l);
      const double con = (2.0 * sd + t.s_c) / (var_a + var_b + t.s_c);
      const double str = (cov + 0.5 * t.s_c) / (sd + 0.5 * t.s_c);
      // weights of one, the usual ones, leave what pow(x, 1) is: x
      return (t.w_l == 1.0 ? lum : pow(lum, t.w_l)) * (t.w_c == 1.0 ? con : pow(con, t.w_c)) * (t.w_s == 1.0 ? str : pow(str, t.w_s));
    }
    default: return 0.0;
  }
}

// sum of `sums` over the workgroup, valid in threads 0 .. kNumSums-1 (thread i returns total i)
__device__ __forceinline__ double group_total(const double* sums, double (*lds)[kNumSums], int waves) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < kNumSums; ++i) {
    double t = wave_sum(sums[i]);
    if (lane == 0) lds[wave][i] = t;
  }
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x < kNumSums)
    for (int w = 0; w < waves; ++w) t += lds[w][threadIdx.x];
  return t;
}

// The requested statistic(s) of segment `segment` from its five sums, `thread` of the first kMaxStatistics threads of a workgroup the
// thread-th one: each is a chain of divisions and roots, nine of which by one thread took 3 us.
constexpr int kMaxStatistics = 9;
__device__ __forceinline__ void write_statistic(const double* fin, const ReduceTail& t, int64_t segment, double K1,
                                                double K2, int thread) {
  ReduceTail one = t;
  if (t.op == kStatistics) {            // mean, variance and norm2 of one array from the same two sums
    if (thread >= 3) return;
    one.op = thread == 0 ? kMean : (thread == 1 ? kVariance : kNorm2);
    t.out[segment * 3 + thread] = finish_statistic(fin, one, K1, K2);
  } else if (t.op == kPairStatistics) { // every statistic of a pair of arrays from the five sums of one pass
    if (thread >= 9) return;
    const int which = (thread - 3) >> 1;
    const bool second = thread >= 3 && ((thread - 3) & 1);          // of the second array: the operands exchanged
    if (thread < 3) one.op = thread == 0 ? kDot : (thread == 1 ? kCosine : kCovariance);
    else one.op = which == 0 ? kMean : (which == 1 ? kVariance : kNorm2);
    const double of[kNumSums] = {fin[kS12], second ? fin[kS22] : fin[kS11], second ? fin[kS11] : fin[kS22],
                                 second ? fin[kD2] : fin[kD1], second ? fin[kD1] : fin[kD2]};
    t.out[segment * 9 + thread] = finish_statistic(of, one, second ? K2 : K1, second ? K1 : K2);
  } else if (thread == 0) {
    t.out[segment] = finish_statistic(fin, t, K1, K2);
  }
}

// grid y runs over the segments of a segmented reduction (1 otherwise).  A segment covered by a single
// workgroup (small arrays) is finished here and needs no second launch; the sums are the same either way.
// K1, K2: the pilot values the sums were shifted by (zero where the pass shifts nothing).  Every workgroup of a
// segment has the same ones; they travel in the partial record (slots kPilot1, kPilot2), so that the final kernel
// finds them in the records it reads anyway instead of fetching N and F of the segment's first block once more.
constexpr int kPilot1 = 5, kPilot2 = 6;
static_assert(kPilot2 < kReducePartialSlots, "record layout");

// waves: of the workgroup, at most kThreads / 64
__device__ __forceinline__ void reduce_tail(double* sums, const ReduceTail& t, double K1, double K2,
                                            int waves = kThreads / 64) {
  __shared__ double lds[kThreads / 64][kNumSums];
  __shared__ double fin[kNumSums];
  const double total = group_total(sums, lds, waves);
  if (gridDim.x == 1) {
    if (threadIdx.x < kNumSums) fin[threadIdx.x] = total;
    __syncthreads();
    if (threadIdx.x < kMaxStatistics) write_statistic(fin, t, blockIdx.y, K1, K2, threadIdx.x);
    return;
  }
  double* record = t.partials + (int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * kReducePartialSlots;
  if (threadIdx.x < kNumSums) record[threadIdx.x] = total;
  if (threadIdx.x == kPilot1) record[kPilot1] = K1;
  if (threadIdx.x == kPilot2) record[kPilot2] = K2;
}

// Whether the sum or the shift of blocks that make no 16-byte vectors goes straight from memory, a wave per block, or through LDS (with which
// the times are compared, as dependent launches of a graph).  Few blocks of 19 to 64 indices, which a wave has in one step: the call is one
// round trip to memory, and the detour is up to 0.4 us more (300 blocks of 63 16-bit indices: sum 3.4 us, 3.8 through LDS, shift 3.1 and
// 3.4; of 33 32-bit ones 3.5 and 3.6; of 65, in two steps, 4.1 and 3.7 to 3.9).  8-bit operands are read straight from memory there, too: only
// shifts of 57 and more (63: 3.1 and 3.4; sums 3.4 and 3.4 to 3.5, of 32 blocks 3.3 and 3.1).  Many blocks of over 14 KiB: three regions leave three waves a compute unit (sum of 6000 blocks of 3600 32-bit indices
// 140 us, 158 through LDS; of 3300 130 and 118; 3500 blocks 120 and 98); one operand's shift never gains more than 2 % there.
inline bool direct_rebin(int64_t n_blocks, int kept, int64_t block_bytes, bool two) {
  if (n_blocks <= 1024) return kept <= 64 && (block_bytes == kept ? !two && kept >= 57 : kept >= 19);
  return two && n_blocks > 4096 && block_bytes > 14 * 1024;
}
// The same of the block-wise statistics.  The covariance has two operands to put into LDS: up to 1024 blocks of up to 160
// indices 0.1-0.4 us more (129 int8 indices: 3.0 us, 3.3 through LDS; from there on the two are alike); two to three words a lane, which 65 to
// 144 indices of 32 bits are, leave lanes idle (5000 blocks of 129: 4.7 and 5.4; 10000: 7.1 and 5.4).  The variance of up to 512 blocks of 33 to
// 65: a wave has them in one step, 0.05-0.3 us less (64 to 512 of 65 16-bit indices: 2.6-2.7 us, 2.9-3.0 through LDS; of 100 8-bit ones, in
// two steps, 2.9-3.0 and 2.7-2.8).  Large blocks go through LDS (4000 of 4095: covariance 75 us and 33, variance 44 and 16).
inline bool direct_blockwise(int64_t n_blocks, int kept, int64_t block_bytes, bool two) {
  if (!two) return n_blocks <= 512 && kept >= 33 && kept <= 65;
  if (block_bytes == 4 * int64_t(kept) && kept > 64 && kept <= 144) return n_blocks <= 5120;
  return n_blocks <= 1024 && kept <= 160;
}
// The same of the reductions, a thread per block: two operands of one or two indices a block (1000 to 30000 blocks of one: pair
// statistics 7.0 us, 7.6 through LDS, dot 5.8 and 6.3; of two 0.2 us less; of three they are alike), except 257 to 512 blocks, which LDS
// lets one workgroup take without a second launch (dot 5.6 and 4.7).
inline bool direct_reduction(int64_t n_blocks, int kept, bool two) {
  return two && kept <= 2 && (n_blocks <= 256 || (n_blocks > 512 && n_blocks <= 32768));
}

// pbz_ops_direct.hip and pbz_ops_staged.hip: any kept count, any alignment.  F2 == nullptr: addition of `shift` to the first
// coefficients.
int launch_rebin_direct(const pbz_codec* c, int64_t n_blocks, const void* N1, const void* F1, const void* N2, const void* F2,
                        void* Nout, void* Fout, double sign2, double shift, hipStream_t s);
int launch_blockwise_direct(const pbz_codec* c, int mode, int64_t n_blocks, const void* N1, const void* F1, const void* N2,
                            const void* F2, double* out, double scale, hipStream_t s);
int launch_reduce_direct(const pbz_codec* c, bool two, bool dc, bool diff, int64_t n_blocks, int n_segments, int max_groups,
                         const void* N1, const void* F1, const void* N2, const void* F2, const ReduceTail& tail, int* groups,
                         hipStream_t s);
int launch_rebin_staged(const pbz_codec* c, int64_t n_blocks, const void* N1, const void* F1, const void* N2, const void* F2,
                        void* Nout, void* Fout, double sign2, double shift, hipStream_t s);
int launch_blockwise_staged(const pbz_codec* c, int mode, int64_t n_blocks, const void* N1, const void* F1, const void* N2,
                            const void* F2, double* out, double scale, hipStream_t s);
// leaves in *groups the workgroups per segment it used (1: the results are written, no final kernel is needed)
int launch_reduce_staged(const pbz_codec* c, bool two, bool dc, bool diff, int64_t n_blocks, int n_segments, int max_groups,
                         const void* N1, const void* F1, const void* N2, const void* F2, const ReduceTail& tail, int* groups,
                         hipStream_t s);

}  // namespace ops
}  // namespace pbz
