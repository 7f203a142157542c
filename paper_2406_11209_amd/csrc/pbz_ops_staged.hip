// Compressed-space operations for kept counts and alignments that the 16-byte-vector kernels of pbz_ops.hip do not
// take: blocks whose indices are no multiple of 16 bytes or of a power of two of them (zonal masks: 19 of 64 int16
// indices are 38 bytes), and F pointers that are not 16-byte aligned (a step in the middle of such a series).
//
// What bounds them is HBM, provided that F moves in 16-byte pieces although blocks start at any element.  A wave
// therefore owns a run of consecutive blocks, whose indices are one contiguous span of F:
//   stage    the span is copied to the wave's own LDS region in aligned 16-byte pieces, at the same phase (address
//            modulo 16) that it has in memory; N goes along, widened to FP64;
//   work     a team of 2^k consecutive lanes takes a block, each a run of consecutive dwords of it: neighbouring aligned LDS words
//            shifted against each other by the block's phase, every word read once, so that the packed arithmetic of the
//            vector kernels applies.  A team is as few lanes as can be (up to 12 dwords each) while that leaves enough waves:
//            what is done once per lane and block, two divisions above all, is spread over as many indices as possible;
//   unstage  new indices collect in LDS at the phase of the output pointer and leave in 16-byte pieces, the span's ends element
//            by element.
// Waves never wait for each other (no workgroup barrier), so the loads of some overlap the arithmetic of others.
// 2M blocks of 19 int16 indices (80 MB of F an operand): add and subtract 56 us, addition of a scalar 48 us (1016 and 592 element by
// element, 85 and 67 with teams of at most four dwords a lane, consecutive lanes consecutive dwords); the reductions are with k_reduce_staged.
// Tried and not kept: dword accesses of LDS at any byte instead of shifting two aligned words (add 99 -> 140 us), spans of 1 or
// 4 KiB per wave and operand (15-35 % slower).
#include "pbz_ops_common.h"
#include "pbz_span.h"
#include "pbz_stage_layout.h"

namespace pbz {
namespace ops {
namespace {

constexpr int kNPerLane = kMaxBlocksPerWave / 64;

// N of `count` (at most kMaxBlocksPerWave) blocks from k0 on: requested, as they are stored, and widened when they are put away,
// so that the requests for the indices do not wait for them
template <int kNType>
struct StagedN {
  typedef typename std::conditional<kNType == PBZ_F64, double, typename std::conditional<kNType == PBZ_F32, float, uint16_t>::type>::type stored_t;
  stored_t raw[kNPerLane];
  double v[kNPerLane];
  __device__ __forceinline__ void request(const void* N, int64_t k0, int count) {
#pragma unroll
    for (int u = 0; u < kNPerLane; ++u) {
      const int i = u * 64 + int(threadIdx.x & 63);
      if (u * 64 < count) raw[u] = static_cast<const stored_t*>(N)[k0 + (i < count ? i : count - 1)];
    }
  }
  __device__ __forceinline__ bool beyond(double limit, int count) const {         // any of the lane's, NaN included
    bool any = false;
#pragma unroll
    for (int u = 0; u < kNPerLane; ++u) any = any || (u * 64 < count && !(fabs(v[u]) < limit));
    return any;
  }
  __device__ __forceinline__ void put(double* lds, int count, bool f16) {
#pragma unroll
    for (int u = 0; u < kNPerLane; ++u) {
      const int i = u * 64 + int(threadIdx.x & 63);
      if (u * 64 < count) v[u] = load_N<kNType>(raw + u, 0, f16);
      if (i < count) lds[i] = v[u];
    }
  }
};

template <int kIType>
struct IndexOf {
  typedef typename std::conditional<kIType == PBZ_I8, int8_t, typename std::conditional<kIType == PBZ_I16, int16_t, int32_t>::type>::type type;
};

// dword d of the block that starts at byte `start` of the LDS region; bytes past the block's end are zero
__device__ __forceinline__ uint32_t block_dword(const uint8_t* lds, int start, int d, int bpb) {
  const int at = start + 4 * d;
  const uint32_t* w = reinterpret_cast<const uint32_t*>(lds) + (at >> 2);
  const uint32_t v = __builtin_amdgcn_alignbyte(w[1], w[0], uint32_t(at & 3));
  const int rest = bpb - 4 * d;
  return rest >= 4 ? v : (rest <= 0 ? 0u : v & ((1u << (8 * rest)) - 1u));
}

// A lane's run of a block: `run` consecutive dwords from byte `start` of the LDS region on, of which `whole` lie in the block, and
// the block's last one, where that is partial and the lane's.
struct LaneRun {
  int run, whole, part;            // part: bytes of the partial dword, zero unless it is this lane's
  uint32_t cut;                    // mask of those bytes
  int start;
  __device__ __forceinline__ LaneRun(const Stage& st, int t) {
    run = st.run;
    start = 4 * t * st.run;
    const int left = (st.bpb >> 2) - t * st.run;            // whole dwords from the lane's first one to the block's end
    whole = left < 0 ? 0 : (left < st.run ? left : st.run);
    part = left >= 0 && left < st.run ? st.bpb & 3 : 0;
    cut = (1u << (8 * part)) - 1u;
  }
};

// f(i, a, b) for the lane's whole dwords i of a block, in order, and then for the partial one, its other bytes zero.  a0, b0: the bytes of the two
// operands' LDS regions at which the lane's run starts (at any alignment).  Every word is read once: a dword is cut from its own
// and the next one.
template <bool kTwo, typename Fn>
__device__ __forceinline__ void for_dwords(const LaneRun& lane, const uint8_t* sa, int a0, const uint8_t* sb, int b0, Fn f) {
  const uint32_t* wa = reinterpret_cast<const uint32_t*>(sa) + (a0 >> 2);
  const uint32_t* wb = reinterpret_cast<const uint32_t*>(sb) + (b0 >> 2);
  const uint32_t ca = uint32_t(a0 & 3), cb = uint32_t(b0 & 3);
  constexpr int kAhead = 4;                                 // words requested together
  uint32_t pa = wa[0], pb = kTwo ? wb[0] : 0u;
  int i0 = 0;
  for (; i0 + kAhead <= lane.run; i0 += kAhead) {
    uint32_t va[kAhead], vb[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      va[u] = wa[i0 + u + 1];
      vb[u] = kTwo ? wb[i0 + u + 1] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const uint32_t a = __builtin_amdgcn_alignbyte(va[u], pa, ca);
      const uint32_t b = kTwo ? __builtin_amdgcn_alignbyte(vb[u], pb, cb) : a;
      if (i0 + u < lane.whole) f(i0 + u, a, b);
      pa = va[u];
      pb = vb[u];
    }
  }
  for (; i0 < lane.run; ++i0) {
    const uint32_t va = wa[i0 + 1], vb = kTwo ? wb[i0 + 1] : 0u;
    const uint32_t a = __builtin_amdgcn_alignbyte(va, pa, ca);
    const uint32_t b = kTwo ? __builtin_amdgcn_alignbyte(vb, pb, cb) : a;
    if (i0 < lane.whole) f(i0, a, b);
    pa = va;
    pb = vb;
  }
  if (lane.part) {
    const int i = lane.whole;
    const uint32_t a = __builtin_amdgcn_alignbyte(wa[i + 1], wa[i], ca) & lane.cut;
    const uint32_t b = kTwo ? __builtin_amdgcn_alignbyte(wb[i + 1], wb[i], cb) & lane.cut : a;
    f(i, a, b);
  }
}

// indices q of a dword to byte `at` of the LDS region; `bytes`: 4, or those of a partial dword
template <int kIType>
__device__ __forceinline__ void put_indices(uint8_t* at, const int* q, int bytes) {
  if (kIType == PBZ_I8) {
    at[0] = uint8_t(q[0]);
    if (bytes > 1) at[1] = uint8_t(q[1]);
    if (bytes > 2) at[2] = uint8_t(q[2]);
    if (bytes > 3) at[3] = uint8_t(q[3]);
  } else if (kIType == PBZ_I16) {
    reinterpret_cast<uint16_t*>(at)[0] = uint16_t(q[0]);
    if (bytes > 2) reinterpret_cast<uint16_t*>(at)[1] = uint16_t(q[1]);
  } else {
    *reinterpret_cast<uint32_t*>(at) = uint32_t(q[0]);
  }
}

// ---------------------------------------------------------------------------------------------
// Algorithms 2 and 4: coefficients from one or two operands, then a new N and new indices; the arithmetic of
// k_add_vec / k_add_scalar_vec, element by element.  kTwo: C = F1 N1 + F2 (sign2 N2); otherwise
// C = N1 F1 / r, the first one moved by `shift`.
// ---------------------------------------------------------------------------------------------
template <int kIType, int kNType, bool kTwo>
struct Rebin {
  static constexpr int kPer = PerDword<kIType>::value;
  static constexpr bool kExactProducts = kNType != PBZ_F64 && kIType != PBZ_I32;
  double n1, n2, r, inv_r, shift;
  // the coefficients of a dword (`head`: the block's first); bytes that are zero come out as zero
  __device__ __forceinline__ void coefficients(uint32_t a, uint32_t b, bool head, double* c) const {
    double fa[kPer], fb[kPer];
    unpack_dword<kIType>(a, fa);
    if (kTwo) unpack_dword<kIType>(b, fb);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (kTwo) {
        c[e] = kExactProducts ? fma(fa[e], n1, fb[e] * n2) : unfused_sum_of_products(fa[e], n1, fb[e], n2);
      } else {
        c[e] = div_by(n1 * fa[e], r, inv_r);
        if (e == 0) c[e] += head ? shift : 0.0;
      }
    }
  }
  // scale: the value an index is a multiple of (kTwo: the new N = max / r; otherwise the maximum itself)
  __device__ __forceinline__ void indices(const double* c, double scale, double inv, int* q) const {
#pragma unroll
    for (int e = 0; e < kPer; ++e) q[e] = rint_to_int(div_by(kTwo ? c[e] : c[e] * r, scale, inv));
  }

  // A block whose numbers are out of reach of the products with reciprocals above, the whole way by division: a scale whose reciprocal is
  // infinite (below 5.6e-309) or whose own rounding leaves quotients beyond r (subnormal), infinite N (whose coefficients
  // div_by would turn into NaN) and NaN.  NaN counts for nothing in the maximum, and becomes the index -r.  One index at a
  // time: the path takes no registers from the others.  a, b, o: the block in LDS; one team of lanes.  Returns the new N.
  // (Other blocks of the tile go this way with it: their indices come out the same.)
  typedef typename IndexOf<kIType>::type index_t;
  __device__ __forceinline__ double far_block(int t, int team, int kept, const uint8_t* a, const uint8_t* b, uint8_t* o) const {
    double m = 0.0, n = 0.0;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
      for (int j = t; j < kept; j += team) {
        const double fa = double(reinterpret_cast<const index_t*>(a)[j]);
        double c;
        if (kTwo) c = unfused_sum_of_products(fa, n1, double(reinterpret_cast<const index_t*>(b)[j]), n2);
        else c = (n1 * fa) / r + (j == 0 ? shift : 0.0);
        m = fmax(m, fabs(c));
        if (pass == 1) {
          const double quo = n > 0.0 ? (kTwo ? c : c * r) / n : 0.0;
          reinterpret_cast<index_t*>(o)[j] = index_t(fmin(fmax(rint(quo), -r), r));
        }
      }
      for (int off = team >> 1; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
      n = kTwo ? m / r : m;
    }
    return n;
  }
};
constexpr double kFarNumber = 0x1p960;             // below it, products with an index and sums of two of them are finite

template <int kIType, int kNType, bool kTwo>
__global__ __launch_bounds__(64 * kMaxWaves) void k_rebin_staged(Stage st, const void* N1, const uint8_t* F1, const void* N2,
                                                                 const uint8_t* F2, void* Nout, uint8_t* Fout, double r,
                                                                 double sign2, double shift, int64_t n_blocks, int n_f16) {
  extern __shared__ __align__(16) uint8_t smem[];
  constexpr int kPer = PerDword<kIType>::value;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  uint8_t* sa = smem + wave * wave_bytes(st, kTwo ? 3 : 2, kTwo ? 2 : 1);
  uint8_t* so = sa + st.region;
  uint8_t* sb = so + st.region;                            // used with two operands only
  double* na = reinterpret_cast<double*>(sa + (kTwo ? 3 : 2) * st.region);
  double* nb = na + st.numbers / 8;
  const int team = 1 << st.team_shift, t = lane & (team - 1), slot = lane >> st.team_shift;
  const int per_round = 64 >> st.team_shift;
  const LaneRun run(st, t);
  const uint8_t* a_end = F1 + n_blocks * st.bpb;
  const uint8_t* b_end = kTwo ? F2 + n_blocks * st.bpb : nullptr;
  const int64_t stride = int64_t(gridDim.x) * waves * st.blocks;
  Rebin<kIType, kNType, kTwo> op;
  op.r = r;
  op.inv_r = 1.0 / r;
  op.shift = shift;
  for (int64_t k0 = (int64_t(blockIdx.x) * waves + wave) * st.blocks; k0 < n_blocks; k0 += stride) {
    const int count = n_blocks - k0 < st.blocks ? int(n_blocks - k0) : st.blocks;
    const int64_t at = k0 * st.bpb;
    const int len = count * st.bpb;
    StagedN<kNType> n1, n2;
    n1.request(N1, k0, count);
    if (kTwo) n2.request(N2, k0, count);
    stage_span<2>(F1, a_end, F1 + at, len, sa);
    if (kTwo) stage_span<2>(F2, b_end, F2 + at, len, sb);
    n1.put(na, count, n_f16 != 0);
    if (kTwo) n2.put(nb, count, n_f16 != 0);
    wave_lds_sync();
    const int pa = phase_of(F1 + at), pb = kTwo ? phase_of(F2 + at) : 0, po = phase_of(Fout + at);
    // a block that needs far_block: after the others, which that keeps out of the registers of this loop
    bool far = n1.beyond(kFarNumber, count) || (kTwo && n2.beyond(kFarNumber, count));
    for (int b0 = 0; b0 < count; b0 += per_round) {        // uniform: the lane exchanges below are convergent
      const int b = b0 + slot;
      const bool live = b < count;
      const int bc = live ? b : count - 1;                 // slots past the end redo the last block and store nothing
      op.n1 = na[bc];
      op.n2 = kTwo ? sign2 * nb[bc] : 0.0;
      double m = 0.0;
      const int from = bc * st.bpb + run.start;
      for_dwords<kTwo>(run, sa, pa + from, sb, pb + from, [&](int i, uint32_t va, uint32_t vb) {
        double c[kPer];
        op.coefficients(va, vb, i == 0 && t == 0, c);
#pragma unroll
        for (int e = 0; e < kPer; ++e) m = fmax(m, fabs(c[e]));
      });
      for (int off = team >> 1; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
      // an all-zero block has scale = inv = 0 and every c = 0, which gives 0; no quotient rounds beyond r
      const double n = kTwo ? m / r : m;
      const double inv = n > 0.0 ? 1.0 / n : 0.0;
      // the coefficients once more: cheaper than a place for them until the maximum is known
      if (live)
        for_dwords<kTwo>(run, sa, pa + from, sb, pb + from, [&](int i, uint32_t va, uint32_t vb) {
          double c[kPer];
          int q[kPer];
          op.coefficients(va, vb, i == 0 && t == 0, c);
          op.indices(c, n, inv, q);
          put_indices<kIType>(so + po + from + 4 * i, q, i < run.whole ? 4 : run.part);
        });
      if (!kTwo || kNType == PBZ_F64) far = far || !(inv < kFarNumber);     // sums of multiples of 2^-149 are within reach
      if (live && t == 0) store_N<kNType>(Nout, k0 + b, n, n_f16 != 0);
    }
    if (__any(far)) {
      wave_lds_sync();                                     // other lanes' writes to the same places precede these
      for (int b = slot; b < count; b += per_round) {
        op.n1 = na[b];
        op.n2 = kTwo ? sign2 * nb[b] : 0.0;
        const double n = op.far_block(t, team, st.kept, sa + pa + b * st.bpb, sb + pb + b * st.bpb, so + po + b * st.bpb);
        if (t == 0) store_N<kNType>(Nout, k0 + b, n, n_f16 != 0);
      }
    }
    wave_lds_sync();
    unstage_span(so, Fout + at, len);
    wave_lds_sync();
  }
}

// The same for blocks that a team holds in registers (at most held_dwords a lane), which is all but the largest.  Every lane takes `run`
// dwords: the last lane's are the block's last ones, which may be another lane's, too (the maximum does not mind, and both write the
// same indices); so is a lane's last dword where the block ends inside one, which starts four bytes before the block's end.
// So no dword is partial, and nothing is masked; the coefficients are computed once, the two divisions of a block by as few
// lanes as can hold it.
// What bounds it: 16 and 32 bits, HBM; their spans go to LDS past the registers, and the new indices take the first operand's
// place there where they are at the same phase, so that five waves fit a SIMD.  8 bits: the FP64 arithmetic (12 instructions an
// index, 2 cycles and more each); the lanes read their dwords straight from memory, at any alignment, which costs the texture path a
// look-up per lane and load (three quarters of its time with 38-byte blocks, where HBM would bind), but spares the detour's instructions.
// 2M blocks of 19 indices, sum and shift: 16 bits 85 and 67 -> 56 and 48 us (both straight from memory 68 and 53), 8 bits 54 and
// 41 -> 32 and 30 (through LDS 42 and 33); 300000 blocks of 33 32-bit ones 43 and 34 -> 28 and 17.  Before: teams of up to 4 dwords a
// lane, masked one by one, and three regions of LDS.  Not kept: waves that stay, with the next tile's loads in flight (16
// bits 78 us and 8 bits 55: 150 registers, three waves a SIMD); coefficients computed twice instead of held (76 and 57); dword stores to LDS at
// any alignment (two thirds of the kernel's time waiting for LDS).
constexpr int held_dwords(int itype, bool two) {          // what leaves five waves a SIMD without spills
  return itype == PBZ_I8 ? (two ? 5 : 6) : (itype == PBZ_I16 && two ? 10 : 12);
}
template <int kIType>
constexpr bool straight_from_memory() { return kIType == PBZ_I8; }

// n (at most kMain, the same in every lane) dwords from p on, at any alignment
template <int kMain>
__device__ __forceinline__ void load_dwords(const uint8_t* p, int n, uint32_t* w) {
#pragma unroll
  for (int j = 0; j < kMain; j += 4) {
    if (j + 4 <= n) {
      raw16 v;
      __builtin_memcpy(&v, p + 4 * j, 16);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j + u < kMain) w[j + u] = v[u];
    } else {
#pragma unroll
      for (int u = j; u < j + 4 && u < kMain; ++u)
        if (u < n) __builtin_memcpy(w + u, p + 4 * u, 4);
    }
  }
}

// A lane's new dwords to its place in the LDS region, whatever its alignment: in whole aligned words and, where it shares one with a
// neighbour, a half.  8-bit indices are put there one by one.
template <int kIType>
struct LaneOut {
  uint32_t* word;            // the next whole one
  uint32_t prev;
  int head;                  // bytes before the first whole word
  __device__ __forceinline__ LaneOut(uint8_t* lds, int at) {
    head = kIType == PBZ_I16 ? at & 2 : 0;
    word = reinterpret_cast<uint32_t*>(lds) + ((at + 3) >> 2);
  }
  __device__ __forceinline__ void put(uint32_t v, bool start) {
    if (!start || kIType == PBZ_I32) *word++ = kIType == PBZ_I32 ? v : __builtin_amdgcn_alignbyte(v, prev, uint32_t(head));
    else if (head) reinterpret_cast<uint16_t*>(word)[-1] = uint16_t(v);
    prev = v;
  }
  __device__ __forceinline__ void some(uint32_t v, int bytes) {
    if (bytes >= 4) *word = v;
    else if (bytes > 0) *reinterpret_cast<uint16_t*>(word) = uint16_t(v);
  }
  // the last dword, of which the first `bytes` count; `start`: it is the first, too
  __device__ __forceinline__ void finish(uint32_t v, int bytes, bool start) {
    if (kIType == PBZ_I32) {
      *word = v;
    } else {
      if (!start) {
        some(__builtin_amdgcn_alignbyte(v, prev, uint32_t(head)), 4 + bytes - head);
        ++word;
      } else if (head) {
        reinterpret_cast<uint16_t*>(word)[-1] = uint16_t(v);
      }
      some(v >> (8 * head), bytes - head);
    }
  }
};

// The bytes at p of a block of less than four in the operand [lo, hi), and others above them: one load, of the operand's last four bytes
// where the block is among those.
__device__ __forceinline__ uint32_t few_bytes(const uint8_t* lo, const uint8_t* hi, const uint8_t* p, int bytes) {
  uint32_t w = 0;
  if (hi - lo >= 4) {
    const uint8_t* q = p + 4 <= hi ? p : hi - 4;
    __builtin_memcpy(&w, q, 4);
    return w >> (8 * int(p - q));
  }
  for (int e = 0; e < bytes; ++e) w |= uint32_t(p[e]) << (8 * e);
  return w;
}

template <int kIType, int kNType, bool kTwo>
__global__ __launch_bounds__(64 * kMaxWaves, 5) void k_rebin_held(Stage st, const void* N1, const uint8_t* F1, const void* N2,
                                                               const uint8_t* F2, void* Nout, uint8_t* Fout, double r,
                                                               double sign2, double shift, int64_t n_blocks, int n_f16, int regions) {
  extern __shared__ __align__(16) uint8_t smem[];
  constexpr int kPer = PerDword<kIType>::value, kMain = held_dwords(kIType, kTwo) - 1;
  constexpr bool kStraight = straight_from_memory<kIType>();
  constexpr bool kLate = kStraight && !kTwo;             // the far blocks found behind the indices: shifts of 8 bits 1-4 % less, sums 1-2 % more
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  // LDS: the first operand, the second, and the result unless it takes the first one's place; of straight_from_memory only the result
  const bool in_place = !kStraight && regions == (kTwo ? 2 : 1);
  uint8_t* sa = smem + wave * regions * st.region;
  uint8_t* sb = sa + st.region;
  uint8_t* so = in_place ? sa : sa + (regions - 1) * st.region;
  const int team = 1 << st.team_shift, t = lane & (team - 1), slot = lane >> st.team_shift;
  const int per_round = 64 >> st.team_shift, run = st.run;
  const int start = 4 * (t * run < st.dwords - run ? t * run : st.dwords - run);
  const int tail = start + 4 * run < st.bpb ? start + 4 * (run - 1) : (st.bpb > 4 ? st.bpb - 4 : 0);      // the lane's last dword
  // bytes of the lane's run that only that dword holds (all of them where the block has no four bytes), and the bits of its others
  const int last_bytes = start + 4 * run < st.bpb ? 4 : st.bpb - start - 4 * (run - 1);
  const int drop = st.bpb < 4 ? 0 : 8 * (4 - last_bytes);
  const uint32_t cut = st.bpb < 4 ? (1u << (8 * st.bpb)) - 1u : ~0u;
  Rebin<kIType, kNType, kTwo> op;
  op.r = r;
  op.inv_r = 1.0 / r;
  op.shift = shift;
  // a tile per wave: memory ends before the largest grid does
  const int64_t k0 = (int64_t(blockIdx.x) * waves + wave) * st.blocks;
  if (k0 >= n_blocks) return;
  const int count = n_blocks - k0 < st.blocks ? int(n_blocks - k0) : st.blocks;
  const int64_t at = k0 * st.bpb;
  const int len = count * st.bpb;
  const uint8_t *a_end = F1 + n_blocks * st.bpb, *b_end = kTwo ? F2 + n_blocks * st.bpb : nullptr;
  if (!kStraight) {
    request_span(F1, a_end, F1 + at, len, sa);
    if (kTwo) request_span(F2, b_end, F2 + at, len, sb);
  }
  const int pa = phase_of(F1 + at), pb = kTwo ? phase_of(F2 + at) : 0, po = phase_of(Fout + at);
  int b0 = 0;
  for (; b0 < count; b0 += per_round) {                  // uniform: the lane exchanges below are convergent
    const int b = b0 + slot;
    const bool live = b < count;
    const int bc = live ? b : count - 1;                 // slots past the end redo the last block and store nothing
    const int base = bc * st.bpb;
    op.n1 = load_N<kNType>(N1, k0 + bc, n_f16 != 0);
    op.n2 = kTwo ? sign2 * load_N<kNType>(N2, k0 + bc, n_f16 != 0) : 0.0;
    uint32_t wa[kMain + 1], wb[kMain + 1];               // the last one's are the last of each
    wb[kMain] = 0;
    if constexpr (kStraight) {
      const uint8_t *a = F1 + at + base, *c = kTwo ? F2 + at + base : nullptr;
      load_dwords<kMain>(a + start, run - 1, wa);
      if (kTwo) load_dwords<kMain>(c + start, run - 1, wb);
      if (st.bpb >= 4) {
        __builtin_memcpy(wa + kMain, a + tail, 4);
        if (kTwo) __builtin_memcpy(wb + kMain, c + tail, 4);
      } else {
        wa[kMain] = few_bytes(F1, a_end, a, st.bpb) & cut;
        if (kTwo) wb[kMain] = few_bytes(F2, b_end, c, st.bpb) & cut;
      }
    } else {
      if (b0 == 0) span_arrived();
      const auto cut_out = [&](const uint8_t* lds, int from, int to, uint32_t* w) __attribute__((always_inline)) {
        const uint32_t* x = reinterpret_cast<const uint32_t*>(lds) + (from >> 2);
        const uint32_t* y = reinterpret_cast<const uint32_t*>(lds) + (to >> 2);
        w[0] = x[0];
#pragma unroll
        for (int u = 0; u < kMain; ++u) {
          if (u + 1 >= run) break;
          w[u + 1] = x[u + 1];
        }
        const uint32_t last = __builtin_amdgcn_alignbyte(y[1], y[0], uint32_t(to & 3)) & cut;
#pragma unroll
        for (int u = 0; u < kMain; ++u) {
          if (u + 1 >= run) break;
          w[u] = __builtin_amdgcn_alignbyte(w[u + 1], w[u], uint32_t(from & 3));
        }
        w[kMain] = last;
      };
      cut_out(sa, pa + base + start, pa + base + tail, wa);
      if (kTwo) cut_out(sb, pb + base + start, pb + base + tail, wb);
    }
    double c[(kMain + 1) * kPer], m = 0.0;
#pragma unroll
    for (int u = 0; u < kMain; ++u) {
      if (u + 1 >= run) break;
      op.coefficients(wa[u], kTwo ? wb[u] : 0u, u == 0 && t == 0, c + u * kPer);
#pragma unroll
      for (int e = 0; e < kPer; ++e) m = fmax(m, fabs(c[u * kPer + e]));
    }
    op.coefficients(wa[kMain], wb[kMain], st.dwords == 1, c + kMain * kPer);
#pragma unroll
    for (int e = 0; e < kPer; ++e) m = fmax(m, fabs(c[kMain * kPer + e]));
    for (int off = team >> 1; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    // an all-zero block has scale = inv = 0 and every c = 0, which gives 0; no quotient rounds beyond r
    const double n = kTwo ? m / r : m;
    const double inv = n > 0.0 ? 1.0 / n : 0.0;
    // A block that needs far_block: its round and those after it go there, behind this loop, whose registers that stays out of.  No N of
    // theirs has been written yet, nor an index where an operand is: both are the operands' still, whatever the result's buffers are.
    bool far = !(fabs(op.n1) < kFarNumber) || (kTwo && !(fabs(op.n2) < kFarNumber));
    if (!kTwo || kNType == PBZ_F64) far = far || !(inv < kFarNumber);     // sums of multiples of 2^-149 are within reach
    if (!kLate && __any(far)) break;
    if (live) {
      LaneOut<kIType> o(so, po + base + start);
#pragma unroll
      for (int u = 0; u < kMain; ++u) {
        if (u + 1 >= run) break;
        int q[kPer];
        op.indices(c + u * kPer, n, inv, q);
        if (kIType == PBZ_I8) put_indices<kIType>(so + po + base + start + 4 * u, q, 4);
        else o.put(pack_dword<kIType>(q), u == 0);
      }
      int q[kPer];
      op.indices(c + kMain * kPer, n, inv, q);
      if (kIType == PBZ_I8) put_indices<kIType>(so + po + base + tail, q, st.bpb < 4 ? st.bpb : 4);
      else o.finish(pack_dword<kIType>(q) >> drop, last_bytes, run == 1);
    }
    if (kLate && __any(far)) break;
    if (live && t == 0) store_N<kNType>(Nout, k0 + b, n, n_f16 != 0);
  }
  wave_lds_sync();
  if (b0 < count) {
    const uint8_t *a = kStraight ? F1 + at : sa + pa, *c = kStraight ? F2 + at : sb + pb;
    for (int b = b0 + slot; b < count; b += per_round) {
      op.n1 = load_N<kNType>(N1, k0 + b, n_f16 != 0);
      op.n2 = kTwo ? sign2 * load_N<kNType>(N2, k0 + b, n_f16 != 0) : 0.0;
      const double n = op.far_block(t, team, st.kept, a + b * st.bpb, kTwo ? c + b * st.bpb : nullptr, so + po + b * st.bpb);
      if (t == 0) store_N<kNType>(Nout, k0 + b, n, n_f16 != 0);
    }
    wave_lds_sync();
  }
  unstage_span(so, Fout + at, len);
}

// ---------------------------------------------------------------------------------------------
// Sums over blocks
// ---------------------------------------------------------------------------------------------
// exact integer sum of products over a lane's dwords of a block (FP64 for 32-bit indices)
template <int kIType>
struct Dot {
  typedef typename std::conditional<kIType == PBZ_I8, int, typename std::conditional<kIType == PBZ_I16, long long, double>::type>::type acc_t;
  static __device__ __forceinline__ acc_t add(acc_t acc, uint32_t a, uint32_t b) {
    if constexpr (kIType == PBZ_I8) return __builtin_amdgcn_sdot4(int(a), int(b), acc, false);
    else if constexpr (kIType == PBZ_I16) return acc + (long long)__builtin_amdgcn_sdot2(as_short2(a), as_short2(b), 0, false);
    else return acc + dot_dword<PBZ_I32>(a, b);
  }
  // the product of two blocks' first indices: taken out of a sum of integers, where that is exact; with 32 bits it is left out instead
  static __device__ __forceinline__ acc_t first(const uint8_t* a, const uint8_t* b) {
    if constexpr (kIType == PBZ_I8) return int(int8_t(*a)) * int(int8_t(*b));
    else if constexpr (kIType == PBZ_I16) return (long long)(int(*reinterpret_cast<const int16_t*>(a)) * int(*reinterpret_cast<const int16_t*>(b)));
    else return 0.0;
  }
};

template <int kIType, int kNType, bool kTwo>
__global__ __launch_bounds__(64 * kMaxWaves) void k_blockwise_staged(Stage st, const void* __restrict__ N1, const uint8_t* __restrict__ F1,
                                                                     const void* __restrict__ N2, const uint8_t* __restrict__ F2,
                                                                     double* __restrict__ out, double scale, int mode,
                                                                     int64_t n_blocks, int n_f16) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  uint8_t* sa = smem + wave * wave_bytes(st, kTwo ? 2 : 1, kTwo ? 2 : 1);
  uint8_t* sb = kTwo ? sa + st.region : sa;
  double* na = reinterpret_cast<double*>(sa + (kTwo ? 2 : 1) * st.region);
  double* nb = kTwo ? na + st.numbers / 8 : na;
  const int team = 1 << st.team_shift, t = lane & (team - 1), slot = lane >> st.team_shift;
  const int per_round = 64 >> st.team_shift;
  const LaneRun run(st, t);
  const uint8_t* a_end = F1 + n_blocks * st.bpb;
  const uint8_t* b_end = kTwo ? F2 + n_blocks * st.bpb : nullptr;
  const int64_t stride = int64_t(gridDim.x) * waves * st.blocks;
  for (int64_t k0 = (int64_t(blockIdx.x) * waves + wave) * st.blocks; k0 < n_blocks; k0 += stride) {
    const int count = n_blocks - k0 < st.blocks ? int(n_blocks - k0) : st.blocks;
    const int64_t at = k0 * st.bpb;
    StagedN<kNType> n1, n2;
    n1.request(N1, k0, count);
    if (kTwo) n2.request(N2, k0, count);
    request_span(F1, a_end, F1 + at, count * st.bpb, sa);
    if (kTwo) request_span(F2, b_end, F2 + at, count * st.bpb, sb);
    n1.put(na, count, n_f16 != 0);
    if (kTwo) n2.put(nb, count, n_f16 != 0);
    span_arrived();
    const int pa = phase_of(F1 + at), pb = kTwo ? phase_of(F2 + at) : pa;
    for (int b0 = 0; b0 < count; b0 += per_round) {
      const int b = b0 + slot;
      const int bc = b < count ? b : count - 1;
      typename Dot<kIType>::acc_t acc = 0;
      const int from = bc * st.bpb + run.start;
      for_dwords<kTwo>(run, sa, pa + from, sb, pb + from, [&](int i, uint32_t va, uint32_t vb) {
        if (kIType != PBZ_I32 || i > 0 || t > 0) acc = Dot<kIType>::add(acc, va, vb);
      });
      if (kIType != PBZ_I32 && t == 0)
        acc -= Dot<kIType>::first(sa + pa + bc * st.bpb, (kTwo ? sb + pb : sa + pa) + bc * st.bpb);
      double sum = double(acc);
      for (int off = team >> 1; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
      if (b < count && t == 0) {
        double res = sum * (na[bc] * nb[bc]) * scale;
        if (mode == kBwStd) res = sqrt(res);
        out[k0 + b] = res;
      }
    }
    wave_lds_sync();
  }
}

// the five sums of a reduction (see pbz_ops_common.h); grid y = segment of n_blocks blocks.  The spans go to LDS past the registers: 2M blocks of
// 19 int16 indices, variance 27 -> 23 us, covariance 50 -> 41 (through registers; 35 and 61 with lanes that took every team's
// dword); the block-wise covariance 40 -> 35 (53), which is what HBM gives.
template <int kIType, int kNType, bool kTwo, bool kDC, bool kDiff>
__global__ __launch_bounds__(64 * kMaxWaves) void k_reduce_staged(Stage st, const void* __restrict__ N1, const uint8_t* __restrict__ F1,
                                                                  const void* __restrict__ N2, const uint8_t* __restrict__ F2,
                                                                  int64_t n_blocks, ReduceTail tail) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  uint8_t* sa = smem + wave * wave_bytes(st, kTwo ? 2 : 1, kTwo ? 2 : 1);
  uint8_t* sb = kTwo ? sa + st.region : sa;
  double* na = reinterpret_cast<double*>(sa + (kTwo ? 2 : 1) * st.region);
  double* nb = kTwo ? na + st.numbers / 8 : na;
  const int team = 1 << st.team_shift, t = lane & (team - 1), slot = lane >> st.team_shift;
  const int per_round = 64 >> st.team_shift;
  const LaneRun run(st, t);
  const int64_t seg0 = int64_t(blockIdx.y) * n_blocks;             // the segment's first block
  F1 += seg0 * st.bpb;
  const uint8_t* a_end = F1 + n_blocks * st.bpb;
  if (kTwo) F2 += seg0 * st.bpb;
  const uint8_t* b_end = kTwo ? F2 + n_blocks * st.bpb : nullptr;
  const double K1 = kDC ? pilot_value(tail.pilot_n1, tail.pilot_f1, tail, blockIdx.y) : 0.0;
  const double K2 = kDC && kTwo ? pilot_value(tail.pilot_n2, tail.pilot_f2, tail, blockIdx.y) : 0.0;
  typedef typename IndexOf<kIType>::type index_t;
  const bool f16 = tail.n_f16 != 0;
  double sums[kNumSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int64_t stride = int64_t(gridDim.x) * waves * st.blocks;
  const int64_t first = (int64_t(blockIdx.x) * waves + wave) * st.blocks;
  const auto take = [&](auto far_t) __attribute__((always_inline)) {
    constexpr bool far = decltype(far_t)::value;
#pragma unroll 1
    for (int64_t k0 = first; k0 < n_blocks; k0 += stride) {
      const int count = n_blocks - k0 < st.blocks ? int(n_blocks - k0) : st.blocks;
      const int64_t at = k0 * st.bpb;
      StagedN<kNType> n1, n2;
      n1.request(N1, seg0 + k0, count);
      if (kTwo) n2.request(N2, seg0 + k0, count);
      request_span(F1, a_end, F1 + at, count * st.bpb, sa);
      if (kTwo) request_span(F2, b_end, F2 + at, count * st.bpb, sb);
      n1.put(na, count, f16);
      if (kTwo) n2.put(nb, count, f16);
      span_arrived();
      const int pa = phase_of(F1 + at), pb = kTwo ? phase_of(F2 + at) : pa;
      for (int b = slot; b < count; b += per_round) {
        const double v1 = na[b], v2 = nb[b];
        typename Dot<kIType>::acc_t s11 = 0, s12 = 0, s22 = 0;
        double diff = 0.0;
        if constexpr (kDiff && far) {
          constexpr int kPer = PerDword<kIType>::value;
#pragma unroll 1
          for (int j = t; j < st.kept; j += team) {
            double fa[kPer], fb[kPer];
            unpack_dword<kIType>(block_dword(sa, pa + b * st.bpb, j / kPer, st.bpb) >> (j % kPer * (32 / kPer)), fa);
            unpack_dword<kIType>(block_dword(sb, pb + b * st.bpb, j / kPer, st.bpb) >> (j % kPer * (32 / kPer)), fb);
            const double x = v1 * fa[0] - v2 * fb[0];
            diff += x * x;
          }
        } else {
          const int from = b * st.bpb + run.start;
          for_dwords<kTwo>(run, sa, pa + from, sb, pb + from, [&](int i, uint32_t va, uint32_t vb) {
            if constexpr (kDiff) {
              constexpr int kPer = PerDword<kIType>::value;
              double fa[kPer], fb[kPer];
              unpack_dword<kIType>(va, fa);
              unpack_dword<kIType>(vb, fb);
#pragma unroll
              for (int e = 0; e < kPer; ++e) {
                const double x = v1 * fa[e] - v2 * fb[e];
                diff += x * x;
              }
            } else if (!kDC || kIType != PBZ_I32 || i > 0 || t > 0) {
              s11 = Dot<kIType>::add(s11, va, va);
              if (kTwo) {
                s12 = Dot<kIType>::add(s12, va, vb);
                s22 = Dot<kIType>::add(s22, vb, vb);
              }
            }
          });
          if (kDC && t == 0) {                      // the first coefficient enters shifted by the pilot value
            const uint8_t *fa = sa + pa + b * st.bpb, *fb = kTwo ? sb + pb + b * st.bpb : fa;
            const double d1 = fma(v1, double(*reinterpret_cast<const index_t*>(fa)), -K1);
            sums[kS11] = fma(d1, d1, sums[kS11]);
            sums[kD1] += d1;
            s11 -= Dot<kIType>::first(fa, fa);
            if (kTwo) {
              const double d2 = fma(v2, double(*reinterpret_cast<const index_t*>(fb)), -K2);
              sums[kS12] = fma(d1, d2, sums[kS12]);
              sums[kS22] = fma(d2, d2, sums[kS22]);
              sums[kD2] += d2;
              s12 -= Dot<kIType>::first(fa, fb);
              s22 -= Dot<kIType>::first(fb, fb);
            }
          }
        }
        if constexpr (kDiff) {
          sums[kS11] += diff;
        } else {
          if constexpr (far) {
            for (int off = team >> 1; off > 0; off >>= 1) {
              s11 += __shfl_xor(s11, off, 64);
              s12 += __shfl_xor(s12, off, 64);
              s22 += __shfl_xor(s22, off, 64);
            }
            if (t != 0) continue;
          }
          sums[kS11] = fma(double(s11), v1 * v1, sums[kS11]);
          if (kTwo) {
            sums[kS12] = fma(double(s12), v1 * v2, sums[kS12]);
            sums[kS22] = fma(double(s22), v2 * v2, sums[kS22]);
          }
        }
      }
      wave_lds_sync();
    }
  };
  take(std::false_type());
  // A lane's sums that are no finite numbers: an infinite N times a zero is NaN, and zero is what a block's padding is, and what
  // the lane's own share of a block's indices may come to.  The wave then takes its blocks once more: without the
  // padding, and with the integer sums of whole blocks.
  bool finite = true;
#pragma unroll
  for (int i = 0; i < kNumSums; ++i) finite = finite && fabs(sums[i]) < INFINITY;
  if (!__all(finite)) {                                      // uniform over the wave
#pragma unroll
    for (int i = 0; i < kNumSums; ++i) sums[i] = 0.0;
    take(std::true_type());
  }
  reduce_tail(sums, tail, K1, K2, blockDim.x >> 6);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
unsigned group_count(int64_t n_blocks, const Stage& st, int waves, int64_t cap) {
  const int64_t per_group = int64_t(st.blocks) * waves;
  int64_t g = (n_blocks + per_group - 1) / per_group;
  return unsigned(g < cap ? g : cap);
}

template <int kIType, int kNType>
void rebin2(bool two, dim3 grid, dim3 block, size_t lds, hipStream_t s, const Stage& st, const void* N1, const void* F1,
            const void* N2, const void* F2, void* Nout, void* Fout, double r, double sign2, double shift, int64_t n_blocks,
            int n_f16, int regions) {
  const uint8_t *a = static_cast<const uint8_t*>(F1), *b = static_cast<const uint8_t*>(F2);
  uint8_t* o = static_cast<uint8_t*>(Fout);
  const bool held = st.run <= held_dwords(kIType, two);
#define PBZ_REBIN(KERNEL, TWO, ...) \
  hipLaunchKernelGGL((KERNEL<kIType, kNType, TWO>), grid, block, lds, s, st, N1, a, N2, b, Nout, o, r, sign2, shift, n_blocks, n_f16, ##__VA_ARGS__)
  if (two && held) PBZ_REBIN(k_rebin_held, true, regions);
  else if (held) PBZ_REBIN(k_rebin_held, false, regions);
  else if (two) PBZ_REBIN(k_rebin_staged, true);
  else PBZ_REBIN(k_rebin_staged, false);
#undef PBZ_REBIN
}

template <int kIType, int kNType>
void blockwise2(bool two, dim3 grid, dim3 block, size_t lds, hipStream_t s, const Stage& st, const void* N1, const void* F1,
                const void* N2, const void* F2, double* out, double scale, int mode, int64_t n_blocks, int n_f16) {
  const uint8_t *a = static_cast<const uint8_t*>(F1), *b = static_cast<const uint8_t*>(F2);
  if (two)
    hipLaunchKernelGGL((k_blockwise_staged<kIType, kNType, true>), grid, block, lds, s, st, N1, a, N2, b, out, scale, mode,
                       n_blocks, n_f16);
  else
    hipLaunchKernelGGL((k_blockwise_staged<kIType, kNType, false>), grid, block, lds, s, st, N1, a, N2, b, out, scale, mode,
                       n_blocks, n_f16);
}

template <int kIType, int kNType>
void reduce2(bool two, bool dc, bool diff, dim3 grid, dim3 block, size_t lds, hipStream_t s, const Stage& st, const void* N1,
             const void* F1, const void* N2, const void* F2, int64_t n_blocks, const ReduceTail& tail) {
  const uint8_t *a = static_cast<const uint8_t*>(F1), *b = static_cast<const uint8_t*>(F2);
#define PBZ_REDUCE(TWO, DC, DIFF) \
  hipLaunchKernelGGL((k_reduce_staged<kIType, kNType, TWO, DC, DIFF>), grid, block, lds, s, st, N1, a, N2, b, n_blocks, tail)
  if (diff) PBZ_REDUCE(true, false, true);
  else if (two && dc) PBZ_REDUCE(true, true, false);
  else if (two) PBZ_REDUCE(true, false, false);
  else if (dc) PBZ_REDUCE(false, true, false);
  else PBZ_REDUCE(false, false, false);
#undef PBZ_REDUCE
}

// CALL<index type, width of N>(arguments) for the codec's types
#define PBZ_BY_TYPES(CALL, ...)                                              \
  do {                                                                       \
    if (c->ftype == PBZ_F64) {                                               \
      if (c->itype == PBZ_I8) CALL<PBZ_I8, PBZ_F64>(__VA_ARGS__);            \
      else if (c->itype == PBZ_I16) CALL<PBZ_I16, PBZ_F64>(__VA_ARGS__);     \
      else CALL<PBZ_I32, PBZ_F64>(__VA_ARGS__);                              \
    } else if (c->ftype == PBZ_F32) {                                        \
      if (c->itype == PBZ_I8) CALL<PBZ_I8, PBZ_F32>(__VA_ARGS__);            \
      else if (c->itype == PBZ_I16) CALL<PBZ_I16, PBZ_F32>(__VA_ARGS__);     \
      else CALL<PBZ_I32, PBZ_F32>(__VA_ARGS__);                              \
    } else {                                                                 \
      if (c->itype == PBZ_I8) CALL<PBZ_I8, kN16>(__VA_ARGS__);               \
      else if (c->itype == PBZ_I16) CALL<PBZ_I16, kN16>(__VA_ARGS__);        \
      else CALL<PBZ_I32, kN16>(__VA_ARGS__);                                 \
    }                                                                        \
  } while (0)

constexpr int kRebinSpan = 2048, kReduceSpan = 4096;       // bytes of F per wave and operand
constexpr int64_t kMinWaves = 4096;                        // 16 per compute unit
constexpr int64_t kSecondLaunchBytes = 28 * 1024;          // of a segment and operand that further workgroups have to spare the first
constexpr int64_t kGroupCap = int64_t(1) << 30;            // the kernels loop beyond that

}  // namespace

int launch_rebin_staged(const pbz_codec* c, int64_t n_blocks, const void* N1, const void* F1, const void* N2, const void* F2,
                        void* Nout, void* Fout, double sign2, double shift, hipStream_t s) {
  const bool two = F2 != nullptr;
  const int team_dwords = held_dwords(c->itype, two);
  const Stage st = make_stage(c->kept, itype_bytes(c->itype), n_blocks, kRebinSpan, kMinWaves, team_dwords);
  const bool held = st.run <= team_dwords;
  const bool same_phase = ((reinterpret_cast<uintptr_t>(F1) ^ reinterpret_cast<uintptr_t>(Fout)) & 15u) == 0;
  const int regions = (two ? 3 : 2) - (held && same_phase ? 1 : 0);
  const int used = held && c->itype == PBZ_I8 ? 1 : regions;
  size_t lds;
  const int waves = waves_for(st, used, held ? 0 : (two ? 2 : 1), &lds);
  const dim3 grid(group_count(n_blocks, st, waves, kGroupCap)), block(64 * waves);
  const int n_f16 = c->ftype == PBZ_F16 ? 1 : 0;
  PBZ_BY_TYPES(rebin2, two, grid, block, lds, s, st, N1, F1, N2, F2, Nout, Fout, c->r, sign2, shift, n_blocks, n_f16, used);
  return hip_status(hipGetLastError());
}

int launch_blockwise_staged(const pbz_codec* c, int mode, int64_t n_blocks, const void* N1, const void* F1, const void* N2,
                            const void* F2, double* out, double scale, hipStream_t s) {
  const bool two = mode == kBwCovariance;
  const Stage st = make_stage(c->kept, itype_bytes(c->itype), n_blocks, kReduceSpan, kMinWaves);
  size_t lds;
  const int waves = waves_for(st, two ? 2 : 1, two ? 2 : 1, &lds);
  const dim3 grid(group_count(n_blocks, st, waves, kGroupCap)), block(64 * waves);
  const int n_f16 = c->ftype == PBZ_F16 ? 1 : 0;
  PBZ_BY_TYPES(blockwise2, two, grid, block, lds, s, st, N1, F1, N2, F2, out, scale, mode, n_blocks, n_f16);
  return hip_status(hipGetLastError());
}

int launch_reduce_staged(const pbz_codec* c, bool two, bool dc, bool diff, int64_t n_blocks, int n_segments, int max_groups,
                         const void* N1, const void* F1, const void* N2, const void* F2, const ReduceTail& tail, int* groups,
                         hipStream_t s) {
  // Up to 256 blocks in 16 KiB (a step of a short series; 12 KiB an operand where there are two: 13 KiB, pair statistics 11.5 us and
  // 9.9): one workgroup, which takes them in a tile per wave or two.  Dealt out to more workgroups they need the second launch
  // (156 blocks of 10 int32 indices, variance: 6.3 us and 8.1).
  const bool few = n_blocks <= 256 && n_blocks * c->kept * itype_bytes(c->itype) <= (two ? 12 : 16) * 1024;
  const Stage st = make_stage(c->kept, itype_bytes(c->itype), n_blocks, kReduceSpan, few ? kMaxWaves : kMinWaves / n_segments);
  size_t lds;
  const int waves = waves_for(st, two ? 2 : 1, two ? 2 : 1, &lds);
  // Four workgroups per compute unit for all segments together: what a workgroup does once, its sums over 64 lanes above all, is
  // spread over as many tiles as can be (16 segments of 18750 blocks of 33 int32 indices: variance 20 -> 16 us, covariance 33 -> 24; eight
  // per compute unit 18 and 27, two 20 and 28).  From some 340 segments on that is two or three of a segment's own, or one: one
  // where the others would spare it little, for they need the second launch (400 segments of 40 KiB, variance: 13.6 us, three 14.6; of
  // 157 KiB 45.8 and 28.3, of 516 KiB 101 and 58).
  const int64_t bytes = n_blocks * st.bpb;
  int64_t share = kReduceGroupsOneSegment / n_segments;
  if (share <= 2) {                        // to the nearest number then (150 segments of 516 KiB, covariance: six 40 us, seven, the nearest, 48)
    share = (kReduceGroupsOneSegment + n_segments / 2) / n_segments;
    if (share < 1 || bytes - bytes / share <= kSecondLaunchBytes) share = 1;
  }
  const unsigned all = group_count(n_blocks, st, waves, max_groups);
  unsigned g = share < int64_t(all) ? unsigned(share) : all;
  if (all <= 2 || few) g = 1;              // two tiles per wave: cheaper than a second launch
  *groups = int(g);
  const dim3 grid(g, unsigned(n_segments)), block(64 * waves);
  PBZ_BY_TYPES(reduce2, two, dc, diff, grid, block, lds, s, st, N1, F1, N2, F2, n_blocks, tail);
  return hip_status(hipGetLastError());
}

}  // namespace ops
}  // namespace pbz
