// General codec kernels for a list of block shapes, any array, working and index type, any mask, any alignment: what the
// specialised families leave to "generic" (4-D and flat blocks, 4x8x8, 8x16, 32x32, 1-D, and the families' shapes with
// types they are not built for).  pbz_tiled.hip takes the shapes that are not listed, and the calls that pays() below leaves it.
// The list is a choice, not a bound: the families' shapes, the cubes, squares and lines that the method is described for, and their
// neighbours.  The template takes any shape of its static_asserts' kind (8x8x4, 16x32 and 2x16 stay tiled at 2-3.4 TB/s); every
// shape adds 0.6 MB to the library, with two or three sizes of tile each way, and some seconds to its build.
//
// Wave autonomous like the families: a wave owns a tile of consecutive blocks, VALUES (8 to 64, by shape and size of the
// call: tiles()) values per lane in registers, no workgroup barrier, LDS private to the wave.  Two layouts, each with whole lines of its dimensions
// in a lane:
//   A  lane (s, b): rows s RA .. s RA + RA - 1 of block b, all of x (a block's rows in row-major order of the other
//      dimensions; RA = VALUES / BX).  How the array is read and written: the rows a lane needs come as 16-byte pieces, the
//      lanes of neighbouring blocks next to each other.  Transforms along x and the dimensions whole in RA rows.
//   B  lane (sr, sx, b): BXB columns of NR rows for every index of the remaining ("outer") dimensions, which are
//      transformed there.  How indices are made and read.
// Blocks of up to VALUES elements stay in layout A, several to a lane if smaller.  Between the layouts the tile passes through
// LDS, 16 bytes a slot, in as many rounds as a lane's BXB columns have slots, so that LDS holds a part of the tile at a time.
// Indices enter and leave F as in the families' kernels for any mask: dropped at their places in the span of F that the
// tile's blocks are, which moves in 16-byte pieces.
// The block shape is a template argument, so every index and bound is a constant but for the lane's own and the block's
// place in the array; types, mask and geometry are arguments, with one uniform branch around each loop.
// Memory bounds the FP32 work (4.3 - 5.1 TB/s of the copy's 5.6; wide blocks less, in the regrouped stores, and 16-bit arrays with
// int16 in 8x8x8 blocks, 2.1), FP64 work what is in flight (four waves per SIMD, two where blocks leave a lane 64 values; 4x4x4x4:
// vector ALUs a quarter busy, waves waiting half of their time).  Measured, us, with pbz_tiled.hip -> here:
//                                      compress      decompress
//   256x512x512 FP32, 4x8x8, i8        110 ->  66    100 ->  67
//   32x64x128x256 FP32, 2x4x8x8, i8    129 ->  66    112 ->  66
//   8192^2 FP32, 4x4, i8               101 ->  68     96 ->  68
//   8192^2 FP32, 8x16, i8               99 ->  68    107 ->  79
//   8192^2 FP32, 32x32, i8             134 ->  85    118 ->  90
//   256x512x512 FP32, 2x8x8, i16       168 ->  87    166 ->  91
//   16x32x128x256 FP64, 4^4, i32        65 ->  44     58 ->  47
//   512x512x256 bf16, 8x8x8, i16       193 ->  81    200 -> 131
//   509x509x251 bf16, 8x8x8, i8        138 ->  52    120 ->  59
//   4 Mi FP32, 64 (dense kernels)      181 ->  10    486 ->  11
#pragma once

#include <type_traits>

#include "pbz_fast_common.h"

namespace pbz {
namespace brick {
namespace {

using fast::bf16_t;
using fast::f16_t;
using fast::get_index;
using fast::put_index;

// n / d for n < 2^31: with s = ceil(log2 d) and m = floor(2^(31 + s) / d) + 1 the product exceeds n 2^(31 + s) / d by less
// than 2^(31 + s) / d, which never carries the quotient to the next integer
struct Divisor {
  uint32_t d, m, shift;
};
Divisor make_divisor(int64_t d) {
  Divisor v;
  uint32_t s = 0;
  while ((int64_t(1) << s) < d) ++s;
  v.d = uint32_t(d);
  v.shift = 31 + s;
  v.m = uint32_t((uint64_t(1) << v.shift) / uint64_t(d)) + 1;
  return v;
}
__device__ __forceinline__ uint32_t divide(uint32_t n, const Divisor& v, uint32_t* rest) {
  const uint32_t q = uint32_t((uint64_t(n) * v.m) >> v.shift);
  *rest = n - q * v.d;
  return q;
}

struct BrickGeom {
  uint32_t n_blocks;
  Divisor gx, gy, gz, gw;              // blocks along each dimension; what precedes them is folded (block extents 1)
  int64_t sy, sz, sw, sb;              // elements from one row, plane, ... to the next
  int lx, ly, lz, lw;                  // entries of the last block along each dimension that lie in the array
  int whole;                           // 1: every block lies in the array; 2: and its rows are whole lines of 128 bytes
  int xtype, ntype, itype, kept;
  int per_round;                       // blocks whose span of F is in LDS at a time
  uint32_t region;                     // bytes of a wave's LDS
  uint32_t run;                        // compressing: neighbouring workgroups that go to one die (group_in_runs)
  double r;
  const uint16_t* places;
};

// Rows whole in a lane that holds v values, and the outer indices that leaves
constexpr int inner_rows(int v, int bw, int bz, int by, int bx) {
  const int rows = bw * bz * by, ra = v / bx;
  return ra >= rows ? rows : (ra % (by * bz) == 0 ? by * bz : (ra % by == 0 ? by : 1));
}
constexpr int outer_rows(int v, int bw, int bz, int by, int bx) { return bw * bz * by / inner_rows(v, bw, bz, by, bx); }
// Whether a lane can hold v values of the block: whole rows, and every index of two outer dimensions at most
constexpr bool fits(int v, int bw, int bz, int by, int bx) {
  if (bx > v || bw * bz * by * bx > 64 * v) return false;
  if (bw * bz * by * bx < v) return true;
  const int in = inner_rows(v, bw, bz, by, bx), outer = (bw > 1 && in < bw * bz * by) + (bz > 1 && in < bz * by) + (by > 1 && in < by);
  return outer <= 2 && outer_rows(v, bw, bz, by, bx) <= v;
}

// Values that a lane holds: `few` for arrays of up to `few_to` elements, `many` for larger ones.
// A wave goes through its tile once, in one run of code as long as its lanes hold values, so that a call whose tiles leave SIMDs
// without a wave takes what one wave takes: few is the least that fits (the block's rows and outer indices allow 16 mostly, 32 for
// 32x32 and 4x8x8, 64 for 8x8x8, 2x2x8x8 and 2x4x8x8; 8 for blocks of 32 and 8x8, which are short enough to gain from it).  Time with
// few / time with 64 values in FP32 work and 32 in FP64 work, 21 shapes, nine types, both directions, geometric means:
//   elements       2^14 - 2^20    2^21    2^22    2^24    2^26
//   FP32 work      0.50 - 0.65    0.70    0.82    1.00    1.10
//   FP64 work      0.65 - 0.90    0.92    0.96    1.02    1.08
// (2^17 elements: 4x4 FP32 / i8 7.1 -> 3.6 us, 4x4x4x4 FP64 / i16 5.7 -> 4.5, 8192x16 FP16 / i16 compress 6 -> 4.3.)
// many: FP64 work holds 32 (16 for blocks of 16, and compressing where runs of two values and more of a row remain to each lane of
// layout B, OUT <= 8: 0.80-0.95 of 32's time), FP32 work 32 (0.85-0.95 of 64's time) but for
//   blocks of 256 and more that 16 does not fit: 64 (4x8x8, 32x32: 32 takes 1.05-1.2 of its time from 2^24 on);
//   FP32 work, blocks of 64, whole in a lane then: 64 (32: 1.03);
//   FP32 work, decompressing, blocks of 16, single rows under many outer indices, FP64 arrays: 64 (2x8x8: 32 takes 1.08 at 2^26; FP64 1.1);
//   FP32 work, compressing, blocks of 16 and FP64 arrays: 16 (0.9).
// few_to, where the two meet, is 4 Mi elements (one or two waves per SIMD with the larger tiles), 2 Mi for lanes of 8, and 8 Mi against
// 64 values of FP32 and for the runs above, decompressing; in FP64 work 16-bit arrays, whose compression waits least, 1 Mi (4x4x8 at 2 and
// 4 Mi: 1.08).
// What those means hide, by shape and mask: each line with the time at these sizes over the larger tiles' of 64
// (FP32 work) and 32 (FP64 work) values:
//   FP32 work, compressing, single rows under many outer indices (2x8x8, 16x8, 16x16): runs of two indices to a lane with 32 values, 1.15-1.45
//     from 2^22 on; with 16, a store each, 0.82-0.98; under a mask 2x8x8 with 32 1.05-1.13 and 64 then (16x8 with 32 0.95-1.0);
//   FP32 work, 4x4x4x4 of up to 32-bit arrays, nothing pruned: compressing 32 1.08-1.24, 16 0.87-1.0 up to 2^24 and 1.06-1.13 beyond, where 64;
//     decompressing 16-bit arrays 32 1.05-1.09, so 64;
//   4x8x8, compressing: 32 1.06-1.16 in FP32 work at 4 Mi (but FP64 arrays), under a mask at 2 Mi already (FP64 work 1.1-1.5); decompressing under
//     one in FP32 work 1.05 at 4 Mi;
//   4x4x8 in FP64 work under a mask, compressing: 16 1.1-1.4 from 1 Mi on;
//   2x8x8 of FP32 and FP64 arrays in FP32 work under a mask, decompressing: 16 1.03-1.08 at 4 Mi;
//   2x4x4x4 and 8x16 of up to 32-bit arrays in FP64 work under a mask, compressing: 16 0.87-1.0 up to 2^24, 1.04-1.07 beyond;
//   FP64 arrays with 8-bit indices: 4x8 and 8x4 compressing 8 1.07-1.1 from 1.5 Mi on; 4x4 decompressing under a mask 16 0.98 up to 2^25, 1.1 beyond.
struct Tiles {
  int few, many;
  int64_t few_to;
};
constexpr Tiles tiles(bool wide, bool compress, int array, int index, bool pruned, int bw, int bz, int by, int bx) {
  constexpr int64_t kMi = int64_t(1) << 20;
  const int rows = bw * bz * by, vol = rows * bx;
  const bool shortest = (vol == 32 && rows > 1) || (bw * bz == 1 && by == 8 && bx == 8);
  const int few = shortest ? 8 : (fits(16, bw, bz, by, bx) ? 16 : (fits(32, bw, bz, by, bx) ? 32 : 64));
  const bool narrow = vol != 32 && few <= 16 && outer_rows(16, bw, bz, by, bx) <= 8;
  const bool single = few == 16 && inner_rows(32, bw, bz, by, bx) == 1 && outer_rows(32, bw, bz, by, bx) > 8;
  const bool flat = bw * bz == 1, tesseract = bw == 4 && vol == 256, slab = few == 32 && vol == 256;
  int many = 32;
  if (bx == 64 || (few >= 32 && vol >= 256)) many = 64;
  else if (wide) many = vol == 16 || (compress && narrow) ? 16 : 32;
  else if (compress && single && (!pruned || !flat)) many = pruned ? 64 : 16;
  else if (compress && tesseract && !pruned && array < 8) many = 64;
  else if (compress) many = vol <= 16 || (array == 8 && few == 16) ? 16 : (vol == 64 ? 64 : 32);
  else if (array == 8 || vol <= 16 || vol == 64 || single || (tesseract && !pruned && array == 2)) many = 64;
  int64_t to = few == 8 ? 2 * kMi : 4 * kMi;
  if (few > 8 && (wide ? !compress && narrow : many == 64)) to = 8 * kMi;
  if (wide && compress && array == 2) to = few == 32 ? 2 * kMi : kMi;
  if (compress) {
    if (slab && pruned) to = 2 * kMi;
    else if (slab && array < 8 && to > 4 * kMi) to = 4 * kMi;
    else if (!wide && tesseract && !pruned && array < 8) to = 16 * kMi;
    else if (!wide && single && pruned && array < 8) to = 4 * kMi;
    else if (wide && pruned && bz == 4 && by == 4 && bx == 8) to = kMi;
    else if (wide && index == 1 && few == 8 && vol == 32) to = 3 * kMi / 2;
    if (wide && pruned && narrow && vol == 128 && array < 8) {
      many = 32;
      to = 16 * kMi;
    }
  } else if (pruned) {
    if (!wide && ((slab && array < 8) || (single && !flat && array > 2))) to = 4 * kMi;
    if (wide && index == 1 && vol == 16 && rows > 1) {
      many = 32;
      to = 32 * kMi;
    }
  }
  return {few, many, few == 64 ? 0 : to};
}
// whether kernels with v values are needed for any types and masks
constexpr bool needed(int v, bool wide, bool compress, int bw, int bz, int by, int bx) {
  for (int array = 2; array <= 8; array *= 2)
    for (int index = 1; index <= 4; index *= 2)
      for (int pruned = 0; pruned < 2; ++pruned) {
        const Tiles t = tiles(wide, compress, array, index, pruned != 0, bw, bz, by, bx);
        if (v == t.many || (v == t.few && t.few_to > 0)) return true;
      }
  return false;
}

template <typename T, int BW_, int BZ_, int BY_, int BX_, int VALUES_>
struct Shape {
  static constexpr int BW = BW_, BZ = BZ_, BY = BY_, BX = BX_;
  static constexpr int ROWS = BW * BZ * BY, VOL = ROWS * BX;
  static constexpr int VALUES = VALUES_;                           // a lane's
  static constexpr int PER_LANE = VOL < VALUES ? VALUES / VOL : 1; // blocks a lane holds
  static constexpr int LANES = VOL < VALUES ? 1 : VOL / VALUES;    // lanes a block takes
  static constexpr int NB = VOL < VALUES ? 64 * PER_LANE : 64 / LANES; // blocks of a tile
  static constexpr int RA = VOL < VALUES ? ROWS : VALUES / BX;     // rows per lane (and block)
  // rows of the dimensions that are whole in layout A, and of the outer ones
  static constexpr int IN = inner_rows(VALUES, BW, BZ, BY, BX);
  static constexpr int OUT = ROWS / IN;
  static_assert(BX <= VALUES && LANES <= 64 && RA % IN == 0, "a lane holds whole rows, and whole inner dimensions");
  static_assert(OUT <= VALUES, "a lane holds every outer index");
  static constexpr int BXB = OUT == 1 ? BX : (VALUES / OUT < BX ? VALUES / OUT : BX);
  static constexpr int NR = OUT == 1 ? RA : VALUES / (OUT * BXB);
  static constexpr int XG = BX / BXB;                              // groups of columns
  // the outer dimensions, from the inside: E1 and E2
  static constexpr int E1 = OUT == 1 ? 1 : (IN == BY * BZ ? BW : (IN == BY ? BZ : BY));
  static constexpr int E2 = OUT / E1;
  static_assert((BW > 1 && IN < ROWS) + (BZ > 1 && IN < BY * BZ) + (BY > 1 && IN < BY) <= 2, "E1 and E2 are one dimension each");
};

template <typename T, typename S>
struct Exchange {
  // Values per slot: 16 bytes, less where that would put the whole tile into LDS at once (16 KiB a wave: two waves per SIMD).
  // In two rounds at least: round trip of a 4-D FP64 field in 4^4 blocks 165 -> 153 us, 4096^2 FP16 / i16 in 32x32 blocks
  // compress 51 -> 33, decompress 77 -> 47
  static constexpr int FIT = 16 / int(sizeof(T)), HALF = S::BXB > 1 ? S::BXB / 2 : 1;
  static constexpr int CH = HALF < FIT ? HALF : FIT;
  static constexpr int ROUNDS = S::BXB / CH;
  static constexpr int BYTES = S::LANES == 1 ? 0 : 64 * S::VALUES / ROUNDS * int(sizeof(T));
  struct __attribute__((aligned(CH * sizeof(T)))) Slot { T v[CH]; };
  // The slots of the lanes that LDS serves at once (256 bytes' worth: 16 lanes of 16 bytes, 32 of 8, 64 of 4) should differ
  // modulo their number on both sides: the bits that vary from lane to lane are above that and folded onto the low ones.
  // At most two lanes meet, for most shapes none
  static __device__ __forceinline__ int slot(int b, int row, int xg) {
    const int q = (b * S::ROWS + row) * S::XG + xg;
    if constexpr (sizeof(Slot) == 16) return q ^ ((q >> 4) & 15) ^ ((q >> 8) & 15);
    else if constexpr (sizeof(Slot) == 8) return q ^ ((q >> 5) & 31);
    else return q ^ ((q >> 6) & 63);
  }
  // kToB: v (layout A) -> u (layout B); otherwise back
  template <bool kToB>
  static __device__ __forceinline__ void run(uint8_t* lds, int lane, T* v, T* u) {
    Slot* st = reinterpret_cast<Slot*>(lds);
    const int b = lane % S::NB, s = lane / S::NB;
    const int sx = s % S::XG, sr = s / S::XG;
#pragma unroll
    for (int rd = 0; rd < ROUNDS; ++rd) {
      if (rd) wave_lds_sync();
      if constexpr (kToB) {
#pragma unroll
        for (int i = 0; i < S::RA; ++i)
#pragma unroll
          for (int xg = 0; xg < S::XG; ++xg) {
            Slot t;
#pragma unroll
            for (int e = 0; e < CH; ++e) t.v[e] = v[i * S::BX + xg * S::BXB + rd * CH + e];
            st[slot(b, s * S::RA + i, xg)] = t;
          }
      } else {
#pragma unroll
        for (int o = 0; o < S::OUT; ++o)
#pragma unroll
          for (int j = 0; j < S::NR; ++j) {
            Slot t;
#pragma unroll
            for (int e = 0; e < CH; ++e) t.v[e] = u[(o * S::NR + j) * S::BXB + rd * CH + e];
            st[slot(b, o * S::IN + sr * S::NR + j, sx)] = t;
          }
      }
      wave_lds_sync();
      if constexpr (kToB) {
#pragma unroll
        for (int o = 0; o < S::OUT; ++o)
#pragma unroll
          for (int j = 0; j < S::NR; ++j) {
            const Slot t = st[slot(b, o * S::IN + sr * S::NR + j, sx)];
#pragma unroll
            for (int e = 0; e < CH; ++e) u[(o * S::NR + j) * S::BXB + rd * CH + e] = t.v[e];
          }
      } else {
#pragma unroll
        for (int i = 0; i < S::RA; ++i)
#pragma unroll
          for (int xg = 0; xg < S::XG; ++xg) {
            const Slot t = st[slot(b, s * S::RA + i, xg)];
#pragma unroll
            for (int e = 0; e < CH; ++e) v[i * S::BX + xg * S::BXB + rd * CH + e] = t.v[e];
          }
      }
    }
    wave_lds_sync();                       // the span of F uses the same LDS
  }
};

// the dimensions whole in layout A, of one block's RA x BX values
template <int TF, typename T, typename S, bool kForward>
__device__ __forceinline__ void inner_transforms(T* v) {
  auto along_x = [&]() {
#pragma unroll
    for (int i = 0; i < S::RA; ++i) {
      if constexpr (kForward) tf_forward<TF, T, S::BX, 1>(v + i * S::BX);
      else tf_inverse<TF, T, S::BX, 1, S::BX>(v + i * S::BX);
    }
  };
  // lines of n rows `stride` rows apart in runs of n * stride rows
  auto along_rows = [&](auto n_tag, auto stride_tag) {
    constexpr int n = decltype(n_tag)::value, stride = decltype(stride_tag)::value;
    if constexpr (n > 1) {
#pragma unroll
      for (int run = 0; run < S::RA / (n * stride); ++run)
#pragma unroll
        for (int k = 0; k < stride * S::BX; ++k) {
          T* line = v + run * n * stride * S::BX + k;
          if constexpr (kForward) tf_forward<TF, T, n, stride * S::BX>(line);
          else tf_inverse<TF, T, n, stride * S::BX, n>(line);
        }
    }
  };
  constexpr int ny = S::IN >= S::BY ? S::BY : 1;
  constexpr int nz = S::IN >= S::BY * S::BZ ? S::BZ : 1;
  constexpr int nw = S::IN >= S::BY * S::BZ * S::BW ? S::BW : 1;
  using y_t = std::integral_constant<int, ny>;
  using z_t = std::integral_constant<int, nz>;
  using w_t = std::integral_constant<int, nw>;
  if constexpr (kForward) {
    along_x();
    along_rows(y_t(), std::integral_constant<int, 1>());
    along_rows(z_t(), std::integral_constant<int, ny>());
    along_rows(w_t(), std::integral_constant<int, ny * nz>());
  } else {
    along_rows(w_t(), std::integral_constant<int, ny * nz>());
    along_rows(z_t(), std::integral_constant<int, ny>());
    along_rows(y_t(), std::integral_constant<int, 1>());
    along_x();
  }
}

template <int TF, typename T, typename S, bool kForward>
__device__ __forceinline__ void outer_transforms(T* u) {
  constexpr int step = S::NR * S::BXB;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const bool first = (pass == 0) == kForward;            // the inner of the two outer dimensions
    if (first) {
      if constexpr (S::E1 > 1) {
#pragma unroll
        for (int o = 0; o < S::E2; ++o)
#pragma unroll
          for (int k = 0; k < step; ++k) {
            if constexpr (kForward) tf_forward<TF, T, S::E1, step>(u + o * S::E1 * step + k);
            else tf_inverse<TF, T, S::E1, step, S::E1>(u + o * S::E1 * step + k);
          }
      }
    } else {
      if constexpr (S::E2 > 1) {
#pragma unroll
        for (int k = 0; k < S::E1 * step; ++k) {
          if constexpr (kForward) tf_forward<TF, T, S::E2, S::E1 * step>(u + k);
          else tf_inverse<TF, T, S::E2, S::E1 * step, S::E2>(u + k);
        }
      }
    }
  }
}

// ---- the array ---------------------------------------------------------------------------------------------------
struct Place {               // of a block, for one lane
  int64_t origin;            // element offset of its first row that the lane holds (clamped rows: of its first row)
  int ly, lz, lw;            // how many of the coordinates from the lane's first row on lie in the array
  bool tail;                 // the last block of its rows
};

// block k; first: the lane's first row in the block
template <typename S>
__device__ __forceinline__ Place place_of(const BrickGeom& g, uint32_t k, int first, int64_t* block_origin) {
  uint32_t kx, ky = 0, kz = 0, kw = 0;
  uint32_t rest = divide(k, g.gx, &kx);
  if (g.gy.d > 1) rest = divide(rest, g.gy, &ky);          // uniform
  if (g.gz.d > 1) rest = divide(rest, g.gz, &kz);
  if (g.gw.d > 1) rest = divide(rest, g.gw, &kw);
  const int64_t at = int64_t(rest) * g.sb + int64_t(kw) * S::BW * g.sw + int64_t(kz) * S::BZ * g.sz +
                     int64_t(ky) * S::BY * g.sy + int64_t(kx) * S::BX;
  *block_origin = at;
  const int y0 = first % S::BY, z0 = first / S::BY % S::BZ, w0 = first / (S::BY * S::BZ);
  Place p;
  p.origin = at + y0 * g.sy + z0 * g.sz + w0 * g.sw;
  p.tail = kx == g.gx.d - 1;
  p.ly = (ky == g.gy.d - 1 ? g.ly : S::BY) - y0;
  p.lz = (kz == g.gz.d - 1 ? g.lz : S::BZ) - z0;
  p.lw = (kw == g.gw.d - 1 ? g.lw : S::BW) - w0;
  return p;
}

// row i of the lane's: offset from its first, and whether it lies in the array
template <typename S>
__device__ __forceinline__ int64_t row_offset(const BrickGeom& g, int i) {
  return (i % S::BY) * g.sy + (i / S::BY % S::BZ) * g.sz + (i / (S::BY * S::BZ)) * g.sw;
}
template <typename S>
__device__ __forceinline__ bool row_inside(const Place& p, int i) {
  bool in = true;
  if (S::BY > 1) in = in && i % S::BY < p.ly;
  if (S::BZ > 1) in = in && i / S::BY % S::BZ < p.lz;
  if (S::BW > 1) in = in && i / (S::BY * S::BZ) < p.lw;
  return in;
}

constexpr int kStoreBytes = 8192;      // of LDS that rows pass through on their way out, unless a row of every lane is more

// pieces of a row: 16 bytes, or the whole row where it is shorter
template <typename XT, typename S>
struct Piece {
  static constexpr int BYTES = S::BX * int(sizeof(XT)) < 16 ? S::BX * int(sizeof(XT)) : 16;
  static constexpr int PER = BYTES / int(sizeof(XT)), COUNT = S::BX / PER;
  struct __attribute__((packed, aligned(sizeof(XT) < 4 ? 2 : 4))) Loose { uint32_t w[BYTES / 4]; };
  struct __attribute__((aligned(BYTES))) Aligned { uint32_t w[BYTES / 4]; };
  typedef uint32_t Words __attribute__((ext_vector_type(4)));      // of a piece of 16 bytes
  template <typename T>
  static __device__ __forceinline__ void unpack(const uint32_t* w, T* out) {
    if constexpr (sizeof(XT) == 8) {
#pragma unroll
      for (int e = 0; e < PER; ++e)
        out[e] = T(__longlong_as_double((long long)((uint64_t(w[2 * e + 1]) << 32) | w[2 * e])));
    } else if constexpr (sizeof(XT) == 4) {
#pragma unroll
      for (int e = 0; e < PER; ++e) out[e] = T(__uint_as_float(w[e]));
    } else {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const uint16_t h = uint16_t(w[e / 2] >> (16 * (e & 1)));
        if constexpr (std::is_same<XT, bf16_t>::value) out[e] = T(bf16_bits_to_float(h));
        else out[e] = T(float(__builtin_bit_cast(_Float16, h)));
      }
    }
  }
  // one rounding from T to the array's type
  template <typename T>
  static __device__ __forceinline__ uint16_t half_bits(T v) {
    if constexpr (std::is_same<XT, bf16_t>::value) return sizeof(T) == 8 ? double_to_bf16_bits(double(v)) : float_to_bf16_bits(float(v));
    else return __builtin_bit_cast(uint16_t, sizeof(T) == 8 ? double_to_f16(double(v)) : _Float16(float(v)));
  }
  template <typename T>
  static __device__ __forceinline__ void pack(const T* v, uint32_t* w) {
    if constexpr (sizeof(XT) == 8) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const uint64_t bits = uint64_t(__double_as_longlong(double(v[e])));
        w[2 * e] = uint32_t(bits);
        w[2 * e + 1] = uint32_t(bits >> 32);
      }
    } else if constexpr (sizeof(XT) == 4) {
#pragma unroll
      for (int e = 0; e < PER; ++e) w[e] = __float_as_uint(float(v[e]));
    } else {
#pragma unroll
      for (int e = 0; e < PER; e += 2) w[e / 2] = uint32_t(half_bits<T>(v[e])) | (uint32_t(half_bits<T>(v[e + 1])) << 16);
    }
  }
};

// the lane's RA rows of a block into v, padding as zeros; sixteen pieces in flight (more would be registers for FP64 arrays
// in FP32 work only)
template <typename T, typename XT, typename S>
__device__ __forceinline__ void load_rows(const BrickGeom& g, const XT* x, const Place& p, int64_t block_origin, T* v) {
  using P = Piece<XT, S>;
  constexpr int ROWS = P::COUNT * S::RA <= 16 ? S::RA : (P::COUNT >= 16 ? 1 : 16 / P::COUNT), N = ROWS * P::COUNT;
  if (g.whole) {                                           // uniform
#pragma unroll
    for (int i0 = 0; i0 < S::RA; i0 += ROWS) {
      typename P::Aligned raw[N];
      if (i0 > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int k = 0; k < P::COUNT; ++k)
          raw[i * P::COUNT + k] =
              *reinterpret_cast<const typename P::Aligned*>(x + p.origin + row_offset<S>(g, i0 + i) + k * P::PER);
#pragma unroll
      for (int i = 0; i < N; ++i) P::template unpack<T>(raw[i].w, v + i0 * S::BX + i * P::PER);
    }
    return;
  }
  // Rows that start anywhere.  Rows outside the array: the block's first one instead, zeroed below.  In the last block of a
  // row a piece that reaches beyond it is read from as much further to the left (a row has a piece's elements at least),
  // and shifted into place.
#pragma unroll
  for (int i0 = 0; i0 < S::RA; i0 += ROWS) {
    typename P::Loose raw[N];
    if (i0 > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int64_t row = row_inside<S>(p, i0 + i) ? p.origin + row_offset<S>(g, i0 + i) : block_origin;
#pragma unroll
      for (int k = 0; k < P::COUNT; ++k) {
        const int over = (k + 1) * P::PER - g.lx;          // uniform
        raw[i * P::COUNT + k] =
            *reinterpret_cast<const typename P::Loose*>(x + row + k * P::PER - (p.tail && over > 0 ? over : 0));
      }
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const bool in = row_inside<S>(p, i0 + i);
#pragma unroll
      for (int k = 0; k < P::COUNT; ++k) {
        T* out = v + (i0 + i) * S::BX + k * P::PER;
        P::template unpack<T>(raw[i * P::COUNT + k].w, out);
        const int over = (k + 1) * P::PER - g.lx;
        if (over > 0) {                                    // uniform
#pragma unroll
          for (int sh = 1; sh < P::PER; sh *= 2)
            if (over & sh) {
#pragma unroll
              for (int e = 0; e < P::PER; ++e)
                out[e] = p.tail ? (e + sh < P::PER ? out[e + sh < P::PER ? e + sh : 0] : T(0)) : out[e];
            }
          if (over >= P::PER) {
#pragma unroll
            for (int e = 0; e < P::PER; ++e) out[e] = p.tail ? T(0) : out[e];
          }
        }
#pragma unroll
        for (int e = 0; e < P::PER; ++e) out[e] = in ? out[e] : T(0);
      }
    }
  }
}

// The lane's RA rows of a block to the array.  Rows of several pieces leave through LDS: written as they are, an instruction
// would store every second to sixteenth piece of the run that neighbouring blocks' rows are (decompress of 8192^2 FP32 in
// 8x16 blocks 110 us, 79 as here; in 32x32 blocks 135 and 90; 4x8x8 of the same size 77 and 67).  Piece k of lane L goes
// to slot L COUNT + k, and 64 consecutive slots are stored at a time, each by a lane that has got lane L's place from it.
// active: the lane's block exists.
// kWhole as BrickGeom::whole.  Where rows are whole lines, pieces of 16 bytes go out with the non-temporal hint: what is written does not stay in the
// caches to be written out beside the reads of the next call.  32x64x128x128 FP64 / i16 in 4^4 blocks, by turns: decompress 62 -> 54 us, the compress of
// another array that follows 89 -> 61.  At any size, as the array's reader is seldom the next kernel.  Time with the hint / without, of six shapes and
// types, arrays one after another (least, mean and largest; us are decompress of 4x8x8 FP32):
//   the array          4 MiB               16 MiB              32-128 MiB          256-512 MiB
//   decompress         0.89 0.94 1.00      0.73 0.79 0.87      0.78 0.84 0.97      0.83 0.87 1.07     (7, 11 -> 9, 15 -> 12 ... 37 -> 32, 68 -> 59)
//   and a pass         1.02 1.02 1.02      0.99 1.03 1.05      0.99 1.05 1.10      0.95 0.97 1.00     (of it that at once reads what was written)
//   and its compress   1.01 1.01 1.02      0.91 0.94 0.99      0.93 1.01 1.09      0.84 0.91 1.03
// Lines that rows only share are written twice then: 92x92x92x88 FP32 in 4^4 blocks (352-byte rows) 1.37 of the time, so not there; nor for loads, whose
// lines would be fetched anew by the next piece (1.1-2.4).  A tile of 4^4 blocks of FP32 with 16 values a lane has half lines, whose other halves the
// next wave stores at about the same time: 0.93-1.01 at 4 MiB, 0.87-0.92 at 16, no worse than the whole lines of larger arrays.
template <int kWhole, typename T, typename XT, typename S>
__device__ __forceinline__ void store_rows(const BrickGeom& g, uint8_t* lds, int lane, XT* y, const Place& p, bool active,
                                           const T* v) {
  using P = Piece<XT, S>;
  constexpr int COUNT = P::COUNT;
  uint32_t rows = 0;                                       // which of the lane's rows lie in the array
#pragma unroll
  for (int i = 0; i < S::RA; ++i) rows |= row_inside<S>(p, i) ? 1u << i : 0u;
  const uint32_t flags = active ? rows | (p.tail ? 1u << 31 : 0u) : 0u;
  static_assert(S::RA <= 16, "rows and the tail's mark share a word");
  auto put_piece = [&](int64_t origin, uint32_t f, int i, int k, const uint32_t* w) {
    XT* at = y + origin + row_offset<S>(g, i) + k * P::PER;
    if constexpr (kWhole) {
      if (f != 0u) {
        typename P::Aligned raw;
#pragma unroll
        for (int e = 0; e < P::BYTES / 4; ++e) raw.w[e] = w[e];
        if constexpr (kWhole == 2 && P::BYTES == 16) {
          const typename P::Words line = {raw.w[0], raw.w[1], raw.w[2], raw.w[3]};
          __builtin_nontemporal_store(line, reinterpret_cast<typename P::Words*>(at));
        } else {
          *reinterpret_cast<typename P::Aligned*>(at) = raw;
        }
      }
    } else if ((f >> i) & 1u) {
      if (!(f >> 31) || (k + 1) * P::PER <= g.lx) {
        typename P::Loose raw;
#pragma unroll
        for (int e = 0; e < P::BYTES / 4; ++e) raw.w[e] = w[e];
        *reinterpret_cast<typename P::Loose*>(at) = raw;
      } else {
#pragma unroll
        for (int e = 0; e < P::PER; ++e)
          if (k * P::PER + e < g.lx) {
            if constexpr (sizeof(XT) == 8) at[e] = __longlong_as_double((long long)((uint64_t(w[2 * e + 1]) << 32) | w[2 * e]));
            else if constexpr (sizeof(XT) == 4) at[e] = __uint_as_float(w[e]);
            else at[e].bits = uint16_t(w[e / 2] >> (16 * (e & 1)));
          }
      }
    }
  };
  if constexpr (COUNT == 1) {
#pragma unroll
    for (int i = 0; i < S::RA; ++i) {
      uint32_t w[P::BYTES / 4];
      P::template pack<T>(v + i * S::BX, w);
      put_piece(p.origin, flags, i, 0, w);
    }
  } else {
    constexpr int FIT = kStoreBytes / (1024 * COUNT);      // rows of every lane that the LDS holds
    constexpr int BATCH = FIT < 1 ? 1 : (FIT < S::RA ? FIT : S::RA);
    auto slot = [](int i) { return i ^ ((i >> 3) & 7) ^ ((i >> 6) & 7); };
    uint4* st = reinterpret_cast<uint4*>(lds);
#pragma unroll
    for (int i0 = 0; i0 < S::RA; i0 += BATCH) {
#pragma unroll
      for (int i = 0; i < BATCH; ++i)
#pragma unroll
        for (int k = 0; k < COUNT; ++k) {
          uint32_t w[4];
          P::template pack<T>(v + (i0 + i) * S::BX + k * P::PER, w);
          st[i * 64 * COUNT + slot(lane * COUNT + k)] = make_uint4(w[0], w[1], w[2], w[3]);
        }
      wave_lds_sync();
      // of the lanes' places in registers at a time (all of them, for all rows: 32x32 blocks 196 registers and 102 us; so 164
      // and 90)
      constexpr int TOGETHER = COUNT < 4 ? COUNT : 4;
#pragma unroll TOGETHER
      for (int t = 0; t < COUNT; ++t) {
        const int from = (t * 64 + lane) / COUNT;
        const int64_t origin = __shfl((long long)p.origin, from, 64);
        const uint32_t f = __shfl(flags, from, 64);
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
          const uint4 q = st[i * 64 * COUNT + slot(t * 64 + lane)];
          const uint32_t w[4] = {q.x, q.y, q.z, q.w};
          put_piece(origin, f, i0 + i, lane % COUNT, w);
        }
      }
      wave_lds_sync();
    }
  }
}

// f(XT()) for the array's type
template <typename F>
__device__ __forceinline__ void by_array_type(int xtype, F f) {
  switch (xtype) {
    case PBZ_F64: f(double()); break;
    case PBZ_F32: f(float()); break;
    case PBZ_BF16: f(bf16_t()); break;
    default: f(f16_t()); break;
  }
}
template <typename F>
__device__ __forceinline__ void by_index_type(int itype, F f) {
  switch (itype) {
    case PBZ_I8: f(int8_t()); break;
    case PBZ_I16: f(int16_t()); break;
    default: f(int32_t()); break;
  }
}

// the places of kCount (1, 2, 4, or a multiple of 8) entries in a row of the table, in 16-bit halves of w
template <int kCount>
__device__ __forceinline__ void load_place_row(const uint16_t* pos, uint32_t* w) {
  if constexpr (kCount == 1) {
    w[0] = pos[0];
  } else if constexpr (kCount == 2) {
    w[0] = *reinterpret_cast<const uint32_t*>(pos);
  } else if constexpr (kCount == 4) {
    const uint2 t = *reinterpret_cast<const uint2*>(pos);
    w[0] = t.x; w[1] = t.y;
  } else {
#pragma unroll
    for (int k = 0; k < kCount / 8; ++k) {
      const uint4 t = reinterpret_cast<const uint4*>(pos)[k];
      w[4 * k] = t.x; w[4 * k + 1] = t.y; w[4 * k + 2] = t.z; w[4 * k + 3] = t.w;
    }
  }
}
template <typename IT>
__device__ __forceinline__ uint32_t place_address(const uint32_t* w, int e, uint32_t base, uint32_t aside) {
  const uint32_t p = (e & 1) ? w[e >> 1] >> 16 : w[e >> 1] & 0xffffu;
  const uint32_t at = base + p * uint32_t(sizeof(IT));
  return at < aside ? at : aside;
}

// kCount packed indices from LDS address `at` (a multiple of 4, or of kCount bytes where that is less)
template <typename IT, int kCount>
__device__ __forceinline__ void put_run(uint8_t* lds, uint32_t at, const uint32_t* q) {
  constexpr int PER = fast::IdxPack<IT>::per;
  if constexpr (kCount < PER) {
#pragma unroll
    for (int e = 0; e < kCount; ++e) put_index<IT>(lds, at + e * uint32_t(sizeof(IT)), q[e]);
  } else {
#pragma unroll
    for (int k = 0; k < kCount / PER; ++k) *reinterpret_cast<uint32_t*>(lds + at + 4 * k) = fast::IdxPack<IT>::pack(q + k * PER);
  }
}
template <typename IT, int kCount>
__device__ __forceinline__ void get_run(const uint8_t* lds, uint32_t at, int* f) {
  constexpr int PER = fast::IdxPack<IT>::per;
  if constexpr (kCount < PER) {
#pragma unroll
    for (int e = 0; e < kCount; ++e) f[e] = get_index<IT>(lds, at + e * uint32_t(sizeof(IT)));
  } else {
#pragma unroll
    for (int k = 0; k < kCount / PER; ++k) {
      const uint32_t w = *reinterpret_cast<const uint32_t*>(lds + at + 4 * k);
#pragma unroll
      for (int e = 0; e < PER; ++e) f[k * PER + e] = fast::IdxPack<IT>::get(w, e);
    }
  }
}

// Walks the lane's values in layout B: f(block of the tile, first entry in the block, first value, count tag) for each
// run of BXB values whose entries are consecutive.
template <typename S, typename F>
__device__ __forceinline__ void each_run(int lane, F f) {
  if constexpr (S::PER_LANE > 1) {
#pragma unroll
    for (int p = 0; p < S::PER_LANE; ++p)
#pragma unroll
      for (int i = 0; i < S::ROWS; ++i) f(p * 64 + lane, i * S::BX, p * S::VOL + i * S::BX);
  } else {
    const int b = lane % S::NB, s = lane / S::NB, sx = s % S::XG, sr = s / S::XG;
#pragma unroll
    for (int o = 0; o < S::OUT; ++o)
#pragma unroll
      for (int j = 0; j < S::NR; ++j)
        f(b, (o * S::IN + sr * S::NR + j) * S::BX + sx * S::BXB, (o * S::NR + j) * S::BXB);
  }
}

// Which tiles a workgroup of compress takes: its own number's, or, with runs (a power of two), those by which `run` neighbours in F are on one die.
// Workgroups go to the eight dies in turn, each with an L2 of its own, and a reduction's workgroups take 32 KiB of F each: what a die wrote, it then
// reads.  The smaller tiles, of 8 and 16 KiB of 32-bit indices, would have given each of its reads halves or quarters of two and four dies.  (Statistics along
// with the compression, 132x206x136 FP32 / i32 in 4x4x8 blocks: with tiles of 32 values a lane 20.2 us, with 16 24.2, with 16 in runs 19.0; the compression alone 12.3, 11.2, 10.6.)
__device__ __forceinline__ uint32_t group_in_runs(uint32_t run) {
  const uint32_t b = blockIdx.x, q = b & (8 * run - 1);
  return run > 1 && (b | (8 * run - 1)) < gridDim.x ? b - q + (q & 7) * run + (q >> 3) : b;
}
template <int TF, typename T, typename S>
__global__ __launch_bounds__(256, 2) void k_compress_brick(BrickGeom g, const void* __restrict__ x, void* __restrict__ N,
                                                        void* __restrict__ F) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  uint8_t* st = smem + (threadIdx.x >> 6) * g.region;
  const uint32_t tile = group_in_runs(g.run) * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t k0 = tile * S::NB;
  if (k0 >= g.n_blocks) return;                            // uniform over the wave
  const int n_active = int(g.n_blocks - k0 < uint32_t(S::NB) ? g.n_blocks - k0 : S::NB);
  T v[S::VALUES], u_[S::LANES > 1 ? S::VALUES : 1];
  T* u = S::LANES > 1 ? u_ : v;
  by_array_type(g.xtype, [&](auto tag) {
    using XT = decltype(tag);
#pragma unroll
    for (int p = 0; p < S::PER_LANE; ++p) {
      const int b = S::PER_LANE > 1 ? p * 64 + lane : lane % S::NB;
      int64_t block_origin;
      const Place at = place_of<S>(g, k0 + (b < n_active ? b : n_active - 1), S::LANES > 1 ? lane / S::NB * S::RA : 0, &block_origin);
      load_rows<T, XT, S>(g, static_cast<const XT*>(x), at, block_origin, v + p * S::VOL);
    }
  });
#pragma unroll
  for (int p = 0; p < S::PER_LANE; ++p) inner_transforms<TF, T, S, true>(v + p * S::VOL);
  if constexpr (S::LANES > 1) {
    Exchange<T, S>::template run<true>(st, lane, v, u);
    outer_transforms<TF, T, S, true>(u);
  }
  fast::Binner<T> binner[S::PER_LANE];
#pragma unroll
  for (int p = 0; p < S::PER_LANE; ++p) {
    constexpr int kValues = S::PER_LANE > 1 ? S::VOL : S::VALUES;
    T m = T(0);
#pragma unroll
    for (int i = 0; i < kValues; ++i) m = fmax(m, fabs(u[p * S::VOL + i]));
    if constexpr (S::LANES > 1) {
#pragma unroll
      for (int off = S::NB; off < 64; off <<= 1) m = fmax(m, __shfl_xor(m, off, 64));
    }
    binner[p] = fast::Binner<T>(m, g.r);
    const int b = S::PER_LANE > 1 ? p * 64 + lane : lane % S::NB;
    if (b < n_active && lane / S::NB == 0) store_float(N, g.ntype, int64_t(k0) + b, m);
  }
  uint32_t q[S::VALUES];
#pragma unroll
  for (int i = 0; i < S::VALUES; ++i) q[i] = binner[S::PER_LANE > 1 ? i / S::VOL : 0].bits(u[i]);
  // once for all index types and before anything is placed: 64 registers less than quotients formed at each place (FP64
  // work: 98 instead of 214; compress of 512x512x256 bf16 / i16 in 8x8x8 blocks 108 -> 80 us)
  __builtin_amdgcn_sched_barrier(0);
  by_index_type(g.itype, [&](auto tag) {
    using IT = decltype(tag);
    if constexpr (sizeof(T) == 8 || sizeof(IT) == 1) {
      const int bytes = g.kept * int(sizeof(IT));
      const uint32_t aside = g.region - 256 + uint32_t(lane) * 4u;
      for (int first = 0; first < n_active; first += g.per_round) {
        const int count = n_active - first < g.per_round ? n_active - first : g.per_round;
        uint8_t* dst = static_cast<uint8_t*>(F) + (int64_t(k0) + first) * bytes;
        const int phase = phase_of(dst);
        const bool runs = g.kept == S::VOL && (phase & 3) == 0;             // uniform: entries are their own places
        each_run<S>(lane, [&](int b, int entry, int value) {
          if (b >= first && b < first + count) {
            const uint32_t base = uint32_t(phase + (b - first) * bytes);
            if (runs) {
              put_run<IT, S::BXB>(st, base + uint32_t(entry) * uint32_t(sizeof(IT)), q + value);
            } else {
              uint32_t places[(S::BXB + 1) / 2];
              load_place_row<S::BXB>(g.places + entry, places);
#pragma unroll
              for (int e = 0; e < S::BXB; ++e) put_index<IT>(st, place_address<IT>(places, e, base, aside), q[value + e]);
            }
          }
        });
        wave_lds_sync();
        unstage_span(st, dst, count * bytes);
        wave_lds_sync();
      }
    }
  });
}

template <int TF, typename T, typename S>
__global__ __launch_bounds__(256, 2) void k_decompress_brick(BrickGeom g, const void* __restrict__ N, const void* __restrict__ F,
                                                          void* __restrict__ y) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  uint8_t* st = smem + (threadIdx.x >> 6) * g.region;
  const uint32_t tile = blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t k0 = tile * S::NB;
  if (k0 >= g.n_blocks) return;                            // uniform over the wave
  const int n_active = int(g.n_blocks - k0 < uint32_t(S::NB) ? g.n_blocks - k0 : S::NB);
  T v[S::VALUES], u_[S::LANES > 1 ? S::VALUES : 1];
  T* u = S::LANES > 1 ? u_ : v;
  constexpr bool kLinesOf64 = S::BX == 64;
  constexpr T kFar = T(18446744073709551616.0);                   // 2^64
  T scale[S::PER_LANE];
  bool small[S::PER_LANE];
#pragma unroll
  for (int p = 0; p < S::PER_LANE; ++p) {
    const int b = S::PER_LANE > 1 ? p * 64 + lane : lane % S::NB;
    const T n = load_float<T>(N, g.ntype, int64_t(k0) + (b < n_active ? b : n_active - 1));
    // Algorithm 3: N F / r, the division hoisted per block.  Where N / r is below the normal numbers it would lose digits that the
    // dense kernels, which divide N F, keep: lines of 64 were theirs, so N is scaled up and the products back down
    small[p] = kLinesOf64 && n < T(1) / kFar;
    scale[p] = (small[p] ? n * kFar : n) / T(g.r);
  }
#pragma unroll
  for (int i = 0; i < S::VALUES; ++i) u[i] = T(0);                // blocks past the end
  by_index_type(g.itype, [&](auto tag) {
    using IT = decltype(tag);
    if constexpr (sizeof(T) == 8 || sizeof(IT) == 1) {
      const int bytes = g.kept * int(sizeof(IT));
      const uint8_t* lo = static_cast<const uint8_t*>(F);
      const uint8_t* hi = lo + int64_t(g.n_blocks) * bytes;
      const uint32_t aside = g.region - 256 + uint32_t(lane) * 4u;
      for (int first = 0; first < n_active; first += g.per_round) {
        const int count = n_active - first < g.per_round ? n_active - first : g.per_round;
        const uint8_t* src = lo + (int64_t(k0) + first) * bytes;
        const int phase = phase_of(src);
        const bool runs = g.kept == S::VOL && (phase & 3) == 0;
        put_index<int32_t>(st, aside, 0u);
        stage_span<4>(lo, hi, src, count * bytes, st);
        wave_lds_sync();
        each_run<S>(lane, [&](int b, int entry, int value) {
          if (b >= first && b < first + count) {
            const int p = S::PER_LANE > 1 ? value / S::VOL : 0;
            const uint32_t base = uint32_t(phase + (b - first) * bytes);
            int f[S::BXB];
            if (runs) {
              get_run<IT, S::BXB>(st, base + uint32_t(entry) * uint32_t(sizeof(IT)), f);
            } else {
              uint32_t places[(S::BXB + 1) / 2];
              load_place_row<S::BXB>(g.places + entry, places);
#pragma unroll
              for (int e = 0; e < S::BXB; ++e) f[e] = get_index<IT>(st, place_address<IT>(places, e, base, aside));
            }
#pragma unroll
            for (int e = 0; e < S::BXB; ++e) {
              u[value + e] = scale[p] * T(f[e]);
              if (kLinesOf64) u[value + e] *= small[p] ? T(1) / kFar : T(1);
            }
          }
        });
        wave_lds_sync();
      }
    }
  });
  if constexpr (S::LANES > 1) {
    outer_transforms<TF, T, S, false>(u);
    Exchange<T, S>::template run<false>(st, lane, v, u);
  }
#pragma unroll
  for (int p = 0; p < S::PER_LANE; ++p) inner_transforms<TF, T, S, false>(v + p * S::VOL);
  by_array_type(g.xtype, [&](auto tag) {
    using XT = decltype(tag);
#pragma unroll
    for (int p = 0; p < S::PER_LANE; ++p) {
      const int b = S::PER_LANE > 1 ? p * 64 + lane : lane % S::NB;
      int64_t block_origin;
      const Place at = place_of<S>(g, k0 + (b < n_active ? b : n_active - 1), S::LANES > 1 ? lane / S::NB * S::RA : 0, &block_origin);
      if (g.whole == 2) store_rows<2, T, XT, S>(g, st, lane, static_cast<XT*>(y), at, b < n_active, v + p * S::VOL);
      else if (g.whole) store_rows<1, T, XT, S>(g, st, lane, static_cast<XT*>(y), at, b < n_active, v + p * S::VOL);
      else store_rows<0, T, XT, S>(g, st, lane, static_cast<XT*>(y), at, b < n_active, v + p * S::VOL);
    }
  });
}

// ---- host side -----------------------------------------------------------------------------------------------------
// fills the geometry; false when the array does not fold into it
bool make_brick(const pbz_codec* c, const Geom& geo, const void* array, int xtype, const DeviceTables* t, int bw, int bz, int by,
                int bx, BrickGeom* g) {
  const int nd = c->ndim;
  const int want[4] = {bw, bz, by, bx};
  int64_t ext[4] = {1, 1, 1, 1}, lead = 1;
  for (int d = 0; d < nd; ++d) {
    const int slot = 4 - (nd - d);
    if (slot < 0) {
      if (c->block[d] != 1) return false;
      lead *= geo.shape[d];
    } else {
      if (c->block[d] != want[slot]) return false;
      ext[slot] = geo.shape[d];
    }
  }
  for (int slot = 0; slot < 4 - nd; ++slot)
    if (want[slot] != 1) return false;
  if (geo.n_blocks >= (int64_t(1) << 31) || (reinterpret_cast<uintptr_t>(array) & 15u) != 0) return false;
  int64_t grid[4];
  bool whole = true;
  int last[4];
  for (int i = 0; i < 4; ++i) {
    grid[i] = (ext[i] + want[i] - 1) / want[i];
    last[i] = int(ext[i] - (grid[i] - 1) * want[i]);
    whole = whole && last[i] == want[i];
  }
  const int piece = bx * ftype_bytes(xtype) < 16 ? bx : 16 / ftype_bytes(xtype);
  if (ext[3] < piece) return false;                        // a row holds a piece's elements at least
  g->n_blocks = uint32_t(geo.n_blocks);
  g->gw = make_divisor(grid[0]);
  g->gz = make_divisor(grid[1]);
  g->gy = make_divisor(grid[2]);
  g->gx = make_divisor(grid[3]);
  g->sy = ext[3];
  g->sz = g->sy * ext[2];
  g->sw = g->sz * ext[1];
  g->sb = g->sw * ext[0];
  g->lw = last[0];
  g->lz = last[1];
  g->ly = last[2];
  g->lx = last[3];
  const bool lines = ext[3] * ftype_bytes(xtype) % 128 == 0 && (reinterpret_cast<uintptr_t>(array) & 127u) == 0;
  g->whole = whole ? (lines ? 2 : 1) : 0;
  g->xtype = xtype;
  g->ntype = int(c->ftype);
  g->itype = int(c->itype);
  g->kept = c->kept;
  g->r = c->r;
  g->places = t ? t->places : nullptr;
  return true;
}

constexpr int kSpanBytes = 8192;                 // of F in LDS at a time, unless one block is larger

template <typename T, typename S, bool kStore>
dim3 brick_launch(BrickGeom* g, int* threads, size_t* lds) {
  const int bytes = g->kept * itype_bytes(g->itype);
  int per = S::NB;
  while (per > 1 && per * bytes > kSpanBytes) per /= 2;
  g->per_round = per;
  const int span = (15 + per * bytes + 15) / 16 * 16 + 256;
  int region = span > Exchange<T, S>::BYTES ? span : Exchange<T, S>::BYTES;
  const int pieces = S::BX * ftype_bytes(g->xtype) / 16;
  if (kStore && pieces > 1) {
    const int rows = 1024 * pieces > kStoreBytes ? 1024 * pieces : kStoreBytes;
    if (region < rows) region = rows;
  }
  g->region = uint32_t(region);
  int waves = 4;
  while (waves > 1 && waves * region > 64 * 1024) waves /= 2;
  *threads = 64 * waves;
  *lds = size_t(region) * waves;
  const int64_t tiles = (int64_t(g->n_blocks) + S::NB - 1) / S::NB;
  return dim3(unsigned((tiles + waves - 1) / waves));
}

template <int TF, typename T, typename S>
void compress_with(BrickGeom g, const void* x, void* N, void* F, hipStream_t s) {
  int threads;
  size_t lds;
  const dim3 grid = brick_launch<T, S, false>(&g, &threads, &lds);
  const int64_t bytes = int64_t(threads / 64) * S::NB * g.kept * 4;      // of F that a workgroup writes, where indices are of 32 bits
  g.run = 1;
  if (g.itype == PBZ_I32 && g.kept == S::VOL && int64_t(g.n_blocks) * g.kept * 4 <= int64_t(1) << 25)      // (beyond, a reduction's workgroups take more)
    while (g.run * bytes < 32 * 1024) g.run *= 2;
  hipLaunchKernelGGL((k_compress_brick<TF, T, S>), grid, dim3(threads), lds, s, g, x, N, F);
}
template <int TF, typename T, typename S>
void decompress_with(BrickGeom g, const void* N, const void* F, void* y, hipStream_t s) {
  int threads;
  size_t lds;
  const dim3 grid = brick_launch<T, S, true>(&g, &threads, &lds);
  hipLaunchKernelGGL((k_decompress_brick<TF, T, S>), grid, dim3(threads), lds, s, g, N, F, y);
}

// Whether blocks of the shape are taken here for the codec's arithmetic.  Lines of 64 in FP64 are not: the dense kernels' direct
// sums are the more accurate there (decompressed values, rms relative to theirs: 4.6e-15 with the split transform; in FP32
// work it is the other way round, 1.6e-7 dense and 9.6e-8 split)
template <typename T, int BX>
constexpr bool kTaken = BX < 64 || sizeof(T) == 4;

// When these kernels take a call, against the tiled ones: a wave does a tile in one long straight run of code, so that one alone
// takes longer than a workgroup with its phases, while many overlap.  First what holds for 64 values a lane (32 in FP64 work), that is beyond few_to
// and for the shapes without smaller tiles.  Decompress, whose rows pass LDS once more, up to some 2^21 elements: 1.05-1.6 of the tiled kernels' time
// (FP64 work with blocks of 256 and more and 16-bit or 32-bit indices: 9 -> 15 us; FP32 work with rows of 8 to 32: 7 -> 9), 0.75-0.95 from 2^22 on, rows of 16 and more in FP32 work and int32 in small flat blocks from
// 2^23; not so rows of 4, 4-D blocks in FP32 work, int8 in FP64 work and small blocks there (0.6-1.03 at any size; FP64 arrays in rows
// of 4: 1.0-1.09).  Under a mask the tiled kernels look every entry up: 8x8, and 16x16 in FP64 work, 0.7-1.0.  Compress: 0.4-1.05 but for
// FP64 arrays in rows of 16 and more in FP32 work (1.1-1.2), 32x32 blocks of FP32 (1.05), and FP64 work that leaves a lane 64
// values, with int32 or FP64 arrays and nothing pruned (1.1-1.6), from 2^14 to 2^20 elements.  32-bit indices of flat blocks with
// nothing pruned stay with the tiled kernels where measured slower at every size above a few blocks: 8x8 both ways (1.05-1.3), 4x8 and
// 8x4 of FP64 arrays decompressing (1.05-1.15); and so do 32x32 blocks of FP64 arrays in FP32 work under a mask, decompressing
// (1.2).
// Rows that are no whole blocks, or no whole 16-byte pieces, the tiled kernels take element by element.  Decompressing, these
// kernels then win at every size: in FP32 work blocks of up to 64 (0.6-0.9; 16-bit arrays 8x8 0.8), 3-D blocks of 16-bit arrays (0.75-0.9) and,
// under a mask, of FP32 arrays (0.9); in FP64 work flat blocks of up to 128 in rows of less than 32 (0.65-0.9; FP64 arrays under a mask only, all of
// them 1.15), 16x16 of 16-bit arrays with nothing pruned (0.9); and the others, too, from 2^22 on.  Compressing, 8x8 of 16-bit arrays with
// 32-bit indices (0.88) and 32x32 of FP32 arrays (0.9).
// Up to few_to elements the smaller tiles win against the tiled kernels throughout (0.57-0.97), but, decompressing under a mask,
//   whole rows of 32x32 blocks of FP32 and 16-bit arrays in FP32 work and of 4x8x8 blocks of 16-bit arrays (1.04-1.09);
//   rows of whole 16-byte pieces, a quarter kept at most, of 4x8x8 blocks of FP32 and FP64 arrays (1.05-1.23 up to 2^20 elements, 0.83-1.0 with a
//   half kept) and of 32x32 blocks, in FP32 work (1.08-1.27) or with the Haar transform (1.1-1.35; and FP64 arrays, FP32 work, with a half: 1.14),
//   of 16-bit and FP32 arrays up to 2^20;
// and 32-bit indices with nothing pruned: lines of 32 decompressing rows of whole pieces (1.0-1.1 up to 2^20, the Haar transform 1.2-1.4 up to 2^22) and
// both ways between 2 and 3 Mi elements (1.0-1.25; 0.75-0.9 on both sides), 4x8x8 of 16-bit arrays.  What follows is for the larger calls and the shapes that hold 64 values at any size.
template <typename T, typename S>
bool pays(const pbz_codec* c, bool compress, int xtype, int64_t elements, int64_t row, const Tiles& t) {
  constexpr int64_t kMi = int64_t(1) << 20;
  constexpr bool kWide = sizeof(T) == 8, kFlat = S::BW == 1 && S::BZ == 1;
  constexpr bool k8x8 = kFlat && S::BY == 8 && S::BX == 8, k4x8 = kFlat && S::VOL == 32 && S::BX < 16;
  const int array = ftype_bytes(xtype), index = itype_bytes(c->itype);
  const bool pruned = c->kept != c->vol, ragged = row % S::BX != 0 || row * array % 16 != 0;
  if (c->route == kRouteShape || S::BX == 64) return true;
  const bool haar = c->transform == PBZ_TRANSFORM_HAAR, in_pieces = row * array % 16 == 0, quarter = 4 * c->kept <= c->vol;
  const bool looked_up = !compress && pruned && t.few == 32 &&
                         ((!ragged && (S::VOL == 1024 ? !kWide && array < 8 : S::VOL == 256 && array == 2)) ||
                          (in_pieces && S::VOL == 256 && array > 2 && quarter && elements <= kMi) ||
                          (in_pieces && S::VOL == 1024 && (array == 8 || elements <= kMi) && (kWide ? haar && quarter : quarter || (haar && array == 8))));
  if (S::ROWS == 1 && S::BX == 32 && kWide && index == 4 && !pruned && elements > 2 * kMi && elements < 3 * kMi) return false;
  const bool rows_of_32 = !compress && kWide && index == 4 && !pruned && in_pieces &&
                          ((S::ROWS == 1 && S::BX == 32 && elements <= (haar ? 4 * kMi : kMi)) ||
                           (!ragged && t.few == 32 && S::VOL == 256 && array == 2 && elements <= kMi / 2));
  const bool large = !compress && !kWide && S::VOL == 1024 && array == 8 && pruned && elements > 4 * kMi;
  if (elements <= t.few_to && !looked_up && !rows_of_32 && !large) return true;
  if (index == 4 && !pruned && ((k8x8 && !(compress && ragged && array == 2)) || (k4x8 && !compress && array == 8))) return false;
  if (compress) {
    const bool enough = elements <= 4096 || elements >= 3 * kMi;
    if (kWide) return pruned || !(t.many == 64 && (index == 4 || array == 8)) || enough;
    return !((array == 8 && S::BX >= 16) || (array == 4 && S::VOL == 1024 && !ragged)) || enough;
  }
  if (!kWide && S::VOL == 1024 && array == 8 && pruned) return false;
  if (S::BX == 4 && (kWide || array < 8 || S::BW > 1 || pruned)) return true;
  if (!kWide && S::BW > 1) return true;
  if (kWide && ((index == 1 && S::VOL < 1024) || (!kFlat && S::VOL <= 128) || (index == 2 && S::VOL <= 32 && S::BX <= 8))) return true;
  if (pruned && (k8x8 || (kWide && kFlat && S::BY == 16 && S::BX == 16))) return true;
  if (ragged && !kWide && array < 8 && (S::VOL <= 64 || (!kFlat && S::VOL <= 512 && (array == 2 || (pruned && S::VOL <= 256))))) return true;
  if (ragged && kWide && kFlat && S::VOL <= 128 && S::BX < 32 && (array < 8 || pruned)) return true;
  if (ragged && kWide && kFlat && S::VOL == 256 && array == 2 && !pruned) return true;
  const bool late = (!kWide && S::BX >= 16 && !pruned) || (index == 4 && kFlat && S::VOL < 256);
  return elements >= (late && !ragged ? 8 * kMi : 3 * kMi);
}

// The shape with the values per lane that the call gets
template <typename T, bool kCompress, int BW, int BZ, int BY, int BX, typename F>
int with_shape(const pbz_codec* c, int xtype, const BrickGeom& g, int64_t row, bool dry_run, F f) {
  constexpr bool kWide = sizeof(T) == 8;
  const Tiles t = tiles(kWide, kCompress, ftype_bytes(xtype), itype_bytes(c->itype), c->kept != c->vol, BW, BZ, BY, BX);
  const int64_t elements = int64_t(g.n_blocks) * BW * BZ * BY * BX;
  if (!pays<T, Shape<T, BW, BZ, BY, BX, 64>>(c, kCompress, xtype, elements, row, t)) return 0;
  if (dry_run) return 1;
  const int v = elements <= t.few_to ? t.few : t.many;
  if constexpr (needed(8, kWide, kCompress, BW, BZ, BY, BX)) if (v == 8) f(Shape<T, BW, BZ, BY, BX, 8>());
  if constexpr (needed(16, kWide, kCompress, BW, BZ, BY, BX)) if (v == 16) f(Shape<T, BW, BZ, BY, BX, 16>());
  if constexpr (needed(32, kWide, kCompress, BW, BZ, BY, BX)) if (v == 32) f(Shape<T, BW, BZ, BY, BX, 32>());
  if constexpr (needed(64, kWide, kCompress, BW, BZ, BY, BX)) if (v == 64) f(Shape<T, BW, BZ, BY, BX, 64>());
  return hipGetLastError() == hipSuccess ? 1 : PBZ_ERR_HIP;
}

template <typename T, int BW, int BZ, int BY, int BX>
int compress_shape(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* x, int xtype, void* N, void* F,
                   hipStream_t s, bool dry_run) {
  if constexpr (kTaken<T, BX>) {
    BrickGeom g;
    if (!make_brick(c, geo, x, xtype, t, BW, BZ, BY, BX, &g)) return 0;
    return with_shape<T, true, BW, BZ, BY, BX>(c, xtype, g, geo.shape[c->ndim - 1], dry_run, [&](auto tag) {
      using S = decltype(tag);
      if (c->transform == PBZ_TRANSFORM_HAAR) compress_with<kTfHaar, T, S>(g, x, N, F, s);
      else compress_with<kTfDct, T, S>(g, x, N, F, s);
    });
  }
  return 0;
}
template <typename T, int BW, int BZ, int BY, int BX>
int decompress_shape(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* N, const void* F, void* y,
                     int ytype, hipStream_t s, bool dry_run) {
  if constexpr (kTaken<T, BX>) {
    BrickGeom g;
    if (!make_brick(c, geo, y, ytype, t, BW, BZ, BY, BX, &g)) return 0;
    return with_shape<T, false, BW, BZ, BY, BX>(c, ytype, g, geo.shape[c->ndim - 1], dry_run, [&](auto tag) {
      using S = decltype(tag);
      if (c->transform == PBZ_TRANSFORM_HAAR) decompress_with<kTfHaar, T, S>(g, N, F, y, s);
      else decompress_with<kTfDct, T, S>(g, N, F, y, s);
    });
  }
  return 0;
}

// Defines the two entry points of a part from its list of shapes X(BW, BZ, BY, BX)
#define PBZ_DEFINE_BRICK_PART(PART, SHAPES)                                                                             \
  int PART##_compress(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* x, int xtype, void* N,    \
                      void* F, hipStream_t s, bool dry_run) {                                                           \
    int r = 0;                                                                                                          \
    SHAPES(PBZ_BRICK_COMPRESS_ROW)                                                                                      \
    return r;                                                                                                           \
  }                                                                                                                     \
  int PART##_decompress(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* N, const void* F,       \
                        void* y, int ytype, hipStream_t s, bool dry_run) {                                              \
    int r = 0;                                                                                                          \
    SHAPES(PBZ_BRICK_DECOMPRESS_ROW)                                                                                    \
    return r;                                                                                                           \
  }
#define PBZ_BRICK_COMPRESS_ROW(W, Z, Y, XX)                                                                             \
  if (r == 0)                                                                                                           \
    r = c->compute_f64 ? compress_shape<double, W, Z, Y, XX>(c, geo, t, x, xtype, N, F, s, dry_run)                              \
                       : compress_shape<float, W, Z, Y, XX>(c, geo, t, x, xtype, N, F, s, dry_run);
#define PBZ_BRICK_DECOMPRESS_ROW(W, Z, Y, XX)                                                                           \
  if (r == 0)                                                                                                           \
    r = c->compute_f64 ? decompress_shape<double, W, Z, Y, XX>(c, geo, t, N, F, y, ytype, s, dry_run)                            \
                       : decompress_shape<float, W, Z, Y, XX>(c, geo, t, N, F, y, ytype, s, dry_run);

}  // namespace

// the parts: a translation unit each
#define PBZ_BRICK_PARTS(X) X(lines) X(small) X(flat) X(wide) X(planes) X(cubes) X(tesseracts) X(long_tesseracts)
#define PBZ_BRICK_DECLARE(PART)                                                                                         \
  int PART##_compress(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* x, int xtype, void* N,    \
                      void* F, hipStream_t s, bool dry_run);                                                            \
  int PART##_decompress(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* N, const void* F,       \
                        void* y, int ytype, hipStream_t s, bool dry_run);
PBZ_BRICK_PARTS(PBZ_BRICK_DECLARE)
#undef PBZ_BRICK_DECLARE

}  // namespace brick
}  // namespace pbz
