// Specialised codec kernels for the block shapes that matter for throughput.
//
// Every kernel here is "wave autonomous": a 64-lane wave owns a run of consecutive blocks along the
// contiguous (last) array dimension, reads whole block rows straight from HBM with 16-byte loads (the
// lanes of a wave cover a contiguous span of every row, which measures at the same bandwidth as a
// linear copy on MI355X), transforms in registers with the even/odd-split DCT of pbz_dct.h or the Haar
// cascade of pbz_haar.h (template switch TF), and writes N and F.  There is no workgroup barrier in the
// compress kernels and LDS, where used, is private to a wave (one exception: the first exchange of "cube16").
//
// Family "lane":   one lane owns one whole block (blocks of at most 64 elements: 8x8, 4x4x4).  Where a block
//                   row is two (four) 16-byte pieces the half-waves (quarter-waves) trade pieces, so that every
//                   load / store instruction of the array covers one contiguous KiB.  Indices leave through a wave-private
//                   LDS transpose when a block's F is 64 bytes or more, for the same reason.
// Family "quad16":  16x16 and 4x16x16 blocks of FP32, 16-bit or FP64 input (int8 in FP32 arithmetic; in FP64 arithmetic FP32 input
//                   with int16 / int32 and FP64 input with int8 to int32), 16 planes of 16x16 per wave.  Each lane first holds a 16-row x
//                   4-column strip (the column transform runs in registers), the wave exchanges through LDS,
//                   then each lane holds four whole rows (row transform, and for 4x16x16 the transform across
//                   the four planes); rows leave as 16-byte pieces in linear order.
// Family "oct8":    8x8x8 blocks of bfloat16, FP16, FP32 or FP64 input (int8 in FP32 arithmetic; in FP64 arithmetic FP32 input
//                   with int16 / int32 and FP64 input with int8 to int32), 8 blocks per wave.  Each lane first holds one z-plane of
//                   a block (x and y transforms), the wave exchanges through LDS, then each lane holds one
//                   y-row of all eight z-planes (z transform).  Decompression needs no exchange: every
//                   lane rebuilds its own z-plane from the block's few kept coefficients; wide arrays use a
//                   variant in which a wave owns one plane of 64 blocks and stores whole 1 KiB row pieces.
// Family "cube16":  16x16x16 blocks of FP32 input (int16 / int32 indices in FP64 arithmetic, int8 in FP32) or FP64 input (int8 in
//                   FP32 arithmetic, int8 to int32 in FP64), two neighbouring blocks
//                   per workgroup of two waves.  Three layouts, one per transformed dimension, with an LDS exchange
//                   between them; the first is how rows are read (eight lanes cover the 128 bytes the two blocks have
//                   in a row), the last how F is written (whole rows of indices).
//
// Variants of every kernel: kRagged (the slower dimensions are not multiples of the block extents), kTailX
// (neither is the last one: rows start at any 4-byte boundary, the last block of a row is partial), kStats
// (compress also leaves the per-wave sums from which mean, variance and norm follow).  N is stored in the
// codec's working type, converted on load / store.
//
// kMasked variants take any pruning mask (and any alignment of F); they serve the settings that differ from a family's
// only in the mask, without statistics, and count as general kernels: pbz_kernel_name says "generic".
//
// Preconditions checked on the host (otherwise the call falls back to the general kernels): the array
// reduces to at most three dimensions (leading dimensions with block extent 1 fold into the slowest one),
// the block shape / types / mask box match an instantiation, rows are at least one 16-byte piece long and
// start on a 4-byte boundary.
// Where the kernels per block shape (pbz_brick.h) are faster they take such calls all the same: shape_kernels_pay() and small_to() below.
// The families live in pbz_fast_lane.hip, pbz_fast_quad16.hip, pbz_fast_oct8.hip and pbz_fast_cube16.hip; this file folds the array
// and asks each family in turn.
#include "pbz_fast_common.h"

namespace pbz {

// When the kernels per block shape (pbz_brick.h) take a call that a family has kernels for.  A family deals out the blocks of a row, 64 (lane), 16
// (quad16) or 8 (oct8) to a wave: where rows have fewer, lanes idle, and a wave does as much for one block as for all; and where rows are no
// whole blocks its lane and FP64 kernels take what is beyond the whole pieces element by element.  The kernels per block shape go by block
// number and shift whole pieces into place.  The family keeps the call while its waves are too few to fill the chip, its own one wave being the
// faster (1.1-1.4), and where a wave is full enough.  Measured for 2^16 to 2^25.5 elements in rows of 1 to 256 blocks, whole and not, family ->
// here: FP32 / i8 in 8x8, 2^24 elements in rows of 2, 8 and 24 blocks, compress 0.13, 0.43, 0.86 of the time, decompress 0.14, 0.44, 0.83;
// FP64 / i16 in 4x4x4 0.16, 0.55, 1.09; in rows that are no whole blocks, of 128 blocks, FP64 / i16 8x8 0.70 and 0.86, FP64 / i8 0.61 and 0.6, FP32 / i16
// 16x16 0.83.  Each constant below is the share of a wave (`fill`) and the number of waves up to which, and from which, calls of that family,
// direction, raggedness, array, index and transform were the faster ones here; nothing else is behind them.  57,670 calls by turns, of the 23,000 that
// come here: lane compress 0.24-0.27 of the family's time, decompress 0.38-0.45, quad16 0.37 and 0.6-0.68, oct8 0.45 and 0.5-0.73 (means); over 1.05 in
// 0.6 % (whole rows of 16x16 decompressing 5.6 %), worst 1.15.  Calls under a mask have MaskedCall's rules.
// The statistics of a compressed array, which a family's kernel leaves along the way, have to be those of the same {N, F}: such calls take this
// route too and read {N, F} once more.  Compressing, the line is therefore where both win: 0.05-0.95 of the time for the statistics inside it, 1.1-1.5
// in the calls outside where compression alone would win (0.75-0.95: small arrays, and rows a third full and more).  Decompressing, for
// calls that are not small() below.
static bool shape_kernels_pay(const pbz_codec* c, const fast::Folded& f, int xtype, bool compress) {
  const fast::FastGeom& g = f.g;
  const bool flat = f.bz == 1, lane = (flat && f.by == 8 && f.bx == 8) || (f.bz == 4 && f.by == 4 && f.bx == 4);
  const bool quad = flat && f.by == 16 && f.bx == 16, oct = f.bz == 8 && f.by == 8 && f.bx == 8;
  if (!lane && !quad && !oct) return false;
  const int per_wave = lane ? 64 : (quad ? 16 : 8);
  const int64_t tiles = (g.gx + per_wave - 1) / per_wave, waves = g.gz * g.gy * tiles;
  const int64_t blocks = g.gz * g.gy * g.gx;
  if (blocks * f.bz * f.by * f.bx < int64_t(1) << 16) return false;      // a few us whichever way
  const double fill = double(g.gx) / double(tiles * per_wave);
  const int array = ftype_bytes(xtype), index = itype_bytes(c->itype);
  const bool ragged = f.tail_x, wide = c->compute_f64, haar = c->transform == PBZ_TRANSFORM_HAAR;
  const auto from = [&](int64_t least_waves, double most_fill) { return waves >= least_waves && fill <= most_fill; };
  constexpr double kAny = 1.0;
  if (lane && compress) {
    if (!ragged) return from(2000, array == 8 ? (flat ? 0.44 : 0.25) : (index == 4 ? 0.15 : 0.2));
    if (!flat) return array == 8 ? g.gx <= (index == 1 ? 48 : (index == 2 ? 20 : 12)) || from(2000, index == 4 ? 0.9 : kAny) : from(1300, 0.32);
    if (array == 8) return g.gx <= 40 || from(2000, kAny) || blocks <= 24 * 1024;
    return index == 1 ? g.gx <= 8 || from(2000, 0.8) : g.gx <= 4 || from(2000, 0.35);
  }
  if (lane && !flat) {
    if (fill <= 0.15) return true;
    if (!ragged) return from(2500, array == 8 && !wide ? 0.35 : (index == 4 ? 0.15 : 0.2));
    return from(2000, index == 2 ? 0.4 : (array == 8 ? 0.3 : 0.25));
  }
  if (lane) {
    if (!ragged) return from(2500, index == 4 || (haar && array < 8) ? 0.15 : (index == 2 && array == 4 ? 0.25 : (array == 8 ? 0.5 : 0.35)));
    if (array == 2) return from(0, 0.6);
    if (array == 8) return from(700, kAny);
    return index == 1 ? from(2800, kAny) : from(2000, haar ? 0.22 : 0.4);
  }
  if (quad && compress) {
    if (!ragged) return from(2000, array == 8 && !wide ? 0.4 : 0.5);
    return from(500, 0.5) || from(4500, array == 8 || index == 4 ? 0.75 : 0.9);
  }
  if (quad) {
    if (array == 8 && wide) return from(2000, index == 4 ? 0.5 : (ragged ? (index == 2 ? 0.8 : 0.65) : 0.95));
    return haar && !ragged ? from(2000, 0.3) : from(0, ragged ? 0.5 : 0.4);
  }
  if (compress) {
    if (ragged && array == 8) return wide || from(2000, kAny);
    return from(4000, 0.25) || (ragged && from(8000, 0.5));
  }
  if (ragged && array == 8) return blocks >= (index == 4 ? 9 * 1024 : 6 * 1024);
  if (ragged) return array == 4 && from(2800, index == 1 ? 0.95 : (index == 4 ? 0.25 : 0.4));
  return from(2800, haar ? 0.15 : (index == 4 ? 0.25 : 0.4));
}

// Up to how many elements the kernels per block shape are the faster ones for any row width, with their smaller tiles: a family's wave holds
// 16 to 32 KiB of the array, so that up to 2^20 elements it is one wave's time that counts, which is the longer the more it holds.  Measured
// for ten types, two aspects, whole rows and not, 2^16 to 2^22.5 elements; here / family, decompressing, full masks:
//             2^17   2^19   2^20   2^21   2^21.5  2^22
//   8x8       0.70   0.80   0.84   1.00   1.18    1.23   rows of no whole blocks 0.60 ... 0.82, 0.95
//   4x4x4     0.87   0.94   0.96   1.03   1.08    1.14   rows of no whole blocks 0.60 ... 0.83, 0.92; FP32 / i8 0.99 at 2^18
//   16x16     0.89   0.93   0.92   0.90   0.97    1.01   rows of no whole blocks 0.70 ... 0.78, 0.90; FP64 arrays 0.88 at 2^22
// and under a mask 0.6-0.8 compressing (1.0 at 2^21.5, 2^22 and 2^22.5), 0.7-0.95 decompressing.  Compressing without one it would be 0.75-0.9 up to
// 2^20, but 1.2-1.4 for the statistics.  With the Haar transform, whose waves are shorter, whole rows of 16x16 decompress in 1.05-1.2 here, of
// 4x4x4 and 8x8 / i8 in 1.0-1.1: they stay.  8x8x8 blocks keep 64 values a lane here (1.1-1.6): not these.
static int64_t small_to(const pbz_codec* c, const fast::Folded& f, int xtype, bool compress) {
  constexpr int64_t kKi = 1024, kMi = kKi * kKi;
  const bool flat = f.bz == 1, masked = c->kept != c->vol, ragged = f.tail_x, wide = c->compute_f64;
  const int array = ftype_bytes(xtype), index = itype_bytes(c->itype);
  const bool haar = c->transform == PBZ_TRANSFORM_HAAR;
  if (compress && !masked) return 0;
  if (flat && f.by == 8 && f.bx == 8) {
    if (ragged || masked) return 2 * kMi;
    if (index == 1 && array < 8) return haar ? 0 : kMi;
    return 3 * kMi / 2;
  }
  if (f.bz == 4 && f.by == 4 && f.bx == 4) {
    if (compress) return 4 * kMi;
    if (ragged) return 2 * kMi;
    if (array < 8 && (haar || !wide)) return haar ? 0 : 256 * kKi;
    return kMi;
  }
  if (flat && f.by == 16 && f.bx == 16) {
    if (compress) return 4 * kMi;
    if (ragged) return 3 * kMi;
    return haar ? 0 : (array == 8 ? 4 * kMi : (wide ? 2 * kMi : kMi));
  }
  return 0;
}
static bool small(const pbz_codec* c, const fast::Folded& f, int xtype, bool compress) {
  return f.g.gz * f.g.gy * f.g.gx * (f.bz * f.by * f.bx) <= small_to(c, f, xtype, compress);
}
// Up to here a family keeps the calls it fits exactly, not for its time: with the smaller tiles such a call takes 0.45-0.9 of it (8x8 0.46 to 0.85 of 4 to
// 10 us, 4x4x4 0.5-0.89, 16x16 0.65-0.91; but 16x16 decompressing with the Haar transform 1.1 and 8x8x8 1.2-1.55).  At these sizes the families' kernels are
// compared with the oracle element by element, by the names that pbz_kernel_name gives, and through no other route would those meet them.
constexpr int64_t kTiny = int64_t(1) << 17;

static bool shape_first(const pbz_codec* c, const fast::Folded& f, int xtype, bool compress) {
  if (!f.ok) return false;
  const bool enough = f.g.gz * f.g.gy * f.g.gx * (f.bz * f.by * f.bx) > kTiny;
  return (enough && small(c, f, xtype, compress)) || shape_kernels_pay(c, f, xtype, compress);
}

int try_compress_shape_first(const pbz_codec* c, const Geom& geo, const void* x, int xtype, void* N, void* F, hipStream_t s, bool dry_run) {
  if (c->kept != c->vol || c->route != kRouteAuto || !fast::aligned16(x) || !fast::aligned16(F)) return 0;
  // no tables: with everything kept and F aligned an entry is its own place
  return shape_first(c, fast::fold(c, geo), xtype, true) ? try_compress_brick(c, geo, nullptr, x, xtype, N, F, s, dry_run) : 0;
}
int try_decompress_shape_first(const pbz_codec* c, const Geom& geo, const void* N, const void* F, void* y, int ytype, hipStream_t s, bool dry_run) {
  if (c->kept != c->vol || c->route != kRouteAuto || !fast::aligned16(y) || !fast::aligned16(F)) return 0;
  return shape_first(c, fast::fold(c, geo), ytype, false) ? try_decompress_brick(c, geo, nullptr, N, F, y, ytype, s, dry_run) : 0;
}

int try_compress_fast(const pbz_codec* c, const Geom& geo, const void* x, int xtype, void* N, void* F, hipStream_t s,
                      bool dry_run, const char** name, double* tile_sums) {
  if (!fast::aligned16(x) || !fast::aligned16(F)) return 0;
  const fast::Folded f = fast::fold(c, geo);
  if (!f.ok) return 0;
  *name = nullptr;
  int r = fast::lane_compress(c, f, xtype, x, N, F, s, dry_run, name, tile_sums);
  if (!*name) r = fast::quad16_compress(c, f, xtype, x, N, F, s, dry_run, name, tile_sums);
  if (!*name) r = fast::oct8_compress(c, f, xtype, x, N, F, s, dry_run, name, tile_sums);
  if (!*name) r = fast::cube16_compress(c, f, xtype, x, N, F, s, dry_run, name, tile_sums);
  return r;
}

int64_t fast_compress_tiles(const pbz_codec* c, const Geom& geo, int xtype) {
  const fast::Folded f = fast::fold(c, geo);
  if (!f.ok) return 0;
  int64_t t = fast::lane_tiles(c, f, xtype);
  if (t < 0) t = fast::quad16_tiles(c, f, xtype);
  if (t < 0) t = fast::oct8_tiles(c, f, xtype);
  if (t < 0) t = fast::cube16_tiles(c, f, xtype);
  return t < 0 ? 0 : t;
}

int try_decompress_fast(const pbz_codec* c, const Geom& geo, const void* N, const void* F, void* y, int ytype,
                        hipStream_t s, bool dry_run, const char** name) {
  if (!fast::aligned16(y) || !fast::aligned16(F)) return 0;
  const fast::Folded f = fast::fold(c, geo);
  if (!f.ok) return 0;
  *name = nullptr;
  int r = fast::lane_decompress(c, f, ytype, N, F, y, s, dry_run, name);
  if (!*name) r = fast::quad16_decompress(c, f, ytype, N, F, y, s, dry_run, name);
  if (!*name) r = fast::oct8_decompress(c, f, ytype, N, F, y, s, dry_run, name);
  if (!*name) r = fast::cube16_decompress(c, f, ytype, N, F, y, s, dry_run, name);
  return r;
}

// The kernels of the same families that take any mask, in the order above.  They are asked after the kernels for one
// mask (everything, or a box), which skip work that these cannot, and before the kernels for any block shape; each
// family's pays() says where it is the faster one (the figures are there and with MaskArgs), above what is small()
int try_compress_masked(const pbz_codec* c, const Geom& geo, const uint16_t* pos, const void* x, int xtype, void* N, void* F,
                        hipStream_t s, bool dry_run) {
  if (c->kept == c->vol || !fast::aligned16(x) || c->route == kRouteShape) return 0;
  const fast::Folded f = fast::fold(c, geo);
  if (!f.ok) return 0;
  if (c->route == kRouteAuto && small(c, f, xtype, true) && try_compress_brick(c, geo, nullptr, x, xtype, N, F, s, true) == 1) return 0;
  int r = fast::lane_compress_masked(c, f, xtype, pos, x, N, F, s, dry_run);
  if (r == 0) r = fast::quad16_compress_masked(c, f, xtype, pos, x, N, F, s, dry_run);
  if (r == 0) r = fast::oct8_compress_masked(c, f, xtype, pos, x, N, F, s, dry_run);
  if (r == 0) r = fast::cube16_compress_masked(c, f, xtype, pos, x, N, F, s, dry_run);
  return r;
}

int try_decompress_masked(const pbz_codec* c, const Geom& geo, const uint16_t* pos, const void* N, const void* F, void* y,
                          int ytype, hipStream_t s, bool dry_run) {
  if (c->kept == c->vol || !fast::aligned16(y) || c->route == kRouteShape) return 0;
  const fast::Folded f = fast::fold(c, geo);
  if (!f.ok) return 0;
  if (c->route == kRouteAuto && small(c, f, ytype, false) && try_decompress_brick(c, geo, nullptr, N, F, y, ytype, s, true) == 1) return 0;
  int r = fast::lane_decompress_masked(c, f, ytype, pos, N, F, y, s, dry_run);
  if (r == 0) r = fast::quad16_decompress_masked(c, f, ytype, pos, N, F, y, s, dry_run);
  if (r == 0) r = fast::oct8_decompress_masked(c, f, ytype, pos, N, F, y, s, dry_run);
  if (r == 0) r = fast::cube16_decompress_masked(c, f, ytype, pos, N, F, y, s, dry_run);
  return r;
}

}  // namespace pbz
