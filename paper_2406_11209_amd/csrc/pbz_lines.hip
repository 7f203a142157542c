// Codec kernels for blocks that are lines of 64 elements in FP64 work (block extents 1 x ... x 1 x 64): signals, and rows of an image taken by
// themselves.  Lines are the one shape whose transform is a plain contraction, [blocks x 64] with the 64 x 64 matrix H, so it goes to the matrix cores:
// v_mfma_f64_16x16x4, a wave per 16 blocks, 64 of them for 1024 elements.
//
// What bounds them: the matrix instructions (64 cycles each: 7 us for 4 Mi elements, 33 for 20 Mi) and HBM in turn.  4 Mi FP64 elements, int8: compress
// 173 -> 19 us, decompress 512 -> 26; 16 Mi 65 and 82; 16384 elements 36 -> 9 (the dense kernels of pbz_generic.hip, which took these calls, loop
// over LDS element by element).  A fast transform would need a third of the operations, but its error is larger than the dense
// sums'.  These have the error they had, 1.4e-16 of N: with the elements in another order, one share of sixteen after the other, it was
// 2.4e-16, and no less in two, four or eight partial sums.
// A step of the sums takes elements 4 s .. 4 s + 3 of a block, one by each quarter of the wave.  A lane loads sixteen consecutive elements, 16
// bytes at a time, and the quarters then trade them in registers: the sums are in the order of the elements, as they were.  The
// matrix stands in LDS so that a step's numbers use all banks.  F leaves and comes through LDS spans like the other kernels', at any kept
// count and alignment.
#include "pbz_fast_common.h"
#include "pbz_span.h"

namespace pbz {
namespace {

using fast::Binner;
using fast::bf16_t;
using fast::f16_t;

constexpr int kLine = 64, kTileBlocks = 16, kMaxWaves = 8;
typedef double f64x4 __attribute__((ext_vector_type(4)));

struct Lines {
  int64_t X, gx, n_blocks, tiles;      // elements and blocks of a row; of all rows together
  double r;
  int kept, ntype, itype, index_bytes;
  int span;                            // bytes of LDS for a tile's F at any phase
};

// where block k starts, and how many elements its row has from there on
struct LinePlace { int64_t at, left; };
__device__ __forceinline__ LinePlace place_of(const Lines& g, int64_t k) {
  const int64_t row = g.gx == g.n_blocks ? 0 : k / g.gx;                 // one row: a uniform branch instead of a division
  const int64_t bx = k - row * g.gx;
  return {row * g.X + bx * kLine, g.X - bx * kLine};
}

__device__ __forceinline__ double widened(double v) { return v; }
__device__ __forceinline__ double widened(float v) { return double(v); }
__device__ __forceinline__ double widened(bf16_t v) { return double(bf16_bits_to_float(v.bits)); }
__device__ __forceinline__ double widened(f16_t v) { return double(float(__builtin_bit_cast(_Float16, v))); }

// sixteen consecutive elements, of which the first `inside` are the array's and the others zero
template <typename XT>
__device__ __forceinline__ void load_share(const XT* p, int64_t inside, double* a) {
  if (inside >= 16) {
    XT v[16];
#pragma unroll
    for (int k = 0; k < int(sizeof(v)) / 16; ++k) {                      // at the element's alignment
      raw16 piece;
      __builtin_memcpy(&piece, reinterpret_cast<const uint8_t*>(p) + 16 * k, 16);
      __builtin_memcpy(reinterpret_cast<uint8_t*>(v) + 16 * k, &piece, 16);
    }
#pragma unroll
    for (int s = 0; s < 16; ++s) a[s] = widened(v[s]);
  } else {
#pragma unroll
    for (int s = 0; s < 16; ++s) a[s] = s < inside ? widened(p[s]) : 0.0;
  }
}

// Where H[m][q] stands in the table.  A step of the forward transform reads sixteen q of four m, one of the inverse four q of sixteen m: both are
// spread over all banks.
template <bool kForward>
__device__ __forceinline__ int table_slot(int m, int q) {
  if (kForward) return m * kLine + (q ^ ((m & 1) << 4));
  return m * kLine + (((q >> 2) ^ (m & 15)) << 2 | (q & 3));
}
template <bool kForward>
__device__ __forceinline__ void fill_table(double* table, const double* __restrict__ H) {
  for (int e = threadIdx.x; e < kLine * kLine; e += blockDim.x) table[table_slot<kForward>(e >> 6, e & 63)] = H[e];
}

// acc[t]: columns 16 t .. of the product of the lanes' numbers (4 s + lane / 16 of block lane % 16) with H or its transpose
template <bool kForward>
__device__ __forceinline__ void multiply(const double* a, const double* table, int lane, f64x4* acc) {
  const int row = lane >> 4, column = lane & 15;
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 4 * s + row, j = 16 * t + column;
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], table[kForward ? table_slot<true>(k, j) : table_slot<false>(j, k)], acc[t], 0, 0, 0);
    }
}

// The lanes' shares (16 g + e of the block, g = lane / 16) become their numbers (4 s + g): the four quarters of the wave trade them
__device__ __forceinline__ void shares_to_numbers(double* a) {
  double out[16];
#pragma unroll
  for (int c = 0; c < 4; c += 2) {
    uint4 p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint64_t u = __builtin_bit_cast(uint64_t, a[4 * c + e]), v = __builtin_bit_cast(uint64_t, a[4 * c + 4 + e]);
      p[e] = make_uint4(uint32_t(u), uint32_t(u >> 32), uint32_t(v), uint32_t(v >> 32));
    }
    fast::transpose_quarter_waves(p[0], p[1], p[2], p[3]);       // p[k] now: what quarter k had in p[g]
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      out[4 * k + c] = __builtin_bit_cast(double, uint64_t(p[k].x) | (uint64_t(p[k].y) << 32));
      out[4 * k + c + 1] = __builtin_bit_cast(double, uint64_t(p[k].z) | (uint64_t(p[k].w) << 32));
    }
  }
#pragma unroll
  for (int s = 0; s < 16; ++s) a[s] = out[s];
}

__device__ __forceinline__ void put(uint8_t* at, int bytes, int64_t v) {
  if (bytes == 1) *at = uint8_t(v);
  else if (bytes == 2) *reinterpret_cast<uint16_t*>(at) = uint16_t(v);
  else *reinterpret_cast<uint32_t*>(at) = uint32_t(v);
}

__global__ __launch_bounds__(64 * kMaxWaves) void k_compress_lines(Lines g, const void* __restrict__ x, int xtype,
                                                                void* __restrict__ N, uint8_t* __restrict__ F,
                                                                const double* __restrict__ H,
                                                                const uint16_t* __restrict__ places) {
  __shared__ double table[kLine * kLine];
  extern __shared__ __align__(16) uint8_t spans[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, share = lane >> 4;
  const int waves = blockDim.x >> 6;
  uint8_t* span = spans + wave * g.span;
  fill_table<true>(table, H);
  int place[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) place[t] = places[16 * t + i] == kPruned ? -1 : int(places[16 * t + i]) * g.index_bytes;
  __syncthreads();
  const int bytes = g.kept * g.index_bytes;
  for (int64_t tile = int64_t(blockIdx.x) * waves + wave; tile < g.tiles; tile += int64_t(gridDim.x) * waves) {
    const int64_t first = tile * kTileBlocks;
    const int count = g.n_blocks - first < kTileBlocks ? int(g.n_blocks - first) : kTileBlocks;
    double a[16];
    {
      const LinePlace p = place_of(g, first + (i < count ? i : count - 1));
      const int64_t inside = i < count ? p.left - 16 * share : 0;
      const int64_t at = p.at + (inside > 0 ? 16 * share : 0);
      switch (xtype) {
        case PBZ_F64: load_share(static_cast<const double*>(x) + at, inside, a); break;
        case PBZ_F32: load_share(static_cast<const float*>(x) + at, inside, a); break;
        case PBZ_BF16: load_share(static_cast<const bf16_t*>(x) + at, inside, a); break;
        default: load_share(static_cast<const f16_t*>(x) + at, inside, a); break;
      }
    }
    shares_to_numbers(a);
    f64x4 c[4];
    multiply<true>(a, table, lane, c);
    // the lane has column 16 t + i of blocks 4 v + share
    const int phase = phase_of(F + first * bytes);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int b = 4 * v + share;
      double m = 0.0;
#pragma unroll
      for (int t = 0; t < 4; ++t) m = fmax(m, fabs(c[t][v]));
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) m = fmax(m, __shfl_xor(m, off, 64));
      if (b >= count) continue;
      if (i == 0) store_float(N, g.ntype, first + b, m);
      const Binner<double> bin(m, g.r);
      uint8_t* at = span + phase + b * bytes;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        // an infinite maximum: what the quotients C r / N are then, limited, gives -r (of NaN)
        const uint32_t q = m < INFINITY ? bin.bits(c[t][v]) : uint32_t(-int64_t(g.r));
        if (place[t] >= 0) put(at + place[t], g.index_bytes, q);
      }
    }
    wave_lds_sync();
    unstage_span(span, F + first * bytes, count * bytes);
    wave_lds_sync();
  }
}

__global__ __launch_bounds__(64 * kMaxWaves) void k_decompress_lines(Lines g, const void* __restrict__ N,
                                                                  const uint8_t* __restrict__ F, void* __restrict__ y, int ytype,
                                                                  const double* __restrict__ H,
                                                                  const uint16_t* __restrict__ places) {
  __shared__ double table[kLine * kLine];
  extern __shared__ __align__(16) uint8_t spans[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, share = lane >> 4;
  const int waves = blockDim.x >> 6;
  uint8_t* span = spans + wave * g.span;
  fill_table<false>(table, H);
  uint32_t place[16];                                                    // of the lane's sixteen entries
#pragma unroll
  for (int k = 0; k < 16; ++k) place[k] = places[4 * k + share];
  __syncthreads();
  const int bytes = g.kept * g.index_bytes;
  const uint8_t* end = F + g.n_blocks * bytes;
  for (int64_t tile = int64_t(blockIdx.x) * waves + wave; tile < g.tiles; tile += int64_t(gridDim.x) * waves) {
    const int64_t first = tile * kTileBlocks;
    const int count = g.n_blocks - first < kTileBlocks ? int(g.n_blocks - first) : kTileBlocks;
    const int mine = i < count ? i : count - 1;                          // lanes past the end redo the last block and store nothing
    const double n = load_float<double>(N, g.ntype, first + mine);
    stage_span<2>(F, end, F + first * bytes, count * bytes, span);
    wave_lds_sync();
    const uint8_t* from = span + phase_of(F + first * bytes) + mine * bytes;
    double a[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      a[s] = place[s] == kPruned ? 0.0 : (n * double(load_index(from, g.itype, place[s]))) / g.r;        // (N F) / r, as it is written
    }
    wave_lds_sync();
    f64x4 c[4];
    multiply<false>(a, table, lane, c);
    const LinePlace own = place_of(g, first + mine);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int b = 4 * v + share;
      const int64_t at = __shfl((long long)own.at, b, 64), left = __shfl((long long)own.left, b, 64);
      if (b >= count) continue;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (16 * t + i < left) store_float(y, ytype, at + 16 * t + i, c[t][v]);
    }
  }
}

// Compressing, eight waves share a table where there are tiles for two workgroups on every compute unit: four waves a SIMD hide each
// other's loads and quotients behind the matrix instructions (16 Mi FP32 elements, int16: 72 -> 61 us).  With fewer tiles four, which spreads
// them over more units, and decompressing, which has its quotients before and its stores after (82 us, 85 with eight).
int lines_waves(const Lines& g, bool compress) { return compress && g.tiles >= 2 * 256 * kMaxWaves ? kMaxWaves : 4; }
dim3 lines_grid(const Lines& g, int waves) {
  const int64_t groups = (g.tiles + waves - 1) / waves, most = waves == kMaxWaves ? 512 : 768;      // what LDS lets stand at once
  const int64_t turns = (groups + most - 1) / most;
  return dim3(unsigned((groups + turns - 1) / turns));
}

Lines lines_of(const pbz_codec* c, const Geom& geo) {
  Lines g;
  g.X = geo.shape[geo.ndim - 1];
  g.gx = geo.grid[geo.ndim - 1];
  g.n_blocks = geo.n_blocks;
  g.tiles = (g.n_blocks + kTileBlocks - 1) / kTileBlocks;
  g.r = c->r;
  g.kept = c->kept;
  g.ntype = int(c->ftype);
  g.itype = int(c->itype);
  g.index_bytes = itype_bytes(c->itype);
  g.span = (16 + kTileBlocks * g.kept * g.index_bytes + 16 + 15) / 16 * 16;
  return g;
}

}  // namespace

bool line_kernels_cover(const pbz_codec* c) {
  for (int d = 0; d + 1 < c->ndim; ++d)
    if (c->block[d] != 1) return false;
  return c->compute_f64 && c->block[c->ndim - 1] == kLine;
}

int launch_compress_lines(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* x, int xtype, void* N, void* F,
                          hipStream_t s) {
  const Lines g = lines_of(c, geo);
  const int waves = lines_waves(g, true);
  hipLaunchKernelGGL(k_compress_lines, lines_grid(g, waves), dim3(64 * waves), size_t(waves) * g.span, s, g, x, xtype, N, static_cast<uint8_t*>(F),
                     t->H + c->h_offset[c->ndim - 1], t->places);
  return hip_status(hipGetLastError());
}

int launch_decompress_lines(const pbz_codec* c, const Geom& geo, const DeviceTables* t, const void* N, const void* F, void* y,
                            int ytype, hipStream_t s) {
  const Lines g = lines_of(c, geo);
  const int waves = lines_waves(g, false);
  hipLaunchKernelGGL(k_decompress_lines, lines_grid(g, waves), dim3(64 * waves), size_t(waves) * g.span, s, g, N, static_cast<const uint8_t*>(F), y, ytype,
                     t->H + c->h_offset[c->ndim - 1], t->places);
  return hip_status(hipGetLastError());
}

}  // namespace pbz
