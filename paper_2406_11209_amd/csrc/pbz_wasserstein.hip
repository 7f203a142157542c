// Approximate Wasserstein distance of two compressed arrays (Sec. IV-A, "Approximate Wasserstein distance",
// Algorithm 13): block-wise means -> softmax unless they already sum to one -> sort -> p-th power mean of the
// differences of the two sorted sequences.
//
// Everything stays on the device and on the caller's stream:
//   1. block means of both operands into the workspace, as unsigned keys in the order of the doubles, with their
//      sums, maxima and sums of exp(x - max) per tile, and how many of a tile's keys fall between which splitters,
//   2. the parameters of the softmax and the decision whether to apply it,
//   3. which of the keys can matter for the distance at all (k_select); the raw means of these are sorted (softmax is
//      increasing, so it commutes with sorting), both operands in the same launches (grid y): a sample sort up to
//      kSampleSortMax keys, a least-significant-digit radix sort of all keys beyond.  Up to kRangeMax keys, where the
//      launches are the time, all are sorted by as few kernels as can do it (launch_few),
//   4. m = max |P_A - P_B| and sum (|P_A - P_B| / m)^p, then m (sum / n)^(1/p): the scaling by m changes
//      nothing in exact arithmetic and keeps orders such as p = 68 .. 80 from underflowing.
// All sums are two-stage with a fixed order, so the result is reproducible run to run.
#include <cmath>
#include <type_traits>

#include "pbz_device.h"
#include "pbz_internal.h"

namespace pbz {
namespace {

constexpr int kThreads = 256;
constexpr int kRadixBits = 8;
constexpr int kBins = 1 << kRadixBits;
constexpr int kSortThreads = 256;                // threads of a sorting workgroup: four waves, one thread per digit
constexpr int kKeysPerLane = 16;
constexpr int kWaveKeys = 64 * kKeysPerLane;     // keys one wave ranks
constexpr int kTileKeys = kSortThreads * kKeysPerLane;   // keys of a tile (one workgroup)
// workgroups per operand in the small reductions, at most
constexpr int kStatGroups = 1024;
constexpr int kMeansPerThread = 8;               // blocks whose N and first index a thread requests together
constexpr int kDistancesInFlight = 2;
constexpr int kKeptDifferences = 12;             // of a thread of k_distance, in LDS until the maximum is known; a multiple of those
constexpr int kKeysInFlight = 8;                 // keys a thread of the passes below requests together

// Sample sort: 2 K to 16 K keys drawn from the n (4096 at most; one from each run of equally many, at a place that depends on the run's number) and
// sorted give K - 1 splitters; one pass counts and one pass scatters the keys into the 2 K - 1 buckets (between two
// splitters, or equal to one: a value that many blocks share fills a bucket that needs no sorting); a workgroup sorts a
// bucket in LDS.  What bounds it: 8-byte scatters and LDS, 16 bytes a key and pass against memory otherwise.
// K = n / 2048 rounded up to a power of two, so that a bucket has some 1024 to 2048 keys: smaller ones would make the
// runs that a tile scatters into a bucket shorter than the 64 bytes they are, larger ones would not fit LDS beside
// three more.  2 x 2M keys, the whole distance: 491 us with eight radix passes, 290 with all buckets sorted, 190 with those that matter
// (of that the means, a line of F each, and the counting 105; samples and splitters 13, k_select 16, scattering 14, sorting 20).
constexpr int kSampleSortMax = 1 << 22;          // 2048 buckets: fewer than two samples each would leave them too uneven
constexpr int kBucketKeys = 2048;                // on average, at most
constexpr int kBucketCap = 4096;                 // keys sorted in LDS at once: larger buckets take more than one round
constexpr int kMaxSamples = 4096;
constexpr int kMaxTiles = 256;                   // tiles per operand of the counting and scattering passes
constexpr int kMinTileKeys = 2048;
constexpr int kSelectMin = 128;                  // buckets from which k_select pays ...
constexpr double kSelectGain = 640.0;            // ... where the gap of the maxima, in shares of the larger, times their square is above this
// Few keys (launch_few): ranges of kRangeKeys on average, found by workgroups that each go through all keys, from kMaxSamples keys on; below, a
// key's rank is counted, and up to kBucketThreads one workgroup does an operand.  What it saves are launches, of 4.5 us in line: nine, or six
// where there was one bucket, are two, three and five.  Whole distance in a captured graph, us, nine or six launches -> now: 256 blocks 22.4 -> 10.1, 1024 25.8 ->
// 13.2, 4096 45 -> 23, 16384 52 -> 26, 65536 of a crowded image 92 -> 38.  At 110 thousand the walk through all keys (48 us) costs more than
// scattering them: 62 -> 70.  Calls through the Python binding one after another take as long (1024 blocks 25.7 -> 13.3, 16384 43.7 -> 25.8, of
// which the host is busy 20 -> 9.8 and 27 -> 17.4), one that is waited for 12 to 15 more.  Ranges of 1024 keys, in two to a thread: 16384 keys 31, 65536 43.
constexpr int kRangeMax = 65536;
constexpr int kRangeKeys = 512;
constexpr int kSampleRun = 32;                   // one sample of as many keys: 8 to 16 a range, so that hardly one has twice the average
static_assert(kRangeMax <= kMaxSamples * kSampleRun, "a sample of each run");
constexpr int kPieceRanks = 512;                 // ranks of a piece of k_distance, at most
constexpr int kPassThreads = 512;
constexpr int kGoingInFlight = 4;
constexpr int kGoing = kPassThreads * kGoingInFlight + 512;      // of the scattering pass: a step's keys and some before them
constexpr double kSumTolerance = 1e-9;           // "the means sum to one" is taken as |sum - 1| <= this

// per operand: written by the one-workgroup kernels, read by everything after them
struct OperandParams {
  double sum, max, exp_sum, use_softmax;
};

// per operand, from k_select: keys from .. to (from > to: none) are in no bucket that matters
struct Gap {
  uint64_t from, to;
};
// for k_distance, from k_select
struct Selection {
  double threshold;        // differences below it do not matter
  int pieces;              // of ranks that may; -1: all do
};

struct Workspace {
  OperandParams* params;   // [2]
  double* partials;        // [2][kStatGroups][2]
  uint64_t* buf0;          // [2][n]: keys; the sorted keys end up here
  uint64_t* buf1;          // [2][n]: keys by bucket, later the differences
  uint32_t* hist;          // sample sort: [2][tiles][2 K]; radix sort: [2][kBins][n_tiles]
  uint32_t* sums;          // [2][2 K] / [2][kBins]: the buckets' / digits' totals
  uint64_t* splitters;     // [2][K]
  uint32_t* rest;          // [2 + 2 K]: the numbers of left-over buckets and of pieces, then the buckets
  uint2* pieces;           // [K]: pieces of buckets of one value (first key of both operands' 2 n, number of keys)
  Gap* gap;                // [2], and the selection
  uint8_t* needed;         // [2][2 K]: the bucket has keys whose order matters
  uint2* ranks;            // pieces of the ranks at which differences matter (first rank, number)
};

struct SortPlan {
  bool sample;             // else radix
  int buckets;             // K
  int tiles;               // of the counting and scattering passes
  int64_t tile_keys;
};

SortPlan sort_plan(int64_t n) {
  SortPlan p;
  p.sample = n <= kSampleSortMax;
  p.buckets = 1;
  if (p.sample && n > kBucketCap)
    while (int64_t(p.buckets) * kBucketKeys < n) p.buckets *= 2;
  int64_t tiles = (n + kMinTileKeys - 1) / kMinTileKeys;
  if (tiles > kMaxTiles) tiles = kMaxTiles;
  p.tile_keys = (n + tiles - 1) / tiles;
  p.tiles = int((n + p.tile_keys - 1) / p.tile_keys);
  return p;
}

size_t align_up(size_t v) { return (v + 255) & ~size_t(255); }

size_t carve(void* base, int64_t n, Workspace* w) {
  // Never less than for fewer blocks, so that a workspace for the largest array serves all: beyond the sample sort's
  // sizes its largest needs count, and tiles count before they are evened out.
  const int64_t sampled = n < kSampleSortMax ? n : kSampleSortMax;
  const size_t buckets = size_t(sort_plan(sampled).buckets);
  const int64_t tiles = (sampled + kMinTileKeys - 1) / kMinTileKeys;
  const size_t sample_counts = size_t(tiles < kMaxTiles ? tiles : kMaxTiles) * 2 * buckets;
  const size_t radix_counts = n > kSampleSortMax ? size_t(kBins) * size_t((n + kTileKeys - 1) / kTileKeys) : 0;
  const size_t counts = sample_counts > radix_counts ? sample_counts : radix_counts;
  const size_t totals = 2 * buckets;
  size_t off = 0;
  char* p = static_cast<char*>(base);
  auto take = [&](size_t bytes) {
    char* q = p ? p + off : nullptr;
    off += align_up(bytes);
    return q;
  };
  char* a = take(sizeof(OperandParams) * 2);
  char* b = take(sizeof(double) * 2 * kStatGroups * 2);
  char* d = take(sizeof(uint64_t) * 2 * size_t(n));
  char* e = take(sizeof(uint64_t) * 2 * size_t(n));
  char* f = take(sizeof(uint32_t) * 2 * counts);
  char* g = take(sizeof(uint32_t) * 2 * totals);
  char* h = take(sizeof(uint64_t) * 2 * buckets);
  char* i = take(sizeof(uint32_t) * (2 + 2 * buckets));
  char* j = take(sizeof(uint2) * buckets);
  char* k = take(sizeof(Gap) * 2 + sizeof(Selection));
  char* l = take(2 * totals);
  char* m = take(sizeof(uint2) * (2 * totals + size_t(sampled) / kPieceRanks + 1));
  if (w) {
    w->params = reinterpret_cast<OperandParams*>(a);
    w->partials = reinterpret_cast<double*>(b);
    w->buf0 = reinterpret_cast<uint64_t*>(d);
    w->buf1 = reinterpret_cast<uint64_t*>(e);
    w->hist = reinterpret_cast<uint32_t*>(f);
    w->sums = reinterpret_cast<uint32_t*>(g);
    w->splitters = reinterpret_cast<uint64_t*>(h);
    w->rest = reinterpret_cast<uint32_t*>(i);
    w->pieces = reinterpret_cast<uint2*>(j);
    w->gap = reinterpret_cast<Gap*>(k);
    w->needed = reinterpret_cast<uint8_t*>(l);
    w->ranks = reinterpret_cast<uint2*>(m);
  }
  return off;
}

// doubles <-> unsigned keys with the same order (negative values: all bits flipped; others: sign bit set).  NaN comes before
// -infinity or after infinity, by its sign; the one whose key would be the largest number, which k_splitters needs free, takes the
// key before it.
__device__ __forceinline__ uint64_t key_of(double v) {
  const uint64_t u = uint64_t(__double_as_longlong(v));
  const uint64_t k = (u >> 63) ? ~u : (u | (uint64_t(1) << 63));
  return k - (k == ~uint64_t(0) ? 1u : 0u);
}
__device__ __forceinline__ double value_of(uint64_t k) {
  const uint64_t u = (k >> 63) ? (k & ~(uint64_t(1) << 63)) : ~k;
  return __longlong_as_double((long long)u);
}

// the largest over the 64 lanes of a wave, all of them active, in every lane; register moves, as wave_sum
template <int kControl, int kRows>
__device__ __forceinline__ double lane_shifted_or_own(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = int(uint32_t(u)), hi = int(uint32_t(u >> 32));
  const uint32_t l = uint32_t(__builtin_amdgcn_update_dpp(lo, lo, kControl, kRows, 0xf, false));
  const uint32_t h = uint32_t(__builtin_amdgcn_update_dpp(hi, hi, kControl, kRows, 0xf, false));
  return __builtin_bit_cast(double, uint64_t(l) | (uint64_t(h) << 32));
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, lane_shifted_or_own<0x111, 0xf>(v));
  v = fmax(v, lane_shifted_or_own<0x112, 0xf>(v));
  v = fmax(v, lane_shifted_or_own<0x114, 0xf>(v));
  v = fmax(v, lane_shifted_or_own<0x118, 0xf>(v));
  v = fmax(v, lane_shifted_or_own<0x142, 0xa>(v));
  v = fmax(v, lane_shifted_or_own<0x143, 0xc>(v));
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), 63));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u >> 32)), 63));
  return __builtin_bit_cast(double, uint64_t(lo) | (uint64_t(hi) << 32));
}

// workgroup totals of two values (sum, max) in thread 0; at most 1024 threads
__device__ __forceinline__ void group_sum_max(double& s, double& m) {
  __shared__ double ls[16], lm[16];
  s = wave_sum(s);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) {
    ls[threadIdx.x >> 6] = s;
    lm[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s = ls[0];
    m = lm[0];
    for (int w = 1; w < int(blockDim.x >> 6); ++w) {
      s += ls[w];
      m = fmax(m, lm[w]);
    }
  }
}

// Block mean N_k F_k0 * scale of both operands (grid y) as doubles: calls f(load) with a function that gives N and the first index of
// block i.  The types are uniform: one branch outside the loops.
template <typename Fn>
__device__ __forceinline__ void with_loads(const void* N, const void* F, int ntype, int itype, int kept, Fn f) {
  auto by_index = [&](auto load_n) {
    if (itype == PBZ_I8) f(load_n, [&](int64_t i) { return double(__builtin_nontemporal_load(static_cast<const int8_t*>(F) + i * kept)); });
    else if (itype == PBZ_I16) f(load_n, [&](int64_t i) { return double(__builtin_nontemporal_load(static_cast<const int16_t*>(F) + i * kept)); });
    else f(load_n, [&](int64_t i) { return double(__builtin_nontemporal_load(static_cast<const int32_t*>(F) + i * kept)); });
  };
  if (ntype == PBZ_F64) by_index([&](int64_t i) { return static_cast<const double*>(N)[i]; });
  else if (ntype == PBZ_F32) by_index([&](int64_t i) { return double(static_cast<const float*>(N)[i]); });
  else if (ntype == PBZ_BF16) by_index([&](int64_t i) { return double(bf16_bits_to_float(static_cast<const uint16_t*>(N)[i])); });
  else by_index([&](int64_t i) { return double(float(static_cast<const _Float16*>(N)[i])); });
}

// One workgroup of an operand: the tiles' {sum, maximum, sum of exp(x - the tile's maximum)} -> parameters.
__device__ __forceinline__ void mean_params(const double* partials, int tiles, OperandParams* params) {
  const double* in = partials + int64_t(blockIdx.y) * kMaxTiles * 4;
  __shared__ double top;
  double s = 0.0, m = -INFINITY;
  for (int g = threadIdx.x; g < tiles; g += blockDim.x) {
    s += in[4 * g];
    m = fmax(m, in[4 * g + 1]);
  }
  group_sum_max(s, m);
  if (threadIdx.x == 0) {
    OperandParams& p = params[blockIdx.y];
    p.sum = s;
    p.max = m;
    p.use_softmax = fabs(s - 1.0) > kSumTolerance ? 1.0 : 0.0;
    top = m;
  }
  __syncthreads();
  m = top;
  double e = 0.0, none = 0.0;
  for (int g = threadIdx.x; g < tiles; g += blockDim.x) e += in[4 * g + 2] * exp(in[4 * g + 1] - m);
  group_sum_max(e, none);
  if (threadIdx.x == 0) params[blockIdx.y].exp_sum = e;
}

// ---- sample sort -----------------------------------------------------------------------------------------------
// 32 bits that look arbitrary from a run's number: products with the golden ratio's, the square root of two's and of three's fractions, folded.  One
// product alone is a lattice over the keys, and with the rows of an image another: places then miss columns (524288 blocks in rows of 725, runs of 256 keys:
// buckets of up to 14137 keys, 4.6 times the expected most, and 111 us for the distance, 92 with half as many samples; simulated over
// 1500 images of any size and width, the largest bucket is at most 3.7 of the average now, 41 with one product).
__device__ __forceinline__ uint32_t scattered(uint32_t i) {
  i *= 2654435761u;
  i ^= i >> 15;
  i *= 1779033703u;
  i ^= i >> 13;
  i *= 3144134277u;
  return i ^ (i >> 16);
}
// sample i of 2^shift <= n (both below 2^23): from the i-th run of the keys, at a place that looks arbitrary
__device__ __forceinline__ int64_t sample_place(int i, int shift, int64_t n) {
  const int64_t lo = (n * i) >> shift, hi = (n * (i + 1)) >> shift;
  return lo + int64_t((uint64_t(scattered(uint32_t(i))) * uint64_t(hi - lo)) >> 32);
}

// the same for up to kRangeMax keys, of every kSampleRun one
__device__ __forceinline__ int64_t sample_of_run(int64_t run, int64_t n) {
  const int64_t lo = run * kSampleRun, length = n - lo < kSampleRun ? n - lo : kSampleRun;
  return lo + int64_t((uint64_t(scattered(uint32_t(run))) * uint64_t(length)) >> 32);
}

// Ascending order of p[0 .. m) by the whole workgroup: bitonic merges whose first step folds a run onto itself, so that every
// exchange is ascending and a count that is no power of two needs no padding.  int_t: wide enough for 4 m.
template <typename int_t>
__device__ __forceinline__ void fold_sort(uint64_t* p, int_t m) {
  for (int_t k = 2; k / 2 < m; k *= 2) {
    for (int_t j = k / 2; j > 0; j /= 2) {
      __syncthreads();
      for (int_t i = threadIdx.x; 2 * i < m + j; i += int_t(blockDim.x)) {
        const int_t lo = 2 * (i & ~(j - 1)) + (i & (j - 1));
        const int_t hi = j == k / 2 ? lo + k - 1 - 2 * (lo & (k - 1)) : lo + j;
        if (hi < m) {
          const uint64_t a = p[lo], b = p[hi];
          if (a > b) {
            p[lo] = b;
            p[hi] = a;
          }
        }
      }
    }
  }
  __syncthreads();
}

// The workgroups rank kRankThreads / kRankLanes samples each, by counting the smaller ones (and the equal ones before them), kRankLanes lanes
// per sample.  The samples are taken from N and F, once (by every ranking workgroup: 27 us for 2 x 2M blocks): the pass that makes all
// keys counts them by bucket already.  (One workgroup sorting the samples in its LDS: 50 us for 4096, at 0.65 us a step of fold_sort.)
// All of up to kMaxSamples keys are sorted like that, too: 4 us for 1024, 9 for 4096 (LDS reads and 64-bit compares, as n squared).
constexpr int kRankLanes = 16;
constexpr int kRankThreads = 512;
__global__ __launch_bounds__(64) void k_samples(const void* __restrict__ N1, const void* __restrict__ F1,
                                                const void* __restrict__ N2, const void* __restrict__ F2, int ntype, int itype,
                                                double scale, int kept, int64_t n, int sample_shift, uint64_t* __restrict__ samples) {
  const int i = int(blockIdx.x) * 64 + int(threadIdx.x);
  if (i >= 1 << sample_shift) return;
  const int64_t at = sample_place(i, sample_shift, n);
  with_loads(blockIdx.y ? N2 : N1, blockIdx.y ? F2 : F1, ntype, itype, kept, [&](auto load_n, auto load_f) {
    const double f = load_f(at), x = load_n(at);
    samples[int64_t(blockIdx.y) * kMaxSamples + i] = key_of(x * f * scale);
  });
}

// Of the workgroup's kRankThreads / kRankLanes keys, the thread's one and its rank among the first `samples` (kMaxSamples at most) of load(i),
// the same in its kRankLanes lanes.
template <typename Load>
__device__ __forceinline__ int rank_among(int samples, Load load, uint64_t* its_key) {
  __shared__ uint64_t sample[kMaxSamples];
  constexpr int kLoads = kMaxSamples / kRankThreads;
  const int mine = int(blockIdx.x) * (kRankThreads / kRankLanes) + int(threadIdx.x) / kRankLanes;
  uint64_t v[kLoads];
#pragma unroll
  for (int u = 0; u < kLoads; ++u) {
    const int i = u * kRankThreads + int(threadIdx.x);
    if (u * kRankThreads < samples) v[u] = load(i < samples ? i : samples - 1);
  }
#pragma unroll
  for (int u = 0; u < kLoads; ++u)
    if (u * kRankThreads < samples)                            // fewer than a step's: padded with what is below no key
      sample[u * kRankThreads + threadIdx.x] = u * kRankThreads + int(threadIdx.x) < samples ? v[u] : ~uint64_t(0);
  __syncthreads();
  const uint64_t key = sample[mine < samples ? mine : 0];
  int rank = 0;
  constexpr int kAhead = 8;                                // look-ups in flight
  static_assert(kMaxSamples % (kRankLanes * kAhead) == 0, "the steps stay inside the samples and what pads them");
  for (int j0 = threadIdx.x % kRankLanes; j0 < samples; j0 += kRankLanes * kAhead) {
    uint64_t other[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) other[u] = sample[j0 + u * kRankLanes];
    // all of these before `mine`: up to and with the equal ones; otherwise the smaller ones, and then equal ones before it
    const uint64_t bound = key + (j0 + (kAhead - 1) * kRankLanes < mine ? 1 : 0);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) rank += other[u] < bound ? 1 : 0;
    if (bound == key && j0 < mine) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) rank += other[u] == key && j0 + u * kRankLanes < mine ? 1 : 0;
    }
  }
#pragma unroll
  for (int off = 1; off < kRankLanes; off <<= 1) rank += __shfl_xor(rank, off, 64);
  *its_key = key;
  return mine < samples ? rank : -1;
}

// splitter b: the sample of rank (b + 1) samples / buckets - 1; at least as many samples as buckets
__global__ __launch_bounds__(kRankThreads) void k_splitters(const uint64_t* __restrict__ keys, int buckets,
                                                            uint64_t* __restrict__ splitters, int samples) {
  const uint64_t* in = keys + int64_t(blockIdx.y) * kMaxSamples;
  uint64_t key;
  const int rank = rank_among(samples, [&](int i) { return in[i]; }, &key);
  if (threadIdx.x % kRankLanes != 0 || rank < 0) return;
  const int b = int((int64_t(rank + 1) * buckets + samples - 1) / samples) - 1;
  if (b >= 0 && b < buckets - 1 && int(int64_t(b + 1) * samples / buckets) - 1 == rank) splitters[int64_t(blockIdx.y) * buckets + b] = key;
}

// All keys are samples, and a key's rank is its place.  The last workgroup along x makes the parameters.
__global__ __launch_bounds__(kRankThreads) void k_rank_sort(const uint64_t* __restrict__ keys, int n, uint64_t* __restrict__ sorted,
                                                            const double* __restrict__ partials, int tiles,
                                                            OperandParams* __restrict__ params) {
  if (blockIdx.x + 1 == gridDim.x) {
    mean_params(partials, tiles, params);
    return;
  }
  const uint64_t* in = keys + int64_t(blockIdx.y) * n;
  uint64_t key;
  const int rank = rank_among(n, [&](int i) { return in[i]; }, &key);
  if (threadIdx.x % kRankLanes == 0 && rank >= 0) sorted[int64_t(blockIdx.y) * n + rank] = key;
}

// buckets of kCount keys: 2 (number of splitters below it), and one more when it equals the next splitter.  The keys take
// the steps of the search together, so that their look-ups are in flight together.
template <int kCount>
__device__ __forceinline__ void buckets_of(const uint64_t* splitters, int buckets, const uint64_t* key, int* bucket) {
#pragma unroll
  for (int u = 0; u < kCount; ++u) bucket[u] = 0;
  for (int step = buckets >> 1; step > 0; step >>= 1)      // buckets - 1 splitters, a power of two less one
#pragma unroll
    for (int u = 0; u < kCount; ++u)
      if (splitters[bucket[u] + step - 1] < key[u]) bucket[u] += step;
#pragma unroll
  for (int u = 0; u < kCount; ++u)
    bucket[u] = 2 * bucket[u] + (bucket[u] < buckets - 1 && splitters[bucket[u]] == key[u] ? 1 : 0);
}

// consecutive workgroups go to the eight dies in turn: each die gets a run of tiles, whose pieces of a bucket are
// neighbours, so that its L2 completes their lines
__device__ __forceinline__ int tile_of_group() { return int(blockIdx.x & 7u) * int(gridDim.x >> 3) + int(blockIdx.x >> 3); }

// The means of a tile as keys, their sum, maximum and sum of exp (rescaled whenever a thread's maximum rises, once for
// kMeansPerThread of them), and with kCount the tile's keys of each bucket.  Where a block's indices fill a 128-byte line or more every
// line of F is fetched for two bytes of it (the L2 asks for whole lines, whatever the load's scope): that is the time, 82 us for 2 x 2M of
// them alone, and the search, the exponentials and the counting run behind it: 106 us, with a pass of its own for these 112 and 27.
// Non-temporal loads: a line is used once (a plain gather 80 us instead of 88).  The next step's loads ahead of this one's work: 112.
// kSample: the key at sample_of_run's place in each run of kSampleRun goes to `samples`, too.
template <bool kCount, int kThreadsOf = kPassThreads, int kPer = kMeansPerThread, bool kSample = false>
__global__ __launch_bounds__(kThreadsOf) void k_means(const void* __restrict__ N1, const void* __restrict__ F1,
                                                        const void* __restrict__ N2, const void* __restrict__ F2, int ntype,
                                                        int itype, double scale, int64_t n, int64_t tile_keys, int tiles, int kept,
                                                        int buckets, const uint64_t* __restrict__ splitters,
                                                        uint64_t* __restrict__ keys, uint32_t* __restrict__ hist,
                                                        uint32_t* __restrict__ rest, double* __restrict__ partials,
                                                        uint64_t* __restrict__ samples) {
  extern __shared__ __align__(16) uint64_t split[];         // [buckets], then the counts [2 buckets]
  uint32_t* count = reinterpret_cast<uint32_t*>(split + buckets);
  __shared__ double top;
  const int tile = tile_of_group();
  if (tile >= tiles) return;                                // uniform over the workgroup
  if (tile == 0 && blockIdx.y == 0 && threadIdx.x < 2) rest[threadIdx.x] = 0;
  if (kCount) {
    for (int i = threadIdx.x; i < buckets - 1; i += kThreadsOf) split[i] = splitters[int64_t(blockIdx.y) * buckets + i];
    for (int i = threadIdx.x; i < 2 * buckets; i += kThreadsOf) count[i] = 0;
    __syncthreads();
  }
  uint64_t* out = keys + int64_t(blockIdx.y) * n;
  const int64_t begin = int64_t(tile) * tile_keys;
  const int64_t end = begin + tile_keys < n ? begin + tile_keys : n;
  double s = 0.0, m = -INFINITY, e = 0.0;
  with_loads(blockIdx.y ? N2 : N1, blockIdx.y ? F2 : F1, ntype, itype, kept, [&](auto load_n, auto load_f) {
    for (int64_t i0 = begin + threadIdx.x; i0 < end; i0 += kThreadsOf * kPer) {
      double v[kPer], f[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int64_t i = i0 + u * kThreadsOf < end ? i0 + u * kThreadsOf : end - 1;
        f[u] = load_f(i);
        v[u] = load_n(i);
      }
      uint64_t key[kPer];
      double most = m;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int64_t i = i0 + u * kThreadsOf;
        v[u] = v[u] * f[u] * scale;
        key[u] = key_of(v[u]);
        if (i < end) {
          out[i] = key[u];
          if (kSample && i == sample_of_run(i / kSampleRun, n)) samples[int64_t(blockIdx.y) * kMaxSamples + i / kSampleRun] = key[u];
          s += v[u];
          most = fmax(most, v[u]);
        }
      }
      e *= most > m ? exp(m - most) : 1.0;
      m = most;
      const double base = fmax(m, -1.7976931348623157e308);      // minus infinity weighs nothing, also where the thread has met nothing else
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const double x = exp(v[u] - base);
        e += i0 + u * kThreadsOf < end ? x : 0.0;
      }
      if (kCount) {
        int b[kPer];
        buckets_of<kPer>(split, buckets, key, b);
#pragma unroll
        for (int u = 0; u < kPer; ++u)
          if (i0 + u * kThreadsOf < end) atomicAdd(&count[b[u]], 1u);
      }
    }
  });
  const double mine = m;
  group_sum_max(s, m);
  if (threadIdx.x == 0) top = m;
  __syncthreads();
  const double tile_max = top;
  double none = 0.0;
  e *= mine < tile_max ? exp(mine - tile_max) : 1.0;         // a thread without keys: nothing times exp(-infinity)
  group_sum_max(e, none);
  if (threadIdx.x == 0) {
    double* p = partials + (int64_t(blockIdx.y) * kMaxTiles + tile) * 4;
    p[0] = s;
    p[1] = tile_max;
    p[2] = e;
  }
  if (kCount) {
    uint32_t* h = hist + (int64_t(blockIdx.y) * tiles + tile) * 2 * buckets;
    for (int i = threadIdx.x; i < 2 * buckets; i += kThreadsOf) h[i] = count[i];   // (group_sum_max has the barrier)
  }
}

// The keys go to their buckets (hist holds the keys of the bucket in earlier tiles).  The order within a bucket does not matter, so
// places are handed out by LDS atomics.  Keys of a gap stay behind: nobody reads their places.
__global__ __launch_bounds__(kPassThreads) void k_scatter(const uint64_t* __restrict__ keys, uint64_t* __restrict__ out,
                                                          int64_t n, int64_t tile_keys, int tiles, int buckets,
                                                          const uint64_t* __restrict__ splitters,
                                                          const uint32_t* __restrict__ hist, const uint32_t* __restrict__ totals,
                                                          const Gap* __restrict__ gaps) {
  extern __shared__ __align__(16) uint64_t split[];         // [buckets], then the cursors [2 buckets]
  uint32_t* count = reinterpret_cast<uint32_t*>(split + buckets);
  const int tile = tile_of_group();
  if (tile >= tiles) return;                                // uniform over the workgroup
  const uint64_t* in = keys + int64_t(blockIdx.y) * n;
  const uint32_t* h = hist + (int64_t(blockIdx.y) * tiles + tile) * 2 * buckets;
  const Gap gap = gaps ? gaps[blockIdx.y] : Gap{1, 0};
  for (int i = threadIdx.x; i < buckets - 1; i += kPassThreads) split[i] = splitters[int64_t(blockIdx.y) * buckets + i];
  {
    // the buckets' first places: every thread adds up a run of totals, the runs are chained over the workgroup
    __shared__ uint32_t wave_total[kPassThreads / 64];
    const uint32_t* t = totals + int64_t(blockIdx.y) * 2 * buckets;
    const int run = (2 * buckets + kPassThreads - 1) / kPassThreads;
    const int first = int(threadIdx.x) * run;
    uint32_t sum = 0;
    for (int i = first; i < first + run && i < 2 * buckets; ++i) sum += t[i];
    uint32_t before = sum;                                  // inclusive over the wave, then exclusive
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(before, off, 64);
      if (int(threadIdx.x & 63) >= off) before += up;
    }
    if ((threadIdx.x & 63) == 63) wave_total[threadIdx.x >> 6] = before;
    __syncthreads();
    before -= sum;
    for (int w = 0; w < int(threadIdx.x >> 6); ++w) before += wave_total[w];
    for (int i = first; i < first + run && i < 2 * buckets; ++i) {
      count[i] = before + h[i];
      before += t[i];
    }
  }
  __syncthreads();
  const int64_t begin = int64_t(tile) * tile_keys;
  const int64_t end = begin + tile_keys < n ? begin + tile_keys : n;
  const auto send = [&](auto count_t, const uint64_t* key, const bool* goes) {
    constexpr int kCount = decltype(count_t)::value;
    int b[kCount];
    uint32_t place[kCount];
    buckets_of<kCount>(split, buckets, key, b);
#pragma unroll
    for (int u = 0; u < kCount; ++u)
      if (goes[u]) place[u] = atomicAdd(&count[b[u]], 1u);
#pragma unroll
    for (int u = 0; u < kCount; ++u)
      if (goes[u]) out[int64_t(blockIdx.y) * n + place[u]] = key[u];
  };
  if (gap.from > gap.to) {
    for (int64_t i0 = begin + threadIdx.x; i0 < end; i0 += kPassThreads * kKeysInFlight) {
      uint64_t key[kKeysInFlight];
      bool goes[kKeysInFlight];
#pragma unroll
      for (int u = 0; u < kKeysInFlight; ++u) {
        const int64_t i = i0 + u * kPassThreads;
        goes[u] = i < end;
        key[u] = in[goes[u] ? i : end - 1];
      }
      send(std::integral_constant<int, kKeysInFlight>(), key, goes);
    }
    return;
  }
  // the few keys beside the gap are collected, and then looked up together
  __shared__ uint64_t going[kGoing];
  __shared__ uint32_t n_going;
  if (threadIdx.x == 0) n_going = 0;
  __syncthreads();
  const auto send_going = [&]() {
    for (uint32_t i0 = threadIdx.x; i0 < n_going; i0 += kPassThreads) {
      const uint64_t key = going[i0];
      const bool goes = true;
      send(std::integral_constant<int, 1>(), &key, &goes);
    }
    __syncthreads();
    if (threadIdx.x == 0) n_going = 0;
    __syncthreads();
  };
  for (int64_t j0 = begin; j0 < end; j0 += kPassThreads * kGoingInFlight) {
    uint64_t key[kGoingInFlight];
#pragma unroll
    for (int u = 0; u < kGoingInFlight; ++u) {
      const int64_t i = j0 + threadIdx.x + u * kPassThreads;
      key[u] = in[i < end ? i : end - 1];
    }
    __syncthreads();
    if (n_going > uint32_t(kGoing - kPassThreads * kGoingInFlight)) send_going();      // uniform: nobody adds between the barriers
    else __syncthreads();
#pragma unroll
    for (int u = 0; u < kGoingInFlight; ++u)
      if (j0 + threadIdx.x + u * kPassThreads < end && (key[u] < gap.from || key[u] > gap.to)) going[atomicAdd(&n_going, 1u)] = key[u];
  }
  __syncthreads();
  send_going();
}

// hist [tile][bucket] -> keys of the bucket in earlier tiles, in place, and the buckets' totals.  A workgroup takes 64
// buckets, wave w the w-th run of tiles; the last workgroup along x makes the parameters.
constexpr int kScanWaves = 16;
__global__ __launch_bounds__(64 * kScanWaves) void k_bucket_scan(uint32_t* __restrict__ hist, int tiles, int bins,
                                                                 uint32_t* __restrict__ totals,
                                                                 const double* __restrict__ partials,
                                                                 OperandParams* __restrict__ params) {
  if (blockIdx.x + 1 == gridDim.x) {
    mean_params(partials, tiles, params);
    return;
  }
  __shared__ uint32_t part[kScanWaves][64];
  constexpr int kRun = kMaxTiles / kScanWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = int(blockIdx.x) * 64 + lane;
  uint32_t* column = hist + int64_t(blockIdx.y) * tiles * bins + (b < bins ? b : bins - 1);
  uint32_t v[kRun];
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < kRun; ++j) {
    const int t = wave * kRun + j;
    v[j] = column[int64_t(t < tiles ? t : tiles - 1) * bins];
  }
#pragma unroll
  for (int j = 0; j < kRun; ++j) sum += wave * kRun + j < tiles ? v[j] : 0u;
  part[wave][lane] = sum;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += part[w][lane];
  if (b < bins) {
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      const int t = wave * kRun + j;
      if (t < tiles) {
        column[int64_t(t) * bins] = before;
        before += v[j];
      }
    }
    if (wave == kScanWaves - 1) totals[int64_t(blockIdx.y) * bins + b] = before;
  }
}

__device__ __forceinline__ double mapped(uint64_t key, const OperandParams& p) {
  const double v = value_of(key);
  return p.use_softmax != 0.0 ? exp(v - p.max) / p.exp_sum : v;
}

// Which buckets matter.  A difference below `least` times the largest one, m, adds nothing to the distance (see k_distance).  The
// buckets' totals say which rank is in which bucket of either operand, and the splitters between which bounds the two values of a rank
// lie: a run of ranks in one bucket of A and one of B whose bounds are closer than `least` times a difference that is certain
// to be reached (by two buckets that lie apart, or by the two maxima) need not be sorted, nor scattered into buckets.  With smooth fields, whose
// largest values differ, that is all but some hundredth of the keys (2 x 2M: scatter 39 -> 15 us, sort 63 -> 22, distance 23 -> 7; this
// kernel 16; 2 x 3.4M of 32-bit indices the whole distance 458 -> 198).  What is found is the
// same: `threshold` is below every difference that counts.
// What it can save grows with the buckets and, of these, with the share that the largest difference reaches past: where the maxima's gap, in shares
// of the larger maximum, times the buckets squared is below kSelectGain, everything is handed on as it is, for 2 us instead of 10 to 16.
// Measured with blocks of one and of 64 indices, with and without the selection: 512 buckets, gap 3.5e-4: 107 us without, 121 with;
// 8e-3: 118 and 86; 1024 buckets, 2e-4: 160 and 176, 1.3e-3: 164 and 150; 2048 buckets, 1e-4: 349 and 374, 1e-3: 339 and 284.  Below
// kSelectMin buckets it does not pay at any gap (64 buckets: 66000 blocks 46 and 57 us, 131072 56 and 67; 128, 6e-2: 65 and 56).  Two
// versions of one field, 1M blocks: 144 us, 164 with the selection made whatever the gap (2M: 245 and 264; 66000: 46 and 58).
// One workgroup.  A run of ranks starts where a bucket of A or of B does: kEach of each per thread, in the order of the buckets.
constexpr int kSelectThreads = 1024;
template <int kEach>
__global__ __launch_bounds__(kSelectThreads) void k_select(int64_t n, int buckets, const uint64_t* __restrict__ splitters,
                                                           const uint32_t* __restrict__ totals,
                                                           const OperandParams* __restrict__ params, double least,
                                                           Gap* __restrict__ gap, uint8_t* __restrict__ needed,
                                                           uint2* __restrict__ ranks) {
  constexpr int kBucketsMax = kEach * kSelectThreads;
  constexpr int kWaves = kSelectThreads / 64;
  __shared__ union {
    uint32_t first[2][kBucketsMax];               // the buckets' first ranks ...
    double value[2][kBucketsMax / 2];             // ... and then the mapped splitters
  } lds;
  __shared__ uint8_t need[2][kBucketsMax];
  __shared__ uint32_t wave_count[2][kWaves];
  __shared__ double wave_low[kWaves], wave_size[kWaves];
  __shared__ int wave_last[2][kWaves];
  __shared__ unsigned long long longest[2];
  const int t = int(threadIdx.x), lane = t & 63, wave = t >> 6, bins = 2 * buckets;
  const OperandParams p[2] = {params[0], params[1]};
  const double inv[2] = {1.0 / p[0].exp_sum, 1.0 / p[1].exp_sum};
  const double top[2] = {p[0].use_softmax != 0.0 ? inv[0] : p[0].max, p[1].use_softmax != 0.0 ? inv[1] : p[1].max};
  if (!(fabs(top[0] - top[1]) * (double(buckets) * buckets) > kSelectGain * fmax(fabs(top[0]), fabs(top[1])))) {
    for (int b = t; b < 2 * bins; b += kSelectThreads) needed[b] = 1;
    if (t < 2) gap[t] = Gap{1, 0};
    if (t == 0) *reinterpret_cast<Selection*>(gap + 2) = Selection{0.0, -1};
    return;
  }
  // first ranks
  uint32_t first[2][kEach], size[2][kEach];
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int b = t * kEach + j;
      size[o][j] = b < bins ? totals[o * bins + b] : 0u;
      sum += size[o][j];
    }
    uint32_t before = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(before, off, 64);
      if (lane >= off) before += up;
    }
    if (lane == 63) wave_count[o][wave] = before;
    first[o][0] = before - sum;
  }
  if (t < 2) longest[t] = 0;
  __syncthreads();
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    for (int w = 0; w < wave; ++w) first[o][0] += wave_count[o][w];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      if (j > 0) first[o][j] = first[o][j - 1] + size[o][j - 1];
      if (t * kEach + j < kBucketsMax) {
        lds.first[o][t * kEach + j] = first[o][j];             // n beyond the last bucket
        need[o][t * kEach + j] = 0;
      }
    }
  }
  __syncthreads();
  // the runs: of thread t's buckets of operand o, the other operand's bucket in which they start, and their lengths
  int other[2][kEach];
  uint32_t length[2][kEach];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      int b = 0;                                              // the last bucket that starts at or before the rank
      for (int step = bins >> 1; step > 0; step >>= 1)
        if (b + step < bins && lds.first[1 - o][b + step] <= first[o][j]) b += step;
      other[o][j] = b;
      const uint32_t end = b + 1 < bins ? lds.first[1 - o][b + 1] : uint32_t(n), mine = first[o][j] + size[o][j];
      length[o][j] = size[o][j] == 0 || (o == 1 && lds.first[0][b] == first[1][j]) ? 0u : (end < mine ? end : mine) - first[o][j];
    }
  __syncthreads();
  // values at the splitters, and the largest magnitude among them
  const auto value_at = [&](double v, int o) { return p[o].use_softmax != 0.0 ? exp(v - p[o].max) * inv[o] : v; };
  double most = fmax(fabs(top[0]), fabs(top[1]));
  for (int i = t; i < 2 * (buckets - 1); i += kSelectThreads) {
    const int o = i >= buckets - 1 ? 1 : 0, b = i - o * (buckets - 1);
    const double v = value_at(value_of(splitters[o * buckets + b]), o);
    lds.value[o][b] = v;
    most = fmax(most, fabs(v));
  }
  __syncthreads();
  const auto low = [&](int o, int b) { return (b & 1) ? lds.value[o][b >> 1] : (b > 0 ? lds.value[o][(b >> 1) - 1] : (p[o].use_softmax != 0.0 ? 0.0 : -INFINITY)); };
  const auto high = [&](int o, int b) { return (b >> 1) < buckets - 1 ? lds.value[o][b >> 1] : top[o]; };
  double reached = fabs(top[0] - top[1]);
  double apart[2][kEach];                                     // how far the run's two values can be from each other
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      apart[o][j] = 0.0;
      if (length[o][j] == 0) continue;
      const int b = t * kEach + j, c = other[o][j];
      apart[o][j] = fmax(high(o, b) - low(1 - o, c), high(1 - o, c) - low(o, b));
      reached = fmax(reached, fmax(low(o, b) - high(1 - o, c), low(1 - o, c) - high(o, b)));
    }
  reached = wave_max(reached);
  most = wave_max(most);
  if (lane == 0) {
    wave_low[wave] = reached;
    wave_size[wave] = most;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    reached = fmax(reached, wave_low[w]);
    most = fmax(most, wave_size[w]);
  }
  // The mapped values are off by a few 2^-53 of the largest; where means or their sums are no finite numbers, everything matters.
  const double slack = 64.0 * 2.220446049250313e-16 * most;
  const bool finite = fabs(p[0].sum) < INFINITY && fabs(p[1].sum) < INFINITY && fabs(p[0].exp_sum) < INFINITY && fabs(p[1].exp_sum) < INFINITY;
  double threshold = least * (reached - slack) * (1.0 - 1e-12);
  if (!finite || !(threshold > slack)) threshold = 0.0;
  uint32_t pieces = 0;
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      if (length[o][j] != 0 && !(apart[o][j] + slack < threshold)) {
        need[o][t * kEach + j] = 1;
        need[1 - o][other[o][j]] = 1;
        pieces += (length[o][j] + kPieceRanks - 1) / kPieceRanks;
      } else {
        length[o][j] = 0;
      }
    }
  uint32_t before = pieces;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t up = __shfl_up(before, off, 64);
    if (lane >= off) before += up;
  }
  if (lane == 63) wave_count[0][wave] = before;
  __syncthreads();
  before -= pieces;
  for (int w = 0; w < wave; ++w) before += wave_count[0][w];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int j = 0; j < kEach; ++j)
      for (uint32_t k = 0; k < length[o][j]; k += kPieceRanks)
        ranks[before++] = make_uint2(first[o][j] + k, length[o][j] - k < uint32_t(kPieceRanks) ? length[o][j] - k : uint32_t(kPieceRanks));
  if (t == kSelectThreads - 1) {
    Selection* sel = reinterpret_cast<Selection*>(gap + 2);
    sel->threshold = threshold;
    sel->pieces = int(before);
  }
  // the longest run of buckets between two that matter, of either operand: its keys need not be looked at again
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    int last = -1;                                            // of the thread's needed buckets, then of all before them
#pragma unroll
    for (int j = 0; j < kEach; ++j)
      if (t * kEach + j < bins && need[o][t * kEach + j]) last = t * kEach + j;
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(last, off, 64);
      if (lane >= off) last = up > last ? up : last;
    }
    if (lane == 63) wave_last[o][wave] = last;
    last = __shfl_up(last, 1, 64);
    if (lane == 0) last = -1;
    __syncthreads();
    for (int w = 0; w < wave; ++w) last = wave_last[o][w] > last ? wave_last[o][w] : last;
    const auto run_below = [&](int b) {
      if (b - last >= 2) atomicMax(&longest[o], (unsigned long long)(b - last) << 32 | (unsigned long long)(last + 1) << 16 | (unsigned long long)b);
    };
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int b = t * kEach + j;
      if (b < bins && need[o][b]) {
        run_below(b);
        last = b;
      }
    }
    if (t == kSelectThreads - 1) run_below(bins);
    for (int b = t; b < bins; b += kSelectThreads) needed[o * bins + b] = need[o][b];
  }
  __syncthreads();
  if (t < 2) {
    const int above = int(longest[t] & 0xffffu), below = int((longest[t] >> 16) & 0xffffu) - 1;
    const uint64_t* split = splitters + t * buckets;
    Gap g = {1, 0};
    if (longest[t] != 0 && (below < 0 || (below >> 1) < buckets - 1)) {      // nothing is above the last splitter's last bucket
      g.from = below < 0 ? 0 : split[below >> 1] + ((below & 1) ? 1u : 0u);
      g.to = above == bins ? ~uint64_t(0) : ((above & 1) ? split[above >> 1] - 1u : split[(above >> 1) - 1]);
    }
    gap[t] = g;
  }
}

constexpr int kBucketThreads = 1024;
constexpr int kBucketWaves = kBucketThreads / 64;
// v of lane (this one ^ kXor), by register moves; all lanes active
template <int kXor>
__device__ __forceinline__ uint32_t across(uint32_t v) {
  if constexpr (kXor == 1) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0xb1, 0xf, 0xf, true));             // quad_perm
  else if constexpr (kXor == 2) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x4e, 0xf, 0xf, true));
  else if constexpr (kXor == 3) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x1b, 0xf, 0xf, true));
  else if constexpr (kXor == 4) return across<7>(across<3>(v));
  else if constexpr (kXor == 7) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x141, 0xf, 0xf, true));       // row_half_mirror
  else if constexpr (kXor == 8) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x128, 0xf, 0xf, true));       // row_ror 8
  else if constexpr (kXor == 15) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x140, 0xf, 0xf, true));      // row_mirror
  else if constexpr (kXor == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
  } else if constexpr (kXor == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
  } else if constexpr (kXor == 31) return across<16>(across<15>(v));
  else return across<32>(across<31>(v));
}
constexpr int top_bit(int v) { return v < 2 ? v : 2 * top_bit(v / 2); }
// the smaller of the thread's key and that of thread (this one ^ kXor), the larger in the upper of the two
template <int kXor>
__device__ __forceinline__ uint64_t ordered(uint64_t mine, uint64_t other) {
  constexpr uint32_t kUpper = uint32_t(top_bit(kXor));
  return (other < mine) != ((threadIdx.x & kUpper) != 0) ? other : mine;
}
template <int kXor>
__device__ __forceinline__ void exchange_in_wave(uint64_t& key) {
  key = ordered<kXor>(key, uint64_t(across<kXor>(uint32_t(key))) | (uint64_t(across<kXor>(uint32_t(key >> 32))) << 32));
}
template <int kXor>
__device__ __forceinline__ void halve_in_wave(uint64_t& key) {        // distances kXor, kXor / 2, ... 1
  exchange_in_wave<kXor>(key);
  if constexpr (kXor > 1) halve_in_wave<kXor / 2>(key);
}
template <int kRun>
__device__ __forceinline__ void sort_in_wave(uint64_t& key) {         // runs of kRun / 2 to runs of kRun, and on to 64
  exchange_in_wave<kRun - 1>(key);
  if constexpr (kRun > 2) halve_in_wave<kRun / 4>(key);
  if constexpr (kRun < 64) sort_in_wave<2 * kRun>(key);
}
// A step between waves: key j of thread t is number j kBucketThreads + t, the exchanges are with number ^ kXor.  kTwo: two buffers in turn, so
// that one barrier a step is enough.
template <int kXor, int kPer, bool kTwo>
__device__ __forceinline__ void exchange_in_group(uint64_t* key, uint64_t* lds, int& turn) {
  constexpr int kOther = kXor / kBucketThreads, kThread = kXor % kBucketThreads;
  uint64_t* at = lds + (kTwo ? turn * kPer * kBucketThreads : 0);
#pragma unroll
  for (int j = 0; j < kPer; ++j) at[j * kBucketThreads + int(threadIdx.x)] = key[j];
  __syncthreads();
  constexpr int kUpper = top_bit(kXor);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint64_t other = at[(j ^ kOther) * kBucketThreads + (int(threadIdx.x) ^ kThread)];
    if constexpr (kUpper >= kBucketThreads) key[j] = (other < key[j]) != ((j & (kUpper / kBucketThreads)) != 0) ? other : key[j];
    else key[j] = ordered<kXor>(key[j], other);
  }
  if (!kTwo) __syncthreads();
  turn ^= 1;
}
template <int kXor, int kPer, bool kTwo>
__device__ __forceinline__ void halve_in_group(uint64_t* key, uint64_t* lds, int& turn) {       // distances kXor, kXor / 2, ... 64
  if constexpr (kXor >= kBucketThreads) {
    constexpr int d = kXor / kBucketThreads;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if ((j & d) == 0) {
        const uint64_t a = key[j], b = key[j | d];
        key[j] = b < a ? b : a;
        key[j | d] = b < a ? a : b;
      }
  } else {
    exchange_in_group<kXor, kPer, kTwo>(key, lds, turn);
  }
  if constexpr (kXor > 64) halve_in_group<kXor / 2, kPer, kTwo>(key, lds, turn);
}
template <int kRun, int kPer, bool kTwo>
__device__ __forceinline__ void merge_in_group(uint64_t* key, int count, uint64_t* lds, int& turn) {
  if (kRun / 2 >= count) return;                           // uniform
  exchange_in_group<kRun - 1, kPer, kTwo>(key, lds, turn);
  if constexpr (kRun > 128) halve_in_group<kRun / 4, kPer, kTwo>(key, lds, turn);
#pragma unroll
  for (int j = 0; j < kPer; ++j)                           // (the waves beyond have nothing but what pads the keys)
    if (j * kBucketThreads + int(threadIdx.x & ~63u) < count) halve_in_wave<32>(key[j]);
  if constexpr (kRun < kPer * kBucketThreads) merge_in_group<2 * kRun, kPer, kTwo>(key, count, lds, turn);
}
// Ascending order of the workgroup's keys, kPer a thread (the largest number from `count` on): bitonic merges whose first step folds a run onto
// itself, so that all exchanges are ascending.  Of the 55 steps of 1024 keys 45 are between lanes, register moves without LDS.  No step depends
// on the keys: 4 us for 1024 and 12 for 4096 whatever they are, where dealing them into intervals takes 7 to 20.  (Many uncrowded buckets, as in
// k_bucket_sort, are the intervals': 1M keys 87 us by exchanges, 83 as there.)  lds: kPer kBucketThreads keys, twice that with kTwo; the first
// half is written first.
template <int kPer, bool kTwo>
__device__ __forceinline__ void sort_group(uint64_t* key, int count, uint64_t* lds) {
  int turn = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (j * kBucketThreads + int(threadIdx.x & ~63u) < count) sort_in_wave<2>(key[j]);
  merge_in_group<128, kPer, kTwo>(key, count, lds, turn);
}

constexpr int kSubs = 2048;
constexpr int kMaxSub = 128;
constexpr int kRestGroups = 64;                  // workgroups of the second sorting kernel
constexpr int kOwnSplitters = 256;               // that a crowded bucket draws from its keys ...
constexpr int kOwnSlots = kSubs / kOwnSplitters; // ... and the intervals below each: the last for the keys that equal it

// cursor[] -> first[]: exclusive prefix sums, by the whole workgroup
__device__ __forceinline__ void scan_intervals(const uint32_t* cursor, uint32_t* first, uint32_t* wave_total) {
  constexpr int kEach = kSubs / kBucketThreads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t c[kEach], sum = 0;
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    c[j] = cursor[int(threadIdx.x) * kEach + j];
    sum += c[j];
  }
  uint32_t before = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t up = __shfl_up(before, off, 64);
    if (lane >= off) before += up;
  }
  if (lane == 63) wave_total[wave] = before;
  __syncthreads();
  before -= sum;
  for (int w = 0; w < wave; ++w) before += wave_total[w];
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    first[int(threadIdx.x) * kEach + j] = before;
    before += c[j];
  }
  if (threadIdx.x == kBucketThreads - 1) first[kSubs] = before;
}

// smallest and largest of the threads' (lo, hi), in every thread
__device__ __forceinline__ void group_bounds(uint64_t& lo, uint64_t& hi, uint64_t* bounds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t l = __shfl_xor((unsigned long long)lo, off, 64), h = __shfl_xor((unsigned long long)hi, off, 64);
    lo = l < lo ? l : lo;
    hi = h > hi ? h : hi;
  }
  if (lane == 0) {
    bounds[2 * wave] = lo;
    bounds[2 * wave + 1] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kBucketWaves; ++w) {
    lo = bounds[2 * w] < lo ? bounds[2 * w] : lo;
    hi = bounds[2 * w + 1] > hi ? bounds[2 * w + 1] : hi;
  }
}

// Bucket b of operand y: its first key and, for 2 b, its number of keys (sums: scratch of one value per wave)
struct BucketPlace { int64_t base, m, equal; };
__device__ __forceinline__ BucketPlace bucket_place(int b, int operand, int buckets, const uint32_t* totals, uint32_t* sums) {
  BucketPlace p;
  const uint32_t* t = totals + int64_t(operand) * 2 * buckets;
  uint32_t sum = 0;
  for (int i = threadIdx.x; i < 2 * b; i += kBucketThreads) sum += t[i];
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = sum;
  __syncthreads();
  p.base = 0;
  for (int w = 0; w < kBucketWaves; ++w) p.base += sums[w];
  p.m = t[2 * b];
  p.equal = t[2 * b + 1];
  return p;
}

// A workgroup sorts bucket 2 b of its operand and copies bucket 2 b + 1, whose keys are equal (one of more than kPieceKeys is left in
// pieces to all workgroups of k_bucket_sort_rest: 2 x 4M equal keys: 1320 -> 233 us for the whole distance, seven values 652 -> 215).  The bucket's keys, at most
// kHeldKeys, are read once and stay in registers.  They are dealt into kSubs equal intervals between the smallest and the
// largest of their values (between neighbouring quantiles the means are spread nearly evenly: one key an interval), put
// together by interval in LDS, at most kBucketCap keys a round, and every key counts the smaller ones of its interval.
// Where that leaves more than kMaxSub keys in one interval (values over many orders of magnitude, as in the first and the last
// bucket) or meets NaN, which has no interval among the values, the intervals are taken between
// splitters drawn from the bucket itself (4096 means of 8x8 blocks: 84 -> 26 us).  Larger buckets and those that
// are crowded even so go to the list of k_bucket_sort_rest.
constexpr int kHeldKeys = 8192;
// above, the pieces of a bucket are at most twice its keys / kPieceKeys, those of both operands at most 2 * 2 n / kPieceKeys <= K
constexpr int kPieceKeys = 4 * kBucketKeys;
static_assert(2 * kSampleSortMax / kBucketKeys >= kBins, "the workspace's totals hold the radix sort's digits");
__device__ __forceinline__ void sort_bucket(int bucket, bool sorts, bool copies, const uint64_t* in_all, uint64_t* out_all, int64_t n,
                                            int buckets, const uint32_t* __restrict__ totals, uint32_t* __restrict__ rest,
                                            uint2* __restrict__ pieces) {
  __shared__ uint64_t key[kBucketCap];
  __shared__ uint32_t first[kSubs + 1], cursor[kSubs];
  __shared__ uint32_t wave_total[kBucketWaves];
  __shared__ double2 bounds[kBucketWaves];
  __shared__ uint64_t split[kOwnSplitters], drawn[kOwnSplitters];
  constexpr int kPerThread = kHeldKeys / kBucketThreads;
  const BucketPlace place = bucket_place(bucket, blockIdx.y, buckets, totals, wave_total);
  const uint64_t* in = in_all + int64_t(blockIdx.y) * n + place.base;
  uint64_t* out = out_all + int64_t(blockIdx.y) * n + place.base;
  if (!copies) {
  } else if (place.equal <= kPieceKeys) {
    for (int64_t i = threadIdx.x; i < place.equal; i += kBucketThreads) out[place.m + i] = in[place.m + i];
  } else if (threadIdx.x == 0) {
    const uint32_t count = uint32_t((place.equal + kPieceKeys - 1) / kPieceKeys), at = atomicAdd(rest + 1, count);
    const int64_t begin = int64_t(blockIdx.y) * n + place.base + place.m;
    for (uint32_t k = 0; k < count; ++k) {
      const int64_t left = place.equal - int64_t(k) * kPieceKeys;
      pieces[at + k] = make_uint2(uint32_t(begin + int64_t(k) * kPieceKeys), uint32_t(left < kPieceKeys ? left : kPieceKeys));
    }
  }
  if (place.m == 0 || !sorts) return;                      // uniform over the workgroup, here and below
  if (place.m > kHeldKeys) {
    if (threadIdx.x == 0) rest[2 + atomicAdd(rest, 1u)] = uint32_t(bucket) * 2 + blockIdx.y;
    return;
  }
  const int m = int(place.m), t = int(threadIdx.x);
  uint64_t held[kPerThread];
#pragma unroll
  for (int j = 0; j < kPerThread; ++j)
    if (j * kBucketThreads < m) held[j] = in[j * kBucketThreads + t < m ? j * kBucketThreads + t : m - 1];
  for (int i = t; i < kSubs; i += kBucketThreads) cursor[i] = 0;
  double least = value_of(held[0]), most = least;
#pragma unroll
  for (int j = 1; j < kPerThread; ++j)
    if (j * kBucketThreads < m) {
      least = fmin(least, value_of(held[j]));
      most = fmax(most, value_of(held[j]));
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    least = fmin(least, __shfl_xor(least, off, 64));
    most = fmax(most, __shfl_xor(most, off, 64));
  }
  if ((t & 63) == 0) bounds[t >> 6] = make_double2(least, most);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kBucketWaves; ++w) {
    least = fmin(least, bounds[w].x);
    most = fmax(most, bounds[w].y);
  }
  // subtraction, product and truncation are all non-decreasing: intervals follow the order of the values
  const double span = most - least;
  const double scale = span > 0.0 ? double(kSubs) / span : 0.0;
  uint32_t where[kPerThread] = {};                         // interval, and the key's number in it above
  bool crowded = false;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j)
    if (j * kBucketThreads + t < m) {
      const double value = value_of(held[j]);
      const int s = int(fmin(fmax((value - least) * scale, 0.0), double(kSubs - 1)));
      // a wave that has many of its first keys in one interval need not have them all counted one after the other there
      if (j == 0 && m > 2 * kMaxSub) crowded = __popcll(__ballot(s == __builtin_amdgcn_readfirstlane(s))) > 24;
      if (crowded) continue;
      const uint32_t at = atomicAdd(&cursor[s], 1u);
      where[j] = uint32_t(s) | (at << 16);
      crowded = crowded || at >= uint32_t(kMaxSub) || value != value;
    }
  bool by_sample = false;
  if (__syncthreads_or(crowded)) {                         // once more, between splitters of the bucket's own
    by_sample = m <= kBucketCap;
    crowded = !by_sample;
    if (by_sample) {
#pragma unroll
      for (int j = 0; j < kPerThread; ++j)
        if (j * kBucketThreads + t < m) key[j * kBucketThreads + t] = held[j];
      for (int i = t; i < kSubs; i += kBucketThreads) cursor[i] = 0;
      __syncthreads();
      if (t < kOwnSplitters) drawn[t] = key[(t * m) / kOwnSplitters];
      __syncthreads();
      constexpr int kParts = kBucketThreads / kOwnSplitters, kEach = kOwnSplitters / kParts;
      const int mine = t / kParts, part = t % kParts;
      const uint64_t value = drawn[mine];
      int rank = 0;
      for (int i = part * kEach; i < (part + 1) * kEach; ++i) rank += drawn[i] < value || (drawn[i] == value && i < mine) ? 1 : 0;
#pragma unroll
      for (int off = 1; off < kParts; off <<= 1) rank += __shfl_xor(rank, off, 64);
      if (part == 0) split[rank] = value;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kPerThread; ++j)
        if (j * kBucketThreads + t < m) {
          int b;
          buckets_of<1>(split, kOwnSplitters, held + j, &b);
          int s = (b >> 1) * kOwnSlots + ((b & 1) ? kOwnSlots - 1 : 0);
          if ((b & 1) == 0 && b > 0 && b < 2 * (kOwnSplitters - 1)) {      // by the key between its two splitters
            const uint64_t lo = split[(b >> 1) - 1], hi = split[b >> 1];
            s += int(fmin(double(held[j] - lo) * (double(kOwnSlots - 1) / double(hi - lo)), double(kOwnSlots - 2)));
          }
          const uint32_t at = atomicAdd(&cursor[s], 1u);
          where[j] = uint32_t(s) | (at << 16);
          crowded = crowded || ((b & 1) == 0 && at >= uint32_t(kMaxSub));
        }
    }
    if (__syncthreads_or(crowded)) {
      if (t == 0) rest[2 + atomicAdd(rest, 1u)] = uint32_t(bucket) * 2 + blockIdx.y;
      return;
    }
  }
  scan_intervals(cursor, first, wave_total);
  __syncthreads();
  for (int s0 = 0; s0 < kSubs;) {
    int s1 = kSubs;                                        // this round: intervals s0 .. s1 - 1, the same in every thread
    if (m > kBucketCap) {
      s1 = s0;
      for (int step = kSubs; step > 0; step >>= 1)
        if (s1 + step <= kSubs && first[s1 + step] - first[s0] <= uint32_t(kBucketCap)) s1 += step;
    }
    const int from = int(first[s0]), count = int(first[s1]) - from;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (j * kBucketThreads + t < m) {
        const int s = int(where[j] & 0xffffu);
        if (s >= s0 && s < s1) key[int(first[s]) - from + int(where[j] >> 16)] = held[j];
      }
    __syncthreads();
    uint32_t rank[kPerThread];                             // among the keys of its interval
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (j * kBucketThreads + t < m) {
        const int s = int(where[j] & 0xffffu);
        rank[j] = 0;
        if (s >= s0 && s < s1) {
          const int a = int(first[s]) - from, b = int(first[s + 1]) - from, self = a + int(where[j] >> 16);
          const auto look = [&](int q) {
            const uint64_t other = key[q];
            rank[j] += other < held[j] || (other == held[j] && q < self) ? 1u : 0u;
          };
          if (by_sample && s % kOwnSlots == kOwnSlots - 1) {
            rank[j] = where[j] >> 16;                      // equal to a splitter
          } else {
            int q = a;
            if (b - a >= 4)                                // an interval has one key on average, in crowded buckets many: 15625 means of an
              for (; q + 4 <= b; q += 4)                   // image 33 -> 26 us; with the loop unrolled for all, 2 x 1M keys 41 -> 44
#pragma unroll
                for (int u = 0; u < 4; ++u) look(q + u);
            for (; q < b; ++q) look(q);
          }
        }
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (j * kBucketThreads + t < m) {
        const int s = int(where[j] & 0xffffu);
        if (s >= s0 && s < s1) key[int(first[s]) - from + int(rank[j])] = held[j];
      }
    __syncthreads();
    for (int i = t; i < count; i += kBucketThreads) out[from + i] = key[i];
    __syncthreads();
    s0 = s1;
  }
}

// grid (buckets, operand): all of them, or those that k_select has marked
__global__ __launch_bounds__(kBucketThreads, 8) void k_bucket_sort(const uint64_t* in_all, uint64_t* out_all, int64_t n,
                                                                   int buckets, const uint32_t* __restrict__ totals,
                                                                   uint32_t* __restrict__ rest, uint2* __restrict__ pieces,
                                                                   const uint8_t* __restrict__ needed) {
  const int bin = int(blockIdx.y) * 2 * buckets + 2 * int(blockIdx.x);
  const bool sorts = !needed || needed[bin] != 0, copies = !needed || needed[bin + 1] != 0;
  if (sorts || copies) sort_bucket(blockIdx.x, sorts, copies, in_all, out_all, n, buckets, totals, rest, pieces);
}

// The pieces of large buckets of one value, and the buckets that k_bucket_sort leaves, listed in rest, any number of keys in
// any distribution.  As there, with the keys read again where they are needed and intervals of one shared value left as
// they are.  Where an interval has more than kMaxSub keys of several values (values over many orders of magnitude), or there
// is NaN or infinity at an end, the intervals are made equal in the keys instead; if that does not help, fold_sort takes over
// (a cluster of two fifths of all keys that the samples miss altogether: 0.9 ms for 70001 keys, 18 for 2^20).  A bucket that
// does not fit LDS takes several rounds.
__global__ __launch_bounds__(kBucketThreads) void k_bucket_sort_rest(const uint64_t* in_all, uint64_t* out_all, int64_t n,
                                                                     int buckets, const uint32_t* __restrict__ totals,
                                                                     const uint32_t* __restrict__ rest,
                                                                     const uint2* __restrict__ pieces) {
  __shared__ uint64_t key[kBucketCap];
  __shared__ uint32_t first[kSubs + 1], cursor[kSubs];
  __shared__ uint32_t wave_total[kBucketWaves];
  __shared__ uint64_t bounds[2 * kBucketWaves];
  constexpr int kPerThread = kBucketCap / kBucketThreads;
  const uint32_t listed = rest[0], cut = rest[1];
  for (uint32_t r = blockIdx.x; r < cut; r += gridDim.x) {
    const uint2 piece = pieces[r];
    const uint64_t value = in_all[piece.x];
    for (uint32_t i = threadIdx.x; i < piece.y; i += kBucketThreads) out_all[piece.x + i] = value;
  }
  for (uint32_t r = blockIdx.x; r < listed; r += gridDim.x) {
    const uint32_t which = rest[2 + r];
    const BucketPlace bucket = bucket_place(int(which >> 1), int(which & 1u), buckets, totals, wave_total);
    const uint64_t* in = in_all + int64_t(which & 1u) * n + bucket.base;
    uint64_t* out = out_all + int64_t(which & 1u) * n + bucket.base;
    const int64_t m = bucket.m;
    if (m <= kBucketCap) {                                 // by exchanges, whatever the values: 12 us where the rounds below took 37 to 46
      uint64_t mine[kPerThread];
#pragma unroll
      for (int j = 0; j < kPerThread; ++j)
        mine[j] = j * kBucketThreads + int(threadIdx.x) < m ? in[j * kBucketThreads + int(threadIdx.x)] : ~uint64_t(0);
      sort_group<kPerThread, false>(mine, int(m), key);
#pragma unroll
      for (int j = 0; j < kPerThread; ++j)
        if (j * kBucketThreads + int(threadIdx.x) < m) out[j * kBucketThreads + int(threadIdx.x)] = mine[j];
      __syncthreads();
      continue;
    }
    // calls f(key) for the thread's keys, kPerThread of them requested together
    auto each = [&](auto f) {
      for (int64_t i0 = threadIdx.x; i0 < m; i0 += kBucketCap) {
        uint64_t v[kPerThread];
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) v[j] = in[i0 + j * kBucketThreads < m ? i0 + j * kBucketThreads : m - 1];
#pragma unroll
        for (int j = 0; j < kPerThread; ++j)
          if (i0 + j * kBucketThreads < m) f(v[j]);
      }
    };
    uint64_t lo = ~uint64_t(0), hi = 0;
    each([&](uint64_t k) {
      lo = k < lo ? k : lo;
      hi = k > hi ? k : hi;
    });
    group_bounds(lo, hi, bounds);
    bool by_value = isfinite(value_of(lo)) && isfinite(value_of(hi));
    for (;;) {
      // subtraction, conversion, product and truncation are all non-decreasing: intervals follow the order of the keys
      const double least = value_of(lo);
      const double span = by_value ? value_of(hi) - least : double(hi - lo);
      const double scale = span > 0.0 ? double(kSubs) / span : 0.0;
      auto sub_of = [&](uint64_t k) {
        return int(fmin((by_value ? value_of(k) - least : double(k - lo)) * scale, double(kSubs - 1)));
      };
      for (int i = threadIdx.x; i < kSubs; i += kBucketThreads) cursor[i] = 0;
      __syncthreads();
      each([&](uint64_t k) { atomicAdd(&cursor[sub_of(k)], 1u); });
      __syncthreads();
      scan_intervals(cursor, first, wave_total);
      __syncthreads();
      bool again = false;
      for (int s0 = 0; s0 < kSubs;) {
        // intervals s0 .. s1 - 1 fit; the same in every thread
        int s1 = s0;
        for (int step = kSubs; step > 0; step >>= 1)
          if (s1 + step <= kSubs && first[s1 + step] - first[s0] <= uint32_t(kBucketCap)) s1 += step;
        if (s1 == s0) {                                      // an interval larger than LDS
          if (by_value) {
            again = true;
            break;
          }
          for (int64_t i = threadIdx.x; i < m; i += kBucketThreads) out[i] = in[i];
          fold_sort<int64_t>(out, m);
          break;
        }
        const uint32_t from = first[s0];
        const int count = int(first[s1] - from);
        for (int i = threadIdx.x; i < kSubs; i += kBucketThreads) cursor[i] = first[i] - from;
        __syncthreads();
        each([&](uint64_t k) {
          const int s = sub_of(k);
          if (s >= s0 && s < s1) key[atomicAdd(&cursor[s], 1u)] = k;
        });
        __syncthreads();
        for (int i = threadIdx.x; i < kSubs; i += kBucketThreads) cursor[i] = 0;      // now: the interval has several values
        __syncthreads();
        for (int i = threadIdx.x; i < count; i += kBucketThreads) {
          const int s = sub_of(key[i]);
          if (key[i] != key[first[s] - from]) cursor[s] = 1;
        }
        __syncthreads();
        uint64_t mine[kPerThread];
        int place[kPerThread];
        bool crowded = false;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
          const int i = j * kBucketThreads + int(threadIdx.x);
          place[j] = -1;
          if (i < count) {
            mine[j] = key[i];
            const int s = sub_of(mine[j]);
            const int a = int(first[s] - from), b = int(first[s + 1] - from);
            place[j] = i;
            if (cursor[s] != 0) {
              crowded = crowded || b - a > kMaxSub;
              if (b - a <= kMaxSub) {
                int p = a;
                for (int q = a; q < b; ++q) {
                  const uint64_t other = key[q];
                  p += other < mine[j] || (other == mine[j] && q < i) ? 1 : 0;
                }
                place[j] = p;
              }
            }
          }
        }
        if (__syncthreads_or(crowded)) {
          if (by_value && s0 == 0) {                         // nothing has been written yet
            again = true;
            break;
          }
          fold_sort<int>(key, count);
        } else {
#pragma unroll
          for (int j = 0; j < kPerThread; ++j)
            if (place[j] >= 0) key[place[j]] = mine[j];
          __syncthreads();
        }
        for (int i = threadIdx.x; i < count; i += kBucketThreads) out[from + i] = key[i];
        __syncthreads();
        s0 = s1;
      }
      if (!again) break;
      by_value = false;
    }
  }
}

// ---- up to kRangeMax keys: each workgroup finds its own range of them -----------------------------------------------
// Up to kBucketThreads blocks: one workgroup of an operand makes the keys, one a thread, the parameters, and the order.
__global__ __launch_bounds__(kBucketThreads) void k_means_in_order(const void* __restrict__ N1, const void* __restrict__ F1, const void* __restrict__ N2,
                                                                   const void* __restrict__ F2, int ntype, int itype, double scale, int n, int kept,
                                                                   uint64_t* __restrict__ sorted, OperandParams* __restrict__ params) {
  __shared__ uint64_t lds[2 * kBucketThreads];
  __shared__ double top;
  const int t = int(threadIdx.x), at = t < n ? t : n - 1;
  double v = 0.0;
  with_loads(blockIdx.y ? N2 : N1, blockIdx.y ? F2 : F1, ntype, itype, kept, [&](auto load_n, auto load_f) {
    const double f = load_f(at), x = load_n(at);
    v = x * f * scale;
  });
  uint64_t key = t < n ? key_of(v) : ~uint64_t(0);
  double s = t < n ? v : 0.0, m = t < n ? fmax(v, -INFINITY) : -INFINITY;
  group_sum_max(s, m);
  if (t == 0) {
    OperandParams& p = params[blockIdx.y];
    p.sum = s;
    p.max = m;
    p.use_softmax = fabs(s - 1.0) > kSumTolerance ? 1.0 : 0.0;
    top = m;
  }
  __syncthreads();
  m = fmax(top, -1.7976931348623157e308);                  // minus infinity weighs nothing
  double e = t < n ? exp(v - m) : 0.0, none = 0.0;
  group_sum_max(e, none);
  if (t == 0) params[blockIdx.y].exp_sum = e;
  sort_group<1, true>(&key, n, lds);
  if (t < n) sorted[int64_t(blockIdx.y) * n + t] = key;
}

// Workgroup b of an operand goes through all of its keys, which its L2 holds, counts those below its own range (between
// two splitters, the upper one included), and sorts those in it: no counting of buckets, no scattering, no list of what is left over.  More than
// kBucketThreads are sorted in two to a thread (one range of some thousand at full size: 65536 blocks with such a range 69 -> 43 us, by another walk
// through all keys before), more than kRangeHeld, and the range ends at one of them instead, and goes on from there: at a place among those that
// were collected that leaves out a third of them at least.  The last workgroup along x makes the parameters.  Bounds: the reads from L2 (64 bytes a
// cycle and compute unit) and the compares, 20 us for 2 x 65536 keys; the exchanges, 4 us, from 16384 keys down (11 us).  74 registers and so one
// workgroup a compute unit: two, in 64 registers, are slower (52000 blocks 38 -> 45 us for the whole distance).
constexpr int kRangeInFlight = 16;
constexpr int kRangeHeld = 2 * kBucketThreads;
__global__ __launch_bounds__(kBucketThreads) void k_range_sort(const uint64_t* __restrict__ keys, uint64_t* __restrict__ sorted, int n, int buckets,
                                                               const uint64_t* __restrict__ splitters, const double* __restrict__ partials,
                                                               int tiles, OperandParams* __restrict__ params) {
  if (int(blockIdx.x) == buckets) {
    mean_params(partials, tiles, params);
    return;
  }
  __shared__ uint64_t lds[2 * kRangeHeld];                  // the second half also: the keys of the range as they come
  __shared__ int counted[3];                               // keys below the range, equal to its end, inside
  __shared__ uint64_t cut;
  const uint64_t* in = keys + int64_t(blockIdx.y) * n;
  uint64_t* out = sorted + int64_t(blockIdx.y) * n;
  const uint64_t* split = splitters + int64_t(blockIdx.y) * buckets;
  const int t = int(threadIdx.x), b = int(blockIdx.x);
  uint64_t from = b > 0 ? split[b - 1] + 1u : 0u;           // (no key is the largest number)
  const uint64_t last = b < buckets - 1 ? split[b] : ~uint64_t(0);
  uint64_t end = last;
  if (from > last) return;                                 // uniform: equal splitters
  for (;;) {
    if (t < 3) counted[t] = 0;
    __syncthreads();
    int below = 0, equal = 0;
    const uint64_t span = end - from;
    for (int i0 = 0; i0 < n; i0 += kBucketThreads * kRangeInFlight) {
      uint64_t k[kRangeInFlight];
#pragma unroll
      for (int u = 0; u < kRangeInFlight; ++u) {           // beyond the last: the largest number, which no key is
        const int i = i0 + u * kBucketThreads + t;
        k[u] = in[i < n ? i : n - 1];
        if (i >= n) k[u] = ~uint64_t(0);
      }
#pragma unroll
      for (int u = 0; u < kRangeInFlight; ++u) {
        below += k[u] < from ? 1 : 0;
        if (k[u] - from <= span) {
          if (k[u] == end) ++equal;                        // (also what is beyond the last, where the range has no end)
          else {
            const int at = atomicAdd(&counted[2], 1);
            if (at < kRangeHeld) lds[kRangeHeld + at] = k[u];
          }
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      below += __shfl_xor(below, off, 64);
      equal += __shfl_xor(equal, off, 64);
    }
    if ((t & 63) == 0) {
      atomicAdd(&counted[0], below);
      atomicAdd(&counted[1], equal);
    }
    __syncthreads();
    const int inside = counted[2], m = inside < kRangeHeld ? inside : kRangeHeld;
    below = counted[0];
    equal = counted[1];
    uint64_t key[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) key[j] = j * kBucketThreads + t < m ? lds[kRangeHeld + j * kBucketThreads + t] : ~uint64_t(0);
    if (m <= kBucketThreads) sort_group<1, true>(key, m, lds);            // uniform
    else sort_group<2, true>(key, m, lds);
    if (inside > kRangeHeld) {
      const int place = int(int64_t(kRangeHeld) * (kRangeHeld * 2 / 3) / inside);
      if (t == place % kBucketThreads) cut = place < kBucketThreads ? key[0] : key[1];
      __syncthreads();
      end = cut;                                           // below the old end
      continue;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (j * kBucketThreads + t < m) out[below + j * kBucketThreads + t] = key[j];
    if (end != ~uint64_t(0))
      for (int i = t; i < equal; i += kBucketThreads) out[below + m + i] = end;
    if (end == last) break;                                // uniform
    from = end + 1u;
    end = last;
    __syncthreads();
  }
}

// ---- radix sort, one pass = histogram per tile, exclusive scan over (digit, tile), stable scatter --------------
// A tile is kTileKeys consecutive keys, ranked by one workgroup of four waves: wave w takes the tile's w-th quarter,
// and element j * 64 + lane of that quarter belongs to lane `lane` in round j, so waves, rounds and, within a
// round, lanes follow the input order.

// the lanes of this round that hold the same digit as this one (valid lanes only)
__device__ __forceinline__ uint64_t same_digit_lanes(uint32_t digit, bool valid) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < kRadixBits; ++b) {
    const uint64_t set = __ballot(valid && ((digit >> b) & 1u));
    peers &= ((digit >> b) & 1u) ? set : ~set;
  }
  return peers;
}

// One count per digit and tile, one LDS atomic per key (measured against one atomic per group of lanes that share a
// digit, found with the ballots of the scatter kernel: 9.9 against 17.4 us for 2 x 2M keys).
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t* __restrict__ keys, int64_t n,
                                                             int64_t n_tiles, int shift, uint32_t* __restrict__ hist) {
  __shared__ uint32_t count[kBins];
  static_assert(kBins == kSortThreads, "one thread per digit");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t* in = keys + int64_t(blockIdx.y) * n;
  uint32_t* h = hist + int64_t(blockIdx.y) * kBins * n_tiles;
  count[threadIdx.x] = 0;
  __syncthreads();
  // which lane counts which key does not matter here: two neighbouring keys per lane and load, all loads first
  const int64_t base = int64_t(blockIdx.x) * kTileKeys + wave * kWaveKeys;
  uint64_t key[kKeysPerLane];
  const bool whole = base + kWaveKeys <= n && (reinterpret_cast<uintptr_t>(in) & 15u) == 0;      // uniform over the wave
  if (whole) {
#pragma unroll
    for (int j = 0; j < kKeysPerLane / 2; ++j) {
      const uint4 two = *reinterpret_cast<const uint4*>(in + base + (j * 64 + lane) * 2);
      key[2 * j] = uint64_t(two.x) | (uint64_t(two.y) << 32);
      key[2 * j + 1] = uint64_t(two.z) | (uint64_t(two.w) << 32);
    }
  } else {
#pragma unroll
    for (int j = 0; j < kKeysPerLane; ++j) {
      const int64_t i = base + j * 64 + lane;
      key[j] = i < n ? in[i] : 0;
    }
  }
#pragma unroll
  for (int j = 0; j < kKeysPerLane; ++j) {
    const bool valid = whole || base + j * 64 + lane < n;
    if (valid) atomicAdd(&count[uint32_t(key[j] >> shift) & (kBins - 1)], 1u);
  }
  __syncthreads();
  h[int64_t(threadIdx.x) * n_tiles + blockIdx.x] = count[threadIdx.x];
}

__device__ __forceinline__ uint32_t group_exclusive_scan(uint32_t v, uint32_t* lds /* blockDim.x entries */,
                                                         uint32_t* total) {
  lds[threadIdx.x] = v;
  __syncthreads();
  for (int off = 1; off < int(blockDim.x); off <<= 1) {
    const uint32_t add = int(threadIdx.x) >= off ? lds[threadIdx.x - off] : 0u;
    __syncthreads();
    lds[threadIdx.x] += add;
    __syncthreads();
  }
  if (total) *total = lds[blockDim.x - 1];
  const uint32_t ex = lds[threadIdx.x] - v;
  __syncthreads();                                        // the buffer may be used again right away
  return ex;
}

// Per digit (grid x) and operand (grid y): the counts of the digit's tiles become their exclusive prefix sums, in
// place, and the digit's total goes to totals.  The scatter kernel adds the totals of the lower digits itself.
__global__ __launch_bounds__(kSortThreads) void k_scan_digit(uint32_t* __restrict__ hist, int64_t n_tiles,
                                                             uint32_t* __restrict__ totals) {
  __shared__ uint32_t lds[kSortThreads];
  uint32_t* row = hist + (int64_t(blockIdx.y) * kBins + blockIdx.x) * n_tiles;
  uint32_t carry = 0;
  for (int64_t t0 = 0; t0 < n_tiles; t0 += kSortThreads) {
    const int64_t t = t0 + threadIdx.x;
    const uint32_t v = t < n_tiles ? row[t] : 0u;
    uint32_t chunk_total;
    const uint32_t ex = group_exclusive_scan(v, lds, &chunk_total);
    if (t < n_tiles) row[t] = carry + ex;
    carry += chunk_total;
  }
  if (threadIdx.x == 0) totals[blockIdx.y * kBins + blockIdx.x] = carry;
}

// The keys of a tile are first put in digit order in LDS (ranks within a wave from lane ballots and a per-wave
// cursor per digit, then the waves' counts are chained), and then written out in that order, so that consecutive
// threads write consecutive keys of a digit's run.  A digit that all n keys share (the sign and exponent bytes of
// block means, typically) leaves the order as it is: the tile is copied.
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint64_t* __restrict__ keys_in,
                                                                uint64_t* __restrict__ keys_out, int64_t n,
                                                                int64_t n_tiles, int shift,
                                                                const uint32_t* __restrict__ hist,
                                                                const uint32_t* __restrict__ totals) {
  __shared__ uint64_t sorted[kTileKeys];
  __shared__ uint32_t cursor[kSortThreads / 64][kBins];   // per wave: count so far, later the wave's offset in its digit
  __shared__ uint32_t tile_first[kBins];                  // position in the tile of the first key with that digit
  __shared__ uint32_t out_first[kBins];                   // position in the output of that key
  __shared__ uint32_t scan[kSortThreads];
  __shared__ uint32_t uniform;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t* in = keys_in + int64_t(blockIdx.y) * n;
  uint64_t* out = keys_out + int64_t(blockIdx.y) * n;
  const int64_t tile_base = int64_t(blockIdx.x) * kTileKeys;
  const int64_t base = tile_base + wave * kWaveKeys;
  uint64_t key[kKeysPerLane];
#pragma unroll
  for (int j = 0; j < kKeysPerLane; ++j) {
    const int64_t i = base + j * 64 + lane;
    key[j] = i < n ? in[i] : 0;
  }
  const uint32_t digit_total = totals[blockIdx.y * kBins + threadIdx.x];
  if (threadIdx.x == 0) uniform = 0;
#pragma unroll
  for (int w = 0; w < kSortThreads / 64; ++w) cursor[w][threadIdx.x] = 0;
  __syncthreads();
  if (int64_t(digit_total) == n) uniform = 1;
  const uint32_t digit_first = group_exclusive_scan(digit_total, scan, nullptr);   // (contains the barrier)
  if (uniform) {
#pragma unroll
    for (int j = 0; j < kKeysPerLane; ++j) {
      const int64_t i = base + j * 64 + lane;
      if (i < n) out[i] = key[j];
    }
    return;
  }
  const uint64_t below = (uint64_t(1) << lane) - 1;      // lanes before this one
  uint32_t local[kKeysPerLane];                          // rank among the wave's keys with the same digit
#pragma unroll
  for (int j = 0; j < kKeysPerLane; ++j) {
    const bool valid = base + j * 64 + lane < n;
    const uint32_t digit = uint32_t(key[j] >> shift) & (kBins - 1);
    const uint64_t peers = same_digit_lanes(digit, valid);
    const uint32_t start = valid ? cursor[wave][digit] : 0u;
    wave_lds_sync();                                       // every lane has read before any leader writes
    const uint32_t rank = uint32_t(__popcll(peers & below));
    if (valid && rank == 0) cursor[wave][digit] = start + uint32_t(__popcll(peers));
    local[j] = start + rank;
    wave_lds_sync();
  }
  __syncthreads();
  {  // thread d: the waves' counts of digit d become the waves' offsets; the tile's count of d is scanned over d
    uint32_t run = 0;
#pragma unroll
    for (int w = 0; w < kSortThreads / 64; ++w) {
      const uint32_t c = cursor[w][threadIdx.x];
      cursor[w][threadIdx.x] = run;
      run += c;
    }
    tile_first[threadIdx.x] = group_exclusive_scan(run, scan, nullptr);
    out_first[threadIdx.x] = digit_first + hist[int64_t(blockIdx.y) * kBins * n_tiles + int64_t(threadIdx.x) * n_tiles + blockIdx.x];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kKeysPerLane; ++j) {
    if (base + j * 64 + lane < n) {
      const uint32_t digit = uint32_t(key[j] >> shift) & (kBins - 1);
      sorted[tile_first[digit] + cursor[wave][digit] + local[j]] = key[j];
    }
  }
  __syncthreads();
  const int64_t left = n - tile_base;
  const int count = left < kTileKeys ? int(left) : kTileKeys;
#pragma unroll
  for (int k = 0; k < kKeysPerLane; ++k) {
    const int i = k * kSortThreads + threadIdx.x;
    if (i < count) {
      const uint64_t v = sorted[i];
      const uint32_t digit = uint32_t(v >> shift) & (kBins - 1);
      out[out_first[digit] + uint32_t(i) - tile_first[digit]] = v;
    }
  }
}

// ---- the distance ------------------------------------------------------------------------------------------
// d = |P_A - P_B| of a workgroup's ranks: their maximum m and the sum of (d / m)^p, in one launch (two, with the differences in memory: 23 us for
// 2 x 2M ranks): the differences wait in LDS, those that do not fit are computed again.  A term with (d / m)^p below
// 2^-100 is left at zero: all of the up to 2^31 of them together are below 2^-69 of the sum, whose largest term is 1, and at the
// orders in use (68 and more) that is every d below a third of m, whose pow would be most of the pass.  `chosen`: the pieces of ranks
// that k_select has left, in its order; otherwise `chunk` ranks per workgroup.
__global__ __launch_bounds__(kThreads) void k_distance(const uint64_t* __restrict__ sorted, int64_t n, int64_t chunk,
                                                       const OperandParams* __restrict__ params, double order, double least,
                                                       const Selection* __restrict__ chosen, const uint2* __restrict__ ranks,
                                                       double* __restrict__ partials) {
  __shared__ double top;
  const OperandParams pa = params[0], pb = params[1];
  const int left = chosen ? chosen->pieces : -1;
  const bool all = left < 0;
  const int pieces = all ? int(gridDim.x) : left;
  __shared__ double kept[kKeptDifferences][kThreads];
  // calls f(d) for the thread's differences from number `skip` on
  const auto each = [&](int skip, auto f) {
    int number = 0;
    for (int k = blockIdx.x; k < pieces; k += gridDim.x) {
      int64_t begin = int64_t(k) * chunk, end = begin + chunk < n ? begin + chunk : n;
      if (!all) {
        const uint2 r = ranks[k];
        begin = r.x;
        end = begin + r.y;
      }
      for (int64_t i0 = begin + threadIdx.x; i0 < end; i0 += kThreads * kDistancesInFlight) {
        if (number + kDistancesInFlight <= skip) {
          number += kDistancesInFlight;
          continue;
        }
        uint64_t a[kDistancesInFlight], b[kDistancesInFlight];
#pragma unroll
        for (int u = 0; u < kDistancesInFlight; ++u) {
          const int64_t i = i0 + u * kThreads < end ? i0 + u * kThreads : end - 1;
          a[u] = sorted[i];
          b[u] = sorted[n + i];
        }
#pragma unroll
        for (int u = 0; u < kDistancesInFlight; ++u, ++number)
          f(number, i0 + u * kThreads < end ? fabs(mapped(a[u], pa) - mapped(b[u], pb)) : 0.0);
      }
    }
    return number;
  };
  double s = 0.0, m = 0.0;
  int held = each(0, [&](int number, double d) {
    m = fmax(m, d);
    if (number < kKeptDifferences) kept[number][threadIdx.x] = d;
  });
  group_sum_max(s, m);
  if (threadIdx.x == 0) top = m;
  __syncthreads();
  m = top;
  s = 0.0;
  const double cut = fmax(chosen ? chosen->threshold : 0.0, least * m);
  const auto add = [&](double d) {
    if (d != d) s += d;
    else if (m > 0.0 && !(d < cut)) {
      const double x = d / m;
      if (!(x < least)) s += pow(x, order);
    }
  };
  for (int k = 0; k < held && k < kKeptDifferences; ++k) add(kept[k][threadIdx.x]);
  if (held > kKeptDifferences) each(kKeptDifferences, [&](int, double d) { add(d); });
  double none = 0.0;
  group_sum_max(s, none);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = s;
    partials[2 * blockIdx.x + 1] = m;
  }
}

// a thread per workgroup's record
__global__ __launch_bounds__(kStatGroups) void k_distance_final(const double* __restrict__ partials, int groups, double n, double order,
                                                                  double* __restrict__ out) {
  __shared__ double top;
  const int g = int(threadIdx.x);
  const double part = g < groups ? partials[2 * g] : 0.0, most = g < groups ? partials[2 * g + 1] : 0.0;
  double s = 0.0, m = most;
  group_sum_max(s, m);
  if (g == 0) top = m;
  __syncthreads();
  m = top;
  // the workgroups' sums are relative to their own maxima
  const double x = most / m;
  s = part != 0.0 && x < 1.0 ? part * pow(x, order) : part;
  double none = 0.0;
  group_sum_max(s, none);
  if (g == 0) out[0] = m > 0.0 ? m * pow(s / n, 1.0 / order) : 0.0;
}

// The same of few ranks, in one workgroup and without a second launch
constexpr int kOneGroupThreads = 1024;
__global__ __launch_bounds__(kOneGroupThreads) void k_distance_of_few(const uint64_t* __restrict__ sorted, int n, const OperandParams* __restrict__ params,
                                                                      double order, double least, double* __restrict__ out) {
  __shared__ double top;
  constexpr int kEach = kMaxSamples / kOneGroupThreads;
  const OperandParams pa = params[0], pb = params[1];
  uint64_t a[kEach], b[kEach];
#pragma unroll
  for (int u = 0; u < kEach; ++u)
    if (u * kOneGroupThreads < n) {
      const int i = u * kOneGroupThreads + int(threadIdx.x) < n ? u * kOneGroupThreads + int(threadIdx.x) : n - 1;
      a[u] = sorted[i];
      b[u] = sorted[n + i];
    }
  double d[kEach], s = 0.0, m = 0.0;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    d[u] = 0.0;
    if (u * kOneGroupThreads < n)
      d[u] = u * kOneGroupThreads + int(threadIdx.x) < n ? fabs(mapped(a[u], pa) - mapped(b[u], pb)) : 0.0;
    m = fmax(m, d[u]);
  }
  group_sum_max(s, m);
  if (threadIdx.x == 0) top = m;
  __syncthreads();
  m = top;
  s = 0.0;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    if (d[u] != d[u]) s += d[u];
    else if (m > 0.0 && !(d[u] < least * m)) {
      const double x = d[u] / m;
      if (!(x < least)) s += pow(x, order);
    }
  }
  double none = 0.0;
  group_sum_max(s, none);
  if (threadIdx.x == 0) out[0] = m > 0.0 ? m * pow(s / double(n), 1.0 / order) : 0.0;
}

// Up to kRangeMax blocks: few launches, of kernels that go through all keys again rather than have them counted and scattered.
int launch_few(int64_t n, int kept, const void* N1, const void* F1, const void* N2, const void* F2, int nt, int it, double scale, double order, double least,
               double* out, const Workspace& w, hipStream_t s) {
  if (n <= kBucketThreads) {
    hipLaunchKernelGGL(k_means_in_order, dim3(1, 2), dim3(kBucketThreads), 0, s, N1, F1, N2, F2, nt, it, scale, int(n), kept, w.buf0, w.params);
    hipLaunchKernelGGL(k_distance_of_few, dim3(1), dim3(kOneGroupThreads), 0, s, w.buf0, int(n), w.params, order, least, out);
    return hip_status(hipGetLastError());
  }
  constexpr int kFewThreads = 256;                         // of k_means, a key each
  static_assert(kRangeMax <= kFewThreads * kMaxTiles && kMaxTiles <= kStatGroups, "a tile of as many keys, and a record of each");
  const int tiles = int((n + kFewThreads - 1) / kFewThreads);
  const int samples = int((n + kSampleRun - 1) / kSampleRun);      // in the sorted keys' place, which have none yet
  const auto means = n <= kMaxSamples ? k_means<false, kFewThreads, 1> : k_means<false, kFewThreads, 1, true>;
  hipLaunchKernelGGL(means, dim3(unsigned((tiles + 7) / 8 * 8), 2), dim3(kFewThreads), 0, s, N1, F1, N2, F2, nt, it, scale, n, int64_t(kFewThreads), tiles, kept, 1,
                     nullptr, w.buf1, nullptr, w.rest, w.partials, w.buf0);
  constexpr int kPerGroup = kRankThreads / kRankLanes;
  if (n <= kMaxSamples) {
    hipLaunchKernelGGL(k_rank_sort, dim3(unsigned((n + kPerGroup - 1) / kPerGroup + 1), 2), dim3(kRankThreads), 0, s, w.buf1, int(n), w.buf0, w.partials, tiles,
                       w.params);
    hipLaunchKernelGGL(k_distance_of_few, dim3(1), dim3(kOneGroupThreads), 0, s, w.buf0, int(n), w.params, order, least, out);
    return hip_status(hipGetLastError());
  }
  int buckets = 1;
  while (int64_t(buckets) * kRangeKeys < n) buckets *= 2;
  // the splitters take the place of the counts, which are not needed here: those are 16 bytes a tile of kMinTileKeys and bucket of kBucketKeys, rounded
  // up to 256 in all, these 16 bytes a range, of which there are at most four for such a bucket, and three or four tiles at least
  uint64_t* splitters = reinterpret_cast<uint64_t*>(w.hist);
  hipLaunchKernelGGL(k_splitters, dim3((samples + kPerGroup - 1) / kPerGroup, 2), dim3(kRankThreads), 0, s, w.buf0, buckets, splitters, samples);
  hipLaunchKernelGGL(k_range_sort, dim3(buckets + 1, 2), dim3(kBucketThreads), 0, s, w.buf1, w.buf0, int(n), buckets, splitters, w.partials, tiles, w.params);
  const int64_t chunk = ((n + kStatGroups - 1) / kStatGroups + kThreads - 1) / kThreads * kThreads;
  const int groups = int((n + chunk - 1) / chunk);
  hipLaunchKernelGGL(k_distance, dim3(groups), dim3(kThreads), 0, s, w.buf0, n, chunk, w.params, order, least, nullptr, w.ranks, w.partials);
  hipLaunchKernelGGL(k_distance_final, dim3(1), dim3((groups + 63) / 64 * 64), 0, s, w.partials, groups, double(n), order, out);
  return hip_status(hipGetLastError());
}

}  // namespace

size_t wasserstein_workspace_bytes(int64_t n_blocks) { return carve(nullptr, n_blocks, nullptr); }

int launch_approximate_wasserstein(const pbz_codec* c, int64_t n, const void* N1, const void* F1, const void* N2,
                                   const void* F2, double order, double* out, void* workspace, hipStream_t s) {
  Workspace w;
  carve(workspace, n, &w);
  const SortPlan plan = sort_plan(n);
  const int64_t chunk = ((n + kStatGroups - 1) / kStatGroups + kThreads - 1) / kThreads * kThreads;
  const int groups = int((n + chunk - 1) / chunk);
  const double scale = 1.0 / (c->r * std::sqrt(double(c->vol)));
  const double least = std::exp2(-100.0 / order);
  const int K = plan.buckets;
  const int nt = int(c->ftype), it = int(c->itype);
  if (n <= kRangeMax) return launch_few(n, c->kept, N1, F1, N2, F2, nt, it, scale, order, least, out, w, s);
  const bool select = plan.sample && K >= kSelectMin;
  const dim3 pass_grid(unsigned((plan.tiles + 7) / 8 * 8), 2);
  const size_t pass_bytes = size_t(K) * 16;
  if (plan.sample) {
    int sample_shift = 0;
    // four a bucket, two where there are 2048 buckets; more where buckets are large on average, as one of over kBucketCap keys that are crowded
    // goes to k_bucket_sort_rest in several rounds (262144 blocks of an image: 114 us with four, 62 with sixteen; where no bucket is like
    // that, more samples cost 2 to 5 us)
    const int per_bucket = n > int64_t(K) * 1400 ? 16 : (n > int64_t(K) * 1100 ? 8 : 4), most = K <= 256 ? 2048 : kMaxSamples;
    while ((1 << sample_shift) < (K <= 256 ? per_bucket : 4) * K && (1 << sample_shift) < most) ++sample_shift;
    constexpr int kPerGroup = kRankThreads / kRankLanes;
    static_assert(kBucketCap >= kMaxSamples, "the samples of both operands fit the keys' place");
    hipLaunchKernelGGL(k_samples, dim3(((1 << sample_shift) + 63) / 64, 2), dim3(64), 0, s, N1, F1, N2, F2, nt, it, scale, c->kept, n,
                       sample_shift, w.buf1);
    hipLaunchKernelGGL(k_splitters, dim3(((1 << sample_shift) + kPerGroup - 1) / kPerGroup, 2), dim3(kRankThreads), 0, s, w.buf1, K,
                       w.splitters, 1 << sample_shift);
    hipLaunchKernelGGL(k_means<true>, pass_grid, dim3(kPassThreads), pass_bytes, s, N1, F1, N2, F2, nt, it, scale, n, plan.tile_keys,
                       plan.tiles, c->kept, K, w.splitters, w.buf0, w.hist, w.rest, w.partials, nullptr);
  } else {
    hipLaunchKernelGGL(k_means<false>, pass_grid, dim3(kPassThreads), 0, s, N1, F1, N2, F2, nt, it, scale, n, plan.tile_keys,
                       plan.tiles, c->kept, K, w.splitters, w.buf0, w.hist, w.rest, w.partials, nullptr);
  }
  const int scan_groups = plan.sample ? (2 * K + 63) / 64 : 0;
  hipLaunchKernelGGL(k_bucket_scan, dim3(scan_groups + 1, 2), dim3(64 * kScanWaves), 0, s, w.hist, plan.tiles, 2 * K, w.sums,
                     w.partials, w.params);
  int st = hip_status(hipGetLastError());
  if (st != PBZ_OK) return st;
  if (plan.sample) {
    if (select) {
      static_assert(2 * (kSampleSortMax / kBucketKeys) <= 4 * kSelectThreads, "four buckets a thread are all");
      const auto k = 2 * K <= kSelectThreads ? k_select<1> : (2 * K <= 2 * kSelectThreads ? k_select<2> : k_select<4>);
      hipLaunchKernelGGL(k, dim3(1), dim3(kSelectThreads), 0, s, n, K, w.splitters, w.sums, w.params, least, w.gap, w.needed, w.ranks);
    }
    hipLaunchKernelGGL(k_scatter, pass_grid, dim3(kPassThreads), pass_bytes, s, w.buf0, w.buf1, n, plan.tile_keys, plan.tiles, K,
                       w.splitters, w.hist, w.sums, select ? w.gap : nullptr);
    hipLaunchKernelGGL(k_bucket_sort, dim3(K, 2), dim3(kBucketThreads), 0, s, w.buf1, w.buf0, n, K, w.sums, w.rest,
                       w.pieces, select ? w.needed : nullptr);
    hipLaunchKernelGGL(k_bucket_sort_rest, dim3(2 * K < kRestGroups ? 2 * K : kRestGroups), dim3(kBucketThreads), 0, s, w.buf1,
                       w.buf0, n, K, w.sums, w.rest, w.pieces);
  } else {
    const int64_t n_tiles = (n + kTileKeys - 1) / kTileKeys;
    uint64_t* src = w.buf0;
    uint64_t* dst = w.buf1;
    for (int pass = 0; pass < 64 / kRadixBits; ++pass) {      // an even number: the sorted keys are back in buf0
      const int shift = pass * kRadixBits;
      hipLaunchKernelGGL(k_radix_hist, dim3(unsigned(n_tiles), 2), dim3(kSortThreads), 0, s, src, n, n_tiles, shift, w.hist);
      hipLaunchKernelGGL(k_scan_digit, dim3(kBins, 2), dim3(kSortThreads), 0, s, w.hist, n_tiles, w.sums);
      hipLaunchKernelGGL(k_radix_scatter, dim3(unsigned(n_tiles), 2), dim3(kSortThreads), 0, s, src, dst, n, n_tiles, shift,
                         w.hist, w.sums);
      uint64_t* t = src;
      src = dst;
      dst = t;
    }
  }
  st = hip_status(hipGetLastError());
  if (st != PBZ_OK) return st;
  hipLaunchKernelGGL(k_distance, dim3(groups), dim3(kThreads), 0, s, w.buf0, n, chunk, w.params, order, least,
                     select ? reinterpret_cast<const Selection*>(w.gap + 2) : nullptr, w.ranks, w.partials);
  hipLaunchKernelGGL(k_distance_final, dim3(1), dim3((groups + 63) / 64 * 64), 0, s, w.partials, groups, double(n), order, out);
  return hip_status(hipGetLastError());
}

}  // namespace pbz
