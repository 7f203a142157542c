// Compressed-space operations straight from memory, element by element: any kept count, any alignment, any type at run time.
// For the sizes at which putting blocks through LDS (pbz_ops_staged.hip) costs more than it saves: few blocks, where a
// call is one memory round trip and the launch, and sums of blocks so large that LDS holds one wave's only.  The rules and both sides' times
// are with direct_rebin, direct_blockwise and direct_reduction.
#include "pbz_ops_common.h"

namespace pbz {
namespace ops {
namespace {

// Algorithms 2 and 4, one wave per block.  kTwo: C = F1 N1 + F2 (sign2 N2), N = max|C| / r, F = rint(C / N); otherwise
// C = N1 F1 / r, the first one moved by `shift`, N = max|C|, F = rint(C r / N).
template <bool kTwo>
__global__ __launch_bounds__(64) void k_rebin_direct(const void* N1, const void* F1, const void* N2, const void* F2, void* Nout,
                                                     void* Fout, int ntype, int itype, double r, double sign2, double shift,
                                                     int64_t n_blocks, int kept) {
  for (int64_t k = blockIdx.x; k < n_blocks; k += gridDim.x) {
    const double n1 = load_float<double>(N1, ntype, k), n2 = kTwo ? sign2 * load_float<double>(N2, ntype, k) : 0.0;
    auto coefficient = [&](int j) {
      const double f1 = double(load_index(F1, itype, k * kept + j));
      if (kTwo) return unfused_sum_of_products(f1, n1, double(load_index(F2, itype, k * kept + j)), n2);
      return (n1 * f1) / r + (j == 0 ? shift : 0.0);
    };
    double m = 0.0;
    for (int j = threadIdx.x; j < kept; j += 64) m = fmax(m, fabs(coefficient(j)));
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    const double n = kTwo ? m / r : m;
    // F_out may alias an operand: every lane re-reads only the entries it then overwrites
    for (int j = threadIdx.x; j < kept; j += 64) {
      const double c = coefficient(j);
      const double t = n > 0.0 ? (kTwo ? c : c * r) / n : 0.0;
      store_index(Fout, itype, k * kept + j, int64_t(fmin(fmax(rint(t), -r), r)));
    }
    if (threadIdx.x == 0) store_float(Nout, ntype, k, n);
  }
}

// one wave per block
__global__ __launch_bounds__(64) void k_blockwise_direct(const void* __restrict__ N1, const void* __restrict__ F1,
                                                         const void* __restrict__ N2, const void* __restrict__ F2, int ntype,
                                                         int itype, double* __restrict__ out, double scale, int mode,
                                                         int64_t n_blocks, int kept) {
  for (int64_t k = blockIdx.x; k < n_blocks; k += gridDim.x) {
    double sum = 0.0;
    for (int j = 1 + threadIdx.x; j < kept; j += 64)
      sum += double(load_index(F1, itype, k * kept + j)) * double(load_index(F2, itype, k * kept + j));
    sum = wave_sum(sum);
    if (threadIdx.x == 0) {
      double res = sum * (load_float<double>(N1, ntype, k) * load_float<double>(N2, ntype, k)) * scale;
      if (mode == kBwStd) res = sqrt(res);
      out[k] = res;
    }
  }
}

// the five sums of a reduction, one thread per block; grid y = segment of n_blocks blocks
__global__ __launch_bounds__(kThreads) void k_reduce_direct(const void* __restrict__ N1, const void* __restrict__ F1,
                                                            const void* __restrict__ N2, const void* __restrict__ F2, int ntype,
                                                            int itype, int64_t n_blocks, int kept, int dc, int diff, ReduceTail tail) {
  double sums[kNumSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int64_t nthreads = int64_t(gridDim.x) * kThreads;
  const int64_t k0 = int64_t(blockIdx.y) * n_blocks;     // first block of this segment
  const double K1 = dc ? pilot_value(tail.pilot_n1, tail.pilot_f1, tail, blockIdx.y) : 0.0;
  const double K2 = dc ? pilot_value(tail.pilot_n2, tail.pilot_f2, tail, blockIdx.y) : 0.0;
  for (int64_t kk = int64_t(blockIdx.x) * kThreads + threadIdx.x; kk < n_blocks; kk += nthreads) {
    const int64_t k = k0 + kk;
    const double n1 = load_float<double>(N1, ntype, k);
    const double n2 = load_float<double>(N2, ntype, k);
    if (diff) {
      double acc = 0.0;
      for (int j = 0; j < kept; ++j) {
        const double d = n1 * double(load_index(F1, itype, k * kept + j)) - n2 * double(load_index(F2, itype, k * kept + j));
        acc += d * d;
      }
      sums[kS11] += acc;
      continue;
    }
    double s11 = 0.0, s12 = 0.0, s22 = 0.0;
    for (int j = dc ? 1 : 0; j < kept; ++j) {       // dc: the first coefficient enters shifted, below
      const double f1 = double(load_index(F1, itype, k * kept + j));
      const double f2 = double(load_index(F2, itype, k * kept + j));
      s11 += f1 * f1;
      s12 += f1 * f2;
      s22 += f2 * f2;
    }
    sums[kS11] += s11 * (n1 * n1);
    sums[kS12] += s12 * (n1 * n2);
    sums[kS22] += s22 * (n2 * n2);
    if (dc) {
      const double d1 = n1 * double(load_index(F1, itype, k * kept)) - K1;
      const double d2 = n2 * double(load_index(F2, itype, k * kept)) - K2;
      sums[kS11] += d1 * d1;
      sums[kS12] += d1 * d2;
      sums[kS22] += d2 * d2;
      sums[kD1] += d1;
      sums[kD2] += d2;
    }
  }
  reduce_tail(sums, tail, K1, K2);
}

dim3 wave_per_block(int64_t n_blocks) { return dim3(unsigned(n_blocks < 65536 ? n_blocks : 65536)); }

}  // namespace

int launch_rebin_direct(const pbz_codec* c, int64_t n_blocks, const void* N1, const void* F1, const void* N2, const void* F2,
                        void* Nout, void* Fout, double sign2, double shift, hipStream_t s) {
  if (F2)
    hipLaunchKernelGGL(k_rebin_direct<true>, wave_per_block(n_blocks), dim3(64), 0, s, N1, F1, N2, F2, Nout, Fout, int(c->ftype),
                       int(c->itype), c->r, sign2, shift, n_blocks, c->kept);
  else
    hipLaunchKernelGGL(k_rebin_direct<false>, wave_per_block(n_blocks), dim3(64), 0, s, N1, F1, N2, F2, Nout, Fout, int(c->ftype),
                       int(c->itype), c->r, sign2, shift, n_blocks, c->kept);
  return hip_status(hipGetLastError());
}

int launch_blockwise_direct(const pbz_codec* c, int mode, int64_t n_blocks, const void* N1, const void* F1, const void* N2,
                            const void* F2, double* out, double scale, hipStream_t s) {
  hipLaunchKernelGGL(k_blockwise_direct, wave_per_block(n_blocks), dim3(64), 0, s, N1, F1, N2, F2, int(c->ftype), int(c->itype),
                     out, scale, mode, n_blocks, c->kept);
  return hip_status(hipGetLastError());
}

int launch_reduce_direct(const pbz_codec* c, bool /*two*/, bool dc, bool diff, int64_t n_blocks, int n_segments, int max_groups,
                         const void* N1, const void* F1, const void* N2, const void* F2, const ReduceTail& tail, int* groups,
                         hipStream_t s) {
  int g = stream_groups(n_blocks, 1);
  if (g > max_groups) g = max_groups;
  *groups = g;
  hipLaunchKernelGGL(k_reduce_direct, dim3(g, n_segments), dim3(kThreads), 0, s, N1, F1, N2, F2, int(c->ftype), int(c->itype),
                     n_blocks, c->kept, dc ? 1 : 0, diff ? 1 : 0, tail);
  return hip_status(hipGetLastError());
}

}  // namespace ops
}  // namespace pbz
