// Second stage of the per-tensor reductions: the sums of the statistics pass's partials and what follows from them. One
// workgroup of k_finalize per tensor, or every workgroup of the strip apply kernel for its own tensor (short lists).
#pragma once

#include "lopt_device.h"
#include "lopt_internal.h"

namespace lopt {

// Adds part[0], part[stride], ... (count terms, 1..B) in double, in index order, term k to acc[k % NS]: B loads issue ahead of
// the adds, those past the end repeat the last term and are dropped.
template <int B, int NS, typename P>
__device__ __forceinline__ void sum_batch(const P* __restrict__ part, int count, size_t stride, double (&acc)[NS]) {
  P t[B];
#pragma unroll
  for (int k = 0; k < B; ++k) t[k] = part[(size_t)min(k, count - 1) * stride];
#pragma unroll
  for (int k = 0; k < B; ++k) acc[k % NS] += k < count ? (double)t[k] : 0.0;
}

// Sums of part[0], part[stride], ... (count terms) in double, always in index order, as NS interleaved sums. Bound by load
// latency: full batches of B loads (32 registers of them), then one batch of the power of two that holds the rest.
template <int NS, typename P>
__device__ __forceinline__ void strided_sums(const P* __restrict__ part, int count, size_t stride, double (&acc)[NS]) {
  constexpr int B = 128 / sizeof(P);
  static_assert(NS <= B && B % NS == 0, "every full batch holds whole rounds of the NS sums");
#pragma unroll
  for (int k = 0; k < NS; ++k) acc[k] = 0.0;
  for (; count > B; count -= B, part += B * stride) sum_batch<B>(part, B, stride, acc);
  if (count > 16) sum_batch<B>(part, count, stride, acc);
  else if (count > 8) sum_batch<16>(part, count, stride, acc);
  else if (count > 4) sum_batch<8>(part, count, stride, acc);
  else if (count > 1) sum_batch<4>(part, count, stride, acc);
  else if (count == 1) acc[0] += (double)part[0];
}

template <typename P>
__device__ __forceinline__ double strided_sum(const P* __restrict__ part, int count, size_t stride) {
  double acc[1];
  strided_sums(part, count, stride, acc);
  return acc[0];
}

// Reduces every partial of a tensor in a fixed order (double accumulation) to s_f and the per-feature scale factors. The 32 sums
// (17 statistics over the tiles, 9 over the row blocks, 6 over the column blocks) are one column of threads each, cut into 32
// interleaved segments: this is a chain of load latencies, and this way it is one batch of loads for up to 1024 tiles
// (k_finalize, 1000x1000: 7.9 -> 4.8 us from eight segments and three such phases; six tensors of 0.3 M elements 5.2 -> 4.9 us).
// A workgroup of 256 threads forms four segments per thread: the order of summation does not depend on the launch.
constexpr int kFinSegs = 32;
constexpr int kFinPerThread = kFinSegs / (kBlock / 32);
static_assert(kFinPerThread == 4, "a narrow workgroup takes four segments per thread");
struct FinLds {
  double part[kFinSegs][32], tot[32];
  float stats[32], scale[32];
};

// s_f and scale of feature f < 32 from the tensor's 32 sums. tot: 0..16 statistics; 17..19 sum r, 20..22 sum r^2, 23..25
// sum 1/(r+eps); 26..28 sum c^2, 29..31 sum 1/(c+eps). The kinds of feature differ in what they select, not in a branch: a branch per
// kind, each with a division in double of its own, was a third of the kernel's time on a short list.
__device__ __forceinline__ void feature_scale(const TensorDev& T, const StepArgs& A, const double* tot, int f, float& sf, float& scale) {
  const double m = (double)T.m, n = (double)T.n;
  const bool fac = (f >= 10 && f < 13) || (f >= 25 && f < 28), clip = f == 28;
  const int k = fac ? (f < 13 ? f - 10 : f - 25) : 0;
  const int q = f < 13 ? f : f < 16 ? 20 + (f - 13) : f < 19 ? 26 + (f - 16) : f < 22 ? 23 + (f - 19) : f < 25 ? 29 + (f - 22)
              : f < 28 ? f - 12 : clip ? 16 : 0;
  const bool row = (f >= 13 && f < 16) || (f >= 19 && f < 22), col = (f >= 16 && f < 19) || (f >= 22 && f < 25);
  const double rbar = tot[17 + k] / m + (double)A.eps_acc;
  double s = tot[q] / (row ? m : col ? n : m * n);
  s = fac ? s * rbar : s;
  s = f < 29 ? s : 0.0;
  const double pre = fac ? sqrt(rbar) : 1.0;  // factor between the raw feature the kernels build and the feature itself
  sf = (float)s;
  scale = (float)(pre / sqrt((double)sf + (double)A.eps_norm));
}

// Where sum q of a tensor finds its terms.
struct FinTerms { const float* base; int count, stride; };
__device__ __forceinline__ FinTerms fin_terms(const TensorDev& T, const float* ws, int q) {
  if (q < kNStat) return FinTerms{ws + T.oStatPart + q, T.nrt * T.nct, kStatStride};
  if (q < 26) return FinTerms{ws + T.oRcPart + (q - kNStat), T.nrpart, kRcStride};
  return FinTerms{ws + T.oRcPart + (size_t)T.nrpart * kRcStride + (q - 26 + 3), T.ncpart, kRcStride};
}

// Sum of the 32 segments of one sum, in a fixed order: part[0], part[32], ...
__device__ __forceinline__ double segment_sum(const double* part) {
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kFinSegs; ++k) s[k % 4] += part[32 * k];
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Called by all threads (1024 or 256). L.stats and L.scale are ready for all of them afterwards; store: to the workspace too.
__device__ __forceinline__ void finalize_scales(const TensorDev& T, float* __restrict__ ws, const StepArgs& A, FinLds& L, bool store) {
  const int q = threadIdx.x & 31, seg = threadIdx.x >> 5, n_seg = blockDim.x >> 5;
  {
    const auto [base0, count, stride] = fin_terms(T, ws, q);
    const float* base = base0;
    // thread (seg, q): terms seg, seg + n_seg, ..., which are those of the segments seg, seg + n_seg, ... < 32 in turn
    const int mine = seg < count ? (count - seg + n_seg - 1) / n_seg : 0;
    base += (size_t)seg * stride;
    if (n_seg == kFinSegs) {
      L.part[seg][q] = strided_sum(base, mine, (size_t)kFinSegs * stride);
    } else {
      double a[kFinPerThread];
      strided_sums(base, mine, (size_t)n_seg * stride, a);
#pragma unroll
      for (int k = 0; k < kFinPerThread; ++k) L.part[seg + n_seg * k][q] = a[k];
    }
  }
  __syncthreads();
  if (threadIdx.x < 32) L.tot[q] = segment_sum(&L.part[0][q]);
  __syncthreads();
  if (threadIdx.x < 32) {
    const int f = threadIdx.x;
    float sf, scale;
    feature_scale(T, A, L.tot, f, sf, scale);
    L.stats[f] = sf;
    L.scale[f] = f < A.F ? scale : 0.f;
    if (store) {
      ws[T.oStats + f] = f < A.F ? sf : 0.f;
      ws[T.oScale + f] = f < A.F ? scale : 0.f;
    }
  }
  __syncthreads();
}

}  // namespace lopt
