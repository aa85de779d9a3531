// Partial sums of smoothing K's channel mean, shared by the FP4 and the INT8 quantizers.
#pragma once
#include "sage_common.h"

namespace sage {

// ---------------------------------------------------------------------------
// Smoothing K, pass 1: per-chunk fp64 column sums.  Block (chunk, bh) sums
// tokens [chunk * KM_CHUNK, ...) of K[bh] for every channel.  The sums are exact,
// and the mean does not depend on their order, while the values' bits and the
// count fit 53: always for fp16 (40 bits of range) up to 2^13 tokens per channel
// at full range and more where it is less; for bf16 while a channel's largest and
// smallest nonzero values are within 2^(45 - log2 N).  Beyond that each addition
// rounds to 2^-53 of the partial sum.
// ---------------------------------------------------------------------------
constexpr int KM_CHUNK = 512;
constexpr int KM_THREADS = 256;

typedef double KmRed[KM_THREADS][9];         // padded against bank conflicts

template <int D, bool BF16>
__device__ __forceinline__ void kmean_partial(const uint16_t* __restrict__ k, double* __restrict__ part, int N,
                                              int nchunk, int chunk, int bh, KmRed& red) {
  constexpr int CG = D / 8;                  // 8-channel groups per row (16 bytes)
  constexpr int RS = KM_THREADS / CG;        // rows handled in parallel
  const int tid = threadIdx.x;
  const int cg = tid % CG, rsub = tid / CG;
  const int t0 = chunk * KM_CHUNK;
  const int t1 = min(N, t0 + KM_CHUNK);
  const uint16_t* kb = k + (size_t)bh * N * D;
  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.0;
  for (int t = t0 + rsub; t < t1; t += RS) {
    uint4 raw = *reinterpret_cast<const uint4*>(kb + (size_t)t * D + cg * 8);
    const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += (double)widen<BF16>(h[i]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[tid][i] = acc[i];
  __syncthreads();
  if (tid < D) {
    const int c = tid, g = c / 8, i = c % 8;
    double s = 0.0;
    for (int r = 0; r < RS; ++r) s += red[r * CG + g][i];
    part[((size_t)bh * nchunk + chunk) * D + c] = s;
  }
}

// Partial sums of up to this many chunks are added by K's quantizer itself
// (each of its workgroups reads them all), more by a pass of their own.  A call
// in us, pass of its own -> inline: 4 heads x 1024, D = 128 (2 chunks) 22.5 ->
// 20.8, D = 64 21.2 -> 18.8, 4 x 4096 (8), D = 128 44.7 -> 42.6, 32 x 4096, D = 64
// 124.2 -> 122.9 (D = 128 170.1 -> 170.9, 128 x 4096 619 -> 622).  With up to 64
// inline the loads of a short sum cost more (32 x 4096 175.6, 128 x 4096 641) and the
// long ones gain nothing: 4 x 8192 (16) 100.7 -> 100.4, 32 x 8192 550 -> 559, 8 x
// 32768 (64) 1955 -> 1977.
constexpr int KM_INLINE = 8;

// mean[c] = fl32(sum of the head's partial sums / N), by the first D threads;
// `store`: also into mu[bh].  Ends with a barrier.
template <int D>
__device__ __forceinline__ void kmean_inline(const double* __restrict__ part, float* __restrict__ mu, int N, int nchunk,
                                             int bh, bool store, float (&mean)[D]) {
  const int tid = threadIdx.x;
  if (tid < D) {
    double p[KM_INLINE], s = 0.0;                // all loads in flight before the first sum (nchunk <= KM_INLINE)
#pragma unroll
    for (int j = 0; j < KM_INLINE; ++j) p[j] = part[((size_t)bh * nchunk + min(j, nchunk - 1)) * D + tid];
#pragma unroll
    for (int j = 0; j < KM_INLINE; ++j)
      if (j < nchunk) s += p[j];
    const float m = (float)(s / (double)N);
    mean[tid] = m;
    if (store) mu[(size_t)bh * D + tid] = m;
  }
  __syncthreads();
}

int kmean_chunks(int N);
hipError_t launch_kmean_partial(const void* k, double* part, int BH, int N, int D, bool bf16, hipStream_t st);
hipError_t launch_kmean_final(const double* part, float* mu, int BH, int N, int D, hipStream_t st);

}  // namespace sage
