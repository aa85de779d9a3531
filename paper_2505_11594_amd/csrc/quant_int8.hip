// INT8 per-block quantization psi for the 8-bit attention of SageBwd
// (Algorithms 2 and 3; Sec. 4.1, Eq. psi) on gfx950.
//
// One scale s = max|X| / 127 per block of R consecutive rows with all D
// channels -- R = 128 query rows for Q and dO (the attention kernels' query
// tile), the KV tile (128 or 64 rows) for K and V -- and codes round(x * fl32(1/s)) to the
// nearest integer, ties to even; an all-zero block gets s = 0 and zero codes.
// K is smoothed first: K' = fl32(K - mean_t K) with the exact mean of the
// FP4 path's k-mean kernels.
//
// Layouts: Q^ [BH, N, D] and K^ [BH, Np, D] token-major (rows >= N of K^ are
// zero); V^T [BH, D, Np] transposed, the tokens of every 32-token group
// stored in the order in which the int8 MFMA of P.V receives P from the
// accumulator of S^T = K^ Q^T: position 16h + 4g + r holds token 8g + 4h + r.
// The backward stores Q^, K^ and dO^ transposed the same way (the A operands
// of dK^T = Q^T dS^, dQ^T = K^T dS^T and dV^T = dO^T P^).
//
// One workgroup per block of rows: each thread owns 8 channels of up to 8 rows
// (one 16-byte load each), the block max is reduced across the wave and through
// LDS, and the codes are formed by one add of 1.5 * 2^23, whose fp32 rounding
// is the round-to-nearest-even to an integer (the code is the low byte).  A
// tensor needed in both layouts (the backward's Q and K) is read once; the
// transpose goes through LDS a dword (four rows of one channel) at a time, on
// padded rows.  HBM-bound on large calls, launch-bound on small ones.
#include <algorithm>
#include <climits>

#include "kmean.h"
#include "sage_common.h"

namespace sage {

constexpr int I8Q_THREADS = 256;
constexpr float kRoundMagic = 12582912.0f;   // 1.5 * 2^23

// V^T storage position of token offset o inside its 32-token group
__device__ __forceinline__ int i8_v_pos(int o) {
  const int g = o >> 3, h = (o >> 2) & 1, r = o & 3;
  return (h << 4) | (g << 2) | r;
}

// the low bytes of four rounded values, packed (element 0 in the low byte)
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0C0C0400u);   // [a.b0, b.b0, 0, 0]
  const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0C0C0400u);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100u);              // [a, b, c, d]
}

constexpr int I8_TRS = 33;   // dwords per channel row of the transpose buffer (128 rows, padded)

template <int D>
union I8qLds {
  uint32_t tr[D * I8_TRS];
  KmRed km;
};

// What a block is read and written as.  ROWS: codes [BH, Nrow, D] row-major;
// COLS: codes [BH, D, Np], tokens permuted per 32.  MEAN: m8 is subtracted first.
// DROW: also D_q = sum_d x[q,d] o[q,d] (fp32) and Lb_q = lse_q log2(e) per row
// (x is dO, o the forward's output), 0 for rows N .. Np - 1.
struct I8Block {
  const uint16_t* x;
  int8_t *rows, *cols;
  float* scales;
  const float *o, *lse;
  float *drow, *lb;
  int N, Nrow, Np, R, nb;
};

template <int D, bool BF16, bool ROWS, bool COLS, bool MEAN, bool DROW>
__device__ __forceinline__ void quant_i8_block(const I8Block& a, const float (&m8)[8], int b, int bh,
                                               uint32_t (&tr)[D * I8_TRS]) {
  constexpr int UPR = D / 8;                      // 16-byte units per row
  constexpr int RSTEP = I8Q_THREADS / UPR;        // rows covered by one pass of the workgroup
  constexpr int MAXU = 128 / RSTEP;               // passes for R = 128
  const int tid = threadIdx.x, cg = tid % UPR, rsub = tid / UPR;   // this thread's channels [8 cg, +8)
  const int r0 = b * a.R;
  // row of pass u; four consecutive rows per thread where they become one dword of the transpose
  auto row_of = [&](int u) { return COLS ? 4 * (rsub + RSTEP * (u >> 2)) + (u & 3) : rsub + u * RSTEP; };
  uint4 raw[MAXU];
#pragma unroll
  for (int u = 0; u < MAXU; ++u) {
    const int row = row_of(u), t = r0 + row;
    raw[u] = row < a.R && t < a.N ? *reinterpret_cast<const uint4*>(a.x + ((size_t)bh * a.N + t) * D + cg * 8)
                                  : make_uint4(0, 0, 0, 0);
  }
  float v[MAXU][8];
  float amax = 0.0f;
#pragma unroll
  for (int u = 0; u < MAXU; ++u) {
    const int row = row_of(u), t = r0 + row;
    const bool in = row < a.R && t < a.N;
    const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw[u]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float x = widen<BF16>(h[i]);
      if (MEAN) x = in ? x - m8[i] : 0.0f;
      v[u][i] = x;
      amax = __builtin_fmaxf(amax, __builtin_fabsf(x));
    }
    if constexpr (DROW) {
      float s = 0.0f;
      if (in) {
        const float* op = a.o + ((size_t)bh * a.N + t) * D + cg * 8;
        const float4 o0 = *reinterpret_cast<const float4*>(op), o1 = *reinterpret_cast<const float4*>(op + 4);
        const float ov[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) s = __builtin_fmaf(v[u][i], ov[i], s);
      }
#pragma unroll
      for (int off = UPR / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (cg == 0) {
        a.drow[(size_t)bh * a.Np + t] = s;
        a.lb[(size_t)bh * a.Np + t] = in ? a.lse[(size_t)bh * a.N + t] * 1.44269504088896340736f : 0.0f;
      }
    }
  }
  // block max: across the wave, then across the 4 waves
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) amax = __builtin_fmaxf(amax, __shfl_xor(amax, off, 64));
  float* red = reinterpret_cast<float*>(tr);
  if ((tid & 63) == 0) red[tid >> 6] = amax;
  __syncthreads();
  amax = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
  const float s = amax / 127.0f;                  // correctly rounded division
  const float r = amax > 0.0f ? 1.0f / s : 0.0f;  // a zero block: codes 0
  if (tid == 0) a.scales[(size_t)bh * a.nb + b] = s;
  if (COLS) __syncthreads();                      // the maxima are read before the transpose overwrites them

#pragma unroll
  for (int u0 = 0; u0 < MAXU; u0 += 4) {
    uint32_t w[4][8];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 8; ++i) w[k][i] = __float_as_uint(v[u0 + k][i] * r + kRoundMagic);
    if constexpr (ROWS) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = row_of(u0 + k), t = r0 + row;
        if (row < a.R && t < a.Nrow)
          *reinterpret_cast<uint2*>(a.rows + ((size_t)bh * a.Nrow + t) * D + cg * 8) =
              make_uint2(pack_low_bytes(w[k][0], w[k][1], w[k][2], w[k][3]), pack_low_bytes(w[k][4], w[k][5], w[k][6], w[k][7]));
      }
    }
    if constexpr (COLS) {
      const int row = row_of(u0);                 // rows row .. row + 3: one dword of each channel
      if (row < a.R) {
        const int q = ((row & ~31) | i8_v_pos(row & 31)) / 4;
#pragma unroll
        for (int i = 0; i < 8; ++i) tr[(cg * 8 + i) * I8_TRS + q] = pack_low_bytes(w[0][i], w[1][i], w[2][i], w[3][i]);
      }
    }
  }
  if constexpr (COLS) {
    __syncthreads();
    const int dw = a.R / 4, sh = a.R == 128 ? 5 : 4;      // dwords per channel row, log2
    for (int idx = tid; idx < D * dw; idx += I8Q_THREADS) {
      const int c = idx >> sh, q = idx & (dw - 1);
      *reinterpret_cast<uint32_t*>(a.cols + ((size_t)bh * D + c) * a.Np + r0 + 4 * q) = tr[c * I8_TRS + q];
    }
  }
}

// Q or another tensor without a mean
template <int D, bool BF16, bool ROWS, bool COLS, bool DROW>
__global__ __launch_bounds__(I8Q_THREADS) void quant_i8_kernel(const I8Block a) {
  __shared__ uint32_t tr[D * I8_TRS];
  const float m8[8] = {};
  quant_i8_block<D, BF16, ROWS, COLS, false, DROW>(a, m8, blockIdx.x, blockIdx.y, tr);
}

// K: the mean is read from mu, or (part given) summed here; mu null: none is subtracted.
template <int D, bool BF16, bool COLS>
__global__ __launch_bounds__(I8Q_THREADS) void quant_i8_k_kernel(const I8Block a, const double* __restrict__ part,
                                                                 float* __restrict__ mu, int nchunk) {
  __shared__ uint32_t tr[D * I8_TRS];
  __shared__ float mean[D];
  const int b = blockIdx.x, bh = blockIdx.y, cg = threadIdx.x % (D / 8);
  float m8[8];
  if (part != nullptr) kmean_inline<D>(part, mu, a.N, nchunk, bh, b == 0, mean);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    m8[i] = mu == nullptr ? 0.0f : part != nullptr ? mean[cg * 8 + i] : mu[(size_t)bh * D + cg * 8 + i];
  quant_i8_block<D, BF16, true, COLS, true, false>(a, m8, b, bh, tr);
}

// Everything that does not depend on the K mean in one launch, for calls whose
// passes are too short to fill the GPU one by one: blocks of tensor a, of tensor
// b, then the K mean's partial sums.  Forward: a = V (COLS), b = Q (ROWS);
// backward: a = dO (COLS, DROW), b = Q (both).
template <int D, bool BF16, bool BWD>
__global__ __launch_bounds__(I8Q_THREADS) void i8_prep_kernel(const I8Block a, const I8Block b, int na, int nbq,
                                                              const uint16_t* __restrict__ k, double* __restrict__ part,
                                                              int nchunk) {
  __shared__ I8qLds<D> lds;
  const float m8[8] = {};
  int w = blockIdx.x;
  if (w < na) {
    quant_i8_block<D, BF16, false, true, false, BWD>(a, m8, w % a.nb, w / a.nb, lds.tr);
    return;
  }
  w -= na;
  if (w < nbq) {
    quant_i8_block<D, BF16, true, BWD, false, false>(b, m8, w % b.nb, w / b.nb, lds.tr);
    return;
  }
  w -= nbq;
  kmean_partial<D, BF16>(k, part, a.N, nchunk, w % nchunk, w / nchunk, lds.km);
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
template <typename F>
static hipError_t i8_dispatch(int D, bool bf16, F&& f) {
  if (D == 128) return bf16 ? f(ic<128>{}, ic<1>{}) : f(ic<128>{}, ic<0>{});
  return bf16 ? f(ic<64>{}, ic<1>{}) : f(ic<64>{}, ic<0>{});
}

static I8Block i8_block(const void* x, void* rows, void* cols, float* scales, int N, int Nrow, int Np, int R, int nb) {
  I8Block a = {};
  a.x = (const uint16_t*)x; a.rows = (int8_t*)rows; a.cols = (int8_t*)cols; a.scales = scales;
  a.N = N; a.Nrow = Nrow; a.Np = Np; a.R = R; a.nb = nb;
  return a;
}

template <bool ROWS, bool COLS, bool DROW>
static hipError_t launch_i8_tensor(const I8Block& a, int BH, int D, bool bf16, hipStream_t st) {
  return i8_dispatch(D, bf16, [&](auto D_, auto B_) {
    hipLaunchKernelGGL((quant_i8_kernel<decltype(D_)::value, decltype(B_)::value != 0, ROWS, COLS, DROW>),
                       dim3((unsigned)a.nb, (unsigned)BH), dim3(I8Q_THREADS), 0, st, a);
    return hipGetLastError();
  });
}

template <bool COLS>
static hipError_t launch_i8_k_rows(const I8Block& a, const double* part, float* mu, int BH, int D, bool bf16, hipStream_t st) {
  const int nchunk = kmean_chunks(a.N);
  if (part != nullptr && nchunk > KM_INLINE) {
    const hipError_t e = launch_kmean_final(part, mu, BH, a.N, D, st);
    if (e != hipSuccess) return e;
    part = nullptr;
  }
  return i8_dispatch(D, bf16, [&](auto D_, auto B_) {
    hipLaunchKernelGGL((quant_i8_k_kernel<decltype(D_)::value, decltype(B_)::value != 0, COLS>),
                       dim3((unsigned)a.nb, (unsigned)BH), dim3(I8Q_THREADS), 0, st, a, part, mu, nchunk);
    return hipGetLastError();
  });
}

// Q: codes [BH, N, D], blocks of 128 rows.
hipError_t launch_quant_i8_q(const void* q, void* codes, float* scales, int BH, int N, int D, bool bf16, hipStream_t st) {
  return launch_i8_tensor<true, false, false>(i8_block(q, codes, nullptr, scales, N, N, 0, 128, (N + 127) / 128), BH, D, bf16, st);
}
// V: codes [BH, D, Np], blocks of R rows.
hipError_t launch_quant_i8_v(const void* v, void* codes, float* scales, int BH, int N, int Np, int D, int R, bool bf16,
                             hipStream_t st) {
  return launch_i8_tensor<false, true, false>(i8_block(v, nullptr, codes, scales, N, 0, Np, R, Np / R), BH, D, bf16, st);
}
// K: codes [BH, Np, D], blocks of R rows; part and mu null without smoothing.
hipError_t launch_quant_i8_k(const void* k, double* part, float* mu, void* codes, float* scales, int BH, int N, int Np,
                             int D, int R, bool bf16, hipStream_t st) {
  if (mu != nullptr) {
    const hipError_t e = launch_kmean_partial(k, part, BH, N, D, bf16, st);
    if (e != hipSuccess) return e;
  }
  return launch_i8_k_rows<false>(i8_block(k, codes, nullptr, scales, N, Np, Np, R, Np / R), mu ? part : nullptr, mu, BH, D,
                                 bf16, st);
}

// Up to this many elements (BH Np D) the tensors share a launch, the FP4 quantizers'
// line.  Forward, D = 128, in us, apart -> shared: 4 heads x 1024 40.5 -> 33.3, 64 x
// 1024 (2^23) 70.2 -> 60.2, 32 x 4096 (2^24) 243 -> 237; backward 111 -> 95, 198 -> 181,
// 959 -> 953.  (Here sharing still gains past it: 256 x 1024, 2^25, 193 -> 185 and
// 673 -> 655; 512 x 1024, 2^26, 370 -> 364 and 1283 -> 1267.)
constexpr long long I8_PREP_MAX_ELEMS = 1LL << 24;

template <bool BWD>
static hipError_t launch_i8_prep(const I8Block& a, const I8Block& b, const void* k, double* part, bool smooth, int BH, int D,
                                 bool bf16, hipStream_t st) {
  if ((long long)BH * a.Np * D > I8_PREP_MAX_ELEMS) {
    hipError_t e = launch_i8_tensor<false, true, BWD>(a, BH, D, bf16, st);
    if (e == hipSuccess) e = launch_i8_tensor<true, BWD, false>(b, BH, D, bf16, st);
    if (e == hipSuccess && smooth) e = launch_kmean_partial(k, part, BH, a.N, D, bf16, st);
    return e;
  }
  const int nchunk = kmean_chunks(a.N), na = a.nb * BH, nb = b.nb * BH, nk = smooth ? nchunk * BH : 0;
  return i8_dispatch(D, bf16, [&](auto D_, auto B_) {
    hipLaunchKernelGGL((i8_prep_kernel<decltype(D_)::value, decltype(B_)::value != 0, BWD>), dim3((unsigned)(na + nb + nk)),
                       dim3(I8Q_THREADS), 0, st, a, b, na, nb, (const uint16_t*)k, part, nchunk);
    return hipGetLastError();
  });
}

// The forward's Q, K and V (K and V in blocks of R rows); part and mu null without smoothing.
hipError_t launch_quant_i8_qkv(const void* q, const void* k, const void* v, void* qc, float* qs, void* kc, float* ks,
                               void* vc, float* vs, double* part, float* mu, int BH, int N, int Np, int D, int R,
                               bool bf16, hipStream_t st) {
  const I8Block a = i8_block(v, nullptr, vc, vs, N, 0, Np, R, Np / R);
  const I8Block b = i8_block(q, qc, nullptr, qs, N, N, Np, 128, (N + 127) / 128);
  const hipError_t e = launch_i8_prep<false>(a, b, k, part, mu != nullptr, BH, D, bf16, st);
  if (e != hipSuccess) return e;
  return launch_i8_k_rows<false>(i8_block(k, kc, nullptr, ks, N, Np, Np, R, Np / R), mu ? part : nullptr, mu, BH, D, bf16, st);
}

// The backward's operands, all in blocks of 128 rows: Q and K in both layouts, dO
// transposed, D_q and Lb_q [BH, Np] (o: the forward's output, lse its L).
hipError_t launch_quant_i8_bwd(const void* q, const void* k, const void* dout, const float* o, const float* lse, void* qc,
                               float* qs, void* qt, void* kc, float* ks, void* kt, void* gt, float* gs, float* drow,
                               float* lb, double* part, float* mu, int BH, int N, int Np, int D, bool bf16,
                               hipStream_t st) {
  I8Block a = i8_block(dout, nullptr, gt, gs, N, 0, Np, 128, Np / 128);
  a.o = o; a.lse = lse; a.drow = drow; a.lb = lb;
  const I8Block b = i8_block(q, qc, qt, qs, N, N, Np, 128, Np / 128);
  const hipError_t e = launch_i8_prep<true>(a, b, k, part, mu != nullptr, BH, D, bf16, st);
  if (e != hipSuccess) return e;
  return launch_i8_k_rows<true>(i8_block(k, kc, kt, ks, N, Np, Np, 128, Np / 128), mu ? part : nullptr, mu, BH, D, bf16, st);
}

}  // namespace sage
