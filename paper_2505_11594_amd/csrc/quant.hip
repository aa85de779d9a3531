// Quantization kernels for gfx950: smoothing-K mean, FP4 microscaling of Q and
// K along the head dimension, and of V along tokens with the transpose fused in.
//
// phi (Sec. 3.1, Eq. microscaling): per 1 x n block, s = max|x| / 6 stored as
// E8M0 (MXFP4, n = 32: the smallest power of two with 6 s >= max) or E4M3
// (n = 16, round to nearest even, saturating at 448); codes are FP4 E2M1
// round-to-nearest-even of x / s.  Smoothing K (Algorithm 1 preprocessing)
// subtracts the per-(b,h) channel mean first, smoothing Q (Algorithm 1) the
// mean of each block of QB query rows; the V transpose is fused into its
// quantization (Appendix, "Transposing V").  For smoothing Q the GEMV of the
// block means with K' is computed here as well.
//
// The quantizers are HBM-bound on large calls and launch-bound on small ones: each element is read once as 16 bits
// (twice for K, which the mean also reads) and written as 4 bits plus 8 bits
// per block.
#include <algorithm>
#include <climits>

#include "kmean.h"
#include "sage_common.h"

namespace sage {

template <int D, bool BF16>
__global__ __launch_bounds__(KM_THREADS) void kmean_partial_kernel(const uint16_t* __restrict__ k,
                                                                   double* __restrict__ part, int N, int nchunk) {
  __shared__ KmRed red;
  kmean_partial<D, BF16>(k, part, N, nchunk, blockIdx.x, blockIdx.y, red);
}

// Pass 2: mu = fl32(fl64(sum) / N).  One workgroup per (b,h): 256 / D
// threads per channel sum strided chunks, then one of them adds the partial
// sums.
template <int D>
__global__ __launch_bounds__(256) void kmean_final_kernel(const double* __restrict__ part, float* __restrict__ mu,
                                                          int N, int nchunk) {
  constexpr int TPC = 256 / D;
  const int bh = blockIdx.x, tid = threadIdx.x, c = tid % D, k = tid / D;
  double s = 0.0;
  for (int j = k; j < nchunk; j += TPC) s += part[((size_t)bh * nchunk + j) * D + c];
  __shared__ double red[256];
  red[tid] = s;
  __syncthreads();
  if (k == 0) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < TPC; ++i) t += red[i * D + c];
    mu[(size_t)bh * D + c] = (float)(t / (double)N);
  }
}

constexpr int QB = 128;   // query rows per smoothing block (= the attention kernel's query tile)

// GEMV of smoothing Q: bias[bh, b, k] = qbar[bh, b, :] . K'[bh, k, :] with
// K' = fl32(K - mu) (K itself without smoothing K), as a chain of fp32 fused
// multiply-adds in order of the channel from 0; keys k >= N get 0.  A
// workgroup takes GK keys and 8 WB query blocks (WB of its four waves along the
// blocks) and walks the channels GC at a time: K' and the means are staged in
// LDS channel-major, the next channels' loads in flight meanwhile.  With WB = 4
// each lane has 8 blocks x 8 keys, four 16-byte LDS reads for 64 independent
// multiply-adds (one key per thread took two for 8, and LDS reads bounded it);
// with WB = 1 one key per lane, for calls too small to fill the GPU with the
// larger tiles.  B4 H32 N4096 D128: 117 -> 100 us (its multiply-adds take 37, K
// and the result move 201 MB); B2 H8 N1000 with 512-key tiles 61 us a call, 44 so.
template <int D, bool BF16, int GK, int WB, int GC>
__global__ __launch_bounds__(256) void qk_bias_kernel(const uint16_t* __restrict__ k, const float* __restrict__ mu,
                                                      const float* __restrict__ qbar, float* __restrict__ bias, int N,
                                                      int Np, int nqb, int nkt) {
  constexpr int GB = 8 * WB, LK = GK * WB / 256, KPT = GK / 256, MPT = GB * GC / 256;
  static_assert(LK == 8 || LK == 1, "keys per lane");
  __shared__ __attribute__((aligned(16))) float kt[GC][GK];
  __shared__ __attribute__((aligned(16))) float qt[GC][GB];
  const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int key0 = (blockIdx.x % nkt) * GK, b0 = (blockIdx.x / nkt) * GB, wb = 8 * (wave % WB);
  const float* qm = qbar + ((size_t)bh * nqb + b0) * D;
  uint4 raw[KPT][GC / 8];
  float mean[MPT];
  auto load = [&](int c0) {
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      const int key = key0 + tid + 256 * e;
#pragma unroll
      for (int h8 = 0; h8 < GC / 8; ++h8)
        raw[e][h8] = key < N ? *reinterpret_cast<const uint4*>(k + ((size_t)bh * N + key) * D + c0 + 8 * h8)
                             : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < MPT; ++e) {
      const int idx = tid + 256 * e, i = idx / GC, c = idx % GC;   // block i, channel c
      mean[e] = (b0 + i < nqb) ? qm[(size_t)i * D + c0 + c] : 0.0f;
    }
  };
  float acc[8][LK];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < LK; ++j) acc[i][j] = 0.0f;
  load(0);
  for (int c0 = 0; c0 < D; c0 += GC) {
    if (c0 > 0) __syncthreads();                   // every wave is done with the previous channels
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      const bool valid = key0 + tid + 256 * e < N;
#pragma unroll
      for (int c = 0; c < GC; ++c) {
        float x = widen<BF16>(reinterpret_cast<const uint16_t*>(&raw[e][c / 8])[c % 8]);
        if (mu != nullptr) x = x - mu[(size_t)bh * D + c0 + c];
        kt[c][tid + 256 * e] = valid ? x : 0.0f;
      }
    }
#pragma unroll
    for (int e = 0; e < MPT; ++e) {
      const int idx = tid + 256 * e;
      qt[idx % GC][idx / GC] = mean[e];
    }
    __syncthreads();
    if (c0 + GC < D) load(c0 + GC);
    if (b0 + wb < nqb) {
#pragma unroll 4
      for (int c = 0; c < GC; ++c) {
        float kk[LK];
        if constexpr (LK == 8) {
          const v4f k0 = *reinterpret_cast<const v4f*>(&kt[c][4 * lane]);
          const v4f k1 = *reinterpret_cast<const v4f*>(&kt[c][256 + 4 * lane]);
#pragma unroll
          for (int j = 0; j < 8; ++j) kk[j] = j < 4 ? k0[j & 3] : k1[j & 3];
        } else {
          kk[0] = kt[c][tid];
        }
        const v4f m0 = *reinterpret_cast<const v4f*>(&qt[c][wb]);
        const v4f m1 = *reinterpret_cast<const v4f*>(&qt[c][wb + 4]);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < LK; ++j) acc[i][j] = __builtin_fmaf(i < 4 ? m0[i & 3] : m1[i & 3], kk[j], acc[i][j]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int b = b0 + wb + i;
    if (b < nqb) {
      float* row = bias + ((size_t)bh * nqb + b) * Np;
      if constexpr (LK == 8) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int key = key0 + 256 * e + 4 * lane;
          if (key < Np)
            *reinterpret_cast<v4f*>(row + key) = v4f{acc[i][4 * e], acc[i][4 * e + 1], acc[i][4 * e + 2], acc[i][4 * e + 3]};
        }
      } else if (key0 + tid < Np) {
        row[key0 + tid] = acc[i][0];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Row quantizers for Q and K (blocks along D).  One lane owns 8 consecutive
// channels (a 16-byte load); the 4 (MXFP4) or 2 (NV16) lanes of a block
// reduce their absolute maxima with cross-lane swaps.  A lane writes its 8
// codes as one 32-bit word.
// ---------------------------------------------------------------------------
// Stored row of K token t.  MXFP4 (32x32x64 block-scaled MFMA): inside each
// 64-token group, offset o = 32h + 16t' + 4g + r goes to 32t' + 8g + 4h + r.
// NV16 (32x32x16 bf16 MFMA after dequantization): inside each 32-token group,
// o = 16h + 4g + r goes to 8g + 4h + r.
template <int FMT>
__device__ __forceinline__ int k_stored_pos(int t) {
  if constexpr (FMT == kFmtMX) {
    const int o = t & 63;
    const int h = o >> 5, tt = (o >> 4) & 1, g = (o >> 2) & 3, r = o & 3;
    return (t & ~63) | (tt << 5) | (g << 3) | (h << 2) | r;
  } else {
    const int o = t & 31;
    const int h = o >> 4, g = (o >> 2) & 3, r = o & 3;
    return (t & ~31) | (g << 3) | (h << 2) | r;
  }
}

// Codes and scale of one unit (8 channels, lane's part of an NB-channel block);
// the lanes of a block are consecutive and all call.
template <int FMT>
__device__ __forceinline__ void quant_unit(const float (&v)[8], uint32_t& word, uint32_t& sbyte) {
  constexpr int LPB = (FMT == kFmtMX ? 32 : 16) / 8;   // lanes per block
  float am = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) am = __builtin_fmaxf(am, __builtin_fabsf(v[i]));
#pragma unroll
  for (int off = 1; off < LPB; off <<= 1) am = __builtin_fmaxf(am, __shfl_xor(am, off, 64));
  float y[8];
  if (FMT == kFmtMX) {
    const int e = e8m0_exponent(am);
    sbyte = (uint32_t)(e + 127);
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = __builtin_ldexpf(v[i], -e);   // exact power-of-two scaling
  } else {
    sbyte = e4m3_encode(am / 6.0f);
    const float s = e4m3_decode(sbyte);
    const float r = s == 0.0f ? 0.0f : 1.0f / s;
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = s == 0.0f ? 0.0f : v[i] * r;
  }
  word = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) word |= cvt_fp4x2(y[2 * i], y[2 * i + 1]) << (8 * i);
}

template <int D, int FMT>
__device__ __forceinline__ void store_unit(uint8_t* codes, uint8_t* scales, long long orow, int cu, uint32_t word,
                                           uint32_t sbyte) {
  constexpr int NB = (FMT == kFmtMX) ? 32 : 16, LPB = NB / 8;
  *reinterpret_cast<uint32_t*>(codes + (size_t)orow * (D / 2) + cu * 4) = word;
  if ((cu % LPB) == 0) scales[(size_t)orow * (D / NB) + cu / LPB] = (uint8_t)sbyte;
}

// Q without smoothing: workgroup blk of nblk takes 256 consecutive units per
// step (one per thread; four, as K takes below, are 4% slower).
template <int D, bool BF16, int FMT>
__device__ __forceinline__ void quant_q(const uint16_t* __restrict__ x, uint8_t* __restrict__ codes,
                                        uint8_t* __restrict__ scales, long long total_units, long long blk,
                                        long long nblk) {
  constexpr int UPR = D / 8;                        // units (lanes) per row
  const long long nsb = (total_units + 255) / 256;
  for (long long sb = blk; sb < nsb; sb += nblk) {
    const long long u = sb * 256 + threadIdx.x;
    if (u >= total_units) break;                    // whole rows, so whole blocks of lanes, leave together
    const uint4 raw = *reinterpret_cast<const uint4*>(x + (size_t)u * 8);
    const uint16_t* hv = reinterpret_cast<const uint16_t*>(&raw);
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = widen<BF16>(hv[i]);
    uint32_t word, sbyte;
    quant_unit<FMT>(v, word, sbyte);
    store_unit<D, FMT>(codes, scales, u / UPR, (int)(u % UPR), word, sbyte);
  }
}

template <int D, bool BF16, int FMT>
__global__ __launch_bounds__(256) void quant_q_kernel(const uint16_t* __restrict__ x, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, long long total_units) {
  quant_q<D, BF16, FMT>(x, codes, scales, total_units, blockIdx.x, gridDim.x);
}

// Q with smoothing (Algorithm 1): qbar[bh, b, c] = mean of Q[bh, t, c] over the
// QB rows t of query block b (the last block holds the remaining rows) -- an
// fp64 sum (exact as the K mean's is, see kmean.h), divided by
// the row count and rounded once to fp32 -- and the codes of Q - qbar.  One
// workgroup per block keeps its rows in registers between the two, so Q is read
// once (a mean pass of its own read it again: 32 us beside the quantizer's 41
// on B4 H32 N4096 D128).
template <int D, bool BF16, int FMT>
__device__ __forceinline__ void quant_q_smooth(const uint16_t* __restrict__ q, float* __restrict__ qbar,
                                               uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, int N,
                                               int nqb, int b, int bh, KmRed& red) {
  constexpr int UPR = D / 8, RS = 256 / UPR, U = QB / RS;   // rows in parallel, rows per thread
  const int tid = threadIdx.x, cg = tid % UPR, rsub = tid / UPR;
  const int t0 = b * QB, rows = min(QB, N - t0);
  const uint16_t* qh = q + ((size_t)bh * N + t0) * D + cg * 8;
  uint4 raw[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int r = rsub + RS * u;
    raw[u] = r < rows ? *reinterpret_cast<const uint4*>(qh + (size_t)r * D) : make_uint4(0, 0, 0, 0);
  }
  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw[u]);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += (double)widen<BF16>(h[i]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[tid][i] = acc[i];
  __syncthreads();
  float* mean = reinterpret_cast<float*>(&red[0][8]);        // the pad column: 18 floats apart
  if (tid < D) {
    const int g = tid / 8, i = tid % 8;
    double s = 0.0;
    for (int r = 0; r < RS; ++r) s += red[r * UPR + g][i];
    const float m = (float)(s / (double)rows);
    qbar[((size_t)bh * nqb + b) * D + tid] = m;
    mean[18 * tid] = m;
  }
  __syncthreads();
  float m8[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) m8[i] = mean[18 * (cg * 8 + i)];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int r = rsub + RS * u;
    if (r >= rows) break;                                    // whole rows leave together
    const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw[u]);
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = widen<BF16>(h[i]) - m8[i];
    uint32_t word, sbyte;
    quant_unit<FMT>(v, word, sbyte);
    store_unit<D, FMT>(codes, scales, (long long)bh * N + t0 + r, cg, word, sbyte);
  }
}

template <int D, bool BF16, int FMT>
__global__ __launch_bounds__(256) void quant_q_smooth_kernel(const uint16_t* __restrict__ q, float* __restrict__ qbar,
                                                             uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                                             int N, int nqb) {
  __shared__ KmRed red;
  quant_q_smooth<D, BF16, FMT>(q, qbar, codes, scales, N, nqb, blockIdx.x, blockIdx.y, red);
}

// K: a workgroup takes KRB rows of one head (four units per thread, all loads
// issued before the first is used, without branches, which would make each wait
// for the one before: B1 H32 N32768 D128 75 us with them, 50.5 without),
// subtracts the head's mean -- read from mu, or (part given, up to
// KM_INLINE chunks) summed here from the partial sums, which saves the pass
// between them -- and stores each token at its permuted position.  Rows N ..
// Np - 1 get zero codes and unit scales.
template <int D, bool BF16, int FMT>
__global__ __launch_bounds__(256) void quant_k_kernel(const uint16_t* __restrict__ x, const double* __restrict__ part,
                                                      float* __restrict__ mu, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, int N, int Np, int nchunk) {
  constexpr int UPR = D / 8, RS = 256 / UPR, U = 4, KRB = RS * U;
  const int nrb = Np / KRB;                                  // Np is a multiple of 128 and KRB 64 or 128
  const int bh = blockIdx.x / nrb, t0 = (blockIdx.x % nrb) * KRB;
  const int tid = threadIdx.x, cg = tid % UPR, rsub = tid / UPR;
  const uint16_t* xh = x + (size_t)bh * N * D + cg * 8;
  uint4 raw[U];
#pragma unroll
  for (int u = 0; u < U; ++u)                                // rows past N: any row, overwritten below
    raw[u] = *reinterpret_cast<const uint4*>(xh + (size_t)min(t0 + rsub + RS * u, N - 1) * D);
  v4f ma = {}, mb = {};
  if (part != nullptr) {
    __shared__ __attribute__((aligned(16))) float mean[D];
    kmean_inline<D>(part, mu, N, nchunk, bh, t0 == 0, mean);
    ma = *reinterpret_cast<const v4f*>(mean + cg * 8);
    mb = *reinterpret_cast<const v4f*>(mean + cg * 8 + 4);
  } else if (mu != nullptr) {
    typedef v4f __attribute__((aligned(4))) v4f_a4;          // the caller's mean is 4-byte aligned
    const v4f_a4* mp = reinterpret_cast<const v4f_a4*>(mu + (size_t)bh * D + cg * 8);
    ma = mp[0];
    mb = mp[1];
  }
  const float m8[8] = {ma[0], ma[1], ma[2], ma[3], mb[0], mb[1], mb[2], mb[3]};
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = t0 + rsub + RS * u;
    const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw[u]);
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = widen<BF16>(h[i]) - m8[i];   // without smoothing m8 is 0: exact
    uint32_t word, sbyte;
    quant_unit<FMT>(v, word, sbyte);
    if (t >= N) {
      word = 0;
      sbyte = FMT == kFmtMX ? 127 : 0;
    }
    store_unit<D, FMT>(codes, scales, (long long)bh * Np + k_stored_pos<FMT>(t), cg, word, sbyte);
  }
}

// ---------------------------------------------------------------------------
// V quantizer with the transpose fused in.  A block of 256 threads stages a
// 128-token x D tile in LDS (coalesced 16-byte loads), then each thread
// quantizes whole token blocks of one channel and writes them contiguously
// into V^T [bh, d, Np/2].  Tokens >= N are zero.  Each block walks a
// contiguous range of per_wg (bh, tile) pairs and keeps the loads of the next
// two tiles in registers while it quantizes the current one.
// ---------------------------------------------------------------------------
constexpr int VT = 128;       // tokens per tile (a V^T row segment of 64 bytes); Np is a multiple of it
// One workgroup per CU, two tiles in flight: 79.7 us on B1 H32 N32768 D128,
// against 96 us for one tile per workgroup and, with the same loop, 92 us at
// two workgroups per CU (one tile ahead: 83.5 us at one per CU, 87, 96 and
// 101 us at two, three and four); with the scale bytes staged, 71.4 us.
constexpr int V_WG_PER_CU = 1;

template <int D, int FMT>
struct VLds {
  // all lanes of a wave read one row (consecutive channels): no padding needed
  uint16_t tile[VT][D];
  // The scale bytes of up to ST_TILES consecutive tiles of one head, per
  // V^T row: one 128-byte segment of the row, stored whole (written one byte
  // per block as they come, a row's line would fill over the workgroup's
  // whole range and partly leave L2 before it is complete).  Rows are 132
  // bytes apart, so the byte writes of a wave's channels fall in different banks.
  static constexpr int SPT = VT / (FMT == kFmtMX ? 32 : 16), ST_TILES = 128 / SPT, ST_ROW = 132;
  __attribute__((aligned(16))) uint8_t sst[D * ST_ROW];
};

// workgroup blk of nblk
template <int D, bool BF16, int FMT>
__device__ __forceinline__ void quant_v(const uint16_t* __restrict__ v, uint8_t* __restrict__ codes,
                                        uint8_t* __restrict__ scales, int N, int Np, int total, int per_wg, int blk,
                                        int nblk, VLds<D, FMT>& lds) {
  using T = VLds<D, FMT>;
  constexpr int NB = (FMT == kFmtMX) ? 32 : 16, SPT = T::SPT, ST_TILES = T::ST_TILES, ST_ROW = T::ST_ROW;
  auto& tile = lds.tile;
  auto& sst = lds.sst;
  const int ntt = (Np + VT - 1) / VT;
  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous
  // range of (bh, tile), so the two 64-byte halves of every 128-byte V^T line
  // are written through the same L2, mostly by one workgroup, one tile apart.
  int w = blk;
  if ((nblk & 7) == 0) w = (blk & 7) * (nblk >> 3) + (blk >> 3);
  const int first = w * per_wg, last = min(total, first + per_wg);
  const int tid = threadIdx.x;
  constexpr int UPR = D / 8, LPT = VT * UPR / 256;   // 16-byte units per row, per thread
  static_assert(LPT * 256 == VT * UPR, "tile loads split evenly");
  uint4 ra[LPT], rb[LPT];
  auto load = [&](int lin, uint4 (&raw)[LPT]) {
    const int t0 = (lin % ntt) * VT;
    const uint16_t* vb = v + (size_t)(lin / ntt) * N * D;
#pragma unroll
    for (int k = 0; k < LPT; ++k) {
      const int i = tid + 256 * k, t = t0 + i / UPR;
      raw[k] = (t < N) ? *reinterpret_cast<const uint4*>(vb + (size_t)t * D + (i % UPR) * 8) : make_uint4(0, 0, 0, 0);
    }
  };
  if (first < last) load(first, ra);
  if (first + 1 < last) load(first + 1, rb);
  // each thread quantizes CPT adjacent channels of BPT token blocks (one
  // 32-bit LDS read per token for two channels)
  constexpr int CPT = (D == 128) ? 2 : 1;
  constexpr int TPG = 256 / (D / CPT);       // threads per channel group
  constexpr int BPT = VT / NB / TPG;         // token blocks per thread
  static_assert(BPT >= 1 && TPG * (D / CPT) == 256, "tile shape");
  const int c0 = (tid % (D / CPT)) * CPT, part = tid / (D / CPT);
  int nst = 0;                               // tiles staged in sst (consecutive, one head)
  auto flush = [&](int lin_last) {           // workgroup-uniform
    __syncthreads();                         // every staged byte is written
    const int lin0 = lin_last - nst + 1;
    const int t0 = (lin0 % ntt) * VT;
    const size_t bh = (size_t)(lin0 / ntt);
    const int ndw = nst * SPT / 4;           // dwords per row (SPT is 4 or 8)
    for (int e = tid; e < D * ndw; e += 256) {
      const int c = e / ndw, i = e % ndw;
      *reinterpret_cast<uint32_t*>(scales + (bh * D + c) * (Np / NB) + t0 / NB + 4 * i) =
          *reinterpret_cast<const uint32_t*>(&sst[c * ST_ROW + 4 * i]);
    }
    nst = 0;                                 // sst is written again only after the next tile's barriers
  };
  auto step = [&](int lin, uint4 (&raw)[LPT]) {
    __syncthreads();                         // every thread is done with the previous tile in LDS
#pragma unroll
    for (int k = 0; k < LPT; ++k) {
      const int i = tid + 256 * k;
      *reinterpret_cast<uint4*>(&tile[i / UPR][(i % UPR) * 8]) = raw[k];
    }
    __syncthreads();
    if (lin + 2 < last) load(lin + 2, raw);  // two tiles in flight while this one is quantized
    const int t0 = (lin % ntt) * VT;
    const size_t bh = (size_t)(lin / ntt);
#pragma unroll
    for (int bb = 0; bb < BPT; ++bb) {
      const int blk = part * BPT + bb;         // token block inside the tile
      if (t0 + blk * NB >= Np) break;          // the last tile may end at Np (a multiple of 128)
      float x[CPT][NB];
      float am[CPT];
#pragma unroll
      for (int k = 0; k < CPT; ++k) am[k] = 0.0f;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int r = blk * NB + j;
        const bool in = t0 + r < N;
        if constexpr (CPT == 2) {
          const uint32_t two = *reinterpret_cast<const uint32_t*>(&tile[r][c0]);
          x[0][j] = in ? widen<BF16>((uint16_t)(two & 0xFFFFu)) : 0.0f;
          x[1][j] = in ? widen<BF16>((uint16_t)(two >> 16)) : 0.0f;
        } else {
          x[0][j] = in ? widen<BF16>(tile[r][c0]) : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < CPT; ++k) am[k] = __builtin_fmaxf(am[k], __builtin_fabsf(x[k][j]));
      }
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        uint32_t sbyte;
        if (FMT == kFmtMX) {
          const int e = e8m0_exponent(am[k]);
          sbyte = (uint32_t)(e + 127);
#pragma unroll
          for (int j = 0; j < NB; ++j) x[k][j] = __builtin_ldexpf(x[k][j], -e);
        } else {
          sbyte = e4m3_encode(am[k] / 6.0f);
          const float s = e4m3_decode(sbyte);
          const float r = (s == 0.0f) ? 0.0f : 1.0f / s;
#pragma unroll
          for (int j = 0; j < NB; ++j) x[k][j] = (s == 0.0f) ? 0.0f : x[k][j] * r;
        }
        uint32_t wd[NB / 8];
#pragma unroll
        for (int q = 0; q < NB / 8; ++q) {
          wd[q] = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) wd[q] |= cvt_fp4x2(x[k][8 * q + 2 * i], x[k][8 * q + 2 * i + 1]) << (8 * i);
        }
        const int c = c0 + k;
        uint8_t* dst = codes + (bh * D + c) * (Np / 2) + (t0 + blk * NB) / 2;
        if (NB == 32) *reinterpret_cast<uint4*>(dst) = make_uint4(wd[0], wd[1], wd[2], wd[3]);
        else *reinterpret_cast<uint2*>(dst) = make_uint2(wd[0], wd[1]);
        sst[c * ST_ROW + nst * SPT + blk] = (uint8_t)sbyte;
      }
    }
    ++nst;
    if (nst == ST_TILES || lin + 1 >= last || (lin + 1) / ntt != lin / ntt) flush(lin);
  };
  for (int lin = first; lin < last; lin += 2) {
    step(lin, ra);
    if (lin + 1 < last) step(lin + 1, rb);
  }
}

template <int D, bool BF16, int FMT>
__global__ __launch_bounds__(256) void quant_v_kernel(const uint16_t* __restrict__ v, uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, int N, int Np, int total,
                                                      int per_wg) {
  __shared__ VLds<D, FMT> lds;
  quant_v<D, BF16, FMT>(v, codes, scales, N, Np, total, per_wg, blockIdx.x, gridDim.x, lds);
}

// ---------------------------------------------------------------------------
// Everything that does not depend on the K mean in one launch: the first nv
// workgroups quantize V, the next nkm form the K mean's partial sums, the rest
// quantize Q.  For calls whose passes are too short to fill the GPU one by one.
// ---------------------------------------------------------------------------
struct PrepArgs {
  const uint16_t *q, *k, *v;
  uint8_t *qc, *qs, *vc, *vs;
  float* qbar;
  double* part;
  long long q_units;
  int N, Np, nchunk, nqb, v_total, v_per_wg, nv, nkm;
};

template <int D, bool BF16, int FMT, bool SQ>
__global__ __launch_bounds__(256) void prep_kernel(const PrepArgs a) {
  __shared__ union Lds {
    VLds<D, FMT> v;
    KmRed red;
  } lds;
  int b = blockIdx.x;
  if (b < a.nv) {
    quant_v<D, BF16, FMT>(a.v, a.vc, a.vs, a.N, a.Np, a.v_total, a.v_per_wg, b, a.nv, lds.v);
    return;
  }
  b -= a.nv;
  if (b < a.nkm) {
    kmean_partial<D, BF16>(a.k, a.part, a.N, a.nchunk, b % a.nchunk, b / a.nchunk, lds.red);
    return;
  }
  b -= a.nkm;
  if constexpr (SQ) quant_q_smooth<D, BF16, FMT>(a.q, a.qbar, a.qc, a.qs, a.N, a.nqb, b % a.nqb, b / a.nqb, lds.red);
  else quant_q<D, BF16, FMT>(a.q, a.qc, a.qs, a.q_units, b, gridDim.x - a.nv - a.nkm);
}

// ---------------------------------------------------------------------------
// Host-side launchers (called by the C ABI in sage_abi.hip).
// ---------------------------------------------------------------------------
int kmean_chunks(int N) { return (N + KM_CHUNK - 1) / KM_CHUNK; }
int qmean_blocks(int N) { return (N + QB - 1) / QB; }

// f(ic<D>, ic<BF16>, ic<FMT>) for run-time values
template <typename F>
static hipError_t quant_dispatch(int D, bool bf16, int fmt, F&& f) {
  if (D == 128) {
    if (fmt == kFmtMX) return bf16 ? f(ic<128>{}, ic<1>{}, ic<kFmtMX>{}) : f(ic<128>{}, ic<0>{}, ic<kFmtMX>{});
    return bf16 ? f(ic<128>{}, ic<1>{}, ic<kFmtNV16>{}) : f(ic<128>{}, ic<0>{}, ic<kFmtNV16>{});
  }
  if (fmt == kFmtMX) return bf16 ? f(ic<64>{}, ic<1>{}, ic<kFmtMX>{}) : f(ic<64>{}, ic<0>{}, ic<kFmtMX>{});
  return bf16 ? f(ic<64>{}, ic<1>{}, ic<kFmtNV16>{}) : f(ic<64>{}, ic<0>{}, ic<kFmtNV16>{});
}

hipError_t launch_kmean_final(const double* part, float* mu, int BH, int N, int D, hipStream_t st) {
  const int nchunk = kmean_chunks(N);
  if (D == 128) hipLaunchKernelGGL((kmean_final_kernel<128>), dim3(BH), dim3(256), 0, st, part, mu, N, nchunk);
  else hipLaunchKernelGGL((kmean_final_kernel<64>), dim3(BH), dim3(256), 0, st, part, mu, N, nchunk);
  return hipGetLastError();
}

hipError_t launch_kmean_partial(const void* k, double* part, int BH, int N, int D, bool bf16, hipStream_t st) {
  const int nchunk = kmean_chunks(N);
  return quant_dispatch(D, bf16, kFmtMX, [&](auto D_, auto B_, auto) {
    hipLaunchKernelGGL((kmean_partial_kernel<decltype(D_)::value, decltype(B_)::value != 0>), dim3(nchunk, BH),
                       dim3(KM_THREADS), 0, st, (const uint16_t*)k, part, N, nchunk);
    return hipGetLastError();
  });
}

// K's codes and scales; mu null without smoothing.  part: the partial sums of
// the mean (mu is then written here), or null when mu holds it already.
static hipError_t launch_quant_k_rows(const void* x, const double* part, float* mu, void* codes, void* scales, int BH,
                                      int N, int Np, int D, int fmt, bool bf16, hipStream_t st) {
  const int nchunk = kmean_chunks(N);
  if (part != nullptr && nchunk > KM_INLINE) {
    const hipError_t e = launch_kmean_final(part, mu, BH, N, D, st);
    if (e != hipSuccess) return e;
    part = nullptr;
  }
  return quant_dispatch(D, bf16, fmt, [&](auto D_, auto B_, auto F_) {
    constexpr int DD = decltype(D_)::value, KRB = 4 * 256 / (DD / 8);
    const long long blocks = (long long)(Np / KRB) * BH;
    if (blocks > INT_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((quant_k_kernel<DD, decltype(B_)::value != 0, decltype(F_)::value>), dim3((unsigned)blocks),
                       dim3(256), 0, st, (const uint16_t*)x, part, mu, (uint8_t*)codes, (uint8_t*)scales, N, Np, nchunk);
    return hipGetLastError();
  });
}

// K with smoothing (mu and part given) or without (both null).
hipError_t launch_quant_k(const void* k, double* part, float* mu, void* codes, void* scales, int BH, int N, int Np,
                          int D, int fmt, bool bf16, hipStream_t st) {
  if (mu != nullptr) {
    const hipError_t e = launch_kmean_partial(k, part, BH, N, D, bf16, st);
    if (e != hipSuccess) return e;
  }
  return launch_quant_k_rows(k, mu ? part : nullptr, mu, codes, scales, BH, N, Np, D, fmt, bf16, st);
}

// Q; qbar [BH, ceil(N/QB), D] receives the block means with smoothing, null without.
hipError_t launch_quant_q(const void* q, float* qbar, void* codes, void* scales, int BH, int N, int D, int fmt,
                          bool bf16, hipStream_t st) {
  return quant_dispatch(D, bf16, fmt, [&](auto D_, auto B_, auto F_) {
    constexpr int DD = decltype(D_)::value, FF = decltype(F_)::value;
    constexpr bool BB = decltype(B_)::value != 0;
    if (qbar != nullptr) {
      hipLaunchKernelGGL((quant_q_smooth_kernel<DD, BB, FF>), dim3((unsigned)qmean_blocks(N), (unsigned)BH), dim3(256), 0,
                         st, (const uint16_t*)q, qbar, (uint8_t*)codes, (uint8_t*)scales, N, qmean_blocks(N));
    } else {
      const long long units = (long long)BH * N * (DD / 8);
      const long long blocks = std::min<long long>((units + 255) / 256, 65536);
      hipLaunchKernelGGL((quant_q_kernel<DD, BB, FF>), dim3((unsigned)blocks), dim3(256), 0, st, (const uint16_t*)q,
                         (uint8_t*)codes, (uint8_t*)scales, units);
    }
    return hipGetLastError();
  });
}

// bias [BH, nqb, Np] fp32; Np is a multiple of 128.  The 512-key tiles are taken
// when they give every CU of a gfx950 (256) a workgroup and more than one wave of each has blocks.
hipError_t launch_qk_bias(const void* k, const float* mu, const float* qbar, float* bias, int BH, int N, int Np, int D,
                          bool bf16, hipStream_t st) {
  const int nqb = qmean_blocks(N);
  const long long big = (long long)((Np + 511) / 512) * ((nqb + 31) / 32) * BH;
  return quant_dispatch(D, bf16, kFmtMX, [&](auto D_, auto B_, auto) {
    constexpr int DD = decltype(D_)::value;
    constexpr bool BB = decltype(B_)::value != 0;
    if (nqb > 8 && big >= 256) {
      const int nkt = (Np + 511) / 512;
      hipLaunchKernelGGL((qk_bias_kernel<DD, BB, 512, 4, 16>), dim3((unsigned)(nkt * ((nqb + 31) / 32)), (unsigned)BH),
                         dim3(256), 0, st, (const uint16_t*)k, mu, qbar, bias, N, Np, nqb, nkt);
    } else {
      const int nkt = (Np + 255) / 256;
      hipLaunchKernelGGL((qk_bias_kernel<DD, BB, 256, 1, 32>), dim3((unsigned)(nkt * ((nqb + 7) / 8)), (unsigned)BH),
                         dim3(256), 0, st, (const uint16_t*)k, mu, qbar, bias, N, Np, nqb, nkt);
    }
    return hipGetLastError();
  });
}

// tiles of the V quantizer, tiles per workgroup and workgroups (Np is a multiple of VT)
static hipError_t v_grid(int BH, int Np, int* total, int* per_wg, int* grid) {
  const long long t = (long long)(Np / VT) * BH;
  if (t > INT_MAX) return hipErrorInvalidValue;
  int dev = 0, ncu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const long long slots = (long long)(ncu > 0 ? ncu : 1) * V_WG_PER_CU;
  *total = (int)t;
  *per_wg = (int)((t + slots - 1) / slots);
  *grid = (int)((t + *per_wg - 1) / *per_wg);
  return hipSuccess;
}

hipError_t launch_quant_v(const void* v, void* codes, void* scales, int BH, int N, int Np, int D, int fmt, bool bf16,
                          hipStream_t st) {
  int total, per_wg, grid;
  const hipError_t e = v_grid(BH, Np, &total, &per_wg, &grid);
  if (e != hipSuccess) return e;
  return quant_dispatch(D, bf16, fmt, [&](auto D_, auto B_, auto F_) {
    hipLaunchKernelGGL((quant_v_kernel<decltype(D_)::value, decltype(B_)::value != 0, decltype(F_)::value>), dim3(grid),
                       dim3(256), 0, st, (const uint16_t*)v, (uint8_t*)codes, (uint8_t*)scales, N, Np, total, per_wg);
    return hipGetLastError();
  });
}

// Up to this many elements (BH Np D) Q, V and K's partial sums share a launch
// (four launches fewer): B1 H4 N4096 D128 61 -> 55 us a call, B2 H24 N1237 60 -> 51,
// B1 H32 N4096 (2^24) 173 -> 170; above it the passes fill the GPU one by one and
// the V part's LDS costs the others occupancy: B2 H32 N4096 326 -> 335.
constexpr long long PREP_MAX_ELEMS = 1LL << 24;

// Q, K and V of one call.  qbar null without smoothing Q; mu and part null
// without smoothing K.
hipError_t launch_quant_qkv(const void* q, const void* k, const void* v, void* qc, void* qs, float* qbar, void* kc,
                            void* ks, double* part, float* mu, void* vc, void* vs, int BH, int N, int Np, int D, int fmt,
                            bool bf16, hipStream_t st) {
  const long long elems = (long long)BH * Np * D;
  if (elems > PREP_MAX_ELEMS) {
    hipError_t e = launch_quant_q(q, qbar, qc, qs, BH, N, D, fmt, bf16, st);
    if (e == hipSuccess) e = launch_quant_k(k, part, mu, kc, ks, BH, N, Np, D, fmt, bf16, st);
    if (e == hipSuccess) e = launch_quant_v(v, vc, vs, BH, N, Np, D, fmt, bf16, st);
    return e;
  }
  PrepArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
  a.qc = (uint8_t*)qc; a.qs = (uint8_t*)qs; a.vc = (uint8_t*)vc; a.vs = (uint8_t*)vs;
  a.qbar = qbar; a.part = part; a.N = N; a.Np = Np; a.nchunk = kmean_chunks(N); a.nqb = qmean_blocks(N);
  hipError_t e = v_grid(BH, Np, &a.v_total, &a.v_per_wg, &a.nv);
  if (e != hipSuccess) return e;
  a.nkm = mu != nullptr ? a.nchunk * BH : 0;
  a.q_units = (long long)BH * N * (D / 8);
  const long long nq = qbar != nullptr ? (long long)a.nqb * BH : (a.q_units + 255) / 256;
  const dim3 grid((unsigned)(a.nv + a.nkm + nq));
  e = quant_dispatch(D, bf16, fmt, [&](auto D_, auto B_, auto F_) {
    constexpr int DD = decltype(D_)::value, FF = decltype(F_)::value;
    constexpr bool BB = decltype(B_)::value != 0;
    if (qbar != nullptr) hipLaunchKernelGGL((prep_kernel<DD, BB, FF, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((prep_kernel<DD, BB, FF, false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
  });
  return e != hipSuccess ? e : launch_quant_k_rows(k, mu ? part : nullptr, mu, kc, ks, BH, N, Np, D, fmt, bf16, st);
}

}  // namespace sage
