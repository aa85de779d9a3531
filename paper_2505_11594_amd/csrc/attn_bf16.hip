// bf16-MFMA comparison kernel for gfx950: FlashAttention forward (Sec. 2)
// with the same work decomposition as the FP4 kernel -- 4 waves x 32 queries
// per workgroup, K and V tiles double-buffered in LDS, online softmax in
// registers -- on v_mfma_f32_32x32x16_bf16:
//   S^T (keys x queries) = K . Q^T     A = K tile (LDS), B = Q (registers)
//   O^T (dims x queries) += V^T . P^T  A = V^T tile (LDS), B = P in bf16
// S is fp32, the softmax is fp32, P is rounded to bf16 (nearest even) for the
// second product.  Layout (32x32x16): lane l holds row/column l%32 and
// K-indices [8*(l/32), +8); the accumulator of lane l holds column l%32 and
// rows 8g + 4*(l/32) + r.
//
// Both tiles go from HBM straight into LDS, row-major as they lie in memory.
// V is transposed by the LDS read: ds_read_b64_tr_b16 gives the 16 lanes of a
// group, each addressing 4 channels of one key, the 4 keys of one channel
// each, and two such reads are the 8 keys 16w + {0, 8} + 4 (l/32) + r of K-step w
// whose scores the lane holds.  (A pre-pass that wrote V^T to a workspace took
// 46 us of 1247 on B4 H32 N4096 D128, and its allocation as much as 370 us of a
// call that starts on an idle GPU.)  MFMA issue bounds it: 1250 -> 1090 us there,
// 1.01 PFLOP/s, against 1.27 that a large bf16 matrix product reaches.
#include "sage_common.h"
#include "bf16_tile.h"

namespace sage {

constexpr int BK = 64;         // keys per tile
constexpr int BW = 4;          // waves per workgroup (32 queries each)

// Chunk swizzle of the V tile (16-byte chunks of a key's row): the 8 keys whose
// chunk pairs one read instruction touches fall on distinct bank groups.
template <int D>
__device__ __forceinline__ int vswz(int row, int ch) {
  return D == 128 ? ch ^ ((row & 7) << 1) : ch ^ (((row >> 1) & 3) << 1);
}

// The A operands (V^T) of one K-step for two channel blocks: per block two
// transposing reads 8 keys apart, at LDS byte addresses a + OFF and a + OFF + 8
// rows.  One asm block with its own wait: for the builtin the compiler first
// waits for every direct-to-LDS load in flight (see sage_common.h).
template <int OFF, int OFF8>
__device__ __forceinline__ void vt_read2(uint32_t a0, uint32_t a1, v8bf& r0, v8bf& r1) {
  v2u x0, x1, x2, x3;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4 offset:%6\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
      "ds_read_b64_tr_b16 %2, %5 offset:%6\n\tds_read_b64_tr_b16 %3, %5 offset:%7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3)
      : "v"(a0), "v"(a1), "n"(OFF), "n"(OFF8)
      : "memory");
  r0 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x0, x1, 0, 1, 2, 3));
  r1 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x2, x3, 0, 1, 2, 3));
}
// The same for four channel blocks, with one wait.
template <int OFF, int OFF8>
__device__ __forceinline__ void vt_read4(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, v8bf& r0, v8bf& r1, v8bf& r2,
                                         v8bf& r3) {
  v2u x0, x1, x2, x3, x4, x5, x6, x7;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %2, %9 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
      "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %10 offset:%13\n\t"
      "ds_read_b64_tr_b16 %6, %11 offset:%12\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3), "=&v"(x4), "=&v"(x5), "=&v"(x6), "=&v"(x7)
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(OFF), "n"(OFF8)
      : "memory");
  r0 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x0, x1, 0, 1, 2, 3));
  r1 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x2, x3, 0, 1, 2, 3));
  r2 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x4, x5, 0, 1, 2, 3));
  r3 = __builtin_bit_cast(v8bf, __builtin_shufflevector(x6, x7, 0, 1, 2, 3));
}

template <int D, bool CAUSAL, bool OUT_F32>
__global__ __launch_bounds__(64 * BW, 2) void attn_bf16_kernel(const uint16_t* __restrict__ q,
                                                               const uint16_t* __restrict__ k,
                                                               const uint16_t* __restrict__ v, void* __restrict__ o,
                                                               int BH, int N, int nqt, float c2) {
  constexpr int NSUB = BK / 32;    // 2 key subtiles
  constexpr int NKS = D / 16;      // QK K-steps
  constexpr int NPK = BK / 16;     // PV K-steps
  constexpr int NDB = D / 32;
  constexpr int ROW = D * 2, CH = ROW / 16;            // bytes and chunks per key row
  constexpr int TB = BK * ROW;                         // bytes of a K (or V) tile
  __shared__ __attribute__((aligned(16))) uint8_t lds[4 * TB];   // stage: K tile, V tile
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, hi = lane >> 5;

  const int total = nqt * BH;
  int lin = blockIdx.x;
  if ((total & 7) == 0) lin = (blockIdx.x & 7) * (total >> 3) + (blockIdx.x >> 3);
  const long long bh = lin / nqt;
  int qt = lin % nqt;
  if (CAUSAL) qt = nqt - 1 - qt;
  const int q0 = qt * (32 * BW), qw = q0 + wave * 32, qi = qw + col;

  v4i qreg[NKS];
  {
    const int qr = min(qi, N - 1);
    const uint16_t* qrow = q + ((size_t)bh * N + qr) * D;
#pragma unroll
    for (int s = 0; s < NKS; ++s) qreg[s] = *reinterpret_cast<const v4i*>(qrow + 16 * s + 8 * hi);
  }
  int ntiles = (N + BK - 1) / BK;
  if (CAUSAL) ntiles = min(ntiles, min(q0 + 32 * BW - 1, N - 1) / BK + 1);

  // Tile loads (see sage_common.h): job J covers 1 KiB of a tile (JR rows), wave
  // J % BW; lane l fills LDS chunk l of the job, which holds the swizzled
  // logical chunk of its row.  Rows past N read zero (those keys are masked).
  constexpr int JR = 1024 / ROW, NJ = BK / JR, JW = (NJ + BW - 1) / BW;
  uint32_t klo[JW], vlo[JW];
#pragma unroll
  for (int i = 0; i < JW; ++i) {
    const int r = (wave + BW * i) * JR + lane / CH;
    klo[i] = (uint32_t)(r * ROW + bswz<CH>(r, lane % CH) * 16);
    vlo[i] = (uint32_t)(r * ROW + vswz<D>(r, lane % CH) * 16);
  }
  const uint8_t* kbase = reinterpret_cast<const uint8_t*>(k) + (size_t)bh * N * ROW;
  const uint8_t* vbase = reinterpret_cast<const uint8_t*>(v) + (size_t)bh * N * ROW;
  auto issue = [&](int j, int stage) {
    const int kb = j * BK;
    uint8_t* L = lds + stage * 2 * TB;
    const uint32_t bytes = (uint32_t)min(N - kb, BK) * ROW;
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(kbase + (size_t)kb * ROW, bytes), rv = make_rsrc(vbase + (size_t)kb * ROW, bytes);
#pragma unroll
    for (int i = 0; i < JW; ++i)
      if (NJ % BW == 0 || wave + BW * i < NJ) {
        buf_load16(rk, klo[i], 0u, L + (wave + BW * i) * 1024);
        buf_load16(rv, vlo[i], 0u, L + TB + (wave + BW * i) * 1024);
      }
  };

  // V^T operand address: this lane of its 16-lane group reads key 4 hi + (lane % 16) / 4 of a
  // K-step, channels [32db + 16 (lane / 16 % 2) + 4 (lane % 4), +4)
  uint32_t vo[NDB];
  {
    const uint32_t l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int r = 4 * hi + (lane & 15) / 4, c0 = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
    for (int db = 0; db < NDB; ++db) vo[db] = l0 + TB + r * ROW + vswz<D>(r, 4 * db + c0) * 16 + 8 * (lane & 1);
  }

  v16f oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = v16f{};
  float m = -INFINITY, l = 0.0f;

  issue(0, 0);
  for (int j = 0; j < ntiles; ++j) {
    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): this wave's loads of tile j have landed
    __syncthreads();                                   // everyone's; every wave is past tile j - 1
    if (j + 1 < ntiles) issue(j + 1, (j + 1) & 1);
    const uint8_t* L = lds + (j & 1) * 2 * TB;
    const int kb = j * BK;
    if (CAUSAL && kb > qw + 31) continue;
    v16f sacc[NSUB];
#pragma unroll
    for (int t = 0; t < NSUB; ++t) {
      const int row = 32 * t + col;
      v16f acc = v16f{};
#pragma unroll
      for (int s = 0; s < NKS; ++s) {
        const v4i a = *reinterpret_cast<const v4i*>(L + row * ROW + bswz<CH>(row, 2 * s + hi) * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf(a), as_bf(qreg[s]), acc, 0, 0, 0);
      }
      sacc[t] = acc;
    }
    if ((kb + BK > N) || (CAUSAL && kb + BK - 1 > qw)) {
      // element (t, v) is key kb + 4 hi + c with c = 32t + 8 (v >> 2) + (v & 3), kept iff
      // c < rem: the sign of c - rem selects its bits or those of -inf (a minimum with
      // -inf would let the NaN of a masked key through)
      const int rem = (CAUSAL ? min(N, qi + 1) : N) - kb - 4 * hi;
#pragma unroll
      for (int t = 0; t < NSUB; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int c = 32 * t + 8 * (e >> 2) + (e & 3);
          const uint32_t keep = (uint32_t)((c - rem) >> 31);
          sacc[t][e] = __uint_as_float((__float_as_uint(sacc[t][e]) & keep) | (0xFF800000u & ~keep));
        }
    }
    float x = sacc[0][0];
#pragma unroll
    for (int t = 0; t < NSUB; ++t)
#pragma unroll
      for (int e = (t == 0 ? 1 : 0); e < 16; ++e) x = smax(x, sacc[t][e]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float m_new = smax(m, smax(__uint_as_float(sw[0]), __uint_as_float(sw[1])));
    const float mc = m_new * c2;
    const float alpha = __builtin_amdgcn_exp2f(m * c2 - mc);      // 0 on the first tile
    m = m_new;
    // rescale only when some row's max moved (alpha == 1 is an exact no-op)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
    }
    uint32_t va[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) va[db] = vo[db] + (uint32_t)((j & 1) * 2 * TB);
    float ps[2] = {0.0f, 0.0f};
    static_for<NPK>([&](auto U_) {
      constexpr int u = decltype(U_)::value, t = u >> 1, base = 8 * (u & 1);
      v8bf a[NDB];
      constexpr int OFF = 16 * u * ROW, OFF8 = OFF + 8 * ROW;
      if constexpr (NDB == 4) vt_read4<OFF, OFF8>(va[0], va[1], va[2], va[3], a[0], a[1], a[2], a[3]);
      else vt_read2<OFF, OFF8>(va[0], va[1], a[0], a[1]);
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[t][base + 2 * i], c2, -mc));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[t][base + 2 * i + 1], c2, -mc));
        ps[i & 1] += p0;
        ps[i & 1] += p1;
        typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
        const v2bf pb = {(__bf16)p0, (__bf16)p1};
        w[i] = __builtin_bit_cast(uint32_t, pb);
      }
      const v4i pk = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
#pragma unroll
      for (int db = 0; db < NDB; ++db)
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[db], as_bf(pk), oacc[db], 0, 0, 0);
    });
    l = l * alpha + (ps[0] + ps[1]);
  }

  const float ltot = l + __shfl_xor(l, 32, 64);
  const float inv = 1.0f / ltot;
  if (qi < N) {
    uint8_t* ob = reinterpret_cast<uint8_t*>(o);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d0 = 32 * db + 8 * g + 4 * hi;
        const size_t idx = ((size_t)bh * N + qi) * D + d0;
        const float a0 = oacc[db][4 * g] * inv, a1 = oacc[db][4 * g + 1] * inv;
        const float a2 = oacc[db][4 * g + 2] * inv, a3 = oacc[db][4 * g + 3] * inv;
        if (OUT_F32) *reinterpret_cast<float4*>(ob + idx * 4) = make_float4(a0, a1, a2, a3);
        else
          *reinterpret_cast<uint2*>(ob + idx * 2) =
              make_uint2((uint32_t)f32_to_bf16_rne(a0) | ((uint32_t)f32_to_bf16_rne(a1) << 16),
                         (uint32_t)f32_to_bf16_rne(a2) | ((uint32_t)f32_to_bf16_rne(a3) << 16));
      }
  }
}

template <int D, bool CAUSAL, bool OUT_F32>
static hipError_t launch_bf16_t(const void* q, const void* k, const void* v, void* o, int BH, int N, float c2,
                                hipStream_t st) {
  const int nqt = (N + 32 * BW - 1) / (32 * BW);
  hipLaunchKernelGGL((attn_bf16_kernel<D, CAUSAL, OUT_F32>), dim3((unsigned)(nqt * BH)), dim3(64 * BW), 0, st,
                     (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, o, BH, N, nqt, c2);
  return hipGetLastError();
}

hipError_t launch_attn_bf16(const void* q, const void* k, const void* v, void* o, int BH, int N, int D, bool causal,
                            bool out_f32, float c2, hipStream_t st) {
#define SAGE_B(DD)                                                                        \
  if (causal) return out_f32 ? launch_bf16_t<DD, true, true>(q, k, v, o, BH, N, c2, st)   \
                             : launch_bf16_t<DD, true, false>(q, k, v, o, BH, N, c2, st); \
  return out_f32 ? launch_bf16_t<DD, false, true>(q, k, v, o, BH, N, c2, st)              \
                 : launch_bf16_t<DD, false, false>(q, k, v, o, BH, N, c2, st)
  if (D == 128) { SAGE_B(128); }
  SAGE_B(64);
#undef SAGE_B
}

}  // namespace sage
