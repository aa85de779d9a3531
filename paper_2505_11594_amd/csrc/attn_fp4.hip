// Microscaled-FP4 attention forward for gfx950 (SageAttention3, Algorithm 1
// without smoothing Q; two-level quantization of P~, Sec. 3.2).
//
// Work decomposition: one workgroup = 4 waves = 128 queries of one (b,h) (8
// waves and 256 queries with SAGE_WG256); each wave owns 32 queries and walks
// all KV tiles (BKV = 64, 128 or 256 keys).
// Both products run on v_mfma_scale_f32_32x32x64_f8f6f4 with FP4 (E2M1)
// operands and E8M0 block scales:
//   S^T (keys x queries) = K^ . Q^T    A = K^ tile (LDS), B = Q^ (registers)
//   O^T (dims x queries) += V^T . P^T  A = V^T tile (LDS), B = P^ (registers)
// MFMA operand layout (32x32x64): lane l holds row/column l%32 and the 32
// consecutive K-indices [32*(l/32), +32) -- exactly one 32-element block and
// its scale byte.  The accumulator of lane l holds column l%32 and rows
// 8g + 4*(l/32) + r.  Because K^ is stored with its tokens permuted inside
// each 64-token group (quant.hip), the 32 scores a lane holds for one
// 64-key group are the original keys [32*(l/32), +32) of that group, in the
// order the B operand of the P.V product expects: S never leaves registers,
// the FP4 block of P is lane-local (its max needs no shuffle), and the row
// max over a tile needs one cross-half swap.
//
// Softmax state per query row (raw score domain): running max m, and the
// accumulator O^T and row sum kept in units of 6 * 2^-f_j of the true
// O_j, l_j, where 2^(delta_j) = 6 s_P1 = 2^{c2 (t_j - m_j)} is split into
// an integer part k_j (folded exactly into P's E8M0 scale) and a fraction
// f_j.  Each tile then rescales the accumulator once by
// gamma_j = 2^{c2 (m_{j-1} - m_j) + f_{j-1} - f_j}.
//
// Data movement: KV tiles go from HBM straight into LDS with loads that write
// LDS (no staging registers), row by row with swizzled 16-byte chunks or in
// MFMA-operand order (see the load jobs); either way operand reads are free of
// bank conflicts.  Two LDS stages and one barrier per tile: after the barrier of tile j every wave has finished
// tile j - 1, and the loads of tile j + 1 go to that stage while tile j runs.
// (Calls with few query tiles take two tiles a step: see KG below.)
//
// What bounds it is instruction issue (exponentials, packs and plain VALU work
// nearly in series with the MFMAs), so the tile's S is computed at its top and
// the registers go to waves instead of a second S: 64- and 128-key tiles run
// three waves per SIMD (four at D = 64 with 64 keys), 256-key tiles, whose S
// takes 128 registers, two.  Against two waves per SIMD with the next tile's S
// computed ahead and three LDS stages, a call on B2 H32 N4096 D128 took 344
// instead of 373 us with 128-key tiles and 387 instead of 408 with 64-key tiles,
// B1 H24 N19200 D64 1766 instead of 1801 us.
#include "sage_common.h"

namespace sage {

__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Swizzle of a tile row's NCH 16-byte chunks: 16 consecutive rows at one chunk fall on distinct bank groups.
template <int NCH>
__device__ __forceinline__ int fp4_swz(int row) {
  return NCH == 8 ? (row >> 1) & 7 : NCH == 4 ? (row >> 2) & 3 : (row >> 3) & 1;
}

__device__ __forceinline__ v8i as_op(const v4i x) { return v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0}; }

// One LDS stage of a KV tile: K^ and V^T codes (in the order of the load jobs in
// the kernel), their scales and, with smoothing Q, the tile's BKV entries of the
// query block's GEMV bias.  Np is a multiple of 128: when the last 256-key tile
// reaches past Np its upper 128 keys are loaded from its lower half (finite
// values, masked as keys >= N), so that no load leaves its tensor.
template <int D, int BKV, bool SQ>
struct Fp4Stage {
  static constexpr int NSUB = BKV / 32;        // 32-key subtiles (S^T rows)
  static constexpr int NKS = D / 64;           // K-steps of S^T = K^ Q^T
  static constexpr int NDB = D / 32;           // 32-dim blocks (O^T rows)
  static constexpr int NG = BKV / 64;          // K-steps of O^T += V^T P^T
  static constexpr int NKB = NSUB * NKS;       // K^ load jobs, 1 KiB each
  static constexpr int NVB = NDB * NG;         // V^T load jobs, 1 KiB each
  static constexpr int KC_OFF = 0;
  static constexpr int VC_OFF = KC_OFF + NKB * 1024;
  static constexpr int KS_OFF = VC_OFF + NVB * 1024;     // K^ scales: BKV rows x D/32 bytes
  static constexpr int KS_BYTES = BKV * (D / 32);
  static constexpr int VW = BKV == 256 ? 2 : 1;          // dwords of V^T scales per dim row (64 keys: half of one)
  static constexpr int VS_OFF = KS_OFF + (KS_BYTES + 255) / 256 * 256;
  static constexpr int BIAS_OFF = VS_OFF + D * 4 * VW;   // smoothing Q: fp32 bias of the tile's keys
  static constexpr int BYTES = BIAS_OFF + (SQ ? BKV * 4 : 0);
  static constexpr int NKSJ = (KS_BYTES / 4 + 63) / 64, NVSJ = D * VW / 64;   // dword-load jobs of 64 lanes
};

// Waves per SIMD that the register budget is set for: a tile's S takes BKV/2
// registers, O D/2; with smoothing Q at D = 128 and 128 keys a third wave would
// spill about 30 registers.  (D = 128, 128 keys and, with smoothing Q, 256 keys
// spill one to four, outside the tile loop.)
constexpr int fp4_waves(int D, int BKV, int W, bool SQ) {
  if (BKV == 256) return 8 / W;
  if (BKV == 128) return D == 128 && SQ ? 2 : 3;
  return D == 128 ? 3 : 4;
}

// LDS of the kernel with two KV groups (KG = 2, below): four stages, then per wave
// three dwords a lane (tile maximum, row sum, block exponents) and the codes of
// P, NG x 16 bytes a lane.  Where that alone keeps a second workgroup off the CU
// (160 KiB), the codes go over the tile's K^ codes instead, behind a barrier.
template <int D, int BKV, bool SQ>
struct Fp4Xchg {
  using T = Fp4Stage<D, BKV, SQ>;
  static constexpr int XS_OFF = 4 * T::BYTES, XP_OFF = XS_OFF + 4 * 768, OWN = 4 * T::NG * 1024;
  static constexpr bool IN_K = XP_OFF <= 81920 && XP_OFF + OWN > 81920;
  static constexpr int BYTES = IN_K ? XP_OFF : XP_OFF + OWN;
  static_assert(2 * T::NG <= T::NKB && BYTES <= 163840, "the codes of two waves fit K^'s, and all fits a CU");
};

// W waves per workgroup (32 queries each).  W = 4 is the default.  W = 8
// (flag SAGE_WG256; non-causal, without smoothing Q, whose GEMV bias rows
// belong to 128-query blocks) shares each K^/V^T tile in LDS between 256
// queries, so a tile is fetched from L2 once per 256 queries instead of per
// 128: about half the fetch traffic.  The two waves on a SIMD then belong to
// one workgroup and meet at the same barrier, so they overlap less: B1 H32 N32768
// D128 7.57 ms against 7.42 with W = 4 on one box, 7.88 against 7.89 on another,
// alternated in one process.
// OUT: 0 = fp32, 1 = bf16, 2 = fp16.  SQ: smoothing Q -- S += qkb[bh, query
// block, key] (Algorithm 1's GEMV of the block mean with K', one row of Np
// floats per 128-query block, which is this workgroup's query tile).
//
// KG: KV groups.  With KG = 2 the workgroup's four waves are two groups of two,
// 64 queries, that take two KV tiles a step: group kg forms S and P of tile
// jj + kg -- P's codes and block scales depend on the tile's own maximum only --
// and leaves the codes, that maximum and the row sum in LDS; then every wave
// runs the softmax state and P.V over both tiles in turn for the channel blocks
// of its half kg.  Every sum keeps the order of KG = 1, so both give the same
// bits, and a head's result does not depend on how many heads share the call.
// For calls with too few 128-query tiles for the GPU; see fp4_kv_groups.
template <int D, int BKV, bool CAUSAL, int OUT, bool SQ, int W, int KG>
__global__ __launch_bounds__(64 * W, KG == 1 ? fp4_waves(D, BKV, W, SQ) : 2) void attn_fp4_mx_kernel(
    const uint8_t* __restrict__ qc, const uint8_t* __restrict__ qs, const uint8_t* __restrict__ kc,
    const uint8_t* __restrict__ ks, const uint8_t* __restrict__ vc, const uint8_t* __restrict__ vs,
    const float* __restrict__ qkb, void* __restrict__ o, int BH, int N, int Np, int nqt, float c2, float log6) {
  using T = Fp4Stage<D, BKV, SQ>;
  constexpr int NSUB = T::NSUB, NKS = T::NKS, NG = T::NG;
  constexpr int NDB = T::NDB / KG;                // channel blocks of this wave
  constexpr int QW = W / KG, AQW = 32 * QW;       // waves along the queries, queries per workgroup
  static_assert((W == 4 || W == 8) && (!SQ || W == 4), "4 or 8 waves; smoothing Q blocks are 128 queries");
  static_assert(KG == 1 || (KG == 2 && W == 4), "one or two KV groups");
  using X = Fp4Xchg<D, BKV, SQ>;
  __shared__ __attribute__((aligned(16))) uint8_t lds[KG == 1 ? 2 * T::BYTES : X::BYTES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % QW;   // wave of its KV group
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / QW;
  const int col = lane & 31, hi = lane >> 5;
  const int total = nqt * BH;
  int lin = blockIdx.x;
  if ((total & 7) == 0) lin = (blockIdx.x & 7) * (total >> 3) + (blockIdx.x >> 3);
  const long long bh = lin / nqt;
  int qt = lin % nqt;
  if (CAUSAL) qt = nqt - 1 - qt;
  const int q0 = qt * AQW;
  const int qw = q0 + wave * 32;
  const int qi = qw + col;

  v4i qreg[NKS];
  uint32_t qsc = 0;
  if (qi < N) {
    const uint8_t* qrow = qc + ((size_t)bh * N + qi) * (D / 2);
#pragma unroll
    for (int s = 0; s < NKS; ++s) qreg[s] = *reinterpret_cast<const v4i*>(qrow + (s + NKS * hi) * 16);
    const uint8_t* srow = qs + ((size_t)bh * N + qi) * (D / 32);
    qsc = (D == 128) ? *reinterpret_cast<const uint32_t*>(srow) : (uint32_t)*reinterpret_cast<const uint16_t*>(srow);
  } else {
#pragma unroll
    for (int s = 0; s < NKS; ++s) qreg[s] = v4i{0, 0, 0, 0};
  }
  qsc >>= 8 * NKS * hi;

  int ntiles = (N + BKV - 1) / BKV;
  if (CAUSAL) ntiles = min(ntiles, min(q0 + AQW - 1, N - 1) / BKV + 1);

  // Load jobs of 1 KiB: wave w of a KV group loads K^ jobs and V^T jobs b = w +
  // QW i and scale dword jobs jb = w + QW i (K^ scale dwords 64jb + lane, then
  // V^T scale dwords 64(jb - NKSJ) + lane, VW per dim row).
  // ROWS (256-key tiles, four waves): a job is whole tile rows as they lie in memory (K^ rows
  // of D/2 bytes, V^T rows of BKV/2), the 16-byte chunks swizzled against bank
  // conflicts by the choice of the chunk each lane loads, so every line is
  // requested once; operand reads then need an address per K-step.  Otherwise a
  // job is one MFMA operand (32 rows x two 16-byte chunks, lane l's bytes at 16 l):
  // a line is requested by up to four jobs, but one lane offset serves all
  // operand reads, and the 128-key kernels have no registers left (D = 128, 8
  // heads x 4096: 76 us a call with ROWS, 65 without; 256-key tiles, 4 heads
  // x 4096 in two KV groups 47.7 -> 45.2, B4 H32 N4096 637 -> 618; 256-query
  // workgroups, which fetch a tile half as often, 7745 -> 7773 on B1 H32 N32768).
  // Each load is a buffer resource over the head's tensor, a uniform offset --
  // tile, job and the tail redirect -- and one of five fixed lane offsets, so
  // a load costs no VALU and no 64-bit address arithmetic.
  constexpr bool ROWS = BKV == 256 && W == 4;
  static_assert(ROWS ? QW % 2 == 0 : QW % NKS == 0 && (QW % NG == 0 || NG % QW == 0), "job layout");
  constexpr int KJ = (T::NKB + QW - 1) / QW, VJ = (T::NVB + QW - 1) / QW, NSJ = T::NKSJ + T::NVSJ, SJ = (NSJ + QW - 1) / QW;
  constexpr int KCH = D / 32, VCH = BKV / 32, VR = 64 / VCH;      // ROWS: chunks per row, V^T rows per job
  // Redirect of a 256-key tile whose upper half lies past Np.  ROWS: V^T by the lane offset, K^ by the uniform
  // one.  Else a wave's V^T jobs (and K^ job, where it has one) lie in one half of the tile: the lane offset is
  // that of the lower half and the uniform offset adds the way up, which the short tile leaves out.
  constexpr bool K_WAVE = !ROWS && BKV == 256 && QW == T::NKB;
  static_assert(ROWS || BKV != 256 || (QW % NG == 0 && (K_WAVE || QW == T::NKB / 2)), "a wave's jobs lie in one half of the tile");
  uint32_t ko0, vo0, vo_back = 0, k_up = 0, v_up = 0;
  if constexpr (ROWS) {
    const int kcl = (lane % KCH) ^ fp4_swz<KCH>(lane / KCH), vcl = (lane % VCH) ^ fp4_swz<VCH>(wave * VR + lane / VCH);
    ko0 = (uint32_t)(lane / KCH * (D / 2) + 16 * kcl);
    vo0 = (uint32_t)(lane / VCH) * (uint32_t)(Np / 2) + 16 * vcl;
    vo_back = vcl >= VCH / 2 ? 64u : 0u;
  } else {
    ko0 = (uint32_t)((32 * (wave / NKS) + col) * (D / 2) + 16 * (wave % NKS) + 16 * NKS * hi);
    vo0 = (uint32_t)((32 * (wave / NG) + col) * (Np / 2) + 32 * (wave % NG) + 16 * hi);
    if constexpr (K_WAVE) k_up = wave >= T::NKB / 2 ? 128u * (D / 2) : 0u;
    if constexpr (BKV == 256) v_up = wave % NG >= NG / 2 ? 64u : 0u;
    ko0 -= k_up;
    vo0 -= v_up;
  }
  const uint32_t kso = (uint32_t)(4 * lane);
  constexpr int VW = T::VW;
  const uint32_t vso = (uint32_t)((lane / VW) * (Np / 32) + 4 * (lane % VW));
  const uint32_t vso_hi = (uint32_t)(4 * (lane % VW));   // the second dword: subtracted when it lies past Np
  const uint8_t* kbase = kc + (size_t)bh * Np * (D / 2);
  const uint8_t* vbase = vc + (size_t)bh * D * (Np / 2);
  const uint8_t* ksbase = ks + (size_t)bh * Np * (D / 32);
  const uint8_t* vsbase = vs + (size_t)bh * D * (Np / 32);
  // buffer resources over this head's K^, V^T codes and scales: every load is
  // the resource, a uniform byte offset and one fixed lane offset
  const __amdgpu_buffer_rsrc_t rk = make_rsrc(kbase, Np * (D / 2)), rv = make_rsrc(vbase, D * (Np / 2));
  const __amdgpu_buffer_rsrc_t rks = make_rsrc(ksbase, Np * (D / 32)), rvs = make_rsrc(vsbase, D * (Np / 32));
  const __amdgpu_buffer_rsrc_t rb =
      make_rsrc(SQ ? qkb + ((size_t)bh * ((N + 127) / 128) + q0 / 128) * Np : nullptr, SQ ? Np * 4 : 0);
  auto issue = [&](int j, int stage) {
    const int kb = j * BKV;
    const bool short_tail = BKV == 256 && kb + BKV > Np;   // keys [kb + 128, kb + 256) lie past Np
    uint8_t* L = lds + (2 * kg + stage) * T::BYTES;
#pragma unroll
    for (int i = 0; i < KJ; ++i) {
      const int b = wave + QW * i;
      if (T::NKB % QW != 0 && b >= T::NKB) break;
      const uint32_t back = (short_tail && b >= T::NKB / 2) ? 128u * (D / 2) : 0u;
      const uint32_t off = ROWS ? (uint32_t)b * 1024u : (uint32_t)i * (32 * QW / NKS) * (D / 2);
      if constexpr (K_WAVE) buf_load16(rk, ko0, (uint32_t)kb * (D / 2) + off + (short_tail ? 0u : k_up), L + T::KC_OFF + b * 1024);
      else buf_load16(rk, ko0, (uint32_t)kb * (D / 2) + off - back, L + T::KC_OFF + b * 1024);
    }
    const uint32_t vo = vo0 - (short_tail ? vo_back : 0u);
#pragma unroll
    for (int i = 0; i < VJ; ++i) {
      const int b = wave + QW * i;
      if (T::NVB % QW != 0 && b >= T::NVB) break;
      const uint32_t off = ROWS ? (uint32_t)(b * VR) * (uint32_t)(Np / 2)
                                : (uint32_t)(QW * i / NG) * 32 * (Np / 2) + 32 * (QW * i % NG);
      if constexpr (BKV == 256 && !ROWS) buf_load16(rv, vo0, (uint32_t)kb / 2 + off + (short_tail ? 0u : v_up), L + T::VC_OFF + b * 1024);
      else buf_load16(rv, vo, (uint32_t)kb / 2 + off, L + T::VC_OFF + b * 1024);
    }
#pragma unroll
    for (int i = 0; i < SJ; ++i) {
      const int jb = wave + QW * i;
      if (jb < T::NKSJ) {
        const uint32_t back = (short_tail && 64 * jb * 4 >= T::KS_BYTES / 2) ? T::KS_BYTES / 2 : 0u;
        if (T::KS_BYTES % 256 == 0 || 256 * jb + 4 * lane < T::KS_BYTES)
          buf_load4(rks, kso, (uint32_t)kb * (D / 32) + 256u * jb - back, L + T::KS_OFF + jb * 256);
      } else if (jb < NSJ) {
        // 64-key tiles: the aligned dword that holds the tile's two scale bytes
        buf_load4(rvs, vso - (short_tail ? vso_hi : 0u), ((uint32_t)kb / 32 & ~3u) + (uint32_t)(jb - T::NKSJ) * (2 / VW) * Np,
              L + T::VS_OFF + (jb - T::NKSJ) * 256);
      }
    }
    if constexpr (SQ) {
      if (wave == 0 && (BKV == 256 || lane < BKV / 4)) buf_load16(rb, 4u * (uint32_t)min(kb + 4 * lane, Np - 4), 0u, L + T::BIAS_OFF);
    }
  };

  // operand addresses in the tile: K^ (key subtile t, K-step s) and V^T (channel block db, K-step g)
  auto k_op = [&](int t, int s) {
    return T::KC_OFF + (ROWS ? (32 * t + col) * (D / 2) + ((s + NKS * hi) ^ fp4_swz<KCH>(col)) * 16
                             : (t * NKS + s) * 1024 + lane * 16);
  };
  auto v_op = [&](int db, int g) {
    return T::VC_OFF + (ROWS ? (32 * db + col) * (BKV / 2) + ((2 * g + hi) ^ fp4_swz<VCH>(col)) * 16
                             : (db * NG + g) * 1024 + lane * 16);
  };
  v16f oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = v16f{};
  float m = -INFINITY, mc_old = -INFINITY, f_old = 0.0f, lsum_acc = 0.0f;

  if (kg < ntiles) issue(kg, 0);
  for (int jj = 0; jj < ntiles; jj += KG) {                // group kg takes tile j = jj + kg
    const int j = jj + kg, stage = (jj / KG) & 1;
    wait_loads();                                          // this wave's loads of tile j have landed
    __syncthreads();                                       // everyone's; every wave is past tile j - KG
    if (j + KG < ntiles) issue(j + KG, stage ^ 1);
    const uint8_t* L = lds + (2 * kg + stage) * T::BYTES;
    const int kb = j * BKV;                                // KG = 2: a group without a tile computes what no one reads
    // the whole tile is above this wave's diagonal (KG = 2: never, 64 queries end inside the last tile)
    if (KG == 1 && CAUSAL && kb > qw + 31) continue;

    // P.V of block g of the tile in Lt: pw the codes of its 32 keys, psb its scale byte
    uint32_t vsw[NDB][VW];
    auto pv = [&](auto G_, const uint8_t* Lt, const v4i pw, int psb) {
      constexpr int g = decltype(G_)::value;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const v4i a = *reinterpret_cast<const v4i*>(Lt + v_op(kg * NDB + db, g));
        oacc[db] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_op(a), as_op(pw), oacc[db], 4, 4, 2 * (g & 1),
                                                                   (int)vsw[db][g >> 1], 0, psb);
      }
    };
    // the softmax state over a tile with row maximum tm (c2 tm = tc): O is
    // rescaled, the tile's V^T scales are read, and the factor of l returned
    int kfold, kf127;
    auto advance = [&](const uint8_t* Lt, int kbt, float tm, float tc) {
      const float m_new = smax(m, tm);
      const float mc = m_new * c2;
      const float delta = tc - mc;
      const float kf = __builtin_floorf(delta);              // c2 (t - m_new) <= 0 split into k and f in [0, 1)
      const float f = delta - kf;
      const float gam = __builtin_amdgcn_exp2f((mc_old - mc) + (f_old - f));
      kfold = (int)__builtin_fmaxf(kf, -300.0f);
      kf127 = kfold + 127;                                   // P's scale byte is e + kfold + 127, clamped at 0
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] *= gam;
      // V^T scale bytes of this lane's dim rows, block 2g + hi of the tile in byte 2(g & 1) of dword g >> 1
      // (read as v2u, not uint2: see sage_common.h; as uint2 this read waited for
      // the whole prefetch of tile j + 1: B4 H32 N4096 D128 681 -> 643 us a call)
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const uint8_t* vp = Lt + T::VS_OFF + (32 * (kg * NDB + db) + col) * 4 * VW;
        if constexpr (VW == 2) {
          const v2u w2 = *reinterpret_cast<const v2u*>(vp);
          vsw[db][0] = w2[0] >> (8 * hi);
          vsw[db][1] = w2[1] >> (8 * hi);
        } else {
          vsw[db][0] = *reinterpret_cast<const uint32_t*>(vp) >> (8 * ((BKV == 64 ? (kbt / 32) & 3 : 0) + hi));
        }
      }
      m = m_new;
      mc_old = mc;
      f_old = f;
      return gam;
    };
    // KG = 2: where the wave of query group `wave` and KV group k leaves P's codes of block g
    auto xp = [&](int k, int g) {
      return (X::IN_K ? lds + (2 * k + stage) * T::BYTES + T::KC_OFF + (wave * NG + g) * 1024
                      : lds + X::XP_OFF + ((k * QW + wave) * NG + g) * 1024) + lane * 16;
    };
    float* const xs = reinterpret_cast<float*>(lds + X::XS_OFF) + lane;
    const int wx = kg * QW + wave;

    // S^T = K^ . Q^T for the tile.  K-step s takes channel block s + NKS hi in
    // lane half hi (blocks s and s + NKS), so each lane's K and Q scale bytes
    // for the NKS steps are one 16-bit half of the row's scale word, selected by
    // op_sel s.  S is exact, so the grouping of blocks into steps does not
    // change it.
    v16f sacc[NSUB];
#pragma unroll
    for (int t = 0; t < NSUB; ++t) {
      uint32_t ksc;
      if constexpr (D == 128) ksc = *reinterpret_cast<const uint16_t*>(L + T::KS_OFF + (32 * t + col) * 4 + 2 * hi);
      else ksc = L[T::KS_OFF + (32 * t + col) * 2 + hi];
      v16f acc = v16f{};
      static_for<NKS>([&](auto S_) {
        constexpr int s = decltype(S_)::value;
        const v4i a = *reinterpret_cast<const v4i*>(L + k_op(t, s));
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_op(a), as_op(qreg[s]), acc, 4, 4, s, (int)ksc, s,
                                                              (int)qsc);
      });
      sacc[t] = acc;
    }
    if constexpr (SQ) {
      // S = fl32(S + bias), elements as below
#pragma unroll
      for (int u = 0; u < NSUB; ++u) {
        const float* bp = reinterpret_cast<const float*>(L + T::BIAS_OFF) + 64 * (u >> 1) + 32 * hi + 16 * (u & 1);
#pragma unroll
        for (int w4 = 0; w4 < 4; ++w4) {
          const v4f b = *reinterpret_cast<const v4f*>(bp + 4 * w4);
#pragma unroll
          for (int r = 0; r < 4; ++r) sacc[u][4 * w4 + r] = sacc[u][4 * w4 + r] + b[r];
        }
      }
    }
    if constexpr (KG == 2 && X::IN_K) lds_barrier();         // K^'s codes have been read
    const bool need_mask = (kb + BKV > N) || (CAUSAL && kb + BKV - 1 > qw);
    if (need_mask) {
      // element (u, v) is key kb + 32 hi + c with c = 64 (u >> 1) + 16 (u & 1) + v;
      // it is kept iff c < rem.  The sign bit of c - rem turns -inf into the
      // bound +inf for kept keys, and min(S, bound) applies it -- plain bit
      // arithmetic, so no per-element lane masks are formed.
      const int rem = (CAUSAL ? min(N, qi + 1) : N) - kb - 32 * hi;
#pragma unroll
      for (int u = 0; u < NSUB; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int c = 64 * (u >> 1) + 16 * (u & 1) + v;
          const float bound = __uint_as_float(0xFF800000u ^ ((uint32_t)(c - rem) & 0x80000000u));
          sacc[u][v] = smin(sacc[u][v], bound);
        }
    }
    // tile row max (raw scores); the max of a P block is lane-local
    float bm[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      float x = sacc[2 * g][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) x = smax(x, sacc[2 * g][v]);
#pragma unroll
      for (int v = 0; v < 16; ++v) x = smax(x, sacc[2 * g + 1][v]);
      bm[g] = x;
    }
    float tl = bm[0];
#pragma unroll
    for (int g = 1; g < NG; ++g) tl = smax(tl, bm[g]);
    // row max over the two lane halves that share a query
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tl), __float_as_uint(tl), false, false);
    const float t = smax(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    const float tc = t * c2;
    float gam = 0.0f;
    if constexpr (KG == 1) gam = advance(L, kb, t, tc);
    const float bias = log6 - tc;                          // P~2 = 2^{fma(S, c2, log2 6 - t c2)}
    float ps[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t ew = 0;                                       // KG = 2: the block exponents, a byte each
    static_for<NG>([&](auto G_) {
      constexpr int g = decltype(G_)::value;
      // smallest e with 6 2^e >= blockmax(P~2) = 6 2^{c2 (bm - t)}; a fully
      // masked block (bm = -inf) takes the floor -126
      const int e = (int)__builtin_fmaxf(__builtin_ceilf((bm[g] - t) * c2), -126.0f);
      const float escale = __builtin_ldexpf(1.0f, e);      // the convert divides by it exactly
      uint32_t w[4];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int tt = 2 * g + half;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          // the four converts write all four bytes, so the word starts from the
          // bits of the first value rather than from a zero
          uint32_t word = 0;
          static_for<4>([&](auto I_) {
            constexpr int i = decltype(I_)::value;
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[tt][8 * q + 2 * i], c2, bias));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[tt][8 * q + 2 * i + 1], c2, bias));
            ps[(2 * half + q) & 3] += p0;
            ps[(2 * half + q) & 3] += p1;
            if constexpr (i == 0) word = __float_as_uint(p0);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, p0, p1, escale, i);
          });
          w[2 * half + q] = word;
        }
      }
      const v4i pw = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
      if constexpr (KG == 1) {
        const int sb = e + kf127;
        pv(G_, L, pw, sb < 0 ? 0 : sb);
      } else {
        *reinterpret_cast<v4i*>(xp(kg, g)) = pw;
        ew |= ((uint32_t)e & 255u) << (8 * g);
      }
    });
    const float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
    if constexpr (KG == 1) {
      lsum_acc = lsum_acc * gam + __builtin_ldexpf(psum, kfold);
    } else {
      xs[wx * 192] = t;
      xs[wx * 192 + 64] = psum;
      xs[wx * 192 + 128] = __uint_as_float(ew);
    }
    if constexpr (KG == 2) {
      lds_barrier();                                       // both tiles' P
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (k == 1 && jj + 1 >= ntiles) break;
        const int wk = k * QW + wave;
        const uint8_t* Lk = lds + (2 * k + stage) * T::BYTES;
        const float tk = xs[wk * 192], pk = xs[wk * 192 + 64];
        const uint32_t ek = __float_as_uint(xs[wk * 192 + 128]);
        const float gam = advance(Lk, (jj + k) * BKV, tk, tk * c2);
        static_for<NG>([&](auto G_) {
          constexpr int g = decltype(G_)::value;
          const int sb = ((int)(ek << (24 - 8 * g)) >> 24) + kf127;
          pv(G_, Lk, *reinterpret_cast<const v4i*>(xp(k, g)), sb < 0 ? 0 : sb);
        });
        lsum_acc = lsum_acc * gam + __builtin_ldexpf(pk, kfold);
      }
    }
  }

  const float ltot = lsum_acc + __shfl_xor(lsum_acc, 32, 64);
  const float inv = 1.0f / ltot;
  if (qi < N) {
    uint8_t* obase = reinterpret_cast<uint8_t*>(o);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d0 = 32 * (kg * NDB + db) + 8 * g + 4 * hi;
        const size_t idx = ((size_t)bh * N + qi) * D + d0;
        const float a0 = oacc[db][4 * g] * inv, a1 = oacc[db][4 * g + 1] * inv;
        const float a2 = oacc[db][4 * g + 2] * inv, a3 = oacc[db][4 * g + 3] * inv;
        if (OUT == 0) {
          *reinterpret_cast<float4*>(obase + idx * 4) = make_float4(a0, a1, a2, a3);
        } else {
          uint16_t h0, h1, h2, h3;
          if (OUT == 1) { h0 = f32_to_bf16_rne(a0); h1 = f32_to_bf16_rne(a1); h2 = f32_to_bf16_rne(a2); h3 = f32_to_bf16_rne(a3); }
          else { h0 = f32_to_fp16_rne(a0); h1 = f32_to_fp16_rne(a1); h2 = f32_to_fp16_rne(a2); h3 = f32_to_fp16_rne(a3); }
          *reinterpret_cast<uint2*>(obase + idx * 2) = make_uint2((uint32_t)h0 | ((uint32_t)h1 << 16), (uint32_t)h2 | ((uint32_t)h3 << 16));
        }
      }
  }
}

template <int D, int BKV, bool CAUSAL, int OUT, bool SQ, int W, int KG>
static hipError_t launch_fp4_t(const void* qc, const void* qs, const void* kc, const void* ks, const void* vc,
                               const void* vs, const float* qkb, void* o, int BH, int N, int Np, float c2, float log6,
                               hipStream_t st) {
  constexpr int AQW = 32 * W / KG;
  const int nqt = (N + AQW - 1) / AQW;
  hipLaunchKernelGGL((attn_fp4_mx_kernel<D, BKV, CAUSAL, OUT, SQ, W, KG>), dim3((unsigned)(nqt * BH)), dim3(64 * W), 0, st,
                     (const uint8_t*)qc, (const uint8_t*)qs, (const uint8_t*)kc, (const uint8_t*)ks, (const uint8_t*)vc,
                     (const uint8_t*)vs, qkb, o, BH, N, Np, nqt, c2, log6);
  return hipGetLastError();
}

template <int D, int BKV, bool CAUSAL, bool SQ, int W, int KG>
static hipError_t launch_fp4_o(int out, const void* qc, const void* qs, const void* kc, const void* ks, const void* vc,
                               const void* vs, const float* qkb, void* o, int BH, int N, int Np, float c2, float log6,
                               hipStream_t st) {
  if (out == 0) return launch_fp4_t<D, BKV, CAUSAL, 0, SQ, W, KG>(qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
  if (out == 1) return launch_fp4_t<D, BKV, CAUSAL, 1, SQ, W, KG>(qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
  return launch_fp4_t<D, BKV, CAUSAL, 2, SQ, W, KG>(qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
}

// KV groups of a call: two where 128-query tiles are too few for the GPU and
// there are at least two KV tiles to share (both give the same bits).  Attention
// alone, N = 4096, one group -> two, in us, by number of 128-query tiles:
//               128           256           384           512
//   D 128, 256 keys  40.2 -> 27.9  42.2 -> 54.2  66 -> 80     (two groups: one workgroup per CU)
//   D 128, 128 keys  43.3 -> 30.7  45.3 -> 46.1  68.4 -> 67   73 -> 85
//     causal         43.5 -> 31.1  44.5 -> 32.9  67.1 -> 53.5 68 -> 54 (N = 16384: 210 -> 236)
//   D 128, 64 keys   55.9 -> 38.2  58.6 -> 52.0  80.8 -> 72.8 86 -> 96
//   D 64, 256 keys   32.5 -> 21.8  33.4 -> 34.2  53.8 -> 49.2 55 -> 63
//   D 64, 128 keys   36.1 -> 25.1  36.9 -> 36.6  57.6 -> 49.9 58 -> 64
//   D 64, 64 keys    46.0 -> 31.8  46.8 -> 45.3  72.4 -> 62.2 71 -> 74
// (N = 16384, D 128, 128 keys: 256 tiles 163 -> 170, 384 250 -> 254.)
static int fp4_kv_groups(int BH, int N, int D, int bkv, bool causal) {
  const long long tiles = (long long)BH * ((N + 127) / 128);
  const int most = D == 128 && (bkv == 256 || (bkv == 128 && !causal)) ? 128 : 384;
  return tiles <= most && N > bkv ? 2 : 1;
}

template <int D, int BKV, bool CAUSAL>
static hipError_t launch_fp4_s(int out, const void* qc, const void* qs, const void* kc, const void* ks, const void* vc,
                               const void* vs, const float* qkb, void* o, int BH, int N, int Np, float c2, float log6,
                               hipStream_t st) {
  if (fp4_kv_groups(BH, N, D, BKV, CAUSAL) == 2)
    return qkb ? launch_fp4_o<D, BKV, CAUSAL, true, 4, 2>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st)
               : launch_fp4_o<D, BKV, CAUSAL, false, 4, 2>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
  return qkb ? launch_fp4_o<D, BKV, CAUSAL, true, 4, 1>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st)
             : launch_fp4_o<D, BKV, CAUSAL, false, 4, 1>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
}

// qkb: smoothing-Q bias [BH, ceil(N/128), Np] fp32, or null without smoothing Q.
hipError_t launch_attn_fp4_mx(const void* qc, const void* qs, const void* kc, const void* ks, const void* vc,
                              const void* vs, const float* qkb, void* o, int BH, int N, int Np, int D, int bkv,
                              bool causal, int out, float c2, float log6, bool wg256, hipStream_t st) {
#define SAGE_A(DD, BB)                                                                                    \
  return causal ? launch_fp4_s<DD, BB, true>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st) \
                : launch_fp4_s<DD, BB, false>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st)
  if (wg256 && fp4_kv_groups(BH, N, D, 256, false) == 1) {
    // 256-query workgroups: 256-key tiles, non-causal, without smoothing Q (checked by the caller); calls
    // with too few tiles for the GPU take two KV groups with the flag too
    if (D == 128) return launch_fp4_o<128, 256, false, false, 8, 1>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
    return launch_fp4_o<64, 256, false, false, 8, 1>(out, qc, qs, kc, ks, vc, vs, qkb, o, BH, N, Np, c2, log6, st);
  }
  if (D == 128) { if (bkv == 256) { SAGE_A(128, 256); } else if (bkv == 128) { SAGE_A(128, 128); } else { SAGE_A(128, 64); } }
  if (bkv == 256) { SAGE_A(64, 256); } else if (bkv == 128) { SAGE_A(64, 128); } else { SAGE_A(64, 64); }
#undef SAGE_A
}

}  // namespace sage
