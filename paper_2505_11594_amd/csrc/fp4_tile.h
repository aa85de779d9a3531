// The FP4 kernel's KV tile in LDS and the loads that fill it, as offsets only:
// plain C++, so that a host program can check every load against its tensor.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define SAGE_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define SAGE_HD inline
#endif

namespace sage {

// Swizzle of a tile row's NCH 16-byte chunks: 16 consecutive rows at one chunk fall on distinct bank groups.
template <int NCH>
SAGE_HD constexpr int fp4_swz(int row) {
  return NCH == 8 ? (row >> 1) & 7 : NCH == 4 ? (row >> 2) & 3 : (row >> 3) & 1;
}

// One LDS stage of a KV tile: K^ and V^T codes (the order inside is the load
// jobs', below), their scales and, with smoothing Q, the tile's BKV entries of
// the query block's GEMV bias.
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

// Load jobs of 1 KiB, shared by the LW waves that load a tile: wave w takes K^
// jobs and V^T jobs b = w + LW i and scale dword jobs jb = w + LW i (K^ scale
// dwords 64jb + lane, then V^T scale dwords 64(jb - NKSJ) + lane, VW per dim row).
// ROWS (256-key tiles, at most four waves): a job is whole tile rows as they lie in memory (K^ rows
// of D/2 bytes, V^T rows of BKV/2), the 16-byte chunks swizzled against bank
// conflicts by the choice of the chunk each lane loads, so every line is
// requested once; operand reads then need an address per K-step.  Otherwise a
// job is one MFMA operand (32 rows x two 16-byte chunks, lane l's bytes at 16 l):
// a line is requested by up to four jobs, but one lane offset serves all
// operand reads, and the 128-key kernels have no registers left (D = 128, 8
// heads x 4096: 76 us a call with ROWS, 65 without; 256-key tiles, 4 heads
// x 4096 in two KV groups 47.7 -> 45.2, B4 H32 N4096 637 -> 618; 256-query
// workgroups, which fetch a tile half as often, 7745 -> 7773 on B1 H32 N32768).
//
// A load's offset from the start of the head's tensor is a lane offset plus a
// uniform one.  Np is a multiple of 128: when the last 256-key tile reaches past
// Np (`tail`), its upper 128 keys are loaded from its lower half (finite values,
// masked as keys >= N), so no load leaves its tensor.
template <int D, int BKV, int LW>
struct Fp4Jobs {
  using T = Fp4Stage<D, BKV, false>;
  static constexpr bool ROWS = BKV == 256 && LW <= 4;
  static constexpr int KJ = (T::NKB + LW - 1) / LW, VJ = (T::NVB + LW - 1) / LW, NSJ = T::NKSJ + T::NVSJ, SJ = (NSJ + LW - 1) / LW;
  static constexpr int KCH = D / 32, VCH = BKV / 32, VR = 64 / VCH;      // ROWS: chunks per row, V^T rows per job
  static_assert(ROWS ? LW % 2 == 0 : LW % T::NKS == 0 && (LW % T::NG == 0 || T::NG % LW == 0), "job layout");
  static_assert(ROWS || BKV < 256 || LW % T::NG == 0, "a wave's V^T jobs lie in one half of a 256-key tile");

  // which 16-byte chunk of its V^T row a lane loads
  SAGE_HD static int v_chunk(int wave, int lane) {
    return ROWS ? (lane % VCH) ^ fp4_swz<VCH>(wave * VR + lane / VCH) : 2 * (wave % T::NG) + (lane >> 5);
  }
  SAGE_HD static uint32_t k_lane(int wave, int lane) {
    if (ROWS) return (uint32_t)(lane / KCH * (D / 2) + 16 * ((lane % KCH) ^ fp4_swz<KCH>(lane / KCH)));
    return (uint32_t)((32 * (wave / T::NKS) + (lane & 31)) * (D / 2) + 16 * (wave % T::NKS) + 16 * T::NKS * (lane >> 5));
  }
  // Whether the tail's redirect of K^ depends on the wave alone (one job each); it is then taken from the lane
  // offset, k_lane - k_back, since the uniform offset may be smaller, else from k_uni.
  static constexpr bool KBACK_LANE = !ROWS && BKV == 256 && LW > T::NKB / 2;
  static_assert(!KBACK_LANE || LW == T::NKB, "one K^ job per wave");
  SAGE_HD static uint32_t k_back(int wave) { return KBACK_LANE && wave >= T::NKB / 2 ? 128u * (D / 2) : 0u; }
  SAGE_HD static uint32_t v_lane(int wave, int lane, int Np) {
    const int row = ROWS ? lane / VCH : 32 * (wave / T::NG) + (lane & 31);
    return (uint32_t)row * (uint32_t)(Np / 2) + 16 * v_chunk(wave, lane);
  }
  // subtracted from v_lane in the tail
  SAGE_HD static uint32_t v_back(int wave, int lane) { return BKV == 256 && v_chunk(wave, lane) >= VCH / 2 ? 64u : 0u; }
  SAGE_HD static uint32_t ks_lane(int lane) { return (uint32_t)(4 * lane); }
  SAGE_HD static uint32_t vs_lane(int lane, int Np) { return (uint32_t)((lane / T::VW) * (Np / 32) + 4 * (lane % T::VW)); }
  SAGE_HD static uint32_t vs_back(int lane) { return (uint32_t)(4 * (lane % T::VW)); }   // the second dword, in the tail
  // uniform offsets of jobs b = wave + LW i and jb of the tile at key kb
  SAGE_HD static bool tail(int kb, int Np) { return BKV == 256 && kb + BKV > Np; }
  SAGE_HD static uint32_t k_uni(int kb, int wave, int i, bool tail) {
    const int b = wave + LW * i;
    const uint32_t back = (!KBACK_LANE && tail && b >= T::NKB / 2) ? 128u * (D / 2) : 0u;
    return (uint32_t)kb * (D / 2) + (ROWS ? (uint32_t)b * 1024u : (uint32_t)i * (32 * LW / T::NKS) * (D / 2)) - back;
  }
  SAGE_HD static uint32_t v_uni(int kb, int wave, int i, int Np) {
    const int b = wave + LW * i;
    return (uint32_t)kb / 2 + (ROWS ? (uint32_t)(b * VR) * (uint32_t)(Np / 2)
                                    : (uint32_t)(LW * i / T::NG) * 32 * (Np / 2) + 32 * (LW * i % T::NG));
  }
  SAGE_HD static uint32_t ks_uni(int kb, int jb, bool tail) {
    const uint32_t back = (tail && 64 * jb * 4 >= T::KS_BYTES / 2) ? T::KS_BYTES / 2 : 0u;
    return (uint32_t)kb * (D / 32) + 256u * jb - back;
  }
  SAGE_HD static bool ks_on(int jb, int lane) { return T::KS_BYTES % 256 == 0 || 256 * jb + 4 * lane < T::KS_BYTES; }
  // 64-key tiles: the aligned dword that holds the tile's two scale bytes
  SAGE_HD static uint32_t vs_uni(int kb, int jb, int Np) {
    return ((uint32_t)kb / 32 & ~3u) + (uint32_t)(jb - T::NKSJ) * (2 / T::VW) * Np;
  }
};

}  // namespace sage
