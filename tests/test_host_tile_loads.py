"""Every KV tile load of the FP4 kernel stays inside its head's tensor: the
kernel's own load code, compiled for the host with a buffer load that checks its
range, and run for every wave, lane, job and tile."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRE = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <initializer_list>
using std::min;
static long long loads = 0, bad = 0;
struct Rsrc { unsigned long long bytes; };
typedef Rsrc __amdgpu_buffer_rsrc_t;
static Rsrc make_rsrc(const void*, uint32_t bytes) { return {bytes}; }
static uint8_t lds[1 << 18];
static uint8_t* stage_end;
static void load(Rsrc r, uint32_t voff, uint32_t soff, int size, int lane, uint8_t* dst) {
  ++loads;
  if ((unsigned long long)voff + soff + size > r.bytes || dst + size * (lane + 1) > stage_end) {
    if (bad++ < 5) printf("%u + %u + %d > %llu\n", voff, soff, size, r.bytes);
  }
}
#define buf_load16(r, v, s, d) load(r, v, s, 16, lane, d)
#define buf_load4(r, v, s, d) load(r, v, s, 4, lane, d)
"""
FN = r"""
template <int D, int BKV, bool SQ, int W, int KG>
static void walk(int N, int step) {
  using T = Fp4Stage<D, BKV, SQ>;
  constexpr int NKS = T::NKS, NG = T::NG, QW = W / KG;
  const int Np = (N + 127) / 128 * 128, ntiles = (N + BKV - 1) / BKV;
  const long long bh = 0;
  const uint8_t *kc = nullptr, *vc = nullptr, *ks = nullptr, *vs = nullptr;
  const float* qkb = nullptr;
  const int q0 = 0;
  for (int kg = 0; kg < KG; ++kg)
    for (int wave = 0; wave < QW; ++wave)
      for (int lane = 0; lane < 64; ++lane) {
        const int col = lane & 31, hi = lane >> 5;
        (void)NG; (void)col; (void)hi;
        @KERNEL@
        for (int j = 0; j < ntiles; j = j == ntiles - 1 ? ntiles : min(j + step, ntiles - 1))
          for (int st = 0; st < 2; ++st) {
            stage_end = lds + (2 * kg + st + 1) * T::BYTES;
            issue(j, st);
          }
      }
}
template <int D> static void all(int N, int step) {
  walk<D, 64, false, 4, 1>(N, step); walk<D, 128, false, 4, 1>(N, step); walk<D, 256, false, 4, 1>(N, step);
  walk<D, 64, true, 4, 2>(N, step); walk<D, 128, true, 4, 2>(N, step); walk<D, 256, true, 4, 2>(N, step);
  walk<D, 256, false, 8, 1>(N, step);
}
int main() {
  for (int N : {1, 64, 65, 128, 129, 255, 256, 257, 384, 385, 640, 1000, 1237}) { all<64>(N, 1); all<128>(N, 1); }
  for (int N : {76800, 1 << 20, (1 << 24) - 127, 1 << 24}) all<128>(N, 1 << 18);   // up to a head of 2^31 elements
  for (int N : {76800, (1 << 25) - 127, 1 << 25}) all<64>(N, 1 << 18);
  printf("%lld loads, %lld out of range\n", loads, bad);
  return bad != 0;
}
"""


@pytest.mark.parametrize("planted", ["", "V", "K"])
def test_fp4_tile_loads_stay_inside_their_tensors(tmp_path, planted):
    """... and the walk finds a tail that is not redirected (planted in a copy)."""
    src = open(os.path.join(ROOT, "paper_2505_11594_amd", "csrc", "attn_fp4.hip")).read()
    swz = src[src.index("template <int NCH>"):src.index("__device__ __forceinline__ v8i as_op")]
    stage = src[src.index("template <int D, int BKV, bool SQ>\nstruct Fp4Stage"):src.index("// Waves per SIMD that the register")]
    code = src[src.index("  constexpr bool ROWS = "):src.index("  // operand addresses in the tile")]
    if planted == "V":
        assert code.count("if constexpr (BKV == 256) v_up = ") == 1
        code = code.replace("if constexpr (BKV == 256) v_up = ", "if constexpr (false) v_up = ")
    if planted == "K":
        assert code.count("if constexpr (K_WAVE) k_up = ") == 1
        code = code.replace("if constexpr (K_WAVE) k_up = ", "if constexpr (false) k_up = ")
    text = PRE + swz + stage + FN.replace("@KERNEL@", code)
    (tmp_path / "t.cpp").write_text(re.sub(r"__device__|__forceinline__", "", text))
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-o", exe, str(tmp_path / "t.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    print(r.stdout)
    assert (r.returncode != 0) == bool(planted), r.stdout
