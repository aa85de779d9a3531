"""Every KV tile load of the FP4 kernel stays inside its head's tensor: the offsets
of csrc/fp4_tile.h, which the kernel uses as they are, walked on the host for
every wave, lane, job and tile."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "fp4_tile.h"
using namespace sage;
static long long loads = 0, bad = 0;
static void in(const char* what, int N, int kb, uint32_t lane, uint32_t uni, uint32_t size, unsigned long long bytes) {
  ++loads;
  if ((unsigned long long)lane + uni + size > bytes && bad++ < 5)
    printf("%s N=%d kb=%d: %u + %u + %u > %llu\n", what, N, kb, lane, uni, size, bytes);
}
template <int D, int BKV, int LW> static void walk(int N, int step) {
  using J = Fp4Jobs<D, BKV, LW>;
  using T = typename J::T;
  const unsigned long long Np = (N + 127) / 128 * 128;
  const int last = (N + BKV - 1) / BKV - 1;
  for (int j = 0; j <= last; j = j == last ? j + 1 : (j + step < last ? j + step : last)) {
    const int kb = j * BKV;
    const bool tail = J::tail(kb, (int)Np);
    for (int w = 0; w < LW; ++w)
      for (int l = 0; l < 64; ++l) {
        for (int i = 0; i < J::KJ && w + LW * i < T::NKB; ++i)
          in("K", N, kb, J::k_lane(w, l) - (tail ? J::k_back(w) : 0), J::k_uni(kb, w, i, tail), 16, Np * D / 2);
        for (int i = 0; i < J::VJ && w + LW * i < T::NVB; ++i)
          in("V", N, kb, J::v_lane(w, l, (int)Np) - (tail ? J::v_back(w, l) : 0), J::v_uni(kb, w, i, (int)Np), 16, Np * D / 2);
        for (int i = 0; i < J::SJ; ++i) {
          const int jb = w + LW * i;
          if (jb < T::NKSJ) {
            if (J::ks_on(jb, l)) in("K scales", N, kb, J::ks_lane(l), J::ks_uni(kb, jb, tail), 4, Np * D / 32);
          } else if (jb < J::NSJ) {
            in("V scales", N, kb, J::vs_lane(l, (int)Np) - (tail ? J::vs_back(l) : 0), J::vs_uni(kb, jb, (int)Np), 4, Np * D / 32);
          }
        }
      }
  }
}
template <int D> static void all(int N, int step) {
  walk<D, 64, 4>(N, step); walk<D, 128, 4>(N, step); walk<D, 256, 4>(N, step); walk<D, 256, 8>(N, step);
  walk<D, 64, 2>(N, step); walk<D, 128, 2>(N, step); walk<D, 256, 2>(N, step);
}
int main() {
  for (int N : {1, 64, 65, 128, 129, 255, 256, 257, 384, 385, 640, 1000, 1237}) { all<64>(N, 1); all<128>(N, 1); }
  for (int N : {76800, 1 << 20, (1 << 24) - 127, 1 << 24}) all<128>(N, 1 << 18);   // up to a head of 2^31 elements
  for (int N : {76800, (1 << 25) - 127, 1 << 25}) all<64>(N, 1 << 18);
  printf("%lld loads, %lld out of range\n", loads, bad);
  return bad != 0;
}
"""


@pytest.mark.parametrize("planted", [False, True])
def test_fp4_tile_loads_stay_inside_their_tensors(tmp_path, planted):
    """... and the walk finds a tail that is not redirected (planted in a copy)."""
    csrc = os.path.join(ROOT, "paper_2505_11594_amd", "csrc")
    hdr = open(os.path.join(csrc, "fp4_tile.h")).read()
    if planted:
        assert hdr.count("return BKV == 256 && v_chunk") == 1
        hdr = hdr.replace("return BKV == 256 && v_chunk", "return ROWS && v_chunk")
    (tmp_path / "fp4_tile.h").write_text(hdr)
    (tmp_path / "t.cpp").write_text(SRC)
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, str(tmp_path / "t.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    print(r.stdout)
    assert (r.returncode != 0) == planted, r.stdout
