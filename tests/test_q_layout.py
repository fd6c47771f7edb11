"""The offsets with which the K-split kernel and the MLGRU step load their rows
(csrc/q_layout.h), walked on the host: the scalar offset of every buffer load
stays inside its resource (the range check is only defined there), every live
row's bytes are read from where they were written, and nothing else is in
range."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "q_layout.h"
using namespace mmf;

#define CHECK(c) do { if (!(c)) { std::printf("%s: M=%d K=%d fm=%d tiled=%d s=%d\n", #c, M, K, fm, tiled, s); std::exit(1); } } while (0)

int main() {
  const int Ks[] = {16, 32, 48, 64, 80, 112, 1024, 1040, 2064, 13824};
  const int Ms[] = {1, 15, 16, 17, 31, 33, 45, 64, 65, 70, 100, 129, 257};
  for (int K : Ks) for (int M : Ms) for (int FM = 1; FM <= 4; ++FM) for (int tiled = 0; tiled < 2; ++tiled)
    for (int m0 = 0; m0 < M; m0 += 16 * FM) {
      const int rows = M - m0 < 16 * FM ? M - m0 : 16 * FM, steps = (K + 63) / 64;
      const uint32_t records = static_cast<uint32_t>(rows) * static_cast<uint32_t>(K);
      for (int fm = 0; fm < FM; ++fm) for (int s = 0; s < steps; ++s) {
        const QBlock b = q_block(rows, fm, K, tiled != 0);
        const uint32_t soff = b.base + static_cast<uint32_t>(s) * b.step;
        CHECK(soff <= records);
        for (int lane = 0; lane < 64; ++lane) {
          const int l16 = lane & 15, g = lane >> 4, r = 16 * fm + l16, k = 64 * s + 16 * g;
          const uint32_t voff = q_lane(l16, g, K, tiled != 0, s == steps - 1);
          if (voff < records - soff) CHECK(voff + 16 <= records - soff);  // whole 16-byte pieces of q
          if (r < rows && k < K) {  // where the row's bytes are
            const int mr = rows - 16 * fm < 16 ? rows - 16 * fm : 16;
            const uint32_t want = tiled ? 16 * fm * K + tiled_q_piece(l16, mr, k, K) : r * K + k;
            CHECK(soff + voff == want);
          }
        }
      }
    }
  // the tiled layout holds every 16-byte piece of a block once
  const int M = 0, fm = 0, tiled = 1, s = 0;
  for (int K : Ks) for (int mr = 1; mr <= 16; ++mr) {
    std::set<int> at;
    for (int r = 0; r < mr; ++r) for (int k = 0; k < K; k += 16) at.insert(tiled_q_piece(r, mr, k, K));
    CHECK(static_cast<int>(at.size()) == mr * (K / 16) && *at.begin() == 0 && *at.rbegin() == mr * K - 16);
  }
  // the gates of a row: f, c and g of vector v, or past the resource
  for (int K : Ks) for (int v = 0; v < 64 * 16 * 4; ++v) {
    const GateRow a = gate_row(v, K);
    const uint32_t so[3] = {a.f, a.c, a.g};
    for (uint32_t i = 0; i < 3; ++i) {
      CHECK(a.bytes == 12u * K && so[i] <= a.bytes);
      if (4 * v < K) CHECK(a.lane + so[i] == 4u * (i * K + 4 * v));
      else CHECK(a.lane >= a.bytes - so[i]);
    }
  }
  std::puts("ok");
}
"""


def test_offsets_stay_inside_their_resources(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2406_02528_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
