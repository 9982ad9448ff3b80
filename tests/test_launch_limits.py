"""Launch geometry and index arithmetic on the CPU: lram_plain.h compiled by the host compiler.

A launch takes fewer than 2^32 work-items; every batch size that the entry points accept (L < 2^31) has to stay below
that in the kernels that cover the batch with lookups_per_wave, and in the access histogram's pieces.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_03474_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "lram_plain.h"
int main() {
  const int64_t items = int64_t(1) << 32;
  for (int s = 0; s <= 31; ++s)
    for (int64_t d = -200; d <= 200; ++d) {
      const int64_t L = (int64_t(1) << s) + d;
      if (L < 1 || L > LMAX) continue;
      for (int waves = 1; waves <= 4; ++waves) for (int64_t rounds : {int64_t(1), int64_t(2), INT64_MAX}) {
        const int32_t lpw = waves == 1 ? lookups_per_wave_k(L) : lookups_per_wave(L, waves, rounds);
        const int64_t blocks = blocks_for(L, lpw);
        if (lpw < 1 || lpw > WAVE || blocks * WAVES * lpw < L || blocks * THREADS >= items)
          std::printf("L = %lld waves = %d: %d lookups per wave, %lld blocks\n", (long long)L, waves, lpw, (long long)blocks);
      }
      int64_t covered = 0;
      for (int64_t l0 = 0; l0 < L; l0 += HIST_PIECE) {
        const int64_t n = std::min(L - l0, HIST_PIECE);
        const int32_t lpw = hist_lookups_per_wave(n);
        const int64_t blocks = blocks_for(n, lpw);
        if (lpw < 1 || (hist_merged(n) && lpw > TILE)) std::printf("histogram L = %lld: %d\n", (long long)L, lpw);
        covered += n;
        if (blocks * THREADS >= items) std::printf("histogram L = %lld: %lld blocks\n", (long long)L, (long long)blocks);
      }
      if (covered != L) std::printf("histogram L = %lld: %lld covered\n", (long long)L, (long long)covered);
    }
  return 0;
}
"""


def run_host(tmp_path, program):
    """Output of a C++ program that includes the library's plain headers."""
    src, exe = tmp_path / "t.cc", tmp_path / "t"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


def test_every_accepted_batch_launches(tmp_path):
    assert run_host(tmp_path, PROGRAM) == ""


SMALL = r"""
#include <cstdio>
#include <initializer_list>
#include "lram_plain.h"
int main() {
  for (int waves = 2; waves <= 4; ++waves)
    for (int64_t L = 1; L <= 200000; ++L) {
      const int64_t room = waves * SIMDS;
      const int32_t lpw = lookups_per_wave(L, waves, 1);
      const bool tile = tile_search(L, waves);
      // one lookup each while there is a wave for each, then two, and tiles above: no more than an even number needs
      bool ok = tile == (L > 2 * room) && (tile || lpw == (L > room ? 2 : 1));
      if (tile) ok = lpw % 2 == 0 && lpw <= TILE && (lpw == 4 || (lpw - 2) * room < L) && (lpw == TILE || lpw * room >= L);
      // evenly over as many rounds as whole tiles need: no more rounds, and no more lookups than they take
      for (int64_t most : {int64_t(2), INT64_MAX}) {
        const int64_t rounds = (L + TILE * room - 1) / (TILE * room);
        const int32_t even = lookups_per_wave(L, waves, most);
        ok = ok && (rounds == 1 || rounds > most ? even == lpw
                                                 : even % 2 == 0 && even <= TILE && even * room * rounds >= L &&
                                                       (even - 2) * room * rounds < L);
      }
      if (!ok) std::printf("%d waves: %lld %d %d\n", waves, (long long)L, tile, lpw);
    }
  return 0;
}
"""


def test_lookups_per_wave_fill_the_simds(tmp_path):
    assert run_host(tmp_path, SMALL) == ""


WRAP = r"""
#include <cstdio>
#include <initializer_list>
#include "lram_plain.h"
int main() {
  for (int K = 2; K <= 8192; K += K < 64 ? 2 : 62)
    for (int h = -K - 3; h <= K + 3; ++h) {
      const uint32_t want = (uint32_t)(((h % K) + K) % K), got = torus_coord((uint32_t)h, (uint32_t)K);
      if (got != want) std::printf("K = %d h = %d: %u, not %u\n", K, h, got, want);
    }
  for (uint32_t K : {2u, 4u, 6u, 8192u})
    for (uint32_t h = 0; h < 0xFFFF0000u; h += 65521u)
      if (torus_coord(h, K) >= K) std::printf("K = %u h = %u: outside\n", K, h);
  return 0;
}
"""


def test_torus_coordinates(tmp_path):
    """The wrap of the per-query tables over the whole range of a point's coordinate, and inside the table for any."""
    assert run_host(tmp_path, WRAP) == ""


@pytest.mark.gpu
def test_histogram_of_a_billion_lookups():
    """2^30 lookups, the first size whose tiles would make 2^32 work-items in one launch, on 2^20 locations: the total
    is the sum of the weights of a sample of the same queries (a fp32 histogram entry sums about 32,768 terms, partly
    merged before: relative error below 2^15 2^-24 = 2e-3)."""
    import torch

    import paper_2107_03474_amd as lram

    K, L, dev = (4, 4, 4, 4, 8, 8, 8, 8), 1 << 30, "cuda"
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 34 GB for the queries")
    g = torch.Generator(device=dev)
    g.manual_seed(0)
    piece = torch.rand((1 << 20, 8), generator=g, device=dev) * torch.tensor(K, device=dev)
    q = piece.repeat(L >> 20, 1)
    hist = lram.access_histogram(q, K).double()
    ref = lram.access_histogram(piece, K).double() * (L >> 20)
    assert ((hist - ref).abs() <= 2e-3 * ref).all()
