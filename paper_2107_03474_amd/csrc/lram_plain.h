// lram_plain.h -- part of liblram.
//
// Launch geometry and index arithmetic in plain C++ (no HIP), so that a host
// compiler can check them over every size the entry points accept.

#pragma once

#include <stdint.h>

namespace {

constexpr int WAVE = 64;
constexpr int WAVES = 4;                 // waves per workgroup
constexpr int THREADS = WAVE * WAVES;
// Lookups that a wave searches together: phase A spreads each over four lanes,
// the tile selection over four lanes of a matrix product's result.
constexpr int TILE = 16;
constexpr int64_t SIMDS = 256 * 4;
constexpr int64_t LMAX = (int64_t(1) << 31) - 1;  // lookups per call

// Whether the closest 32 of a batch are searched tile by tile, or one lookup per
// wave by the general search: a tile's selection is a longer chain than one
// lookup's scan, and two lookups on a wave scatter one after the other, so it pays
// once a SIMD would have more than four waves (two behind the activation
// layer's inline coordinates, whose kernels are built for two).  us, tiles with
// two lookups per wave / general search with one (2^16 rows, m = 32 fp32): forward of
// 300 lookups 9.8 / 6.9, of 2,048 9.7 / 7.3, of 4,096 10.4 / 9.0; backward 12.9 / 8.3, 14.3 /
// 12.8, 19.9 / 19.6; flags 9.1 / 6.3, 9.0 / 6.7, 9.7 / 8.1.  From 4,097 on two lookups
// share a wave either way: forward 10.1 / 12.7, backward 22.6 / 26.4.  Activation
// layer, forward (2^18 rows, m = 64 fp32): 2,048 lookups 9.3 / 8.9, 3,072 11.9 / 13.9.
constexpr bool tile_search(int64_t L, bool inline_theta) { return L > (inline_theta ? 2 : 4) * SIMDS; }

// Lookups per wave.  A wave that searches tiles spends a tile's cost whatever
// the tile holds (about 900 instructions; 120 more for each pair of lookups), so
// small batches put two lookups on a wave, more once every SIMD has two
// waves, up to a whole tile from 32,768 lookups on.  Forward, lookups per
// wave 2 / 4 / 8 / 16 / 32 / 64: 16,384 lookups 28 / 21 / 19.9 / 22 / 37 / - us; 65,536 95 / 67 / 55 /
// 51 / 57 / 87; 262,144 (2^20 rows, m = 64 fp32) - / 352 / 309 / 304 / 305 / 320.  The
// general search (tile = false) costs the same for every lookup: one each until
// every SIMD has four waves, then up to 64.  From 2^30 lookups on a wave takes 64
// either way: 32 would make a grid of 2^32 work-items, which no launch accepts.
constexpr int32_t lookups_per_wave(int64_t L, bool tile) {
  if (!tile || L >= (int64_t(1) << 30)) {
    const int64_t lpw = (L + 4 * SIMDS - 1) / (4 * SIMDS);
    return (int32_t)(lpw < 1 ? 1 : (lpw > WAVE ? WAVE : lpw));
  }
  const int64_t lpw = ((L + 2 * SIMDS - 1) / (2 * SIMDS) + 1) / 2 * 2;
  const int64_t top = L < (int64_t(1) << 19) ? TILE : 2 * TILE;
  return (int32_t)(lpw < 2 ? 2 : (lpw > top ? top : lpw));
}

// h mod K for K even, at least 2, and h in [-K - 3, K + 3] (as uint32_t: two's
// complement): a parity for K = 2; otherwise h + 2 K lies in [K - 3, 3 K + 3], never
// negative, and three periods come off one by one, each by an unsigned minimum (a
// step too far leaves the range).  The last minimum keeps any other h
// below K, so that nothing can address outside the table.
constexpr uint32_t torus_coord(uint32_t h, uint32_t K) {
  auto least = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
  uint32_t Y = h + 2u * K;
  Y = least(Y, Y - K);
  Y = least(Y, Y - K);
  Y = least(Y, Y - K);
  return K == 2u ? (h & 1u) : least(Y, K - 1u);
}

// Workgroups that cover L lookups, lpw to a wave.
constexpr int64_t blocks_for(int64_t L, int32_t lpw) {
  const int64_t per_block = (int64_t)lpw * WAVES;
  return (L + per_block - 1) / per_block;
}

// The access histogram: whether a batch's pairs are merged per workgroup before
// they are added (measured beside k_access_hist), and the lookups per wave.
constexpr bool hist_merged(int64_t L) { return L >= 16384; }
constexpr int32_t hist_lookups_per_wave(int64_t L) {
  if (!hist_merged(L)) return lookups_per_wave(L, tile_search(L, false));
  const int32_t lpw = lookups_per_wave(L, false);
  return L < 98304 ? (lpw < TILE / 2 ? lpw : TILE / 2) : TILE;
}

// Lookups per launch of the access histogram, whose waves take one tile each:
// four work-items per lookup.  Larger batches are launched in pieces.
constexpr int64_t HIST_PIECE = int64_t(1) << 29;

}  // namespace
