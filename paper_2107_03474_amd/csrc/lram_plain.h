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

// Lookups per wave of a kernel that is built for `waves` waves per SIMD: as few as
// fill them.  A batch that leaves a wave at most two takes the general search,
// one lookup after the other (tile_search false): a tile's selection is a longer
// chain than the scans of two lookups.  Above, a wave searches tiles, and spends a
// tile's cost whatever the tile holds (about 900 instructions; 120 more for each
// pair of lookups), so it takes an even number, a whole tile at most below 524,288
// lookups and two from there on.  us, tiles of 2 / tiles of 4 / general search with 1 (up to
// 4,096) or 2 lookups per wave, m = 64 bf16, 2^24 rows: forward of 300 lookups 7.7 / - / 6.7, of 2,048
// 9.9 / - / 7.6, of 5,000 12.2 / 12.0 / 10.4, of 8,192 14.5 / 13.3 / 12.1; backward with row atomics
// 14.6 / - / 9.8, 25.5 / - / 22.9, 51.2 / 53.4 / 51.9, 66.3 / 66.2 / 67.4; flags of 300 (2^16 rows) 9.1 / - /
// 6.3, of 8,192 13.2 / 11.7 / 11.5.  General search with four: 15.1, 69.9 and 13.6 at 8,192.
// Three waves per SIMD (m = 64 fp32): forward of 6,000 13.0 / 13.4 / 11.1, of 7,000 15.9 / 12.8 / 15.9; two
// (inline activation layer) of 2,048 9.3 / - / 8.9, of 3,072 11.9 / - / 13.9 with one lookup.
// Tiles of 2 / 4 / 6 / 8 / 12 / 16, forward: 16,384 lookups 22.5 / 17.2 / 16.7 / 17.1 / 19.8 / 22.2; 24,576
// 28.4 / 25.3 / 19.9 / 20.1 / 21.2 / 23.8; 32,768 35.9 / 28.0 / 29.1 / 23.3 / 24.5 / 24.7; 49,152 50.5 / 40.0 / 34.1 /
// 35.6 / 31.4 / 32.1; backward: 12,000 109 / 104 / 106 / 110 / - / -; 32,768 277 / 277 / 288 / 275 / 281 / 284.  Forward of
// 262,144 (2^20 rows, m = 64 fp32), 4 / 8 / 16 / 32 / 64 to a wave: 352 / 309 / 304 / 305 / 320.  Batches below
// 524,288 that need a few rounds of waves (max_rounds at most: 2, any number where row atomics hide the
// tiles' cost, none where a batch is merged) spread evenly over them; whole tiles leave the last
// round nearly empty: 70,000 lookups, whole tiles / evenly, forward (2^24 rows, m = 32 bf16) 61.1 / 51.6,
// backward with row atomics (2^20, m = 64 bf16) 511 / 464.  From 2^30 lookups on
// a wave takes 64: 32 would make a grid of 2^32 work-items, which no launch accepts.
constexpr int64_t fill_waves(int64_t L, int waves) { return (L + waves * SIMDS - 1) / (waves * SIMDS); }
constexpr bool tile_search(int64_t L, int waves) { return fill_waves(L, waves) > 2; }
constexpr int32_t lookups_per_wave(int64_t L, int waves, int64_t max_rounds) {
  const int64_t n = fill_waves(L, waves);
  if (n <= 2) return (int32_t)(n < 1 ? 1 : n);
  if (L < (int64_t(1) << 19)) {
    const int64_t rounds = (n + TILE - 1) / TILE;
    return rounds > max_rounds ? TILE : (int32_t)(((n + rounds - 1) / rounds + 1) / 2 * 2);
  }
  return L < (int64_t(1) << 30) ? 2 * TILE : WAVE;
}
// Lists other than the closest 32, whose search costs the same for every lookup (64 at most, and
// evenly over the rounds of waves).
constexpr int32_t lookups_per_wave_k(int64_t L) {
  const int64_t n = fill_waves(L, 4), rounds = (n + WAVE - 1) / WAVE;
  return (int32_t)(n < 1 ? 1 : (n + rounds - 1) / rounds);
}

// h mod K for K even, at least 2, and h in [-K - 3, K + 3] (as uint32_t: two's
// complement): a parity for K = 2, otherwise up to two periods up or one down.  The
// minimum keeps any other h below K, so that nothing can address outside the table.
constexpr uint32_t torus_coord(uint32_t h, uint32_t K) {
  int32_t y = (int32_t)h;
  y += y < 0 ? (int32_t)K : 0;
  y += y < 0 ? (int32_t)K : 0;
  y -= y >= (int32_t)K ? (int32_t)K : 0;
  return K == 2u ? (h & 1u) : ((uint32_t)y < K - 1u ? (uint32_t)y : K - 1u);
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
  const int32_t lpw = lookups_per_wave(L, 4, INT64_MAX);
  return !hist_merged(L) || lpw < TILE / 2 ? lpw : (L < 98304 ? TILE / 2 : (lpw < TILE ? lpw : TILE));
}

// Lookups per launch of the access histogram, whose waves take one tile each:
// four work-items per lookup.  Larger batches are launched in pieces.
constexpr int64_t HIST_PIECE = int64_t(1) << 29;

}  // namespace
