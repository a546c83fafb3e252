// The tiles of gemm_lds_k (gemm_lds.hip) and which of them a problem gets.  Host arithmetic only, so that the choice can be
// checked without a GPU.
#pragma once
#include <stdint.h>

namespace hift {

// bm x bn outputs per workgroup, `ring` stages of 64 k in LDS; then what a round costs, in 10 ns (see lds_tile).
struct LdsTile { int bm, bn, ring, alone, stage, fixed; };
constexpr LdsTile LDS_TILES[] = {
    {128, 128, 2, 87, 39, 300}, {128, 64, 3, 35, 24, 300}, {64, 128, 3, 35, 24, 300}, {64, 64, 3, 19, 18, 138},
    {64, 64, 4, 15, 22, 153},   {64, 32, 4, 23, 19, 70},   {32, 64, 4, 23, 19, 70},   {32, 32, 4, 20, 10, 90},
    {256, 256, 2, 97, 85, 1500}};
constexpr int N_LDS_TILES = sizeof(LDS_TILES) / sizeof(LDS_TILES[0]);

// Estimated time of a problem on a tile, in 10 ns.
inline int64_t lds_cost(const LdsTile& t, int64_t M, int64_t N, int64_t K, int64_t nz) {
  const int64_t rounds = ((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn) * nz + 255) / 256;
  return rounds * ((K + 63) / 64 * (rounds == 1 ? t.alone : t.stage) + t.fixed);
}

// The tile with the least estimated time: a round of tiles over the 256 compute units takes (stages x time of a stage + what a
// tile costs besides); a stage takes longer when the round is the only one and the workgroup has its compute unit to itself.
// The constants are a fit to measured times of all the tiles in the four layouts (83 sizes: 8 to 65536 rows, 8 to 100000
// columns, k 56 to 11008; 18 batches of 24 to 2048 products): the tile chosen is on average 1.4 % slower than the best and at
// most 1.23 times.  It was made with operands in the caches: where the weights come from HBM a stage takes up to 1.5 times as long (231 x 4096,
// k 11008: 27 us by the fit, 40 measured).  A ring of four 64 x 64 stages is the better one when it runs alone (231 x 4096, k 11008: 40 us, 47 with
// three), three otherwise (three workgroups per compute unit: 1024 x 2304, k 768: 11.3 us, 12.6 with four).  256 x 256 draws half
// the operand bytes per product of 128 x 128, but has a compute unit to itself and hides nothing of its start and end: the better
// one where its rounds are long and nearly full (2048 x 32000, k 4096: 442 us, 128 x 128: 594), not for 2048 x 4096, k 4096 (half
// a round: 83 and 69) nor short k (16384 x 16384, k 256: 275 and 246).
inline int lds_tile(int64_t M, int64_t N, int64_t K, int64_t nz) {
  int best = 0;
  int64_t least = INT64_MAX;
  for (int i = 0; i < N_LDS_TILES; ++i) {
    const int64_t cost = lds_cost(LDS_TILES[i], M, N, K, nz);
    if (cost < least) { least = cost; best = i; }
  }
  return best;
}

// Rings of three stages that leave a compute unit room for one workgroup only, for long k whose tiles are one round.  The loads of a
// stage are then all of its time (231 x 4096, k 22016: 114 of 116 us without products and LDS reads), and what they cost follows the
// bytes that a compute unit draws: twice the tile halves them, and two rounds of smaller tiles become one.  Microseconds before and
// now, weights from HBM: 231 x 12288, k 4096 53 and 46; 231 x 11008, k 4096 (transposed) 55 and 42; 231 x 22016, k 4096 81 and 64;
// 1024 x 4096, k 11008 138 and 109; 1500 x 4096, k 11008 190 and 144; 2048 x 4096, k 4096 77 and 67.
constexpr LdsTile LDS_LONG_TILES[] = {{128, 128, 3, 44, 0, 800}, {256, 128, 3, 60, 0, 1000}};
constexpr int N_LDS_LONG_TILES = sizeof(LDS_LONG_TILES) / sizeof(LDS_LONG_TILES[0]);

// Which of them a problem gets, or -1: none.  The constants put the line where it was measured, by the scale of the fit above (their
// times with weights from HBM are 1.3 times as long): over 115 sizes (64 to 2048 rows, k 1536 to 11008, three layouts) that
// take one, it is 1.19 times as fast as lds_tile's choice, 1.23 with other work beside it, and at worst 3.5 % slower; as 2 to 32 problems in a launch 1.17 to
// 1.26 (56 sizes, at worst 7 % slower: 32 of 1904 x 128, k 1688); with A transposed and B k-major 1.27 (28 sizes, none slower); with GELU or its
// derivative the contractions of a model take 0.84 to 1.02 of the time (36 models of width 1536 to 3072, 231 to 1430 tokens).  Below k 1536 the start
// and the end of a tile, which nothing hides here, are too much of it (720 x 4096, k 1024: 13.2 and 14.5 us).
inline int lds_long_tile(int64_t M, int64_t N, int64_t K, int64_t nz) {
  if (K < 1536) return -1;
  int64_t least = lds_cost(LDS_TILES[lds_tile(M, N, K, nz)], M, N, K, nz);
  int best = -1;
  for (int i = 0; i < N_LDS_LONG_TILES; ++i) {
    const LdsTile& t = LDS_LONG_TILES[i];
    if ((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn) * nz > 256) continue;
    const int64_t cost = lds_cost(t, M, N, K, nz);
    if (cost < least) { least = cost; best = i; }
  }
  return best;
}

}  // namespace hift
