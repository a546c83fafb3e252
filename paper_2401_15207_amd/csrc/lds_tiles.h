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
  const int64_t nk = (K + 63) / 64;
  int best = 0;
  int64_t least = INT64_MAX;
  for (int i = 0; i < N_LDS_TILES; ++i) {
    const LdsTile& t = LDS_TILES[i];
    const int64_t rounds = ((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn) * nz + 255) / 256;
    const int64_t cost = rounds * (nk * (rounds == 1 ? t.alone : t.stage) + t.fixed);
    if (cost < least) { least = cost; best = i; }
  }
  return best;
}

}  // namespace hift
