// The update of matrices that the model multiplies from MFMA fragment-order copies: optimizer and packing in one pass.
//
// opt_pack_k: a workgroup updates a tile of 32 rows x 256 columns (rows of 1 KB in every fp32 array, read and written once), leaves the
// rounded new values in LDS, and writes from there the tile's part of the forward copy (one 32-row block, 16 k-steps: 16 KB in a row) and
// of the transposed one (eight blocks, two k-steps each), as pack_b_tile_k does (gemm.hip).  Memory bound: AdamW reads 16 and writes 12
// bytes of fp32 a parameter, and 2 per copy.  The packers by themselves read the new master weights again for each copy, 8 bytes a
// parameter more: a layer of 202 M parameters took 1.03 ms in opt_k and 0.45 in the packers, and takes 1.04 or 1.13 here, in a step, by how the arrays happen to lie.  Loads
// go out in batches of two rows a wavefront with AdamW, four with the optimizers that read fewer arrays, of two wavefronts a SIMD: 64 KB and less in flight in
// a compute unit.  More of them only make memory change rows more often (22016 x 4096 alone: 539 us with four rows and wavefronts, 508 with two wavefronts,
// 495 with two rows as well; one row 530, eight rows 513; momentum at width 4096, updates of a sweep: 2.64 ms with two rows, 2.53 with four).  The copies
// of a launch stay in the caches, where the next step's forward pass finds them (updates of a sweep at width 2048 1.59 -> 1.45 ms, of an encoder of width
// 1024 0.67 -> 0.64), unless they are more than fits there: from COPIES_PAST_CACHES on they go past, as all else here does (22016 x 4096
// alone 495 -> 474 us; in a step the update is 2 % slower and what follows as much faster).
#include "common.h"
#include "kernels.h"
#include "optimizer.h"
#include "packed_layout.h"

namespace hift {
namespace {

constexpr int BLK = 256, TILE_ROWS = 32, TILE_COLS = 256;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef hift_u32x4 u32x4;

struct OptPackTensor {
  OptTensor o;
  int64_t rows, cols;
  u32x4 *fwd, *bwd;   // copies of W and of its transpose, either may be null
  const bf16* gain;   // folded into the forward copy, or null
  int order;          // of the forward copy's blocks
  int tiles_inner;    // tiles along a row
};
constexpr int OPT_PACK_TABLE = 8;
constexpr int64_t COPIES_PAST_CACHES = int64_t(300) << 20;  // (of a launch; the last-level cache has 256 MB)
struct OptPackTable {
  OptPackTensor t[OPT_PACK_TABLE];
  int n;
};

template <int KIND, bool PAST>
__global__ void __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(2, 2))) opt_pack_k(OptHyper h, OptPackTable table) {
  constexpr int PITCH = TILE_COLS * 2 + 16;  // bytes per tile row in LDS; the pad spreads 16-byte reads of one column over the banks
  constexpr int NB = KIND == 0 ? 2 : 4;      // rows of a wavefront whose loads are in flight together
  __shared__ __attribute__((aligned(16))) unsigned char tile[TILE_ROWS * PITCH];
  int q = 0;
  while (q + 1 < table.n && blockIdx.x >= table.t[q + 1].o.block0) ++q;  // uniform over the block
  const OptPackTensor& t = table.t[q];
  const int at = (int)(blockIdx.x - t.o.block0), to = at / t.tiles_inner, ti = at % t.tiles_inner;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = (int64_t)to * TILE_ROWS + wave, col = (int64_t)ti * TILE_COLS + lane * 4;
  const bool col_in = col < t.cols;  // columns come in whole fours
#pragma unroll 1
  for (int batch = 0; batch < TILE_ROWS / 4 / NB; ++batch) {
    float th[NB][4], g[NB][4], a[NB][4], b[NB][4];
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const int64_t row = row0 + (batch * NB + p) * 4, i = row * t.cols + col;
      if (!(col_in && row < t.rows)) continue;
      ldnt<4>(t.o.master + i, th[p]);
      ldnt<4>(t.o.grad + i, g[p]);
      if (KIND != 3) ldnt<4>(t.o.s1 + i, a[p]);
      if (KIND == 0) ldnt<4>(t.o.s2 + i, b[p]);
    }
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const int r = wave + (batch * NB + p) * 4;
      const int64_t row = row0 + (batch * NB + p) * 4, i = row * t.cols + col;
      Vec<bf16, 4> w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w.v[e] = static_cast<bf16>(0.f);  // the copies are zero past the matrix
      if (col_in && row < t.rows) {
        opt_math<KIND, 4>(h, t.o, th[p], g[p], a[p], b[p]);
        stnt<4>(t.o.master + i, th[p]);
        if (KIND != 3) stnt<4>(t.o.s1 + i, a[p]);
        if (KIND == 0) stnt<4>(t.o.s2 + i, b[p]);
#pragma unroll
        for (int e = 0; e < 4; ++e) w.v[e] = from_f32<bf16>(th[p][e]);
        if (t.o.cc) {
          if (PAST) stnt<4>(t.o.cc + i, th[p]);
          else *reinterpret_cast<Vec<bf16, 4>*>(t.o.cc + i) = w;
        }
      }
      *reinterpret_cast<Vec<bf16, 4>*>(tile + r * PITCH + lane * 8) = w;
    }
  }
  __syncthreads();
  const auto put = [](u32x4* at, u32x4 v) __attribute__((always_inline)) {
    if (PAST) __builtin_nontemporal_store(v, at);
    else *at = v;
  };
  if (t.fwd) {
    const int64_t k_steps = t.cols / 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kkl = wave * 4 + j;
      const int64_t kk = (int64_t)ti * 16 + kkl;
      if (kk >= k_steps) continue;
      u32x4 v = *reinterpret_cast<const u32x4*>(tile + pi_row(lane & 31) * PITCH + (kkl * 16 + (lane >> 5) * 8) * 2);
      if (t.gain) v = scale8(v, *reinterpret_cast<const u32x4*>(t.gain + kk * 16 + (lane >> 5) * 8));
      put(t.fwd + (pk_block_pos(to, t.order, t.rows / 64) * k_steps + kk) * 64 + lane, v);
    }
  }
  if (t.bwd) {
    const int64_t k_steps = t.rows / 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int idx = wave * 4 + j, nbl = idx >> 1, kkl = idx & 1;
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[e] = *reinterpret_cast<const bf16*>(tile + (kkl * 16 + (lane >> 5) * 8 + e) * PITCH + (nbl * 32 + pi_row(lane & 31)) * 2);
      put(t.bwd + (((int64_t)ti * 8 + nbl) * k_steps + to * 2 + kkl) * 64 + lane, __builtin_bit_cast(u32x4, v));
    }
  }
}

inline bool al16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

}  // namespace

// Arrays in 16-byte pieces, and a shape whose copies pack_b builds from whole pieces.  A copy's rows past the matrix are never written
// here but within a tile: they stay the zeros that the first packing left.
bool update_packs(const OptItem& it, const PackItem& pk) {
  const bool aligned = al16(it.master) && al16(it.grad) && al16(it.s1) && al16(it.s2) && al16(it.compute_copy) && al16(pk.fwd) &&
                       al16(pk.bwd) && al16(pk.gain);
  const bool shapes = pk.rows * pk.cols == it.n && pk.cols % 4 == 0 && (!pk.fwd || packed_b_bytes(pk.rows, pk.cols) > 0) &&
                      (!pk.bwd || packed_b_bytes(pk.cols, pk.rows) > 0);
  const int64_t tiles = (pk.rows + TILE_ROWS - 1) / TILE_ROWS * ((pk.cols + TILE_COLS - 1) / TILE_COLS);
  return aligned && shapes && (pk.fwd || pk.bwd) && tiles > 0 && tiles < (int64_t(1) << 28);
}

hipError_t optimizer_update_packed(const OptArgs& o, const OptItem* items, const PackItem* packs, int n_items, hipStream_t st) {
  if (o.kind < 0 || o.kind > 3) return hipErrorInvalidValue;
  const OptHyper h = opt_hyper(o);
  for (int done = 0; done < n_items;) {
    OptPackTable table;
    table.n = 0;
    int64_t blocks = 0, copied = 0;
    for (; done < n_items && table.n < OPT_PACK_TABLE; ++done) {
      const PackItem& pk = packs[done];
      if (!update_packs(items[done], pk)) return hipErrorInvalidValue;
      OptPackTensor& t = table.t[table.n];
      t.rows = pk.rows; t.cols = pk.cols;
      t.tiles_inner = (int)((pk.cols + TILE_COLS - 1) / TILE_COLS);
      const int64_t more = (pk.rows + TILE_ROWS - 1) / TILE_ROWS * t.tiles_inner;
      if (table.n > 0 && blocks + more > 0x7FFFFFFF) break;
      t.o = opt_tensor(o, items[done]);
      t.o.block0 = (uint32_t)blocks;
      t.fwd = reinterpret_cast<u32x4*>(pk.fwd); t.bwd = reinterpret_cast<u32x4*>(pk.bwd);
      t.gain = reinterpret_cast<const bf16*>(pk.gain);
      t.order = pk.order;
      copied += 2 * items[done].n * ((t.fwd != nullptr) + (t.bwd != nullptr) + (t.o.cc != nullptr));
      blocks += more;
      ++table.n;
    }
    const dim3 grid((unsigned)blocks);
    const bool past = copied >= COPIES_PAST_CACHES;
    switch (opt_kind(o)) {
      case 0: (past ? opt_pack_k<0, true> : opt_pack_k<0, false>)<<<grid, BLK, 0, st>>>(h, table); break;
      case 1: (past ? opt_pack_k<1, true> : opt_pack_k<1, false>)<<<grid, BLK, 0, st>>>(h, table); break;
      case 2: (past ? opt_pack_k<2, true> : opt_pack_k<2, false>)<<<grid, BLK, 0, st>>>(h, table); break;
      default: (past ? opt_pack_k<3, true> : opt_pack_k<3, false>)<<<grid, BLK, 0, st>>>(h, table); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hift
