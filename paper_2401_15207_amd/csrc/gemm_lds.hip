// Contractions of bf16 operands whose tiles do not fill the chip by themselves: the linear layers of small and ragged
// batches in all three directions, weight gradients that gemm_tt_k does not take, batched attention products, the
// low-rank adapters' products.
//
// Both operands travel from memory into LDS with direct-to-LDS loads, as they lie (no registers, no turning around on
// the way), into a ring of stages of 64 k; a k-major operand (rows of 64 k, 128 bytes) is read back as MFMA fragments with
// 16-byte LDS reads, a transposed one (rows of k, the tile's columns side by side) with transposing LDS reads
// (ds_read_b64_tr_b16, see gemm_tt_k for their lane layout).
//
// What bounds it is the rate at which a compute unit draws operands out of L2 (about 50 bytes per clock) and, for the
// smallest problems, latency: a stage is a barrier, LDS reads and few products.  So up to 128 x 128 every tile's ring leaves room
// for two or more workgroups in a compute unit's LDS (they hide each other's waits: 2048 x 4096, k 4096 takes 71 us with a ring of two
// stages of 128 x 128 tiles, 88 us with four stages and one workgroup), and a stage's fragments are all read into registers
// one stage ahead, under the products of the stage before (231 x 4096, k 11008: 40 us, 50 with fragments read one k-step
// ahead).  256 x 256 tiles, for products of several full rounds, work differently (see Tile); long k whose tiles are one round has
// tiles of its own (LDS_LONG_TILES).  An output's sum runs over k in one chain, in ascending order, whatever the tile.
// Measured against the kernel before it (operands through registers, turned around on the way, 128 x 128 tiles): 1024 tokens,
// 768 -> 3072 with input and weight gradients 12 + 50 + 26 us, now 11 + 13 + 13; 231 tokens, 4096 -> 12288: 49 + 185 + 348 us,
// now 37 + 45 + 63.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "lds_tiles.h"

namespace hift {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

struct LdsP {
  int64_t M, N, K;
  const bf16* A; int64_t lda;
  const bf16* B; int64_t ldb;
  void* C; int64_t ldc;
  const bf16* bias;
  const void* R; int64_t ldr;
  int nh;
  int64_t sa1, sa2, sb1, sb2, sc1, sc2;
  int tiles_m, tiles_n, band;
  int vec;  // rows of C and R can be moved in 16-byte pieces (but for what is left of them at N)
  int past_caches;  // (fp32, no bias, no residual, vec) C is written past the caches
  bf16* C2; int64_t ldc2;  // EPI_GELU, EPI_GELU_BWD
};

constexpr int LK = 64;       // k extent of a stage
constexpr uint32_t OUT_OF_RANGE = 0xFFFFFFF0u;  // beyond every buffer below: such a lane's 16 bytes arrive as zeros
constexpr uint32_t BUF_BYTES = OUT_OF_RANGE;    // lds_gemm_applies keeps every valid offset below this

// One operand's tile, ROWS rows (of C: rows for A, columns for B) x 64 k per stage.
// k-major: LDS row = tile row, 128 bytes, 16-byte piece c at position c ^ ((row / 2) % 8): sixteen consecutive rows of a
// piece fall into sixteen different 16-byte bank groups.
// transposed: LDS row = k, 2 ROWS bytes; the piece index is XOR-ed so that the four consecutive k-rows a transposing read
// touches (64 bytes of each) fall into the four 64-byte bank groups.
// Wavefront w requests 1 KB pieces w NL ..+NL-1 of the stage.  Rows past the edge and k past the end are zeroed lane by
// lane through their offset; the base moves along k with the scalar unit, so offsets stay small whatever the matrix size.
template <int ROWS, bool KMAJOR, int NW>
struct Operand {
  static constexpr int NL = ROWS / 8 / NW;  // load instructions per wavefront and stage
  static constexpr int BYTES = ROWS * 128;
  static constexpr int PPR = KMAJOR ? 8 : ROWS / 8;  // 16-byte pieces per LDS row
  uint32_t voff[NL];
  int kpos[NL];  // k of the piece (k-major: of its first value) within the stage
  uint64_t base;
  uint64_t step;  // bytes from one stage to the next

  static __device__ __forceinline__ int swizzle(int row) {
    if (KMAJOR) return (row >> 1) & 7;
    if (ROWS >= 128) return (row & 3) << 2;
    if (ROWS == 64) return ((row >> 1) & 1) << 2;
    return 0;  // 64-byte rows: four of them are four bank groups
  }

  __device__ __forceinline__ void init(const bf16* src, int64_t ld, int64_t row0, int64_t nrows, int wave, int lane) {
    base = reinterpret_cast<uint64_t>(src) + (KMAJOR ? row0 * ld : row0) * 2;
    step = KMAJOR ? LK * 2 : (uint64_t)ld * (LK * 2);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = (wave * NL + i) * (64 / PPR) + lane / PPR;  // LDS row
      const int c = (lane % PPR) ^ swizzle(r);                  // the piece this lane fetches
      const int64_t row = row0 + (KMAJOR ? r : c * 8);          // (a piece of a transposed operand is wholly in or out)
      kpos[i] = KMAJOR ? c * 8 : r;
      voff[i] = row < nrows ? (uint32_t)((r * ld + c * 8) * 2) : OUT_OF_RANGE;
    }
  }

  // stage `st` (k from st * 64 on; `left` = K - st * 64 > 0 values remain) into LDS at `lds`
  __device__ __forceinline__ void request(int st, int left, uint32_t lds, int wave) const {
    const uint64_t a = base + (uint64_t)st * step;
    const u32x4 rsrc = {(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, BUF_BYTES, 0x00020000u};
#pragma unroll
    for (int i = 0; i < NL; ++i)
      load_to_lds_b128(rsrc, lds + (uint32_t)(wave * NL + i) * 1024, kpos[i] < left ? voff[i] : OUT_OF_RANGE, 0);
  }
};

// MFMA fragments of a 32-row block: lane l holds row l % 32, the eight k-values 8 (l / 32) ..+7 of a 16-k step.
template <int ROWS, bool KMAJOR>
struct Fragments {
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef short v8i16 __attribute__((ext_vector_type(8)));

  __device__ __forceinline__ bf16x8 read(const unsigned char* stage, int row0, int ks, int lane) const {
    if constexpr (KMAJOR) {
      const int r = row0 + (lane & 31);
      return *reinterpret_cast<const bf16x8*>(stage + r * 128 + (((ks * 2 + (lane >> 5)) ^ Operand<ROWS, true, 1>::swizzle(r)) * 16));
    } else {
      v4i16 h[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int kr = ks * 16 + 8 * (lane >> 5) + 4 * q + ((lane & 15) >> 2);
        const int col = row0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        const int at = kr * (ROWS * 2) + (((col >> 3) ^ Operand<ROWS, false, 1>::swizzle(kr)) * 16) + (col & 7) * 2;
        h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4i16 __attribute__((address_space(3)))*)(stage + at));
      }
      const v8i16 both = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
      return __builtin_bit_cast(bf16x8, both);
    }
  }
};

// Wavefronts of a tile: 2 x 2, fewer where a tile has fewer than four 32 x 32 blocks; 2 x 4 for 256 x 256 and 4 x 2 for 256 x 128, whose
// accumulators leave room for the fragments of one k-step ahead instead of a whole stage (two wavefronts a SIMD: 2048 x 32000,
// k 4096 takes 442 us, with 2 x 2 of them, one a SIMD, 461) and whose outputs pass through LDS in two halves.
template <int BM, int BN, int RING>
struct Tile {
  static constexpr bool LARGE = BM * BN > 128 * 128;
  static constexpr int SWN = LARGE ? BN / 64 : (BN >= 64 ? 2 : 1), SWM = LARGE ? 8 / SWN : (BM >= 64 ? 2 : 1), NW = SWM * SWN;
  static constexpr int WM = BM / SWM, WN = BN / SWN;
  static constexpr int OUT_PASSES = LARGE ? 2 : 1;
  static constexpr int RING_BYTES = RING * (BM + BN) * 128, OUT_BYTES = BM / OUT_PASSES * BN * 4;
  static constexpr int LDS = RING_BYTES > OUT_BYTES ? RING_BYTES : OUT_BYTES;
};

// EPI_GELU: C (or nothing, if null) receives the pre-activations, C2 gelu of them; EPI_GELU_BWD: the product is d act, C2 holds
// the forward's pre-activations, C receives d act gelu'(pre).  Either takes the value rounded to bf16 as its argument and the
// library's erff, as the separate kernels do that it replaces (6 us each at 1024 x 3072 and two trips of the matrix to memory):
// the same bits, and a 12-layer encoder of width 768 passes through its layers' sweep in 28.6 ms instead of 29.2.
template <int BM, int BN, int RING, bool AK, bool BKM, typename OutT, int EPI>
__global__ void __launch_bounds__((64 * Tile<BM, BN, RING>::NW), (Tile<BM, BN, RING>::LARGE ? 1 : 2)) gemm_lds_k(LdsP p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef Tile<BM, BN, RING> T;
  constexpr int NW = T::NW, WM = T::WM, WN = T::WN, MT = WM / 32, NT = WN / 32, KSP = LK / 16;
  typedef Operand<BM, AK, NW> OpA;
  typedef Operand<BN, BKM, NW> OpB;
  constexpr int STG = OpA::BYTES + OpB::BYTES, NL = OpA::NL + OpB::NL;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::SWN, wn = wave % T::SWN;
  // Workgroups are dealt round-robin to the 8 XCDs: every XCD gets a contiguous run of tiles, walked down bands of 8 tile
  // rows, so that the tiles it works on at a time share operand tiles in its L2.
  const int ntile = p.tiles_m * p.tiles_n;
  const int xcd = blockIdx.x & 7, share = ntile >> 3, more = ntile & 7;
  const int tile = xcd * share + min(xcd, more) + (int)(blockIdx.x >> 3);
  const int band = tile / (8 * p.tiles_n), in_band = tile - band * 8 * p.tiles_n;
  const int band_rows = min(8, p.tiles_m - band * 8);
  const int tm = band * 8 + in_band % band_rows, tn = in_band / band_rows;
  const int z = blockIdx.y, zb = z / p.nh, zh = z % p.nh;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  // stages [kb, ke) of this output tile; a band hint (causal attention) shortens the range
  const int K = (int)p.K, nk = (K + LK - 1) / LK;
  int kb = 0, ke = nk;
  if (p.band == BAND_SKIP_UPPER && n0 >= m0 + BM) return;  // uniform over the workgroup
  if (p.band == BAND_K_UPTO_ROW) ke = min(nk, (int)((m0 + BM + LK - 1) / LK));
  if (p.band == BAND_K_FROM_ROW) kb = min(nk - 1, (int)(m0 / LK));

  OpA sa;
  OpB sb;
  sa.init(p.A + zb * p.sa1 + zh * p.sa2, p.lda, m0, p.M, wave, lane);
  sb.init(p.B + zb * p.sb1 + zh * p.sb2, p.ldb, n0, p.N, wave, lane);
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem);
  auto slot = [](int st) __attribute__((always_inline)) { return RING & (RING - 1) ? st % RING : st & (RING - 1); };
  auto request = [&](int st) __attribute__((always_inline)) {
    const int left = K - st * LK;
    const uint32_t at = lds0 + (uint32_t)slot(st) * STG;
    sa.request(st, left, at, wave);
    sb.request(st, left, at + OpA::BYTES, wave);
  };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  Fragments<BM, AK> ra;
  Fragments<BN, BKM> rb;
  auto read = [&](bf16x8(&a)[MT], bf16x8(&b)[NT], int st, int ks) __attribute__((always_inline)) {
    const unsigned char* at = smem + slot(st) * STG;
#pragma unroll
    for (int i = 0; i < MT; ++i) a[i] = ra.read(at, wm * WM + i * 32, ks, lane);
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = rb.read(at + OpA::BYTES, wn * WN + j * 32, ks, lane);
  };
  auto multiply = [&](const bf16x8(&a)[MT], const bf16x8(&b)[NT]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };

  // Nothing is asked for past the end, so what is in flight shrinks over the last RING stages and the waits there are for all of
  // it (TAIL; a loop of its own, as a branch in the main one costs a tenth).  Stages of zeros past the end, which keep one count
  // throughout, cost a tile of one or two stages a quarter of its time (see the store below).
#pragma unroll
  for (int s = 0; s < RING; ++s)
    if (kb + s < ke) request(kb + s);
  if (kb + RING <= ke) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 1) * NL) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // Past this the stage after `st` has landed (all but the younger stages' requests), and this stage's buffer, whose last
  // fragments every wavefront has, is free for the stage a whole ring further on.
  auto next_stage = [&](int st, auto tail) __attribute__((always_inline)) {
    if (!decltype(tail)::value || st + RING <= ke) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 2) * NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // (Fragments read past the end are never multiplied.)
  if constexpr (T::LARGE) {
    // One stage: the next k-step's fragments are read under the products of the one before.
    bf16x8 fa[2][MT], fb[2][NT];
    auto stage = [&](int st, auto tail) __attribute__((always_inline)) {
#pragma unroll
      for (int ks = 0; ks < KSP - 1; ++ks) {
        read(fa[(ks + 1) & 1], fb[(ks + 1) & 1], st, ks + 1);
        multiply(fa[ks & 1], fb[ks & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      next_stage(st, tail);
      read(fa[0], fb[0], st + 1, 0);
      if (!decltype(tail)::value || st + RING < ke) request(st + RING);
      multiply(fa[1], fb[1]);
      __builtin_amdgcn_sched_barrier(0);
    };
    read(fa[0], fb[0], kb, 0);
    int st = kb;
    for (; st + RING < ke; ++st) stage(st, std::false_type());
    for (; st < ke; ++st) stage(st, std::true_type());
  } else {
    // One stage: its fragments are in registers (or on their way there), the next one's are read under its products.
    bf16x8 fa[2][KSP][MT], fb[2][KSP][NT];
    auto read_stage = [&](bf16x8(&a)[KSP][MT], bf16x8(&b)[KSP][NT], int st) __attribute__((always_inline)) {
#pragma unroll
      for (int ks = 0; ks < KSP; ++ks) read(a[ks], b[ks], st, ks);
    };
    auto stage = [&](int st, int cur, auto tail) __attribute__((always_inline)) {
      next_stage(st, tail);
      read_stage(fa[cur ^ 1], fb[cur ^ 1], st + 1);
      if (!decltype(tail)::value || st + RING < ke) request(st + RING);
#pragma unroll
      for (int ks = 0; ks < KSP; ++ks) multiply(fa[cur][ks], fb[cur][ks]);
    };
    read_stage(fa[0], fb[0], kb);
    int st = kb;
    for (; st + 1 + RING < ke; st += 2) {
      stage(st, 0, std::false_type());
      stage(st + 1, 1, std::false_type());
    }
    for (; st + 1 < ke; st += 2) {
      stage(st, 0, std::true_type());
      stage(st + 1, 1, std::true_type());
    }
    if (st < ke) stage(st, 0, std::true_type());
  }
  __syncthreads();  // every wavefront has its last fragments, and every request has landed (waited for in the last stages)

  // ---- out: the tile into LDS as fp32 rows, then row by row: bias and residual in fp32, one rounding, 16-byte stores.
  // 16-byte piece `ch` of a row sits at `place`: XOR-ed by the row, so that the 16 rows that a store takes at a time fall into
  // different banks, and the second 256 bytes with their lowest bit turned, so that the every other piece that a read takes does
  // (it read the same banks twice before).  512 x 512, k 128, 128 of them: 37.1 us with that and the stages of zeros, 31.4 now.
  constexpr int CH = BN / 4 < 16 ? BN / 4 : 16;  // pieces that the XOR permutes
  auto place = [](int row, int ch) __attribute__((always_inline)) { return ch ^ (row & (CH - 1)) ^ ((ch >> 4) & 1); };
  constexpr int PMT = MT / T::OUT_PASSES, PWM = PMT * 32;  // blocks and rows of a wavefront that leave per pass
  OutT* C = reinterpret_cast<OutT*>(p.C) + zb * p.sc1 + zh * p.sc2;
  const OutT* R = p.R ? reinterpret_cast<const OutT*>(p.R) + zb * p.sc1 + zh * p.sc2 : nullptr;
#pragma unroll
  for (int pass = 0; pass < T::OUT_PASSES; ++pass) {
    if (pass) __syncthreads();
    {
      const int frow = lane & 31, fh = lane >> 5;
#pragma unroll
      for (int ii = 0; ii < PMT; ++ii)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int i = pass * PMT + ii, row = wm * PWM + ii * 32 + frow, ch = place(row, wn * (WN / 4) + j * 8 + 2 * g + fh);
            const f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
            *reinterpret_cast<f32x4*>(smem + row * (BN * 4) + ch * 16) = v;
          }
    }
    __syncthreads();
    if constexpr (sizeof(OutT) == 4 && EPI == EPI_NONE) {
      if (p.past_caches) {  // a wavefront's store is 1 KB of whole lines
        constexpr int CPR = BN / 4, UNITS = BM / T::OUT_PASSES * CPR;
#pragma unroll 2
        for (int u = tid; u < UNITS; u += 64 * NW) {
          const int r = u / CPR, c = (u % CPR) * 4;
          const int64_t row = m0 + r / PWM * WM + pass * PWM + r % PWM, col = n0 + c;
          if (row >= p.M || col >= p.N) continue;
          f32x4 v = *reinterpret_cast<const f32x4*>(smem + r * (BN * 4) + place(r, c / 4) * 16);
          __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(C + row * p.ldc + col));
        }
        continue;
      }
    }
    constexpr int CPR = BN / 8, UNITS = BM / T::OUT_PASSES * CPR;
#pragma unroll 2
    for (int u = tid; u < UNITS; u += 64 * NW) {
      const int r = u / CPR, c = (u % CPR) * 8;
      const int64_t row = m0 + r / PWM * WM + pass * PWM + r % PWM, col = n0 + c;
      if (row >= p.M || col >= p.N) continue;
      const unsigned char* src = smem + r * (BN * 4);
      f32x4 lo = *reinterpret_cast<const f32x4*>(src + place(r, c / 4) * 16);
      f32x4 hi = *reinterpret_cast<const f32x4*>(src + place(r, c / 4 + 1) * 16);
      if constexpr (EPI != EPI_NONE) {  // bf16 in 16-byte pieces, no residual
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = e < 4 ? lo[e & 3] : hi[e & 3];
        if (p.bias) {
          const bf16x8 t = *reinterpret_cast<const bf16x8*>(p.bias + col);
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += static_cast<float>(t[e]);
        }
        bf16x8 t, o;
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = static_cast<__bf16>(x[e]);
        if constexpr (EPI == EPI_GELU) {
          if (p.C) *reinterpret_cast<bf16x8*>(C + row * p.ldc + col) = t;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(gelu_f(static_cast<float>(t[e])));
          *reinterpret_cast<bf16x8*>(p.C2 + row * p.ldc2 + col) = o;
        } else {
          const bf16x8 pre = *reinterpret_cast<const bf16x8*>(p.C2 + row * p.ldc2 + col);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(static_cast<float>(t[e]) * gelu_df(static_cast<float>(pre[e])));
          *reinterpret_cast<bf16x8*>(C + row * p.ldc + col) = o;
        }
      } else if (p.vec && col + 8 <= p.N) {
        if (p.bias) {
          const bf16x8 t = *reinterpret_cast<const bf16x8*>(p.bias + col);
#pragma unroll
          for (int e = 0; e < 4; ++e) { lo[e] += static_cast<float>(t[e]); hi[e] += static_cast<float>(t[4 + e]); }
        }
        if constexpr (sizeof(OutT) == 2) {
          if (R) {
            const bf16x8 rv = *reinterpret_cast<const bf16x8*>(R + row * p.ldr + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) { lo[e] += static_cast<float>(rv[e]); hi[e] += static_cast<float>(rv[4 + e]); }
          }
          bf16x8 t;
#pragma unroll
          for (int e = 0; e < 4; ++e) { t[e] = static_cast<__bf16>(lo[e]); t[4 + e] = static_cast<__bf16>(hi[e]); }
          *reinterpret_cast<bf16x8*>(C + row * p.ldc + col) = t;
        } else {
          if (R) {
            lo += *reinterpret_cast<const f32x4*>(R + row * p.ldr + col);
            hi += *reinterpret_cast<const f32x4*>(R + row * p.ldr + col + 4);
          }
          *reinterpret_cast<f32x4*>(C + row * p.ldc + col) = lo;
          *reinterpret_cast<f32x4*>(C + row * p.ldc + col + 4) = hi;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (col + e >= p.N) break;
          float v = e < 4 ? lo[e & 3] : hi[e & 3];
          if (p.bias) v += static_cast<float>(p.bias[col + e]);
          if (R) v += to_f32(R[row * p.ldr + col + e]);
          C[row * p.ldc + col + e] = from_f32<OutT>(v);
        }
      }
    }
  }
}

inline bool al16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

template <int I, bool AK, bool BKM, typename OutT, int EPI, bool LONG = false>
hipError_t launch(LdsP& p, int nz, hipStream_t st) {
  constexpr LdsTile TILE = LONG ? LDS_LONG_TILES[I] : LDS_TILES[I];
  constexpr int BM = TILE.bm, BN = TILE.bn, RING = TILE.ring;
  constexpr int LDS = Tile<BM, BN, RING>::LDS;
  static_assert(LDS <= 160 * 1024, "LDS of a gfx950 compute unit");
  static bool attr_done = false;  // one flag per instantiation
  auto kern = gemm_lds_k<BM, BN, RING, AK, BKM, OutT, EPI>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  p.tiles_m = (int)((p.M + BM - 1) / BM);
  p.tiles_n = (int)((p.N + BN - 1) / BN);
  kern<<<dim3((unsigned)(p.tiles_m * p.tiles_n), (unsigned)nz), 64 * Tile<BM, BN, RING>::NW, LDS, st>>>(p);
  return hipGetLastError();
}

template <bool AK, bool BKM, typename OutT, int EPI = EPI_NONE>
hipError_t pick_tile(LdsP& p, int nz, hipStream_t st) {
  static_assert(N_LDS_TILES == 9 && N_LDS_LONG_TILES == 2, "one case per tile");
  switch (p.band == BAND_NONE ? lds_long_tile(p.M, p.N, p.K, nz) : -1) {
    case 0: return launch<0, AK, BKM, OutT, EPI, true>(p, nz, st);
    case 1: return launch<1, AK, BKM, OutT, EPI, true>(p, nz, st);
    default: break;
  }
  switch (lds_tile(p.M, p.N, p.K, nz)) {
    case 0: return launch<0, AK, BKM, OutT, EPI>(p, nz, st);
    case 1: return launch<1, AK, BKM, OutT, EPI>(p, nz, st);
    case 2: return launch<2, AK, BKM, OutT, EPI>(p, nz, st);
    case 3: return launch<3, AK, BKM, OutT, EPI>(p, nz, st);
    case 4: return launch<4, AK, BKM, OutT, EPI>(p, nz, st);
    case 5: return launch<5, AK, BKM, OutT, EPI>(p, nz, st);
    case 6: return launch<6, AK, BKM, OutT, EPI>(p, nz, st);
    case 7: return launch<7, AK, BKM, OutT, EPI>(p, nz, st);
    default: return launch<8, AK, BKM, OutT, EPI>(p, nz, st);
  }
}

}  // namespace

// Operands in 16-byte pieces along their contiguous direction, and offsets within a stage's rows (up to 256 of a k-major operand,
// 64 of a transposed one) below BUF_BYTES.
bool lds_gemm_applies(const Gemm& g) {
  if (g.dtype != DT_BF16 || g.K < 8) return false;
  const auto fits = [&](bool kmajor, int64_t rows, int64_t ld) {
    const int64_t in_stage = kmajor ? (rows < 256 ? rows : 256) : (g.K < LK ? g.K : LK);
    return ld < (int64_t(1) << 31) && in_stage * ld * 2 <= BUF_BYTES;
  };
  // A's contiguous direction may end inside a piece where zeros follow: as k they meet rows of B that are zeroed (or, k-major, are not there:
  // refused), as rows of C they are not stored.
  const int64_t along = g.a_kmajor ? g.K : g.M;
  const bool whole = along % 8 == 0 || (g.zero_tail && g.lda >= (along + 7) / 8 * 8 && !(g.a_kmajor && g.b_kmajor));
  const bool a_ok = al16(g.A) && g.lda % 8 == 0 && g.sa1 % 8 == 0 && g.sa2 % 8 == 0 && whole;
  const bool b_ok = al16(g.B) && g.ldb % 8 == 0 && g.sb1 % 8 == 0 && g.sb2 % 8 == 0 && (g.b_kmajor ? g.K % 8 == 0 : g.N % 8 == 0);
  return a_ok && b_ok && fits(g.a_kmajor, g.M, g.lda) && fits(g.b_kmajor, g.N, g.ldb) && g.K < (int64_t(1) << 30) && g.M < (int64_t(1) << 30) &&
         g.N < (int64_t(1) << 30) && ((g.M + 31) / 32) * ((g.N + 31) / 32) < (int64_t(1) << 31);
}

// GELU or its derivative on the way out: one bf16 problem whose rows move in 16-byte pieces, in the layout of the pass it belongs to.
bool lds_gelu_applies(const Gemm& g) {
  const bool fwd = g.epi == EPI_GELU;
  return lds_gemm_applies(g) && (fwd || g.epi == EPI_GELU_BWD) && !g.out_f32 && !g.R && g.nb * g.nh == 1 && g.a_kmajor && g.b_kmajor == fwd &&
         (fwd || (g.C && !g.bias)) && g.N % 8 == 0 && g.ldc % 8 == 0 && al16(g.C) && g.C2 && al16(g.C2) && g.ldc2 % 8 == 0 && al16(g.bias);
}

hipError_t gemm_lds(const Gemm& g, hipStream_t st) {
  LdsP p{};
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.A = reinterpret_cast<const bf16*>(g.A); p.lda = g.lda;
  p.B = reinterpret_cast<const bf16*>(g.B); p.ldb = g.ldb;
  p.C = g.C; p.ldc = g.ldc;
  p.bias = reinterpret_cast<const bf16*>(g.bias);
  p.R = g.R; p.ldr = g.ldr;
  p.nh = g.nh; p.sa1 = g.sa1; p.sa2 = g.sa2; p.sb1 = g.sb1; p.sb2 = g.sb2; p.sc1 = g.sc1; p.sc2 = g.sc2;
  p.band = g.band;
  p.vec = g.ldc % 8 == 0 && al16(g.C) && (!g.R || (g.ldr % 8 == 0 && al16(g.R))) && g.sc1 % 8 == 0 &&
          g.sc2 % 8 == 0 && (!g.bias || al16(g.bias));
  const int nz = g.nb * g.nh;
  // As in gemm_tt_k (231 tokens, decoder of width 4096: 7.66 -> 7.52 ms a sweep).
  p.past_caches = g.out_f32 && p.vec && g.N % 4 == 0 && !g.bias && !g.R && g.M * g.N * nz * 4 >= PAST_CACHES_BYTES;
  if (g.epi != EPI_NONE) {
    if (!lds_gelu_applies(g)) return hipErrorInvalidValue;
    p.C2 = reinterpret_cast<bf16*>(g.C2); p.ldc2 = g.ldc2;
    return g.epi == EPI_GELU ? pick_tile<true, true, bf16, EPI_GELU>(p, nz, st) : pick_tile<true, false, bf16, EPI_GELU_BWD>(p, nz, st);
  }
#define LAYOUT(OutT)                                                                   \
  (g.a_kmajor ? (g.b_kmajor ? pick_tile<true, true, OutT>(p, nz, st) : pick_tile<true, false, OutT>(p, nz, st))     \
              : (g.b_kmajor ? pick_tile<false, true, OutT>(p, nz, st) : pick_tile<false, false, OutT>(p, nz, st)))
  return g.out_f32 ? LAYOUT(float) : LAYOUT(bf16);
#undef LAYOUT
}

}  // namespace hift
