// Contractions of fp32 operands, and of bf16 operands that do not lie in 16-byte pieces: any sizes, strides and alignment.
//
// v_mfma_f32_16x16x4_f32 adds its four products one after the other in ascending k, each a fused multiply-add with one rounding,
// denormals kept: an output is the same chain of multiply-adds over ascending k, bit for bit, that a loop of fmaf gives (checked
// over 246 thousand outputs of operands of like and of unlike size and of denormal ones), at twice the rate of the vector unit and with each LDS
// value read feeding 16 products instead of 1 or 4.
//
// A workgroup of four wavefronts computes BT x BT outputs, a wavefront a quarter of them.  Elements travel one by one through
// registers (converted to fp32 there) into LDS rows of KC k-values, the next pass's on their way while one is multiplied.
// What bounds it: small problems, a trip to memory per pass, so that 32 x 32 tiles take up to 256 k in one pass (256 x 1024, k 1024
// in the three layouts of a linear layer 11 us; a kernel of fused multiply-adds on the vector unit with passes of 64 took
// 31 to 43); large ones, element-wise loads and LDS writes: 2048 x 2048, k 2048 145 to 151 us, 114 TFLOP/s, before 287 to 297.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace hift {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct F32P {
  int64_t M, N, K;
  const void* A; int64_t lda;
  const void* B; int64_t ldb;
  void* C; int64_t ldc;
  const void* bias;
  const void* R; int64_t ldr;
  int nh;
  int64_t sa1, sa2, sb1, sb2, sc1, sc2;
  int tiles_m;
  void* C2; int64_t ldc2;  // EPI_GELU, EPI_GELU_BWD (see Gemm in kernels.h)
  int vec;  // rows of C, R and bias can be moved four values at a time
};

// Where k lies in an LDS row: within 16, the order in which a lane's 16-byte read gives it one k of each of four products (product
// j takes k = 4 j + g of lane group g).
__device__ __forceinline__ int f32_place(int k) { return (k & ~15) | ((k & 3) << 2) | ((k >> 2) & 3); }

__device__ __forceinline__ float f32_load(__amdgpu_buffer_rsrc_t r, uint32_t at, const float*) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0));
}
__device__ __forceinline__ bf16 f32_load(__amdgpu_buffer_rsrc_t r, uint32_t at, const bf16*) {
  return __builtin_bit_cast(bf16, __builtin_amdgcn_raw_buffer_load_b16(r, at, 0, 0));
}

// One operand's share of a pass for a thread: NLD elements at fixed distances, so that neighbouring threads take neighbours along
// the operand's contiguous direction.  KMAJOR: element i is row tid / KC + i 256 / KC at k = tid % KC.  Else row tid % BT; four
// elements after one another are k = c, c + 4, c + 8, c + 12 of one sixteen, which lie side by side in LDS and leave as one 16-byte
// write (one by one, the 64 rows of a write would share 16 banks: 512 x 1024, k 256 with transposed operands 21 us, 9 so).
// LDS rows are KC + 4 floats: the 16 rows of a 16-byte access fall into different banks.
// Elements outside arrive as zeros, for which the loads are bounded: the direction that the elements of a thread advance in by the length
// of the buffer, the other one by an offset beyond it (with pointers and a branch per element at the edges, 26 KB of code for a pass of
// 256 k and 6 now, 256 x 1024, k 1024 took 17 us and 2048 x 2048, k 2048 193).  Lengths and offsets stay below 2^31 (f32_fits); WIDE, for rows too far apart for that, goes by pointers.
constexpr uint32_t F32_OUTSIDE = 0x80000000u;
template <int BT, int KC, bool KMAJOR, bool WIDE, typename T>
struct F32Operand {
  static constexpr int NLD = BT * KC / 256, STEP = KMAJOR ? 256 / KC : 256 / BT, LD = KC + 4;
  static_assert(KMAJOR || (STEP % 4 == 0 && NLD % 4 == 0), "a thread's elements come in fours");
  const T* base;
  const T* tile;  // the tile's first element in this pass
  int64_t ld;
  int r0, k0, rows;  // first row and k of this thread within the tile and pass; rows of the tile inside the matrix
  T v[NLD];
  static __device__ __forceinline__ constexpr int row(int i) { return KMAJOR ? i * STEP : 0; }
  static __device__ __forceinline__ constexpr int kk(int i) { return KMAJOR ? 0 : i / 4 * (4 * STEP) + i % 4 * 4; }
  __device__ __forceinline__ void init(const T* src, int64_t ld_, int64_t row0, int64_t nrows, int tid) {
    base = src;
    ld = ld_;
    r0 = KMAJOR ? tid / KC : tid % BT;
    k0 = KMAJOR ? tid % KC : tid / BT / 4 * 16 + tid / BT % 4;
    rows = (int)(nrows - row0 < BT ? nrows - row0 : BT);
    tile = src + (KMAJOR ? row0 * ld : row0);
  }
  __device__ __forceinline__ void load(int64_t left) {  // left: k-values that remain from this pass on
    const int ks = (int)(left < KC ? left : KC);
    if constexpr (WIDE) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int r = r0 + row(i), k = k0 + kk(i);
        const bool in = r < rows && k < ks;
        const T t = *(in ? tile + (KMAJOR ? r * ld + k : k * ld + r) : base);
        v[i] = in ? t : T();
      }
    } else {
      const uint32_t ld32 = (uint32_t)ld * (uint32_t)sizeof(T);
      const __amdgpu_buffer_rsrc_t buf =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(tile), 0, (int)((KMAJOR ? rows : ks) * ld32), 0x00020000);
      const bool in = KMAJOR ? k0 < ks : r0 < rows;
      const uint32_t at = in ? (KMAJOR ? r0 * ld32 + k0 * (uint32_t)sizeof(T) : k0 * ld32 + r0 * (uint32_t)sizeof(T)) : F32_OUTSIDE;
#pragma unroll
      for (int i = 0; i < NLD; ++i) v[i] = f32_load(buf, at + (uint32_t)(KMAJOR ? row(i) : kk(i)) * ld32, static_cast<const T*>(nullptr));
    }
    tile += KMAJOR ? KC : KC * ld;
  }
  __device__ __forceinline__ void store(float* dst) const {
    float* to = dst + r0 * LD + f32_place(k0);
    if constexpr (KMAJOR) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) to[row(i) * LD] = to_f32(v[i]);
    } else {
#pragma unroll
      for (int i = 0; i < NLD; i += 4)
        *reinterpret_cast<f32x4*>(to + kk(i)) = f32x4{to_f32(v[i]), to_f32(v[i + 1]), to_f32(v[i + 2]), to_f32(v[i + 3])};
    }
  }
};
// What the buffers of the largest tile and pass (64 rows of k-major operands, 256 k of others) need.
bool f32_fits(bool kmajor, int64_t ld, int64_t size) { return ld < (int64_t(1) << 31) && (kmajor ? 64 : 256) * ld * size <= 0x7FF00000; }

// BUFS: LDS buffers; with one the next pass waits in registers until every wavefront has multiplied this one.
template <int BT, int KC, int BUFS, bool AK, bool BKM, bool WIDE, typename T, typename OutT, int EPI>
__global__ void __launch_bounds__(256) gemm_f32_k(F32P p) {
  constexpr int WT = BT / 2, MT = WT / 16, LD = KC + 4, OP = BT * LD;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  const int tile = blockIdx.x;
  const int tm = tile % p.tiles_m, tn = tile / p.tiles_m;
  const int z = blockIdx.y, zb = z / p.nh, zh = z % p.nh;
  const int64_t m0 = (int64_t)tm * BT, n0 = (int64_t)tn * BT;
  F32Operand<BT, KC, AK, WIDE, T> a;
  F32Operand<BT, KC, BKM, WIDE, T> b;
  a.init(reinterpret_cast<const T*>(p.A) + zb * p.sa1 + zh * p.sa2, p.lda, m0, p.M, tid);
  b.init(reinterpret_cast<const T*>(p.B) + zb * p.sb1 + zh * p.sb2, p.ldb, n0, p.N, tid);
  f32x4 acc[MT][MT] = {};
  if (p.K > 0) {
    a.load(p.K);
    b.load(p.K);
    a.store(lds);
    b.store(lds + OP);
  }
  __syncthreads();
  const int frag = (lane & 15) * LD + (lane >> 4) * 4;  // lane l: row l % 16, the k-values that its group takes of four products
  int buf = 0;
  for (int64_t left = p.K; left > 0; left -= KC) {
    const bool more = left > KC;
    if (more) {
      a.load(left - KC);
      b.load(left - KC);
    }
    const float* at = lds + buf * 2 * OP + wm * WT * LD + frag;
    const float* bt = lds + buf * 2 * OP + OP + wn * WT * LD + frag;
    f32x4 x[MT], y[MT];
    auto read = [&](int k) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < MT; ++i) x[i] = *reinterpret_cast<const f32x4*>(at + i * 16 * LD + k);
#pragma unroll
      for (int j = 0; j < MT; ++j) y[j] = *reinterpret_cast<const f32x4*>(bt + j * 16 * LD + k);
    };
    auto multiply = [&](int e) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[j][e], x[i][e], acc[i][j], 0, 0, 0);
    };
    if (left >= KC) {
#pragma unroll
      for (int k = 0; k < KC; k += 16) {
        read(k);
#pragma unroll
        for (int e = 0; e < 4; ++e) multiply(e);
      }
    } else {
      // (a 16-byte read may bring k past the last four, which nothing was stored to: never multiplied)
      for (int k = 0; k < (int)left; k += 16) {
        read(k);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k + 4 * e < (int)left) multiply(e);
      }
    }
    if (BUFS == 1) __syncthreads();
    else buf ^= 1;
    if (more) {
      a.store(lds + buf * 2 * OP);
      b.store(lds + buf * 2 * OP + OP);
    }
    __syncthreads();  // the next pass is complete, this one is no longer read
  }
  // lane l, element e of block (i, j): row i 16 + l % 16, column j 16 + 4 (l / 16) + e
  OutT* C = reinterpret_cast<OutT*>(p.C) + zb * p.sc1 + zh * p.sc2;
  const OutT* R = p.R ? reinterpret_cast<const OutT*>(p.R) + zb * p.sc1 + zh * p.sc2 : nullptr;
  const T* bias = reinterpret_cast<const T*>(p.bias);
  const int64_t row0 = m0 + wm * WT + (lane & 15), col0 = n0 + wn * WT + (lane >> 4) * 4;
  float* C2 = reinterpret_cast<float*>(p.C2);  // of the GELU epilogues: fp32, no residual, no batch; the library's erff, as the separate kernels take it: the same bits
  if (p.vec && m0 + BT <= p.M && n0 + BT <= p.N) {
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      f32x4 add = {0.f, 0.f, 0.f, 0.f};
      if (bias) {
        const Vec<T, 4> t = *reinterpret_cast<const Vec<T, 4>*>(bias + col0 + j * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) add[e] = to_f32(t.v[e]);
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int64_t row = row0 + i * 16;
        f32x4 v = acc[i][j] + add;
        if (R) {
          const Vec<OutT, 4> t = *reinterpret_cast<const Vec<OutT, 4>*>(R + row * p.ldr + col0 + j * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += to_f32(t.v[e]);
        }
        if constexpr (EPI != EPI_NONE) {
          Vec<float, 4>* const c2 = reinterpret_cast<Vec<float, 4>*>(C2 + row * p.ldc2 + col0 + j * 16);
          Vec<float, 4> t;
          if constexpr (EPI == EPI_GELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) t.v[e] = gelu_f(v[e]);
            *c2 = t;
            if (!p.C) continue;
          } else {
            t = *c2;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= gelu_df(t.v[e]);
          }
        }
        Vec<OutT, 4> out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out.v[e] = from_f32<OutT>(v[e]);
        *reinterpret_cast<Vec<OutT, 4>*>(C + row * p.ldc + col0 + j * 16) = out;
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int64_t row = row0 + i * 16;
    if (row >= p.M) continue;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t col = col0 + j * 16 + e;
        if (col >= p.N) continue;
        float v = acc[i][j][e] + (bias ? to_f32(bias[col]) : 0.f);
        if (R) v += to_f32(R[row * p.ldr + col]);
        if constexpr (EPI == EPI_GELU) {
          C2[row * p.ldc2 + col] = gelu_f(v);
          if (!p.C) continue;
        } else if constexpr (EPI == EPI_GELU_BWD) {
          v *= gelu_df(C2[row * p.ldc2 + col]);
        }
        C[row * p.ldc + col] = from_f32<OutT>(v);
      }
    }
  }
}

template <int BT, int KC, int BUFS, bool AK, bool BKM, bool WIDE, typename T, typename OutT, int EPI>
hipError_t launch(F32P& p, int nz, hipStream_t st) {
  constexpr int LDS = BUFS * 2 * BT * (KC + 4) * (int)sizeof(float);
  static_assert(LDS <= 160 * 1024, "LDS of a gfx950 compute unit");
  auto kern = gemm_f32_k<BT, KC, BUFS, AK, BKM, WIDE, T, OutT, EPI>;
  if (LDS > 64 * 1024) {
    static bool attr_done = false;  // one flag per instantiation
    if (!attr_done) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
      if (e != hipSuccess) return e;
      attr_done = true;
    }
  }
  p.tiles_m = (int)((p.M + BT - 1) / BT);
  const int tiles_n = (int)((p.N + BT - 1) / BT);
  kern<<<dim3((unsigned)(p.tiles_m * tiles_n), (unsigned)nz), 256, LDS, st>>>(p);
  return hipGetLastError();
}

// 64 x 64 tiles where they give every compute unit one (1024 x 1024, k 256: 10.4 us), else 32 x 32 (512 x 1024: 7.9), whose passes are no
// longer than k needs: elements past its end cost their loads.
// WIDE, whose loads are bounded one by one, takes 32 x 32 tiles also there (1024 x 1024, k 1024 in rows of 2.2 M values 39 us, 64 x 64: 47; k 256
// 12.4 and 12.8), but for a single pass of 16 k (5.6 us, 64 x 64: 4.2).
template <bool AK, bool BKM, typename T, typename OutT, int EPI = EPI_NONE>
hipError_t pick(F32P& p, int nz, hipStream_t st) {
  const bool fills = ((p.M + 63) / 64) * ((p.N + 63) / 64) * nz >= 256;
  if (!f32_fits(AK, p.lda, sizeof(T)) || !f32_fits(BKM, p.ldb, sizeof(T))) {
    if constexpr (EPI != EPI_NONE) return hipErrorInvalidValue;
    else if (fills && p.K <= 16) return launch<64, 16, 2, AK, BKM, true, T, OutT, EPI>(p, nz, st);
    else return launch<32, 64, 1, AK, BKM, true, T, OutT, EPI>(p, nz, st);
  }
  if (fills) {
    if (p.K <= 16) return launch<64, 16, 2, AK, BKM, false, T, OutT, EPI>(p, nz, st);
    return launch<64, 32, 2, AK, BKM, false, T, OutT, EPI>(p, nz, st);
  }
  if (p.K <= 64) return launch<32, 64, 1, AK, BKM, false, T, OutT, EPI>(p, nz, st);
  if (p.K <= 128) return launch<32, 128, 1, AK, BKM, false, T, OutT, EPI>(p, nz, st);
  return launch<32, 256, 1, AK, BKM, false, T, OutT, EPI>(p, nz, st);
}

template <typename T, typename OutT>
hipError_t pick_layout(const Gemm& g, F32P& p, int nz, hipStream_t st) {
  if (g.a_kmajor) return g.b_kmajor ? pick<true, true, T, OutT>(p, nz, st) : pick<true, false, T, OutT>(p, nz, st);
  return g.b_kmajor ? pick<false, true, T, OutT>(p, nz, st) : pick<false, false, T, OutT>(p, nz, st);
}

}  // namespace

// GELU or its derivative on the way out: one fp32 problem in the layout of the pass it belongs to.
bool f32_gelu_applies(const Gemm& g) {
  const bool fwd = g.epi == EPI_GELU;
  return g.dtype == DT_F32 && (fwd || g.epi == EPI_GELU_BWD) && !g.R && g.nb * g.nh == 1 && g.a_kmajor && g.b_kmajor == fwd && g.C2 &&
         (fwd || (g.C && !g.bias)) && f32_fits(true, g.lda, sizeof(float)) && f32_fits(fwd, g.ldb, sizeof(float));
}

hipError_t gemm_f32(const Gemm& g, hipStream_t st) {
  F32P p{};
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.A = g.A; p.lda = g.lda; p.B = g.B; p.ldb = g.ldb; p.C = g.C; p.ldc = g.ldc;
  p.bias = g.bias; p.R = g.R; p.ldr = g.ldr;
  p.nh = g.nh; p.sa1 = g.sa1; p.sa2 = g.sa2; p.sb1 = g.sb1; p.sb2 = g.sb2; p.sc1 = g.sc1; p.sc2 = g.sc2;
  const int nz = g.nb * g.nh;
  const size_t in = dt_size(g.dtype), out = g.out_f32 || g.dtype == DT_F32 ? 4 : 2;
  const auto fours = [](const void* q, size_t size, int64_t ld) { return !q || (reinterpret_cast<uintptr_t>(q) % (4 * size) == 0 && ld % 4 == 0); };
  p.vec = fours(g.C, out, g.ldc) && g.sc1 % 4 == 0 && g.sc2 % 4 == 0 && fours(g.R, out, g.ldr) && fours(g.bias, in, 0) && fours(g.C2, 4, g.ldc2);
  if (g.epi != EPI_NONE) {
    if (!f32_gelu_applies(g)) return hipErrorInvalidValue;
    p.C2 = g.C2; p.ldc2 = g.ldc2;
    return g.epi == EPI_GELU ? pick<true, true, float, float, EPI_GELU>(p, nz, st) : pick<true, false, float, float, EPI_GELU_BWD>(p, nz, st);
  }
  if (g.dtype == DT_F32) return pick_layout<float, float>(g, p, nz, st);
  return g.out_f32 ? pick_layout<bf16, float>(g, p, nz, st) : pick_layout<bf16, bf16>(g, p, nz, st);
}

}  // namespace hift
