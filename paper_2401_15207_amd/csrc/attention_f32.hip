// Attention of fp32 models (and of nothing else: bf16 has attention.hip): heads up to 64 wide, sequences up to 64.
//
// A wavefront owns 16 query rows of one (batch, head).  Their scores against all keys stay in its registers: in the layout of
// v_mfma_f32_16x16x4_f32 lane l holds, of row l % 16, four consecutive keys of every sixteen; an exchange among the four lanes of a row
// (exchange below) turns them into what the next product wants from it.  So scores, softmax and the product with V (or, backward, with K)
// follow each other without LDS, without a barrier and without anything of size S x S in memory; operands come straight from L2.
// What bounds it: launches.  In fp32 models of a few tokens a launch costs the host 3 to 4 us and the GPU 3; scores, softmax and context
// were three of them a layer, and seven in the backward pass, three now (this query-major kernel leaves P and dS to two contractions
// for dV and dK).  With GELU in the contractions' epilogues and the column sums in one launch each, a sweep of two layers, 2 x 32 tokens
// of width 64, takes 155 launches instead of 217: 1.14 -> 0.83 ms, gemm_f32_k's part included.
// Every sum has the order that the separate contractions and softmax kernels give it, so the bits are theirs: chains over ascending
// k, and a row's sums in the tree of a wavefront whose lanes hold four consecutive keys each (QUADS: S a multiple of four) or one.  AdamW
// makes a full step of a gradient that is nothing but rounding (a key's bias), so other bits would show.
#include "common.h"
#include "kernels.h"

namespace hift {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct AttF {
  int H, S, hd;
  int causal;
  float scale;
  const float* qkv; int64_t ld;
  float* ctx; int64_t ldc;     // forward: context out
  const float* dctx;           // backward (rows ldc apart): gradient of the context
  float *prob, *dprob;         // backward: P and dS out, [B, H, S, S]
  float* dqkv;                 // backward: dq out (rows ld apart)
};

// Fragment of row `row` of m (rows ld apart): element j of part b is column 16 b + 4 j + lane / 16.  Rows from S on and columns from
// hd on are zeros.
template <int NK>
__device__ __forceinline__ void row_frag(f32x4 (&f)[NK], const float* m, int64_t ld, int row, const AttF& p, int lane) {
#pragma unroll
  for (int b = 0; b < NK; ++b)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = b * 16 + 4 * j + (lane >> 4);
      f[b][j] = row < p.S && c < p.hd ? m[(int64_t)row * ld + c] : 0.f;
    }
}

// out[e] of block c: sum over the columns of (row lane % 16 of x) and (key 16 c + 4 (lane / 16) + e of m)
template <int NK>
__device__ __forceinline__ f32x4 against_keys(const float* m, int64_t ld, int c, const f32x4 (&x)[NK], const AttF& p, int lane) {
  f32x4 k[NK], acc = {0.f, 0.f, 0.f, 0.f};
  row_frag<NK>(k, m, ld, c * 16 + (lane & 15), p, lane);
#pragma unroll
  for (int b = 0; b < NK; ++b)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(k[b][j], x[b][j], acc, 0, 0, 0);
  return acc;
}

// The four lanes of a row (l % 16 alike) hold a 4 x 4 square: element e of lane group g becomes element g of lane group e.
__device__ __forceinline__ f32x4 exchange(f32x4 v, int lane) {
#pragma unroll
  for (int step = 1; step <= 2; step *= 2) {
    const bool hi = lane & (16 * step);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int lo_e = step == 1 ? 2 * q : q, hi_e = lo_e + step;
      const float got = __shfl_xor(hi ? v[lo_e] : v[hi_e], 16 * step, 64);
      if (hi) v[lo_e] = got;
      else v[hi_e] = got;
    }
  }
  return v;
}

// Sum over a row of a (DOT: of a b), in the order of softmax_fwd_reg_k and softmax_bwd_reg_k (QUADS) or softmax_fwd_k and
// softmax_bwd_k: there the lane of key j is j / 4 or j, here those lanes are (block, lane group) or (block, lane group, element).
template <int NB, bool QUADS, bool DOT>
__device__ __forceinline__ float row_sum(const f32x4 (&a)[NB], const f32x4 (&b)[NB]) {
  auto add = [&](float t, int c, int e) __attribute__((always_inline)) { return DOT ? fmaf(a[c][e], b[c][e], t) : t + a[c][e]; };
  if constexpr (QUADS) {
    float t[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      t[c] = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) t[c] = add(t[c], c, e);
    }
#pragma unroll
    for (int w = NB / 2; w > 0; w /= 2)
#pragma unroll
      for (int c = 0; c < w; ++c) t[c] += t[c + w];
    float v = t[0];
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
    return v;
  } else {
    float t[NB][4];
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) t[c][e] = add(0.f, c, e);
#pragma unroll
    for (int w = NB / 2; w > 0; w /= 2)
#pragma unroll
      for (int c = 0; c < w; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[c][e] += t[c + w][e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      t[0][e] += __shfl_xor(t[0][e], 32, 64);
      t[0][e] += __shfl_xor(t[0][e], 16, 64);
    }
    return (t[0][0] + t[0][2]) + (t[0][1] + t[0][3]);
  }
}

// rows of x (lane: row lane % 16, values by key as the scores lie) times the keys' rows of m -> out (rows ldo apart)
template <int NK, int NB>
__device__ __forceinline__ void times_keys(const f32x4 (&x)[NB], int nb, const float* m, int64_t ld, float* out, int64_t ldo, int row,
                                           const AttF& p, int lane) {
  const int r = lane & 15, g = lane >> 4;
  f32x4 o[NK];
#pragma unroll
  for (int b = 0; b < NK; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NB; ++c)
    if (c < nb) {
      const f32x4 xc = exchange(x[c], lane);
      float v[NK][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int key = c * 16 + 4 * j + g;
#pragma unroll
        for (int b = 0; b < NK; ++b) v[b][j] = key < p.S && b * 16 + r < p.hd ? m[(int64_t)key * ld + b * 16 + r] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < NK; ++b) o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[b][j], xc[j], o[b], 0, 0, 0);
    }
  if (row < p.S) {
#pragma unroll
    for (int b = 0; b < NK; ++b)
      if (b * 16 + g * 4 < p.hd) *reinterpret_cast<f32x4*>(out + (int64_t)row * ldo + b * 16 + g * 4) = o[b];
  }
}

// NK: sixteens of the head's width; NB: sixteens of keys, a power of two.
template <int NK, int NB, bool QUADS, bool BWD>
__global__ void __launch_bounds__(64) attn_f32_k(AttF p) {
  const int lane = threadIdx.x, g = lane >> 4;
  const int blk = (int)(gridDim.x - 1 - blockIdx.x);  // the rows with the most keys first
  const int64_t bh = blockIdx.y, zb = bh / p.H, zh = bh % p.H;
  const int64_t d = (int64_t)p.H * p.hd;
  const float* q = p.qkv + zb * p.S * p.ld + zh * p.hd;
  const float *k = q + d, *v = q + 2 * d;
  const int row = blk * 16 + (lane & 15);
  const int nb = p.causal ? blk + 1 : (p.S + 15) / 16;  // uniform: sixteens of keys that any of the rows sees
  const int n = p.causal && row < p.S ? row + 1 : p.S;  // keys that the row sees
  auto seen = [&](int c, int e) __attribute__((always_inline)) { return c * 16 + 4 * g + e < n; };
  f32x4 s[NB];
  float mx = -INFINITY;
  {
    f32x4 x[NK];
    row_frag<NK>(x, q, p.ld, row, p, lane);
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      s[c] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (c < nb) {
        const f32x4 t = against_keys<NK>(k, p.ld, c, x, p, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float scaled = seen(c, e) ? t[e] * p.scale : -INFINITY;
          mx = fmaxf(mx, scaled);
          s[c][e] = QUADS ? scaled : t[e];
        }
      }
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[c][e] = c < nb && seen(c, e) ? expf(QUADS ? s[c][e] - mx : fmaf(s[c][e], p.scale, -mx)) : 0.f;
  const float inv = 1.0f / row_sum<NB, QUADS, false>(s, s);
#pragma unroll
  for (int c = 0; c < NB; ++c) s[c] *= inv;
  if constexpr (!BWD) {
    times_keys<NK, NB>(s, nb, v, p.ld, p.ctx + zb * p.S * p.ldc + zh * p.hd, p.ldc, row, p, lane);
  } else {
    f32x4 ds[NB];
    {
      f32x4 x[NK];
      row_frag<NK>(x, p.dctx + zb * p.S * p.ldc + zh * p.hd, p.ldc, row, p, lane);
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        ds[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (c < nb) {
          const f32x4 t = against_keys<NK>(v, p.ld, c, x, p, lane);
#pragma unroll
          for (int e = 0; e < 4; ++e) ds[c][e] = seen(c, e) ? t[e] : 0.f;
        }
      }
    }
    const float dot = row_sum<NB, QUADS, true>(s, ds);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) ds[c][e] = p.scale * s[c][e] * (ds[c][e] - dot);
    if (row < p.S) {
      const int64_t at = (bh * p.S + row) * p.S;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const int key = c * 16 + 4 * g;
        if (QUADS) {
          if (key < p.S) {
            *reinterpret_cast<f32x4*>(p.prob + at + key) = s[c];
            *reinterpret_cast<f32x4*>(p.dprob + at + key) = ds[c];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (key + e < p.S) {
              p.prob[at + key + e] = s[c][e];
              p.dprob[at + key + e] = ds[c][e];
            }
        }
      }
    }
    times_keys<NK, NB>(ds, nb, k, p.ld, p.dqkv + zb * p.S * p.ld + zh * p.hd, p.ld, row, p, lane);
  }
}

template <int NK, int NB, bool BWD>
void launch_nb(const AttF& p, dim3 grid, hipStream_t st) {
  if (p.S % 4 == 0) attn_f32_k<NK, NB, true, BWD><<<grid, 64, 0, st>>>(p);
  else attn_f32_k<NK, NB, false, BWD><<<grid, 64, 0, st>>>(p);
}
template <int NK, bool BWD>
void launch(const AttF& p, int B, hipStream_t st) {
  const dim3 grid((unsigned)((p.S + 15) / 16), (unsigned)(B * p.H));
  if (p.S <= 32) launch_nb<NK, 2, BWD>(p, grid, st);
  else launch_nb<NK, 4, BWD>(p, grid, st);
}
template <bool BWD>
hipError_t run(const AttF& p, int B, hipStream_t st) {
  if (p.hd <= 16) launch<1, BWD>(p, B, st);
  else if (p.hd <= 32) launch<2, BWD>(p, B, st);
  else launch<4, BWD>(p, B, st);
  return hipGetLastError();
}
bool al16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

}  // namespace

// Sequences of up to 64 tokens, heads in whole 16-byte pieces.  Beyond 64 the separate contractions and softmax are the faster way
// whatever the number of heads: a wavefront here walks its blocks of keys one after the other and there are only S / 16 a head, while they
// spread over many tiles.  Sweeps of four layers, one kernel / separate ones, ms: heads of 16, 1 x 8 of them, 64 tokens 1.76 / 1.89, 128
// 2.04 / 1.95, 256 2.51 / 2.11; heads of 64, 1 x 2, 32 tokens 1.69 / 1.85, 64 1.90 / 1.90, 100 2.23 / 1.99, 256 3.08 / 2.04; 4 x 8,
// 32 2.86 / 2.97, 64 3.35 / 3.30, 256 6.76 / 5.96.
bool attention_f32_applies(int dt, int B, int H, int S, int hd, int64_t ld, int64_t ldc, const void* qkv, const void* ctx) {
  return dt == DT_F32 && S >= 1 && S <= 64 && hd >= 4 && hd <= 64 && hd % 4 == 0 && ld % 4 == 0 && ldc % 4 == 0 && al16(qkv) && al16(ctx) &&
         (int64_t)B * H <= 65535;
}
hipError_t attention_fwd_f32(int B, int H, int S, int hd, bool causal, const void* qkv, int64_t ld, void* ctx, int64_t ldc, hipStream_t st) {
  AttF p{};
  p.H = H; p.S = S; p.hd = hd; p.causal = causal; p.scale = 1.0f / sqrtf((float)hd);
  p.qkv = (const float*)qkv; p.ld = ld; p.ctx = (float*)ctx; p.ldc = ldc;
  return run<false>(p, B, st);
}
hipError_t attention_bwd_f32(int B, int H, int S, int hd, bool causal, const void* qkv, int64_t ld, const void* dctx, int64_t ldc, void* prob,
                             void* dprob, void* dqkv, hipStream_t st) {
  AttF p{};
  p.H = H; p.S = S; p.hd = hd; p.causal = causal; p.scale = 1.0f / sqrtf((float)hd);
  p.qkv = (const float*)qkv; p.ld = ld; p.dctx = (const float*)dctx; p.ldc = ldc;
  p.prob = (float*)prob; p.dprob = (float*)dprob; p.dqkv = (float*)dqkv;
  return run<true>(p, B, st);
}

}  // namespace hift
