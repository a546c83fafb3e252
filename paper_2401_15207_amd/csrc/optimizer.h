// The group-local update's arithmetic and what a launch knows of a tensor: shared by opt_k (elementwise.hip), which writes row-major
// copies of the new values, and opt_pack_k (update_pack.hip), which writes them in MFMA fragment order.
#pragma once
#include <math.h>

#include "common.h"
#include "kernels.h"

namespace hift {
namespace {

// fp32 loads and stores of data that is touched once per step (master weights, gradients, moments): non-temporal,
// so that 6 GB of them do not push everything else out of the caches
template <int V>
__device__ __forceinline__ void ldnt(const float* p, float (&f)[V]) {
  typedef float vt __attribute__((ext_vector_type(V)));
  if constexpr (V == 1) {
    f[0] = __builtin_nontemporal_load(p);
  } else {
    const vt t = __builtin_nontemporal_load(reinterpret_cast<const vt*>(p));
#pragma unroll
    for (int e = 0; e < V; ++e) f[e] = t[e];
  }
}
template <int V>
__device__ __forceinline__ void stnt(float* p, const float (&f)[V]) {
  typedef float vt __attribute__((ext_vector_type(V)));
  if constexpr (V == 1) {
    __builtin_nontemporal_store(f[0], p);
  } else {
    vt t;
#pragma unroll
    for (int e = 0; e < V; ++e) t[e] = f[e];
    __builtin_nontemporal_store(t, reinterpret_cast<vt*>(p));
  }
}

// ... and of rounded copies of the new weights that are too large to stay in the last-level cache until the next step reads them
template <int V>
__device__ __forceinline__ void stnt(bf16* p, const float (&f)[V]) {
  typedef bf16 vt __attribute__((ext_vector_type(V)));
  if constexpr (V == 1) {
    *p = from_f32<bf16>(f[0]);
  } else {
    vt t;
#pragma unroll
    for (int e = 0; e < V; ++e) t[e] = from_f32<bf16>(f[e]);
    __builtin_nontemporal_store(t, reinterpret_cast<vt*>(p));
  }
}

struct OptTensor {
  int64_t n;       // parameters
  float* master;
  const float* grad;
  float *s1, *s2;
  bf16* cc;        // where the rounded new values go, or null
  float wd, inv_bc1, inv_bc2;
  int first;       // the tensor's first update
  uint32_t block0; // first block of the launch that works on it
  int vec;         // opt_k: pieces of four are 16-byte aligned in every array
  int grad_fused;  // AdamW: which product of a moment's sum is fused
  int cc_nt;       // opt_k: the copy is written past the caches
  const int32_t* stamps;  // opt_k: see OptItem
  int32_t stamp;
  uint32_t row4;   // pieces of four to a row
};
struct OptHyper {
  float lr, b1, omb1, b2, omb2, eps, mu;
};

// The update of V parameters from their gradients; a, b: the state arrays (KIND 0 AdamW with decoupled decay, 1 AdaGrad, 2 SGD with
// momentum, 3 plain SGD).
// Each of AdamW's moments is a sum of two products, one of them rounded and one fused.  Which one is not left to the compiler
// but is the caller's to say (grad_fused: the gradient's, else the old moment's), and must not depend on where the arrays happen to
// lie: state resident or parked on the host, the same update gives the same bits.
template <int KIND, int V>
__device__ __forceinline__ void opt_math(const OptHyper& h, const OptTensor& t, float (&th)[V], const float (&g)[V], float (&a)[V], float (&b)[V]) {
#pragma unroll
  for (int e = 0; e < V; ++e) {
    if (KIND == 0) {
      th[e] -= h.lr * t.wd * th[e];
      const float g2 = h.omb2 * g[e];
      a[e] = t.grad_fused ? fmaf(h.omb1, g[e], h.b1 * a[e]) : fmaf(h.b1, a[e], h.omb1 * g[e]);
      b[e] = t.grad_fused ? fmaf(g2, g[e], h.b2 * b[e]) : fmaf(h.b2, b[e], g2 * g[e]);
      th[e] -= h.lr * (a[e] * t.inv_bc1) / (sqrtf(b[e] * t.inv_bc2) + h.eps);
    } else if (KIND == 1) {
      const float gg = g[e] + t.wd * th[e];
      a[e] += gg * gg;
      th[e] -= h.lr * gg / (sqrtf(a[e]) + h.eps);
    } else {
      float gg = g[e] + t.wd * th[e];
      if (KIND == 2) {
        a[e] = t.first ? gg : h.mu * a[e] + gg;
        gg = a[e];
      }
      th[e] -= h.lr * gg;
    }
  }
}

inline int opt_kind(const OptArgs& o) { return o.kind == 2 && o.momentum == 0.0 ? 3 : o.kind; }
inline OptHyper opt_hyper(const OptArgs& o) {
  return OptHyper{(float)o.lr, (float)o.beta1, (float)(1.0 - o.beta1), (float)o.beta2, (float)(1.0 - o.beta2), (float)o.eps, (float)o.momentum};
}
inline OptTensor opt_tensor(const OptArgs& o, const OptItem& it) {
  OptTensor t{};
  t.n = it.n; t.master = it.master; t.grad = it.grad; t.s1 = it.s1; t.s2 = it.s2; t.cc = (bf16*)it.compute_copy;
  t.wd = it.decay ? (float)o.wd : 0.f;
  t.inv_bc1 = (float)(1.0 / (1.0 - pow(o.beta1, (double)it.t)));
  t.inv_bc2 = (float)(1.0 / (1.0 - pow(o.beta2, (double)it.t)));
  t.first = it.t == 1 ? 1 : 0;
  t.grad_fused = it.grad_fused;
  t.stamps = it.stamps; t.stamp = it.stamp; t.row4 = (uint32_t)(it.row / 4);
  return t;
}

}  // namespace
}  // namespace hift
