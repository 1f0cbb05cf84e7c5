// Device code of the SGD update that more than one kernel uses: the update kernel itself (pointwise.hip) and the
// weight-gradient kernels that apply the update to the parameters whose gradients they have just completed.
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"
#include "common.h"

namespace omni {

struct Lambdas {
  float v[OMNI_MAX_WORKERS];
};

inline Lambdas lambdas_of(const Segments& seg) {
  Lambdas lam{};
  const double B = (double)seg.off[seg.K];
  for (int k = 0; k < seg.K; ++k) lam.v[k] = (float)((double)(seg.off[k + 1] - seg.off[k]) / B);
  return lam;
}

struct Optim {
  float lr, momentum, weight_decay;
};

// d = g + wd*theta;  v = mu*v + d;  theta -= lr*v   (MOM), or theta -= lr*g
template <bool MOM, typename V>
__device__ inline void apply_update(V& th, V& v, const V& g, const Optim& o) {
  if (MOM) {
    const V d = g + o.weight_decay * th;
    v = o.momentum * v + d;
    th = th - o.lr * v;
  } else {
    th = th - o.lr * g;
  }
}

}  // namespace omni
