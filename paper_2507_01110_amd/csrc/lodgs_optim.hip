// Adam step on the cut set (init/training appendix: a view updates only the
// parameters of its cut set).  One launch: every parameter group has a share
// of the workgroups, and in it one thread per (selected node, chunk) with
// chunks of 4 floats for rows of a multiple of 4 floats (quaternions, SH of
// degree 1 and 3) and of 1 float otherwise: the gradient rows are read by
// selection position (coalesced), the parameter and its two moments by node
// row; d_idx holds every node at most once, so no two threads touch one
// element.  Bound by memory (seven words moved for each parameter); the four
// narrow groups take little, but not with a launch each: 15.5 us in five
// launches at 333 x 171 (5.9 in one), 68 for a 1080p iteration (56).
#include "lodgs_internal.h"

#include <algorithm>
#include <cmath>

namespace lodgs {
namespace {

struct AdamGroup {
  float* p;
  const float* g;
  float* m;
  float* v;
  int32_t w;
  float step_size;  // lr / (1 - beta1^step)
};

struct AdamConst {
  float b1, b2, eps, bc2_sqrt;  // bc2_sqrt = sqrt(1 - beta2^step)
};

__device__ __forceinline__ void adam_element(const AdamConst& a, float step_size, float g, float& p, float& m,
                                             float& v) {
  m = a.b1 * m + (1.0f - a.b1) * g;
  v = a.b2 * v + (1.0f - a.b2) * (g * g);
  p = p - step_size * m / (__builtin_sqrtf(v) / a.bc2_sqrt + a.eps);
}

struct AdamGroups {
  AdamGroup g[5];
  uint32_t first[6];  // each group's first workgroup
};

template <int W>
__device__ __forceinline__ void adam_rows(const AdamGroup& G, const AdamConst& a, const int32_t* idx, int64_t n,
                                          int64_t n_nodes, int64_t t0, int64_t stride) {
  constexpr int V = W % 4 == 0 ? 4 : 1, C = W / V;
  for (int64_t e = t0; e < n * C; e += stride) {
    const int64_t i = e / C;
    const int c = (int)(e - i * C);
    const int64_t node = idx[i];
    if (node < 0 || node >= n_nodes) continue;
    if (V == 4) {
      const float4 g = reinterpret_cast<const float4*>(G.g + i * W)[c];
      float4* pp = reinterpret_cast<float4*>(G.p + node * W) + c;
      float4* mp = reinterpret_cast<float4*>(G.m + node * W) + c;
      float4* vp = reinterpret_cast<float4*>(G.v + node * W) + c;
      float4 p = *pp, m = *mp, v = *vp;
      adam_element(a, G.step_size, g.x, p.x, m.x, v.x);
      adam_element(a, G.step_size, g.y, p.y, m.y, v.y);
      adam_element(a, G.step_size, g.z, p.z, m.z, v.z);
      adam_element(a, G.step_size, g.w, p.w, m.w, v.w);
      *mp = m;
      *vp = v;
      *pp = p;
    } else {
      const int64_t o = node * W + c;
      float p = G.p[o], m = G.m[o], v = G.v[o];
      adam_element(a, G.step_size, G.g[i * W + c], p, m, v);
      G.m[o] = m;
      G.v[o] = v;
      G.p[o] = p;
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_adam_cut(AdamGroups A, AdamConst a, const int32_t* idx,
                                                     const int32_t* d_count, int64_t cap, int64_t n_nodes) {
  int64_t n = *d_count;
  n = n < 0 ? 0 : (n > cap ? cap : n);
  int k = 0;  // block-uniform
  while (blockIdx.x >= A.first[k + 1]) ++k;
  const AdamGroup G = A.g[k];
  const int64_t t0 = (int64_t)(blockIdx.x - A.first[k]) * kBlock + threadIdx.x;
  const int64_t stride = (int64_t)(A.first[k + 1] - A.first[k]) * kBlock;
  switch (G.w) {
    case 1: adam_rows<1>(G, a, idx, n, n_nodes, t0, stride); break;
    case 3: adam_rows<3>(G, a, idx, n, n_nodes, t0, stride); break;
    case 4: adam_rows<4>(G, a, idx, n, n_nodes, t0, stride); break;
    case 12: adam_rows<12>(G, a, idx, n, n_nodes, t0, stride); break;
    case 27: adam_rows<27>(G, a, idx, n, n_nodes, t0, stride); break;
    default: adam_rows<48>(G, a, idx, n, n_nodes, t0, stride); break;
  }
}

}  // namespace
}  // namespace lodgs

extern "C" int lodgs_adam_cut(const lodgs_grads* params, const lodgs_grads* grads, const lodgs_grads* exp_avg,
                              const lodgs_grads* exp_avg_sq, const lodgs_adam* hp, const int32_t* d_idx,
                              const int32_t* d_count, int64_t capacity, int64_t n_nodes, lodgs_stream stream) {
  using namespace lodgs;
  if (!params || !grads || !exp_avg || !exp_avg_sq || !hp || !d_idx || !d_count)
    return set_error(LODGS_E_INVALID, "lodgs_adam_cut: null argument");
  if (hp->step < 1 || !(hp->beta1 >= 0.0f && hp->beta1 < 1.0f) || !(hp->beta2 >= 0.0f && hp->beta2 < 1.0f) ||
      !(hp->eps >= 0.0f) || hp->sh_degree < 0 || hp->sh_degree > 3 || capacity < 0 || n_nodes < 0)
    return set_error(LODGS_E_INVALID, "lodgs_adam_cut: hyper-parameters out of range");
  float* const lodgs_grads::*members[5] = {&lodgs_grads::d_means, &lodgs_grads::d_log_scales, &lodgs_grads::d_quats,
                                          &lodgs_grads::d_opacity_logits, &lodgs_grads::d_sh};
  const int32_t widths[5] = {3, 3, 4, 1, 3 * (hp->sh_degree + 1) * (hp->sh_degree + 1)};
  const double bc1 = 1.0 - std::pow((double)hp->beta1, (double)hp->step);
  const double bc2 = 1.0 - std::pow((double)hp->beta2, (double)hp->step);
  AdamGroups grp{};
  int n_groups = 0;
  for (int k = 0; k < 5; ++k) {
    float* p = params->*members[k];
    if (!p) continue;
    const float* g = grads->*members[k];
    float* m = exp_avg->*members[k];
    float* v = exp_avg_sq->*members[k];
    if (!g || !m || !v)
      return set_error(LODGS_E_INVALID, "lodgs_adam_cut: a group has parameters but no gradient or moments");
    if (widths[k] % 4 == 0 && ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(g) |
                                reinterpret_cast<uintptr_t>(m) | reinterpret_cast<uintptr_t>(v)) & 15u))
      return set_error(LODGS_E_INVALID, "lodgs_adam_cut: quaternion and SH arrays must be 16-byte aligned");
    grp.g[n_groups++] = AdamGroup{p, g, m, v, widths[k], (float)((double)hp->lr[k] / bc1)};
  }
  const AdamConst a{hp->beta1, hp->beta2, hp->eps, (float)std::sqrt(bc2)};
  if (n_groups == 0 || capacity == 0) return LODGS_OK;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // one thread per chunk of the capacity, up to 4096 workgroups for the SH rows
  // and 1024 for each narrow group (a selection fills few of a large capacity)
  for (int k = 0; k < 5; ++k) {
    int64_t blocks = 0;
    if (k < n_groups) {
      const int32_t w = grp.g[k].w, chunks = w % 4 == 0 ? w / 4 : w;
      blocks = std::min<int64_t>((capacity * chunks + kBlock - 1) / kBlock, w > 4 ? 4096 : 1024);
    }
    grp.first[k + 1] = grp.first[k] + (uint32_t)blocks;
  }
  hipLaunchKernelGGL(k_adam_cut, dim3(grp.first[5]), dim3(kBlock), 0, st, grp, a, d_idx, d_count, capacity, n_nodes);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? LODGS_OK : hip_fail(e, "lodgs_adam_cut");
}
