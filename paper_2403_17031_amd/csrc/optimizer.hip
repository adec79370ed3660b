// AdamW step of the PPO update, fused over everything an update touches: fp32 master weights, both
// moments, and the bf16 storage copy of the weights (a bf16 model's matrices reach the forward passes through
// the fp16 image that rlhf_refresh_weights rebuilds from that copy).  Pure streaming work
// (16 bytes read, 12 to 14 written per element): 4 elements per lane, 16-byte accesses.
//
// One launch takes up to kAdamwTensors tensors.  A model's step is some 12 tensors a layer, most of them a bias or a gain that
// is no work at all but a launch and the gap after it.  The 160M shape's 150 tensors: 6.0 ms per four steps in 600 launches ->
// 3.85 in 20 (5.4 TB/s in the launch with the embeddings).  A step of one tensor has arguments for one.
#include <algorithm>

#include "common.h"

namespace rlhf {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;  // NaN stays NaN
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// The tensors of a launch: tensor i has the blocks from first[i] on, of chunk4 float4s each.
template <int N>
struct AdamwArgs {
  AdamwTensor t[N];
  uint32_t first[N];
  int count;
  uint32_t chunk4;
  AdamwScalars c;
};

template <typename T>
using global_ptr = __attribute__((address_space(1))) T*;

template <int N>
__global__ void __launch_bounds__(256) adamw_kernel(AdamwArgs<N> a) {
  int at = 0;  // this block's tensor: the last with first[at] <= blockIdx.x
#pragma unroll
  for (int step = N / 2; step; step /= 2)
    if (at + step < a.count && a.first[at + step] <= blockIdx.x) at += step;
  const auto p = (global_ptr<float>)a.t[at].p;
  const auto g = (global_ptr<const float>)a.t[at].g;
  const auto m = (global_ptr<float>)a.t[at].m;
  const auto v = (global_ptr<float>)a.t[at].v;
  const auto p_bf16 = (global_ptr<uint16_t>)a.t[at].p_bf16;
  const size_t n = a.t[at].n, n4 = n >> 2, chunk = blockIdx.x - a.first[at];
  const AdamwScalars c = a.c;
  auto upd = [&](float pv, float gv, float& mv, float& vv) {
    gv *= c.grad_scale;
    pv *= c.decay;
    mv = c.beta1 * mv + c.omb1 * gv;
    vv = c.beta2 * vv + c.omb2 * gv * gv;
    const float denom = sqrtf(vv) * c.inv_sqrt_bias2 + c.eps;
    return pv - c.step_size * (mv / denom);
  };
  const size_t end = std::min(n4, (chunk + 1) * a.chunk4);
  for (size_t i = chunk * a.chunk4 + threadIdx.x; i < end; i += 256) {
    f32x4_t pv = ((global_ptr<const f32x4_t>)p)[i];
    const f32x4_t gv = ((global_ptr<const f32x4_t>)g)[i];
    f32x4_t mv = ((global_ptr<const f32x4_t>)m)[i], vv = ((global_ptr<const f32x4_t>)v)[i];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float m1 = mv[u], v1 = vv[u];
      pv[u] = upd(pv[u], gv[u], m1, v1);
      mv[u] = m1;
      vv[u] = v1;
    }
    ((global_ptr<f32x4_t>)p)[i] = pv;
    ((global_ptr<f32x4_t>)m)[i] = mv;
    ((global_ptr<f32x4_t>)v)[i] = vv;
    if (p_bf16) {
      u32x2_t o;
      o[0] = f32_to_bf16_rne(pv[0]) | (f32_to_bf16_rne(pv[1]) << 16);
      o[1] = f32_to_bf16_rne(pv[2]) | (f32_to_bf16_rne(pv[3]) << 16);
      ((global_ptr<u32x2_t>)p_bf16)[i] = o;
    }
  }
  // ragged tail (n not a multiple of 4): one element per thread of the tensor's first block
  if (chunk == 0 && threadIdx.x < (n & 3)) {
    const size_t i = (n4 << 2) + threadIdx.x;
    float mv = m[i], vv = v[i];
    const float pv = upd(p[i], g[i], mv, vv);
    p[i] = pv;
    m[i] = mv;
    v[i] = vv;
    if (p_bf16) p_bf16[i] = (uint16_t)f32_to_bf16_rne(pv);
  }
}

// The step of the `count` tensors ts[idx[0]], ts[idx[1]], ...
template <int N>
static hipError_t adamw_group(const AdamwTensor* ts, const int* idx, int count, const AdamwScalars& c, hipStream_t s) {
  AdamwArgs<N> a;
  a.c = c;
  a.count = count;
  size_t n4 = 0;
  for (int i = 0; i < count; ++i) n4 += ts[idx[i]].n >> 2;
  // One float4 per thread up to 2^25 elements, four beyond.  us with one / four: 1 M elements 5.9 / 7.7, 2.4 M 10.8 / 12.2, 20 M
  // 96 / 103; one per thread but no more than 16384 blocks: 40 M 237, 100 M 625, where four are 227 and 563.
  a.chunk4 = n4 <= (size_t)1 << 23 ? 256 : 1024;
  uint32_t blocks = 0;
  for (int i = 0; i < count; ++i) {
    a.t[i] = ts[idx[i]];
    a.first[i] = blocks;
    blocks += (uint32_t)std::max<size_t>(1, ((a.t[i].n >> 2) + a.chunk4 - 1) / a.chunk4);
  }
  hipLaunchKernelGGL(adamw_kernel<N>, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_adamw(const AdamwTensor* ts, int count, const AdamwScalars& c, hipStream_t s) {
  int idx[kAdamwTensors], n = 0;
  for (int i = 0; i < count; ++i) {
    if (ts[i].n) idx[n++] = i;
    if (n && (n == kAdamwTensors || i + 1 == count)) {
      const hipError_t e = n == 1 ? adamw_group<1>(ts, idx, n, c, s) : adamw_group<kAdamwTensors>(ts, idx, n, c, s);
      if (e != hipSuccess) return e;
      n = 0;
    }
  }
  return hipSuccess;
}

}  // namespace rlhf
