// Kernels of a decode pass of few sequences (see run_decode_few in api.hip): the LayerNorm that also closes the
// previous layer, and single-query attention with the rotary turn and the K / V store as its prologue.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rlhf {

typedef __attribute__((ext_vector_type(8))) _Float16 dc_f16x8_t;
typedef __attribute__((ext_vector_type(4))) _Float16 dc_f16x4_t;
typedef __attribute__((ext_vector_type(2))) _Float16 dc_f16x2_t;
typedef __attribute__((ext_vector_type(4))) float dc_f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t dc_u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t dc_u32x2_t;

__device__ __forceinline__ dc_f32x4_t load4(const bf16_t* p) {
  const dc_u32x2_t v = *(const dc_u32x2_t*)p;
  return (dc_f32x4_t){__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xFFFF0000u), __uint_as_float(v[1] << 16),
                      __uint_as_float(v[1] & 0xFFFF0000u)};
}
__device__ __forceinline__ dc_f32x4_t load4(const float* p) { return *(const dc_f32x4_t*)p; }
__device__ __forceinline__ void store4(half_t* p, dc_f32x4_t v) {
  dc_f16x4_t o;
#pragma unroll
  for (int u = 0; u < 4; ++u) o[u] = from_f32<half_t>(v[u]);
  *(dc_f16x4_t*)p = o;
}
__device__ __forceinline__ void store4(float* p, dc_f32x4_t v) { *(dc_f32x4_t*)p = v; }

// Softmax weights: the bare instruction where they multiply fp16 values, expf in fp32 (weights of
// scores 50 to 80 below the maximum: 5e-7 off at most, against 4.4e-6).
__device__ __forceinline__ float softmax_exp(half_t, float x) { return __expf(x); }
__device__ __forceinline__ float softmax_exp(float, float x) { return expf(x); }

// One block per row, one float4 per thread (d <= 4096).  With KS > 0, x <- x + sum of KS fp32 slabs (in order) +
// bias_a + bias_b first: the layer's out-projection and FC2, left as partial sums by their product.  The outputs are
// packed operands (packed_index).  The kernel is
// latency and nothing else (one row per CU), so everything it reads is requested before the first sum.
template <typename WT, typename AT, int KS>
__global__ void __launch_bounds__(1024)
    ln_decode_kernel(float* __restrict__ x, int d, float eps, const WT* __restrict__ g1, const WT* __restrict__ b1,
                     AT* __restrict__ out1, const WT* __restrict__ g2, const WT* __restrict__ b2, AT* __restrict__ out2,
                     const float* __restrict__ part, size_t slab, const WT* __restrict__ bias_a,
                     const WT* __restrict__ bias_b, int write_x) {
  __shared__ __attribute__((aligned(16))) float sh[2][16];
  const int r = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  if (lane < 32 && wave == 0 && (lane & 15) >= waves) sh[lane >> 4][lane & 15] = 0.f;
  const int c = 4 * threadIdx.x;
  const bool in = c < d;
  const int cc = in ? c : 0;
  dc_f32x4_t v = *(const dc_f32x4_t*)(x + (size_t)r * d + cc);
  dc_f32x4_t t[KS > 0 ? KS : 1], bb;
  if (KS > 0) {
#pragma unroll
    for (int z = 0; z < KS; ++z) t[z] = *(const dc_f32x4_t*)(part + z * slab + (size_t)r * d + cc);
    bb = load4(bias_a + cc) + load4(bias_b + cc);
  }
  const dc_f32x4_t vg1 = load4(g1 + cc), vb1 = load4(b1 + cc);
  dc_f32x4_t vg2 = vg1, vb2 = vb1;
  if (out2) {
    vg2 = load4(g2 + cc);
    vb2 = load4(b2 + cc);
  }
  if (KS > 0) {
    dc_f32x4_t sum = t[0];
#pragma unroll
    for (int z = 1; z < KS; ++z) sum += t[z];
    v += sum + bb;
    if (write_x && in) *(dc_f32x4_t*)(x + (size_t)r * d + c) = v;
  }
  auto block_sum = [&](float s, float* buf) {
    s = wave_sum(s);
    if (lane == 0) buf[wave] = s;
    __syncthreads();
    // (buf is zero past the block's waves, so that all sixteen are read at once)
    dc_f32x4_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = *(const dc_f32x4_t*)(buf + 4 * i);
    float tot = t[0][0];
#pragma unroll
    for (int w = 1; w < 16; ++w) tot += t[w >> 2][w & 3];
    return tot;
  };
  const float mean = block_sum(in ? (v[0] + v[1]) + (v[2] + v[3]) : 0.f, sh[0]) / (float)d;
  v -= mean;
  const float q = in ? (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]) : 0.f;
  const float rstd = 1.0f / sqrtf(block_sum(q, sh[1]) / (float)d + eps);
  if (!in) return;
  const size_t o = packed_index<AT>(r, c, d);
  const dc_f32x4_t n = v * rstd;
  store4(out1 + o, n * vg1 + vb1);
  if (out2) store4(out2 + o, n * vg2 + vb2);
}

bool ln_decode_supported(int d) { return (d & 3) == 0 && d <= 4096; }

template <typename M>
static void ln_decode_launch(float* x, int rows, int d, float eps, const void* g1, const void* b1, void* out1,
                             const void* g2, const void* b2, void* out2, const float* part, int ks, size_t slab,
                             const void* bias_a, const void* bias_b, bool write_x, hipStream_t s) {
  typedef typename M::W WT;
  typedef typename M::A AT;
  const dim3 block((d / 4 + 63) / 64 * 64);
#define RLHF_LN(KS_)                                                                                                \
  hipLaunchKernelGGL((ln_decode_kernel<WT, AT, KS_>), dim3(rows), block, 0, s, x, d, eps, (const WT*)g1, (const WT*)b1, \
                     (AT*)out1, (const WT*)g2, (const WT*)b2, (AT*)out2, part, slab, (const WT*)bias_a,             \
                     (const WT*)bias_b, write_x ? 1 : 0)
  switch (ks) {
    case 0: RLHF_LN(0); break;
    case 1: RLHF_LN(1); break;
    case 2: RLHF_LN(2); break;
    case 4: RLHF_LN(4); break;
    default: RLHF_LN(8); break;
  }
#undef RLHF_LN
}

hipError_t launch_ln_decode(int dtype, float* x, int rows, int d, float eps, const void* g1, const void* b1, void* out1,
                            const void* g2, const void* b2, void* out2, const float* part, int ks, size_t slab,
                            const void* bias_a, const void* bias_b, bool write_x, hipStream_t s) {
  if (!ln_decode_supported(d) || ks < 0 || ks > 8 || (ks & (ks - 1)) != 0 || (slab & 3) != 0) return hipErrorInvalidValue;
  if (dtype == 0)
    ln_decode_launch<ModeF32>(x, rows, d, eps, g1, b1, out1, g2, b2, out2, part, ks, slab, bias_a, bias_b, write_x, s);
  else
    ln_decode_launch<ModeBF16>(x, rows, d, eps, g1, b1, out1, g2, b2, out2, part, ks, slab, bias_a, bias_b, write_x, s);
  return hipGetLastError();
}

// =================================================================================================
// Single-query attention with the rotary turn.  Block = one (head, sequence), WV waves.
//   The new token's q, k and v slices come from the row-major [rows, 3d] product; q and k are turned in LDS, k and v
//   are stored to the cache, and the row joins the sum from LDS.
//   The cached rows are a flat stream of 16-byte chunks, dealt to the waves in groups of U wave instructions; each
//   wave runs an online softmax over its own rows, so K and V of a group are requested together and no wave waits
//   for another before the end.  (A kernel in phases -- all scores, softmax, all of V -- has one memory round trip
//   more and two block-wide waits, which is what a small grid spends its time on.)
// lane = (g, part): part = chunk within a row (CPR per row), g = row within a wave instruction.
// =================================================================================================
template <typename T, int HD, int WV>
__global__ void __launch_bounds__(64 * WV)
    attn_decode_rope_kernel(const T* __restrict__ qkv, T* __restrict__ kc, T* __restrict__ vc, long kv_extra,
                            const int* __restrict__ len, int step, const int* __restrict__ kvoff, int H, int half,
                            const float* __restrict__ cos_t, const float* __restrict__ sin_t, float scale,
                            T* __restrict__ out, int out_cols) {
  constexpr int EPC = 16 / (int)sizeof(T), CPR = HD / EPC, G = 64 / CPR, ACTIVE = G * CPR, U = 4;
  constexpr bool POW2 = (CPR & (CPR - 1)) == 0;
  constexpr bool ADJ = sizeof(T) == 2;         // fp16 path: rotary pairs are neighbours
  constexpr int PDS = (CPR + 3) & ~3;          // floats per row of the partial-dot scratch
  __shared__ __attribute__((aligned(16))) T s_row[3][HD];
  __shared__ __attribute__((aligned(16))) float s_pd[POW2 ? 4 : WV * U * G * PDS];
  __shared__ __attribute__((aligned(16))) float s_acc[WV * G * HD];
  __shared__ float s_m[WV], s_l[WV];
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane / CPR, part = lane - g * CPR;
  const bool active = lane < ACTIVE;
  const int n = len[b], ctx = n + step, d = H * HD;  // ctx cached rows; the new one is row ctx
  const size_t base = ((size_t)kvoff[b] * H + (size_t)h * (n + kv_extra)) * HD;
  T* kb = kc + base;
  T* vb = vc + base;

  dc_u32x4_t kr[U], vr[U];
  auto load_rows = [&](int j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t o = (size_t)min(j0 + u * G + g, ctx - 1) * HD + (active ? part : 0) * EPC;
      kr[u] = *(const dc_u32x4_t*)(kb + o);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t o = (size_t)min(j0 + u * G + g, ctx - 1) * HD + (active ? part : 0) * EPC;
      vr[u] = *(const dc_u32x4_t*)(vb + o);
    }
  };
  const int j_first = wave * (U * G);
  // ---- the new row: load, turn, store.  Its loads are issued ahead of the cache's: loads retire in order, so nothing
  //      below waits for the first group of K and V before it is needed.
  dc_u32x4_t nrow = {0, 0, 0, 0};
  if (tid < 3 * CPR) {
    const int sec = tid / CPR, ch = tid - sec * CPR;
    nrow = *(const dc_u32x4_t*)(qkv + (size_t)b * 3 * d + (size_t)sec * d + (size_t)h * HD + ch * EPC);
  }
  const int turn = tid < 2 * half ? tid : -1, tsec = turn >= half ? 1 : 0, ti = turn - tsec * half;  // 2 * half <= HD <= 256
  float co = 0.f, si = 0.f;
  if (turn >= 0) {
    co = cos_t[(size_t)ctx * half + ti];
    si = sin_t[(size_t)ctx * half + ti];
  }
  if (j_first < ctx) load_rows(j_first);
  if (!POW2)
    for (int c = tid; c < (POW2 ? 0 : WV * U * G * PDS); c += 64 * WV) s_pd[c] = 0.f;
  if (tid < 3 * CPR) {
    const int sec = tid / CPR, ch = tid - sec * CPR;
    *(dc_u32x4_t*)(&s_row[sec][ch * EPC]) = nrow;
  }
  __syncthreads();
  if (turn >= 0) {
    T& lo = s_row[tsec][ADJ ? 2 * ti : ti];
    T& hi = s_row[tsec][ADJ ? 2 * ti + 1 : ti + half];
    const float a = to_f32(lo), e = to_f32(hi);
    lo = from_f32<T>(a * co - e * si);
    hi = from_f32<T>(e * co + a * si);
  }
  __syncthreads();
  if (tid < 2 * CPR) {
    const int sec = tid / CPR, ch = tid - sec * CPR;
    *(dc_u32x4_t*)((sec ? vb : kb) + (size_t)ctx * HD + ch * EPC) = *(const dc_u32x4_t*)(&s_row[1 + sec][ch * EPC]);
  }
  dc_u32x4_t qr = {0, 0, 0, 0};
  if (active) qr = *(const dc_u32x4_t*)(&s_row[0][part * EPC]);

  auto dot = [&](dc_u32x4_t k) {
    float pd = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (ADJ) {
        pd = __builtin_amdgcn_fdot2(__builtin_bit_cast(dc_f16x2_t, (uint32_t)k[i]), __builtin_bit_cast(dc_f16x2_t, (uint32_t)qr[i]), pd, false);
      } else {
        pd = fmaf(__uint_as_float(k[i]), __uint_as_float(qr[i]), pd);
      }
    }
    return pd;
  };
  // sums over the CPR lanes of a row, left in all of them
  float* pdw = s_pd + (POW2 ? 0 : wave * (U * G * PDS));
  auto row_sums = [&](float* pd, auto nu) {
    constexpr int NU = decltype(nu)::value;
    if constexpr (POW2) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (CPR > 1) pd[u] += lane_xor<1>(pd[u]);
        if (CPR > 2) pd[u] += lane_xor<2>(pd[u]);
        // (the value repeats every 4, 8 lanes by now: mirroring a half row, a row, is the exchange with lane ^ 4, ^ 8)
        if (CPR > 4) pd[u] += __int_as_float(dpp_mov<0x141>(__float_as_int(pd[u])));
        if (CPR > 8) pd[u] += __int_as_float(dpp_mov<0x140>(__float_as_int(pd[u])));
        if (CPR > 16) pd[u] += lane_xor<16>(pd[u]);
        if (CPR > 32) pd[u] += lane_xor<32>(pd[u]);
      }
    } else {
      __builtin_amdgcn_wave_barrier();
      if (active) {
#pragma unroll
        for (int u = 0; u < NU; ++u) pdw[(u * G + g) * PDS + part] = pd[u];
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const int gg = active ? g : 0;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        dc_f32x4_t t = *(const dc_f32x4_t*)(pdw + (u * G + gg) * PDS);
#pragma unroll
        for (int k = 4; k < PDS; k += 4) t += *(const dc_f32x4_t*)(pdw + (u * G + gg) * PDS + k);
        pd[u] = (t[0] + t[1]) + (t[2] + t[3]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  };
  float m_run = -INFINITY, l_run = 0.f, acc[EPC];
#pragma unroll
  for (int i = 0; i < EPC; ++i) acc[i] = 0.f;
  auto add_v = [&](float p, dc_u32x4_t v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (ADJ) {
        const dc_f16x2_t x = __builtin_bit_cast(dc_f16x2_t, (uint32_t)v[i]);
        acc[(2 * i) % EPC] = fmaf(p, (float)x[0], acc[(2 * i) % EPC]);
        acc[(2 * i + 1) % EPC] = fmaf(p, (float)x[1], acc[(2 * i + 1) % EPC]);
      } else {
        acc[i % EPC] = fmaf(p, __uint_as_float(v[i]), acc[i % EPC]);
      }
    }
  };
  if (wave == 0) {  // the new row, counted once: by the first group
    float pd[1] = {active ? dot(*(const dc_u32x4_t*)(&s_row[1][part * EPC])) : 0.f};
    row_sums(pd, std::integral_constant<int, 1>{});
    m_run = __shfl(pd[0] * scale, 0, 64);
    if (g == 0) {
      l_run = 1.f;
      add_v(1.f, *(const dc_u32x4_t*)(&s_row[2][part * EPC]));
    }
  }
  for (int j0 = j_first; j0 < ctx; j0 += WV * U * G) {
    float pd[U];
#pragma unroll
    for (int u = 0; u < U; ++u) pd[u] = active ? dot(kr[u]) : 0.f;
    row_sums(pd, std::integral_constant<int, U>{});
    float mx = m_run;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      pd[u] = active && j0 + u * G + g < ctx ? pd[u] * scale : -INFINITY;
      mx = fmaxf(mx, pd[u]);
    }
    mx = wave_max(mx);  // finite: row j0 is real
    const float alpha = softmax_exp(T(), m_run - mx);
    m_run = mx;
    l_run *= alpha;
#pragma unroll
    for (int i = 0; i < EPC; ++i) acc[i] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float p = softmax_exp(T(), pd[u] - mx);
      l_run += p;
      add_v(p, vr[u]);
    }
    if (j0 + WV * U * G < ctx) load_rows(j0 + WV * U * G);  // (a second group in flight measured the same)
  }
  // ---- merge: waves bring their sums to the common maximum, then the waves' rows are added
  {
    const float l = wave_sum(active && part == 0 ? l_run : 0.f);
    if (lane == 0) {
      s_m[wave] = m_run;
      s_l[wave] = l;
    }
  }
  float* aw = s_acc + (size_t)wave * G * HD;
  if (active) {
#pragma unroll
    for (int i = 0; i < EPC; i += 4) *(dc_f32x4_t*)(aw + g * HD + part * EPC + i) = (dc_f32x4_t){acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
  }
  __syncthreads();
  float m = s_m[0];
#pragma unroll
  for (int w = 1; w < WV; ++w) m = fmaxf(m, s_m[w]);
  float den = 0.f;
#pragma unroll
  for (int w = 0; w < WV; ++w) den += s_l[w] * softmax_exp(T(), s_m[w] - m);
  const float f = softmax_exp(T(), m_run - m);
  for (int e = lane; e < HD; e += 64) {
    float o = 0.f;
#pragma unroll
    for (int r = 0; r < G; ++r) o += aw[r * HD + e];
    aw[e] = o * f;  // column e of this wave's rows is read and written by this lane only
  }
  __syncthreads();
  const float inv = 1.0f / den;
  for (int e = tid; e < HD; e += 64 * WV) {
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < WV; ++w) o += s_acc[(size_t)w * G * HD + e];
    out[packed_index<T>(b, h * HD + e, out_cols)] = from_f32<T>(o * inv);
  }
}

bool attn_decode_rope_supported(int hd, int r) {
  return (hd == 16 || hd == 64 || hd == 80 || hd == 128 || hd == 256) && (r & 1) == 0 && r <= hd;
}

template <typename T, int HD>
static void launch_adr(const void* qkv, void* kc, void* vc, long kv_extra, int B, const int* len, int step, int ctx_max,
                       const int* kvoff, int H, int r, const float* cos_t, const float* sin_t, void* out, int out_cols,
                       hipStream_t s) {
  constexpr int CPR = HD / (16 / (int)sizeof(T)), ROWS = 4 * (64 / CPR);  // rows a wave takes at a time
  // Waves per block: about twenty waves fit a CU (registers), so sixteen while there is at most one block per CU, eight
  // for two, else four; fewer once a context gives that many waves nothing to do.
  int wv = B * H <= 256 ? 16 : (B * H <= 512 ? 8 : 4);
  while (wv > 4 && wv / 2 * ROWS >= ctx_max) wv /= 2;
#define RLHF_ADR(WV_)                                                                                                  \
  hipLaunchKernelGGL((attn_decode_rope_kernel<T, HD, WV_>), dim3(H, B), dim3(64 * WV_), 0, s, (const T*)qkv, (T*)kc,   \
                     (T*)vc, kv_extra, len, step, kvoff, H, r / 2, cos_t, sin_t, 1.0f / sqrtf((float)HD), (T*)out,     \
                     out_cols)
  if (wv == 4) RLHF_ADR(4);
  else if (wv == 8) RLHF_ADR(8);
  else RLHF_ADR(16);
#undef RLHF_ADR
}

hipError_t launch_attn_decode_rope(int dtype, const void* qkv, void* kc, void* vc, long kv_extra, int B, const int* len,
                                   int step, int ctx_max, const int* kvoff, int H, int hd, int r, const float* cos_t,
                                   const float* sin_t, void* out, int out_cols, hipStream_t s) {
#define RLHF_HD(HD_)                                                                                                    \
  case HD_:                                                                                                             \
    if (dtype == 0)                                                                                                     \
      launch_adr<float, HD_>(qkv, kc, vc, kv_extra, B, len, step, ctx_max, kvoff, H, r, cos_t, sin_t, out, out_cols, s);  \
    else                                                                                                                \
      launch_adr<half_t, HD_>(qkv, kc, vc, kv_extra, B, len, step, ctx_max, kvoff, H, r, cos_t, sin_t, out, out_cols, s); \
    return hipGetLastError();
  switch (hd) {
    RLHF_HD(16) RLHF_HD(64) RLHF_HD(80) RLHF_HD(128) RLHF_HD(256)
    default: return hipErrorInvalidValue;
  }
#undef RLHF_HD
}

}  // namespace rlhf
