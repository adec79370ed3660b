// What PPO consumes after a rollout, computed on the device from the outputs of rollout_generate
// and score_sequences: per-token rewards (KL penalty per kept token, reward-model score on the last
// kept token, a constant in place of the score when the response has no EOS), generalised advantage
// estimates with returns, batch whitening, and the clipped objective with its gradient with respect
// to the model's outputs.  The arrays are tiny (batch x 53), so the kernels are
// latency-bound by construction: one wave per row, sums and recursions in double and in a fixed
// order (bit-reproducible; no atomics).
#include "common.h"

namespace rlhf {

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

template <int O>
__device__ __forceinline__ double add_lane_xor(double v) {
  const int lo = lane_xor<O>(__double2loint(v)), hi = lane_xor<O>(__double2hiint(v));
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_d(double v) {
  v = add_lane_xor<32>(v);
  v = add_lane_xor<16>(v);
  v = add_lane_xor<8>(v);
  v = add_lane_xor<4>(v);
  v = add_lane_xor<2>(v);
  return add_lane_xor<1>(v);
}

// One wave per row.  first = index of the first pad in the response (N if none); the row's kept
// tokens are t <= last = first - 1 (N - 1 if none), which is also where the reward model is read.
// What a chain of dependent loads costs is all there is here, so the first 64 columns of every input are requested at
// once, before the row's length is known (64 rows of 53 tokens: 7.4 -> 5.2 us).
__global__ void __launch_bounds__(64)
    ppo_rewards_kernel(const float* __restrict__ lp, const float* __restrict__ ref_full,
                       const float* __restrict__ rm_full, const int* __restrict__ tokens, int Lq, int N, int eos_id,
                       int pad_id, float beta, float miss, float* __restrict__ rewards, float* __restrict__ scores,
                       float* __restrict__ kl_out, int* __restrict__ kept) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const size_t L = (size_t)Lq + N;
  const int* tok = tokens + b * L + Lq;
  const float* ref = ref_full + b * L + Lq;
  const float* rm = rm_full + b * L + Lq;
  const float* row = lp + (size_t)b * N;
  const int t0 = min(lane, N - 1);
  const int tok0 = tok[t0];
  const float lp0 = row[t0], ref0 = ref[t0], rm0 = rm[t0];
  int first = lane < N && tok0 == pad_id ? lane : N;
  for (int t = lane + 64; t < N; t += 64)
    if (tok[t] == pad_id) first = min(first, t);
  first = wave_min_i(first);
  const int last = first - 1;  // -1: nothing was generated for this row
  float score = 0.f;
  if (last >= 0) {
    const int tok_l = last < 64 ? __shfl(tok0, last & 63, 64) : tok[last];
    const float rm_l = last < 64 ? __shfl(rm0, last & 63, 64) : rm[last];
    score = tok_l == eos_id ? rm_l : miss;
  }
  double kl = 0.0;
  for (int t = lane; t < N; t += 64) {
    float r = 0.f;
    if (t <= last) {
      const float x = t < 64 ? lp0 : row[t], y = t < 64 ? ref0 : ref[t];
      r = -beta * (x - y);
      if (t == last) r += score;
      kl += (double)x - (double)y;
    }
    rewards[(size_t)b * N + t] = r;
  }
  kl = wave_sum_d(kl);
  if (lane == 0) {
    kl_out[b] = (float)kl;
    scores[b] = score;
    kept[b] = last + 1;
  }
}

// One wave per row: A_t = delta_t + gamma * lambda * A_{t+1}, delta_t = r_t + gamma * V_{t+1} - V_t,
// V = 0 beyond the last kept token; returns = A + V.  Lane t holds token t of a run of 64: the loads and the deltas of a
// run are one step, and only the recursion itself is serial, every lane following it with the deltas broadcast from
// their lanes (a thread per row waited for two loads per token: 20 -> 6.1 us for 64 rows of 53 tokens).
__global__ void __launch_bounds__(64)
    ppo_gae_kernel(const float* __restrict__ rewards, const float* __restrict__ values, long vstride,
                   const int* __restrict__ kept, int N, float gamma, float lam, float* __restrict__ adv,
                   float* __restrict__ ret) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int L = __builtin_amdgcn_readfirstlane(min(max(kept[b], 0), N));
  const float* r = rewards + (size_t)b * N;
  const float* v = values + (size_t)b * vstride;
  float* const a_out = adv + (size_t)b * N;
  float* const r_out = ret + (size_t)b * N;
  for (int t = lane; t < N; t += 64)
    if (t >= L) {
      a_out[t] = 0.f;
      r_out[t] = 0.f;
    }
  const double gl = (double)gamma * (double)lam;
  double running = 0.0;
  float v_next = 0.f;  // the value after the run (0 beyond the last kept token)
  for (int c = (L - 1) & ~63; c >= 0; c -= 64) {
    const int t = c + lane, n = min(64, L - c);
    const float rt = t < L ? r[t] : 0.f, vf = t < L ? v[t] : 0.f;
    const float vn = __shfl_down(vf, 1, 64);
    const double vt = vf;
    const double delta = (double)rt + (double)gamma * (double)(lane == 63 ? v_next : vn) - vt;
    double mine = 0.0;
    for (int j = n - 1; j >= 0; --j) {
      const double dj = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(delta), j),
                                         __builtin_amdgcn_readlane(__double2loint(delta), j));
      running = dj + gl * running;
      if (lane == j) mine = running;
    }
    if (t < L) {
      a_out[t] = (float)mine;
      r_out[t] = (float)(mine + vt);
    }
    v_next = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(vf)));
  }
}

// Sums of K values over a block of 1024, one barrier: trees within the waves, then the waves in order.  sh is written
// once per call, so successive calls take arrays of their own.
template <int K>
__device__ __forceinline__ void block_sums_1024_d(double (&v)[K], double (&sh)[K][16]) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = wave_sum_d(v[k]);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += sh[k][i];
    v[k] = t;
  }
}

// Positions tid, tid + 1024, ... of a [B, N] array as (row, column), without a division per element.
struct Walk1024 {
  int row, col, dr, dc, N;
  __device__ explicit Walk1024(int n) : dr(1024 / n), dc(1024 % n), N(n) {
    row = (int)threadIdx.x / n;
    col = (int)threadIdx.x - row * n;
  }
  __device__ void next() {
    row += dr;
    col += dc;
    if (col >= N) {
      col -= N;
      ++row;
    }
  }
};

// One block: (x - mean) * rsqrt(var + 1e-8) over the kept positions, biased variance; the mean is
// added back when shift_mean is 0.  Positions that are not kept get 0.
// A thread's first WR elements stay in registers over the three passes (64 rows of 53 tokens: 9.2 -> 6.4 us, where
// 64-bit divisions for an element's row were most of it).
__global__ void __launch_bounds__(1024)
    ppo_whiten_kernel(const float* __restrict__ x, const int* __restrict__ kept, int B, int N, int shift_mean,
                      float* __restrict__ out) {
  constexpr int WR = 4;
  __shared__ double sh1[2][16], sh2[1][16];
  const size_t total = (size_t)B * N, tid = threadIdx.x;
  float xr[WR];
  bool kr[WR];
  Walk1024 rest(N);
#pragma unroll
  for (int e = 0; e < WR; ++e, rest.next()) {
    const size_t i = tid + e * (size_t)1024;
    kr[e] = i < total && (!kept || rest.col < kept[rest.row]);
    xr[e] = i < total ? x[i] : 0.f;
  }
  auto each_kept = [&](auto f) {
#pragma unroll
    for (int e = 0; e < WR; ++e)
      if (kr[e]) f(xr[e]);
    Walk1024 w = rest;
    for (size_t i = tid + WR * (size_t)1024; i < total; i += 1024, w.next())
      if (!kept || w.col < kept[w.row]) f(x[i]);
  };
  double s[2] = {0.0, 0.0};
  each_kept([&](float v) {
    s[0] += v;
    s[1] += 1.0;
  });
  block_sums_1024_d<2>(s, sh1);
  const double n = s[1], mean = n > 0 ? s[0] / n : 0.0;
  double q[1] = {0.0};
  each_kept([&](float v) {
    const double dlt = v - mean;
    q[0] += dlt * dlt;
  });
  block_sums_1024_d<1>(q, sh2);
  const double var = n > 0 ? q[0] / n : 0.0;
  const double rstd = 1.0 / sqrt(var + 1e-8);
  auto white = [&](float v) {
    double w = (v - mean) * rstd;
    if (!shift_mean) w += mean;
    return (float)w;
  };
#pragma unroll
  for (int e = 0; e < WR; ++e)
    if (tid + e * (size_t)1024 < total) out[tid + e * (size_t)1024] = kr[e] ? white(xr[e]) : 0.f;
  Walk1024 w = rest;
  for (size_t i = tid + WR * (size_t)1024; i < total; i += 1024, w.next())
    out[i] = (!kept || w.col < kept[w.row]) ? white(x[i]) : 0.f;
}

// One block: the clipped PPO objective over the kept response tokens and its gradient with respect
// to the new log-probs and the new values.  Branch choice and sums in double, fixed order.
// stats: loss, pg_loss, vf_loss, approx_kl, pg_clipfrac, vf_clipfrac, ratio_mean, n_tokens.
// The token count comes from the rows' lengths, and the first LR elements of a thread are requested before it is formed;
// the six sums share one reduction (64 rows of 53 tokens: 19.8 -> 8.1 us).
__global__ void __launch_bounds__(1024)
    ppo_loss_kernel(const float* __restrict__ lp, const float* __restrict__ lp0, const float* __restrict__ adv,
                    const float* __restrict__ v, const float* __restrict__ v0, const float* __restrict__ ret,
                    const int* __restrict__ kept, int B, int N, float eps, float eps_v, float c1,
                    float* __restrict__ d_lp, float* __restrict__ d_v, float* __restrict__ stats) {
  constexpr int LR = 4;
  __shared__ double sh1[1][16], sh2[6][16];
  const size_t total = (size_t)B * N, tid = threadIdx.x;
  struct In {
    float lp, lp0, adv, v, v0, ret;
  };
  auto load = [&](size_t i) { return In{lp[i], lp0[i], adv[i], v[i], v0[i], ret[i]}; };
  In in[LR];
  bool kr[LR];
  Walk1024 w(N);
#pragma unroll
  for (int e = 0; e < LR; ++e, w.next()) {
    const size_t i = tid + e * (size_t)1024;
    kr[e] = i < total && w.col < kept[w.row];
    in[e] = load(min(i, total - 1));
  }
  double cnt[1] = {0.0};
  for (int b = threadIdx.x; b < B; b += 1024) cnt[0] += (double)min(max(kept[b], 0), N);
  block_sums_1024_d<1>(cnt, sh1);
  const double n = cnt[0];
  const double inv_n = n > 0 ? 1.0 / n : 0.0;
  double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // pg, vf, kl, ratio, clipped pg, clipped vf
  auto one = [&](size_t i, bool is_kept, const In& x) {
    float g_lp = 0.f, g_v = 0.f;
    if (is_kept) {
      const double diff = (double)x.lp - (double)x.lp0;
      const double ratio = exp(diff);
      const double ratio_c = fmin(fmax(ratio, 1.0 - (double)eps), 1.0 + (double)eps);
      const double a = x.adv;
      const double pg1 = -a * ratio, pg2 = -a * ratio_c;
      sum[0] += fmax(pg1, pg2);
      if (pg2 > pg1) sum[4] += 1.0;
      else g_lp = (float)(-a * ratio * inv_n);
      const double vv = x.v, vo = x.v0, r = x.ret;
      const double v_c = fmin(fmax(vv, vo - (double)eps_v), vo + (double)eps_v);
      const double vf1 = (vv - r) * (vv - r), vf2 = (v_c - r) * (v_c - r);
      sum[1] += 0.5 * fmax(vf1, vf2);
      if (vf2 > vf1) sum[5] += 1.0;
      else g_v = (float)((double)c1 * (vv - r) * inv_n);
      sum[2] += 0.5 * diff * diff;
      sum[3] += ratio;
    }
    d_lp[i] = g_lp;
    d_v[i] = g_v;
  };
#pragma unroll
  for (int e = 0; e < LR; ++e)
    if (tid + e * (size_t)1024 < total) one(tid + e * (size_t)1024, kr[e], in[e]);
  for (size_t i = tid + LR * (size_t)1024; i < total; i += 1024, w.next()) one(i, w.col < kept[w.row], load(i));
  block_sums_1024_d<6>(sum, sh2);
  if (threadIdx.x == 0) {
    const double pg = sum[0] * inv_n, vf = sum[1] * inv_n;
    stats[0] = (float)(pg + (double)c1 * vf);
    stats[1] = (float)pg;
    stats[2] = (float)vf;
    stats[3] = (float)(sum[2] * inv_n);
    stats[4] = (float)(sum[4] * inv_n);
    stats[5] = (float)(sum[5] * inv_n);
    stats[6] = (float)(sum[3] * inv_n);
    stats[7] = (float)n;
  }
}

hipError_t launch_ppo_loss(const float* lp, const float* lp0, const float* adv, const float* v, const float* v0,
                           const float* ret, const int* kept, int B, int N, float eps, float eps_v, float c1,
                           float* d_lp, float* d_v, float* stats, hipStream_t s) {
  hipLaunchKernelGGL(ppo_loss_kernel, dim3(1), dim3(1024), 0, s, lp, lp0, adv, v, v0, ret, kept, B, N, eps, eps_v, c1,
                     d_lp, d_v, stats);
  return hipGetLastError();
}

hipError_t launch_ppo_rewards(const float* lp, const float* ref_full, const float* rm_full, const int* tokens, int B,
                              int Lq, int N, int eos_id, int pad_id, float beta, float miss, float* rewards,
                              float* scores, float* kl, int* kept, hipStream_t s) {
  hipLaunchKernelGGL(ppo_rewards_kernel, dim3(B), dim3(64), 0, s, lp, ref_full, rm_full, tokens, Lq, N, eos_id,
                     pad_id, beta, miss, rewards, scores, kl, kept);
  return hipGetLastError();
}

hipError_t launch_ppo_gae(const float* rewards, const float* values, long vstride, const int* kept, int B, int N,
                          float gamma, float lam, float* adv, float* ret, hipStream_t s) {
  hipLaunchKernelGGL(ppo_gae_kernel, dim3(B), dim3(64), 0, s, rewards, values, vstride, kept, N, gamma, lam, adv, ret);
  return hipGetLastError();
}

hipError_t launch_ppo_whiten(const float* x, const int* kept, int B, int N, int shift_mean, float* out,
                             hipStream_t s) {
  hipLaunchKernelGGL(ppo_whiten_kernel, dim3(1), dim3(1024), 0, s, x, kept, B, N, shift_mean, out);
  return hipGetLastError();
}

// ---- glue of the update loop ------------------------------------------------------------------------------
__global__ void ppo_slice_kernel(const float* __restrict__ lp_full, const float* __restrict__ val_full, int L, int Lq,
                                 int N, float* __restrict__ new_lp, float* __restrict__ new_v) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < N; j += blockDim.x) {
    new_lp[(size_t)b * N + j] = lp_full[(size_t)b * L + Lq + j];
    new_v[(size_t)b * N + j] = (Lq - 1 + j >= 0) ? val_full[(size_t)b * L + Lq - 1 + j] : 0.f;
  }
}

hipError_t launch_ppo_slice(const float* lp_full, const float* val_full, int B, int L, int Lq, int N, float* new_lp,
                            float* new_v, hipStream_t s) {
  hipLaunchKernelGGL(ppo_slice_kernel, dim3(B), dim3(64), 0, s, lp_full, val_full, L, Lq, N, new_lp, new_v);
  return hipGetLastError();
}

__global__ void ppo_pack_grads_kernel(const int32_t* __restrict__ tokens, int L, int Lq, int N,
                                      const int* __restrict__ start, const int* __restrict__ len,
                                      const int* __restrict__ cu, const float* __restrict__ d_lp,
                                      const float* __restrict__ d_v, int32_t* __restrict__ targets,
                                      float* __restrict__ gl, float* __restrict__ gv) {
  const int b = blockIdx.x;
  const int st = start[b], n = len[b], base = cu[b];
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int c = st + i;
    const bool nxt = i + 1 < n;  // the next token of the row is real
    const int jr = c + 1 - Lq;   // response index of the token this row predicts
    const int jv = c - (Lq - 1); // response index whose value is read at this position
    targets[base + i] = nxt ? tokens[(size_t)b * L + c + 1] : -1;
    gl[base + i] = (nxt && jr >= 0 && jr < N) ? d_lp[(size_t)b * N + jr] : 0.f;
    gv[base + i] = (jv >= 0 && jv < N) ? d_v[(size_t)b * N + jv] : 0.f;
  }
}

hipError_t launch_ppo_pack_grads(const int32_t* tokens, int B, int L, int Lq, int N, const int* start, const int* len,
                                 const int* cu, const float* d_lp, const float* d_v, int32_t* targets, float* gl,
                                 float* gv, hipStream_t s) {
  hipLaunchKernelGGL(ppo_pack_grads_kernel, dim3(B), dim3(256), 0, s, tokens, L, Lq, N, start, len, cu, d_lp, d_v,
                     targets, gl, gv);
  return hipGetLastError();
}

}  // namespace rlhf
