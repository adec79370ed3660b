// Stand-alone driver for the few-rows (decode) products of a model layer: the QKV, out-projection, FC1, FC2 and
// LM-head shapes at M rows (the batch), through the library's own launch_gemm.  Each shape is checked on sampled
// outputs against a double-precision dot product on the host, then timed with HIP events twice: on one weight
// matrix (warm: it stays in the caches) and rotating over more than 1 GB of weight copies (cold: every launch
// streams its weights from HBM, as a decode pass does).  Like the other drivers it exists because hardware
// counters (rocprofv3 --pmc) can be collected on a small native process where they cannot on the Python benchmark.
// Up to 256 rows the three product launches of a few-rows decode pass follow, cold, as that pass makes them (packed A,
// QKV and FC1 in one launch, out-projection and FC2 as one product left as slabs, LM head), and again with row-major A.
//   usage: dec_driver [M=256] [d_model=2560] [reps=96] [max_split=0] [timed_phase=0] [pad_a=0] [pad_w=0]
//   (pad_a / pad_w: elements added to the row strides of A / W, to see what the address-to-channel mapping costs)
//   (timed_phase 1 times the partial products alone, as the decode loop runs them: their reductions are folded
//   into the kernels that consume them)
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "common.h"

using namespace rlhf;

#define CK(x)                                                                               \
  do {                                                                                      \
    hipError_t e_ = (x);                                                                    \
    if (e_ != hipSuccess) {                                                                 \
      printf("HIP error %s at %s:%d\n", hipGetErrorString(e_), __FILE__, __LINE__);         \
      return 1;                                                                             \
    }                                                                                       \
  } while (0)

static uint16_t f2h(float f) { _Float16 h = (_Float16)f; uint16_t u; memcpy(&u, &h, 2); return u; }
static float h2f(uint16_t u) { _Float16 h; memcpy(&h, &u, 2); return (float)h; }
static uint16_t f2bf(float f) { unsigned u; memcpy(&u, &f, 4); u += 0x7FFF + ((u >> 16) & 1); return (uint16_t)(u >> 16); }
static float bf2f(uint16_t h) { unsigned u = ((unsigned)h) << 16; float f; memcpy(&f, &u, 4); return f; }

// The few-rows launches.  W: R copies of wmax elements, of which QKV | FC1 | (W_o | W_fc2) of a layer, or the LM head, are
// the first.  Returns the number of wrong outputs.
static int few_rows_part(int M, int d, int F, int V, int reps, int R, size_t wmax, const std::vector<uint16_t>& hW,
                         const uint16_t* dW, const std::vector<uint16_t>& hb, const uint16_t* db, float* dO, hipEvent_t e0,
                         hipEvent_t e1) {
  const size_t rows = (size_t)(M + 15) / 16 * 16;
  std::vector<uint16_t> hA(rows * (d + F));  // read as [rows, d] or [rows, d + F], packed or row-major
  for (auto& x : hA) x = f2h((rand() % 2001 - 1000) / 1000.0f);
  uint16_t *dA, *dF;
  CK(hipMalloc(&dA, hA.size() * 2)); CK(hipMalloc(&dF, hA.size() * 2));
  CK(hipMemcpy(dA, hA.data(), hA.size() * 2, hipMemcpyHostToDevice));
  auto at = [](int m, int k, int K) { return ((size_t)(m >> 4) * (K / 8) + k / 8) * 128 + (m & 15) * 8 + k % 8; };
  const size_t o_fc1 = (size_t)3 * d * d, o_out = o_fc1 + (size_t)F * d;
  int bad = 0;
  for (int which = 0; which < 3; ++which)
    for (int packed = 1; packed >= 0; --packed) {
      const int K = which == 1 ? d + F : d, N = which == 1 ? d : (which == 2 ? V : 3 * d);
      FewRowsArgs a;
      a.M_max = M;
      auto point = [&](const uint16_t* w) {
        fr_seg(1, a.p[0].seg[0], dA, which == 1 ? w + o_out : w, K, packed ? -K : 0, 0);
        if (which == 0) fr_seg(1, a.p[1].seg[0], dA, w + o_fc1, d, packed ? -d : 0, 0);
      };
      point(dW);
      a.p[0].out = dO; a.p[0].N = a.p[0].ldo = N; a.p[0].epilogue = which ? EPI_F32 : EPI_BIAS;
      if (which == 0) {
        a.p[0].bias = a.p[1].bias = db;
        a.p[1].out = dF; a.p[1].N = F; a.p[1].epilogue = EPI_BIAS_GELU; a.p[1].packed_K = d + F; a.p[1].packed_k0 = d;
      }
      if (which == 1) { a.p[0].slab = (size_t)M * d; a.p[0].ksplit = few_rows_splits(d, a.p[0].seg[0].steps); }
      const int prods = which ? 1 : 2, ks = a.p[0].ksplit;
      CK(launch_few_rows(1, a, prods, 0)); CK(hipDeviceSynchronize());
      std::vector<uint16_t> o16((size_t)M * N), f16(hA.size());
      std::vector<float> o32((size_t)ks * M * N);
      if (which) CK(hipMemcpy(o32.data(), dO, o32.size() * 4, hipMemcpyDeviceToHost));
      else {
        CK(hipMemcpy(o16.data(), dO, o16.size() * 2, hipMemcpyDeviceToHost));
        CK(hipMemcpy(f16.data(), dF, f16.size() * 2, hipMemcpyDeviceToHost));
      }
      for (int t = 0; t < 600; ++t) {
        const bool fc1 = which == 0 && t % 2;
        const int r = rand() % M, c = rand() % (fc1 ? F : N);
        const uint16_t* w = hW.data() + (which == 1 ? o_out : (fc1 ? o_fc1 : 0)) + (size_t)c * K;
        double acc = 0, got = 0;
        for (int k = 0; k < K; ++k) acc += (double)h2f(hA[packed ? at(r, k, K) : (size_t)r * K + k]) * h2f(w[k]);
        if (which == 0) acc += bf2f(hb[c]);
        if (fc1) acc = 0.5 * acc * (1 + erf(acc / sqrt(2.0)));
        if (which) for (int z = 0; z < ks; ++z) got += o32[((size_t)z * M + r) * N + c];
        else got = h2f(fc1 ? f16[at(r, d + c, d + F)] : o16[(size_t)r * N + c]);
        if (fabs(got - acc) > (which ? 4e-3 : 8e-3 * fmax(1.0, fabs(acc)))) {
          printf("MISMATCH few rows, launch %d, packed %d: r=%d c=%d got %f want %f\n", which, packed, r, c, got, acc);
          ++bad;
          break;
        }
      }
      for (int i = 0; i < 8; ++i) { point(dW + (size_t)(i % R) * wmax); CK(launch_few_rows(1, a, prods, 0)); }
      CK(hipEventRecord(e0, 0));
      for (int i = 0; i < reps; ++i) { point(dW + (size_t)(i % R) * wmax); CK(launch_few_rows(1, a, prods, 0)); }
      CK(hipEventRecord(e1, 0)); CK(hipEventSynchronize(e1));
      float ms; CK(hipEventElapsedTime(&ms, e0, e1)); ms /= reps;
      const double wb = 2.0 * (which == 0 ? (double)(3 * d + F) * d : (double)N * K);
      printf("few rows %-9s M=%d K=%d split %d, %s A: cold %.1f us (%.2f TB/s of weights)\n",
             which == 0 ? "qkv+fc1" : (which == 1 ? "out+fc2" : "lm_head"), M, K, ks, packed ? "packed" : "row-major", ms * 1e3,
             wb / ms / 1e9);
      fflush(stdout);
    }
  CK(hipFree(dA)); CK(hipFree(dF));
  return bad;
}

int main(int argc, char** argv) {
  const int M = argc > 1 ? atoi(argv[1]) : 256;
  const int d = argc > 2 ? atoi(argv[2]) : 2560, F = 4 * d, V = 50304;
  const int reps = argc > 3 ? atoi(argv[3]) : 96;
  const int max_split = argc > 4 ? atoi(argv[4]) : 0;
  const int timed_phase = argc > 5 ? atoi(argv[5]) : 0;
  const int pad_a = argc > 6 ? atoi(argv[6]) : 0, pad_w = argc > 7 ? atoi(argv[7]) : 0;
  if (M <= 0 || M > 512 || d % 64 != 0) { printf("M must be 1..512 and d_model a multiple of 64\n"); return 1; }
  struct Shape { const char* name; int N, K, epi; } shapes[] = {
      {"qkv", 3 * d, d, EPI_BIAS}, {"out", d, d, EPI_BIAS_RESADD}, {"fc1", F, d, EPI_BIAS_GELU}, {"fc2", d, F, EPI_BIAS_RESADD},
      {"lm_head", V, d, EPI_F32}};
  const size_t wmax = (size_t)std::max(F, V) * (d + pad_w) + (size_t)d * (F + pad_w);  // elements of the largest matrix, padded
  const int R = (int)(((size_t)1200 << 20) / (wmax * 2)) + 1;  // copies: more than 1.2 GB in all
  std::vector<uint16_t> hA((size_t)M * (F + pad_a)), hW(wmax), hb(std::max(F, V));
  srand(1);
  for (auto& x : hA) x = f2h((rand() % 2001 - 1000) / 1000.0f);
  for (auto& x : hW) x = f2h((rand() % 2001 - 1000) / 25000.0f);
  for (auto& x : hb) x = f2bf((rand() % 2001 - 1000) / 5000.0f);
  uint16_t *dA, *dW, *db; void *dO, *dsk;
  const size_t skb = (size_t)16 * 512 * F * 4;
  CK(hipMalloc(&dA, hA.size() * 2)); CK(hipMalloc(&dW, wmax * 2 * R)); CK(hipMalloc(&db, hb.size() * 2));
  CK(hipMalloc(&dO, (size_t)M * std::max(std::max(F, V), 8 * d) * 4)); CK(hipMalloc(&dsk, skb));
  CK(hipMemcpy(dA, hA.data(), hA.size() * 2, hipMemcpyHostToDevice));
  for (int r = 0; r < R; ++r) CK(hipMemcpy(dW + (size_t)r * wmax, hW.data(), wmax * 2, hipMemcpyHostToDevice));
  CK(hipMemcpy(db, hb.data(), hb.size() * 2, hipMemcpyHostToDevice));
  hipEvent_t e0, e1; CK(hipEventCreate(&e0)); CK(hipEventCreate(&e1));
  int bad = 0;
  for (auto& s : shapes) {
    GemmArgs g;
    g.A = dA; g.W = dW; g.bias = s.epi == EPI_F32 ? nullptr : db; g.out = dO;
    g.M_max = M; g.M_dev = nullptr; g.N = s.N; g.K = s.K; g.ldo = s.N; g.epilogue = s.epi;
    g.splitk_ws = dsk; g.splitk_ws_bytes = skb; g.max_split = max_split;
    g.lda = s.K + pad_a; g.ldw = s.K + pad_w;
    const int ks = gemm_splitk_factor(1, g);
    const bool f32out = s.epi == EPI_BIAS_RESADD || s.epi == EPI_F32;
    // the residual epilogue adds into the output: start from a known value
    std::vector<float> init((size_t)M * s.N, 0.25f);
    if (f32out) CK(hipMemcpy(dO, init.data(), init.size() * 4, hipMemcpyHostToDevice));
    CK(launch_gemm(1, g, 0)); CK(hipDeviceSynchronize());
    std::vector<uint16_t> ho16; std::vector<float> ho32;
    if (f32out) { ho32.resize((size_t)M * s.N); CK(hipMemcpy(ho32.data(), dO, ho32.size() * 4, hipMemcpyDeviceToHost)); }
    else { ho16.resize((size_t)M * s.N); CK(hipMemcpy(ho16.data(), dO, ho16.size() * 2, hipMemcpyDeviceToHost)); }
    double maxerr = 0;
    for (int t = 0; t < 600; ++t) {
      const int r = t < 8 ? (t % 2 ? M - 1 : 0) : rand() % M, c = t < 8 ? (t % 4 < 2 ? 0 : s.N - 1) : rand() % s.N;
      double acc = 0;
      for (int k = 0; k < s.K; ++k) acc += (double)h2f(hA[(size_t)r * g.lda + k]) * h2f(hW[(size_t)c * g.ldw + k]);
      if (s.epi != EPI_F32) acc += bf2f(hb[c]);
      if (s.epi == EPI_BIAS_GELU) acc = 0.5 * acc * (1 + erf(acc / sqrt(2.0)));
      if (s.epi == EPI_BIAS_RESADD) acc += 0.25;
      const double got = f32out ? ho32[(size_t)r * s.N + c] : h2f(ho16[(size_t)r * s.N + c]);
      const double tol = f32out ? 4e-3 : 8e-3 * fmax(1.0, fabs(acc));
      const double err = fabs(got - acc);
      if (err > maxerr) maxerr = err;
      if (err > tol) { printf("MISMATCH %s r=%d c=%d got %f want %f\n", s.name, r, c, got, acc); ++bad; break; }
    }
    float ms_w = 0, ms_c = 0;
    if (ks > 1) g.phase = timed_phase;
    for (int mode = 0; mode < 2; ++mode) {
      for (int i = 0; i < 8; ++i) { g.W = dW + (mode ? (size_t)(i % R) * wmax : 0); CK(launch_gemm(1, g, 0)); }
      CK(hipEventRecord(e0, 0));
      for (int i = 0; i < reps; ++i) { g.W = dW + (mode ? (size_t)(i % R) * wmax : 0); CK(launch_gemm(1, g, 0)); }
      CK(hipEventRecord(e1, 0)); CK(hipEventSynchronize(e1));
      float ms; CK(hipEventElapsedTime(&ms, e0, e1)); (mode ? ms_c : ms_w) = ms / reps;
    }
    const double wb = 2.0 * s.N * s.K, fl = 2.0 * M * s.N * s.K;
    printf("%-7s M=%d N=%d K=%d split %d: warm %.1f us  cold %.1f us (%.2f TB/s of weights, %.0f TFLOP/s)  max |err| %.2e\n",
           s.name, M, s.N, s.K, ks, ms_w * 1e3, ms_c * 1e3, wb / ms_c / 1e9, fl / ms_c / 1e9, maxerr);
    fflush(stdout);
  }
  if (M <= 256 && (size_t)4 * d * d + (size_t)2 * d * F <= wmax)
    bad += few_rows_part(M, d, F, V, reps, R, wmax, hW, dW, hb, db, (float*)dO, e0, e1);
  return bad ? 2 : 0;
}
