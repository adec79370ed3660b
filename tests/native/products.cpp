// Host-side checks of the library's product launchers, built by the tests against the library itself.
//   products errors   the launch calls of the runtime are replaced by ones that always fail: every route through
//                     launch_gemm reports it
//   products aligned  the few-rows kernel, which moves 16 bytes at a time, is not given addresses that are no multiple
//   products forms dtype d F V rows   the kernels that the product launches of a decode pass take
//   products many d F V rows    the kernels that the products of a pass over many rows take in fp32 mode
//   products bias2    a second bias is taken by the one epilogue that reads it and refused elsewhere, never dropped
//   products split    a decode product of few rows that is given split-K scratch is cut over K until it covers the chip
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "common.h"

using namespace rlhf;

// The runtime's launch calls, for this program and the library in it: nothing is launched, every launch fails, and the
// error stays until hipGetLastError takes it, as the runtime's own does.
static hipError_t last_error = hipSuccess;
static int launches = 0;
static const void* last_kernel = nullptr;
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
extern "C" hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t, hipStream_t) {
  ++launches;
  last_kernel = kernel;
  return last_error = hipErrorLaunchFailure;
}
extern "C" hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}

static GemmArgs product(int M, int N, int K, int epilogue) {
  GemmArgs g;
  g.A = g.W = (const void*)4096;  // never dereferenced: nothing is launched
  g.bias = nullptr;
  g.out = (void*)4096;
  g.M_max = M; g.M_dev = nullptr; g.N = N; g.K = K; g.ldo = N; g.epilogue = epilogue;
  return g;
}

static int errors() {
  int bad = 0;
  const int epilogues[] = {EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESADD, EPI_F32};
  const int rows[] = {1, 64, 65, 600};
  for (int dtype = 0; dtype < 2; ++dtype)
    for (int epi : epilogues)
      for (int M : rows) {
        const hipError_t e = launch_gemm(dtype, product(M, 256, 256, epi), nullptr);
        printf("dtype %d epilogue %d rows %d: %d launches, status %d\n", dtype, epi, M, launches, (int)e);
        bad += e != hipErrorLaunchFailure || launches == 0;
        launches = 0;
      }
  return bad ? 1 : 0;
}

static int aligned() {
  int bad = 0;
  const int epilogues[] = {EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESADD, EPI_F32};
  for (int dtype = 0; dtype < 2; ++dtype)
    for (int epi : epilogues)
      for (int which = 0; which < 4; ++which)
        for (int off = dtype ? 2 : 4; off < 16; off *= 2) {
          GemmArgs g = product(8, 256, 256, epi);
          const void* moved = (const char*)4096 + off;
          if (which == 0) g.A = moved;
          if (which == 1) g.W = moved;
          if (which == 2) g.out = (void*)moved;
          if (which == 3) g.bias = moved;  // read by single values
          const bool half_out = dtype == 1 && (epi == EPI_BIAS || epi == EPI_BIAS_GELU);
          const bool want = which == 3 || (which == 2 && half_out && off == 8);
          if (few_rows_takes(dtype, g) != want) {
            printf("dtype %d epilogue %d operand %d offset %d\n", dtype, epi, which, off);
            ++bad;
          }
        }
  return bad ? 1 : 0;
}

static int kernel_of(hipError_t e, int split, int steps, int rows) {
  Dl_info info;
  if (e != hipErrorLaunchFailure || !dladdr(last_kernel, &info) || !info.dli_sname) return 1;
  printf("%s split %d steps %d rows %d\n", info.dli_sname, split, steps, rows);
  return 0;
}

static int forms(int dtype, int d, int F, int V, int rows) {
  const void* p = (const void*)4096;
  FewRowsArgs in, out, head;
  in.M_max = out.M_max = head.M_max = rows;
  fr_seg(dtype, in.p[0].seg[0], p, p, d, -d, 0);
  in.p[0].N = in.p[0].ldo = 3 * d; in.p[0].epilogue = EPI_BIAS;
  fr_seg(dtype, in.p[1].seg[0], p, p, d, -d, 0);
  in.p[1].N = F; in.p[1].epilogue = EPI_BIAS_GELU; in.p[1].packed_K = d + F; in.p[1].packed_k0 = d;
  if (dtype) {
    fr_seg(dtype, out.p[0].seg[0], p, p, d + F, -(d + F), 0);
  } else {  // the caller's two matrices
    fr_seg(dtype, out.p[0].seg[0], p, p, d, -(d + F), d);
    fr_seg(dtype, out.p[0].seg[1], p, p, F, -(d + F), F);
  }
  const int steps = out.p[0].seg[0].steps + out.p[0].seg[1].steps;
  out.p[0].N = out.p[0].ldo = d; out.p[0].epilogue = EPI_F32; out.p[0].slab = (size_t)rows * d;
  out.p[0].ksplit = few_rows_splits(d, steps);
  fr_seg(dtype, head.p[0].seg[0], p, p, d, -d, 0);
  head.p[0].N = head.p[0].ldo = V; head.p[0].epilogue = EPI_F32;
  for (FewRowsArgs* a : {&in, &out, &head}) {
    const hipError_t e = launch_few_rows(dtype, *a, a == &in ? 2 : 1, nullptr);
    if (kernel_of(e, a->p[0].ksplit, a == &out ? steps : a->p[0].seg[0].steps, rows)) return 1;
  }
  return 0;
}

static int many(int d, int F, int V, int rows) {
  const int shapes[][3] = {{3 * d, d, EPI_BIAS}, {d, d, EPI_BIAS_RESADD}, {F, d, EPI_BIAS_GELU}, {d, F, EPI_BIAS_RESADD}, {V, d, EPI_F32}};
  for (auto& q : shapes) {
    const GemmArgs g = product(rows, q[0], q[1], q[2]);
    if (few_rows_takes(0, g) && kernel_of(launch_gemm(0, g, nullptr), 1, q[1] / 32, rows)) return 1;
  }
  return 0;
}

static int split() {
  int bad = 0;
  const int shapes[][2] = {{3072, 3072}, {3072, 12288}, {2048, 8192}, {5120, 20480}};  // out-projection and FC2
  for (auto& nk : shapes)
    for (int M : {1, 16, 33, 64}) {
      GemmArgs g = product(M, nk[0], nk[1], EPI_BIAS_RESADD);
      g.splitk_ws = (void*)4096;
      g.splitk_ws_bytes = (size_t)16 * M * 3 * nk[1] * sizeof(float);
      const int ks = gemm_splitk_factor(1, g);
      g.splitk_ws = nullptr;
      printf("rows %d, %d x %d: split %d\n", M, nk[0], nk[1], ks);
      bad += ks < 2 || !few_rows_takes(1, g);
    }
  return bad ? 1 : 0;
}

static int bias2() {
  int bad = 0;
  const int epilogues[] = {EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESADD, EPI_F32, EPI_LSE, EPI_QKV};
  LseArgs lse = {};
  QkvArgs qkv = {};
  qkv.H = 4; qkv.hd = 64; qkv.r = 16;
  for (int epi : epilogues)
    for (int M : {64, 600})
      for (int sliced = 0; sliced < 2; ++sliced) {
        GemmArgs g = product(M, 768, 4096, epi);
        g.bias = sliced ? nullptr : (const void*)4096;
        g.bias2 = (const void*)8192;
        g.lse = &lse;
        g.qkv = &qkv;
        g.long_k = sliced != 0;
        g.splitk_ws = sliced ? (void*)4096 : nullptr;
        g.splitk_ws_bytes = (size_t)1 << 30;
        const bool takes = epi == EPI_BIAS_RESADD && M > 512;
        launches = 0;
        const hipError_t e = launch_gemm(1, g, nullptr);
        // (one launch: slices of K and their sum, which adds no bias, are two)
        if (e != (takes ? hipErrorLaunchFailure : hipErrorInvalidValue) || launches != (takes ? 1 : 0) ||
            gemm_takes_bias2(1, g) != takes) {
          printf("epilogue %d rows %d sliced %d: status %d, %d launches\n", epi, M, sliced, (int)e, launches);
          ++bad;
        }
      }
  return bad ? 1 : 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && !strcmp(argv[1], "errors")) return errors();
  if (argc > 1 && !strcmp(argv[1], "aligned")) return aligned();
  if (argc > 6 && !strcmp(argv[1], "forms"))
    return forms(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]));
  if (argc > 5 && !strcmp(argv[1], "many")) return many(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]));
  if (argc > 1 && !strcmp(argv[1], "split")) return split();
  if (argc > 1 && !strcmp(argv[1], "bias2")) return bias2();
  return 2;
}
