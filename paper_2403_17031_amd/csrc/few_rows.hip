// Products of few rows, C[M,N] = A[M,K] * W[N,K]^T: the decode passes of run_decode_few (up to 64 sequences; up to 256
// where the model is narrow, in tiles of 64 rows), other products of up to 64 rows that come without split-K scratch, and
// products of any number of rows in the fp32 check mode (K a multiple of 32, aligned operands).
//
// Such a product is its weights' bytes and nothing else: at M = 64 the matrix cores need a tenth of the time the
// weights take to arrive.  What the kernel is built around is bytes in flight and few launches:
//   * A block of four waves (eight in one form) owns 32 to 128 output columns for all K of its split; the waves divide K, each holding the
//     weights of its next PF steps (128 bytes of every weight row per step; PF is two to four) in registers.  At K = 2560
//     a wave has ten steps.
//   * Both operands go global -> registers: 16 weight rows x 128 bytes per step, lane (l16, q) taking the 32 bytes at
//     32q of row l16.  No LDS and no barrier until the waves' partial tiles are added at the end.  Such a load touches
//     sixteen rows.  The weights, which HBM delivers, can afford that; A, read from L2 once per column block, cannot: its
//     producers in a decode pass write it packed (packed_index), and a wave's load is contiguous.  QKV + FC1 at width
//     2560 with packed / row-major A, in the forms of two column tiles: 8 rows 24 / 26 us, 30 rows 30 / 39, 64 rows 40 / 57.
//   * The sum over K stays in the block (bias, GELU and the fp16 rounding are its epilogue) unless a product has too
//     few column tiles to cover the chip: then K is cut over blocks into fp32 slabs that the consumer adds in order.
//   * Two products that are ready together (QKV and FC1 of a parallel-residual layer) share one launch.
// Width 2560, cold weights (dec_driver): QKV + FC1 21 us for one row (4.4 TB/s), 21 for 16, 24 for 30, 29 for 64;
// out-projection + FC2 13 to 18; LM head 49 us for one row (5.3 TB/s), 73 for 64.  The weight-streaming kernel of
// gemm_skinny.hip took 17.6 us for a QKV product alone and left slabs to add; the plain fp32 tile kernel 50 us for each
// product of the 70M shape at two rows (now 4 to 9).
#include <algorithm>

#include "common.h"

namespace rlhf {

typedef __attribute__((ext_vector_type(8))) _Float16 fr_f16x8_t;
typedef __attribute__((ext_vector_type(4))) float fr_f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t fr_u32x4_t;

#define FR_GLOBAL __attribute__((address_space(1)))  // (pointers that come as plain words would be generic ones)
typedef const FR_GLOBAL char* fr_in_t;

template <typename T>
struct FrTypes;
template <>
struct FrTypes<half_t> {
  typedef bf16_t P;
  typedef uint64_t B;  // four columns' bias as stored
};
template <>
struct FrTypes<float> {
  typedef float P;
  typedef fr_f32x4_t B;
};

// Bias of columns n .. n + 3 (0 past N), kept as stored until it is used; vec: the array is aligned for one load and N a
// multiple of 4.
__device__ __forceinline__ uint64_t load_bias(const FR_GLOBAL bf16_t* b, int n, int N, bool vec) {
  if (vec) return n < N ? *(const FR_GLOBAL uint64_t*)(b + n) : 0;
  uint64_t v = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (n + u < N) v |= (uint64_t)b[n + u].bits << (16 * u);
  return v;
}
__device__ __forceinline__ fr_f32x4_t load_bias(const FR_GLOBAL float* b, int n, int N, bool vec) {
  fr_f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (vec) {
    if (n < N) v = *(const FR_GLOBAL fr_f32x4_t*)(b + n);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (n + u < N) v[u] = b[n + u];
  }
  return v;
}
__device__ __forceinline__ fr_f32x4_t bias_f32(uint64_t r) {
  const uint32_t lo = (uint32_t)r, hi = (uint32_t)(r >> 32);
  return (fr_f32x4_t){__uint_as_float(lo << 16), __uint_as_float(lo & 0xFFFF0000u), __uint_as_float(hi << 16),
                      __uint_as_float(hi & 0xFFFF0000u)};
}
__device__ __forceinline__ fr_f32x4_t bias_f32(fr_f32x4_t v) { return v; }

// 16 bytes of 16 weight rows (first operand) and of 16 rows of A: accumulator element e of lane (l16, q) is
// (n = 4q + e, m = l16).
__device__ __forceinline__ fr_f32x4_t fr_mfma(half_t, fr_u32x4_t w, fr_u32x4_t a, fr_f32x4_t acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(fr_f16x8_t, w), __builtin_bit_cast(fr_f16x8_t, a), acc,
                                                0, 0, 0);
}
__device__ __forceinline__ fr_f32x4_t fr_mfma(float, fr_u32x4_t w, fr_u32x4_t a, fr_f32x4_t acc) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[j]), __uint_as_float(a[j]), acc, 0, 0, 0);
  return acc;
}

// A product as the kernel reads it: 128 bytes, fetched by two scalar loads, with every division done by the host.  Coming
// field by field, each group's address waiting for the one before, the arguments kept a block 1.5 to 2.7 us from its first
// weight load, and a bias read after the sum kept it another 1 to 2 us from its end (clock readings inside the kernels of a
// decode pass).  With both moved: 64 rows of width 768 QKV + FC1 7.1 -> 6.1 us, out-projection + FC2 5.8 -> 5.3; 37 of
// 2048 18.2 -> 17.4, 11.6 -> 11.0; one of 2560 23.9 -> 22.5, 15.2 -> 14.9 (dec_driver, cold).
struct __attribute__((aligned(64))) FrProd {
  fr_in_t W, A, W1, A1;  // segment 0, segment 1
  fr_in_t bias;
  FR_GLOBAL char* out;
  uint32_t ldw, ldw1;           // row strides of W, bytes
  int steps0, steps, per_block, ks_shift;  // steps of segment 0, of both, of a block; log2 of the K split
  uint32_t a_tile, a_row, a_half, a_q, a_step;
  int N, ldo, epilogue, packed_K, packed_k0, bias_vec;  // bias_vec: four columns' bias with one load
  uint32_t slab;
};
struct FrArgs {
  FrProd p[2];
  int blocks0, M_max, M_sub, pad;
  const int* M_dev;
};
static_assert(sizeof(FrProd) == 128, "two loads of 16 dwords");

// WV: waves per block (they divide K); MT x CT: 16x16 accumulator tiles along M and N per block; PF: steps held in
// registers; OCC: waves per SIMD the registers are sized for; TWO: K runs over a second pair of operands after the
// first.
template <typename T, int WV, int MT, int CT, int PF, int OCC, bool TWO>
__global__ void __launch_bounds__(64 * WV, OCC) few_rows_kernel(FrArgs args) {
  typedef typename FrTypes<T>::P P;
  typedef __attribute__((ext_vector_type(16))) uint32_t u16x_t;
  __shared__ fr_f32x4_t red[WV * MT * CT * 64];
  const int M = args.M_dev ? min(args.M_max, *args.M_dev - args.M_sub) : args.M_max;
  const int m0 = blockIdx.y * (16 * MT);
  if (m0 >= M) return;
  const bool second = (int)blockIdx.x >= args.blocks0;
  FrProd p;
  {
    const u16x_t* src = (const u16x_t*)&args.p[second ? 1 : 0];
    u16x_t both[2] = {src[0], src[1]};
    __builtin_memcpy(&p, both, sizeof(p));
  }
  const int bid = blockIdx.x - (second ? args.blocks0 : 0);
  const int tile = bid >> p.ks_shift, z = bid - (tile << p.ks_shift);
  const int n0 = tile * (16 * CT);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4;

  const int steps0 = p.steps0, steps = p.steps;
  const int b0 = z * p.per_block, b1 = min(steps, b0 + p.per_block);
  const int per_wave = (b1 - b0 + WV - 1) / WV;
  const int s0 = b0 + wave * per_wave, s1 = min(b1, s0 + per_wave);

  // The outputs of this thread: result tile ti = wave + it * WV of the block's CT x MT, its lane's four columns of one row.
  // Their bias is requested ahead of everything else (TWO: products without one): after the sum it would be a cold load
  // with nothing to hide it.
  constexpr int IT = (CT * MT + WV - 1) / WV;
  typename FrTypes<T>::B bias[IT] = {};
#pragma unroll
  for (int it = 0; it < IT && !TWO; ++it)
    if (p.bias) bias[it] = load_bias((const FR_GLOBAL P*)p.bias, n0 + 16 * ((wave + it * WV) / MT) + 4 * q, p.N, p.bias_vec != 0);

  // Weight rows: the block's first one as a 64-bit address, a lane's own as a 32-bit offset from it (an output embedding
  // may be larger than 4 GiB, a block's rows are not: few_rows_takes for 64, fr_form for more).
  uint32_t woff[TWO ? 2 : 1][CT], aoff[TWO ? 2 : 1][MT];
#pragma unroll
  for (int g = 0; g < (TWO ? 2 : 1); ++g) {
    const uint32_t row = g ? p.ldw1 : p.ldw;
#pragma unroll
    for (int c = 0; c < CT; ++c) woff[g][c] = (uint32_t)min(16 * c + l16, p.N - 1 - n0) * row + 32 * q;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = min(m0 + 16 * i + l16, M - 1);
      aoff[g][i] = (uint32_t)(m >> 4) * p.a_tile + (m & 15) * p.a_row + q * p.a_q;
    }
  }
  const fr_in_t wbase[2] = {p.W + (size_t)n0 * p.ldw, TWO ? p.W1 + (size_t)n0 * p.ldw1 : p.W};
  fr_u32x4_t w[PF][CT][2], a[PF][MT][2];
  auto load = [&](int buf, int s) {
    const bool g = TWO && s >= steps0;
    const size_t k = (size_t)(s - (g ? steps0 : 0));
    const fr_in_t wb = wbase[TWO && g ? 1 : 0] + k * 128, ab = (TWO && g ? p.A1 : p.A) + k * p.a_step, ab2 = ab + p.a_half;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const fr_in_t r = wb + (TWO && g ? woff[TWO ? 1 : 0][c] : woff[0][c]);
      w[buf][c][0] = *(const FR_GLOBAL fr_u32x4_t*)r;
      w[buf][c][1] = *(const FR_GLOBAL fr_u32x4_t*)(r + 16);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const uint32_t o = TWO && g ? aoff[TWO ? 1 : 0][i] : aoff[0][i];
      a[buf][i][0] = *(const FR_GLOBAL fr_u32x4_t*)(ab + o);
      a[buf][i][1] = *(const FR_GLOBAL fr_u32x4_t*)(ab2 + o);
    }
  };
  fr_f32x4_t acc[CT][MT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[c][i] = (fr_f32x4_t){0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[c][i] = fr_mfma(T(), w[buf][c][hh], a[buf][i][hh], acc[c][i]);
  };
  if (s0 < s1) {
#pragma unroll
    for (int b = 0; b < PF; ++b) load(b, min(s0 + b, s1 - 1));
    int s = s0;
    for (; s + 2 * PF <= s1; s += PF) {
#pragma unroll
      for (int b = 0; b < PF; ++b) {
        compute(b);
        load(b, s + PF + b);
      }
    }
    // fewer than 2 * PF steps are left, the first PF of them already requested
#pragma unroll
    for (int b = 0; b < PF; ++b) {
      if (s + b < s1) compute(b);
      if (s + PF + b < s1) load(b, s + PF + b);
    }
#pragma unroll
    for (int b = 0; b < PF; ++b)
      if (s + PF + b < s1) compute(b);
  }
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int i = 0; i < MT; ++i) red[((wave * CT + c) * MT + i) * 64 + lane] = acc[c][i];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int ti = wave + it * WV;
    if (ti >= CT * MT) break;
    const int item = ti * 64 + lane;
    fr_f32x4_t v = red[item];
#pragma unroll
    for (int k = 1; k < WV; ++k) v += red[k * CT * MT * 64 + item];
    const int c = ti / MT, i = ti - c * MT;
    const int m = m0 + 16 * i + l16, n = n0 + 16 * c + 4 * q;
    if (m >= M || n >= p.N) continue;
    const size_t o = (size_t)m * p.ldo + n;
    const bool vec = n + 4 <= p.N && (p.packed_K || (p.ldo & 3) == 0);
    if (p.epilogue == EPI_F32) {
      FR_GLOBAL float* out = (FR_GLOBAL float*)p.out + (size_t)z * p.slab + o;
      if (vec) *(FR_GLOBAL fr_f32x4_t*)out = v;
      else
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (n + u < p.N) out[u] = v[u];
      continue;
    }
    if (p.bias) v += bias_f32(TWO ? load_bias((const FR_GLOBAL P*)p.bias, n, p.N, p.bias_vec != 0) : bias[it]);
    if (p.epilogue == EPI_BIAS_RESADD) {
      FR_GLOBAL float* out = (FR_GLOBAL float*)p.out + o;
      if (vec) *(FR_GLOBAL fr_f32x4_t*)out += v;
      else
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (n + u < p.N) out[u] += v[u];
      continue;
    }
    if (p.epilogue == EPI_BIAS_GELU) {  // the erf form for fp16 too: gelu_f16out is many fp16 steps off below -2
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = gelu_erf(v[u]);
    }
    FR_GLOBAL T* out = (FR_GLOBAL T*)p.out + (p.packed_K ? packed_index<T>(m, p.packed_k0 + n, p.packed_K) : o);
    typedef __attribute__((ext_vector_type(4))) T t4_t;
    const t4_t t = {from_f32<T>(v[0]), from_f32<T>(v[1]), from_f32<T>(v[2]), from_f32<T>(v[3])};
    if (vec) *(FR_GLOBAL t4_t*)out = t;
    else
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (n + u < p.N) out[u] = t[u];
  }
}

static int fr_step(int dtype) { return dtype == 0 ? 32 : 64; }  // K elements per step (128 bytes)

// Both operands are read, and four columns of a row written, with one instruction: addresses that are no multiple of its
// size (an fp32 caller's own arrays may have any) stay with the other kernels, which move single floats.
// (A bf16 product that comes with split-K scratch is not taken: see few_rows_layer in api.hip.)
bool few_rows_takes(int dtype, const GemmArgs& a) {
  const size_t esz = dtype == 0 ? 4 : 2, lda = a.lda ? a.lda : a.K, ldw = a.ldw ? a.ldw : a.K;
  const uintptr_t out_mask = dtype == 1 && (a.epilogue == EPI_BIAS || a.epilogue == EPI_BIAS_GELU) ? 7 : 15;
  if ((((uintptr_t)a.A | (uintptr_t)a.W) & 15) != 0 || ((uintptr_t)a.out & out_mask) != 0) return false;
  return (dtype == 0 || !a.splitk_ws) && a.M_max > 0 && a.M_max <= (dtype == 0 ? 1 << 20 : kFewRows) && a.K > 0 && a.K % fr_step(dtype) == 0 && !a.bias2 &&
         !a.k_major && a.epilogue >= EPI_BIAS && a.epilogue <= EPI_F32 && (lda * esz) % 16 == 0 && (ldw * esz) % 16 == 0 &&
         (size_t)a.M_max * lda * esz < (1ull << 32) && (size_t)std::min(a.N, 64) * ldw * esz < (1ull << 32) &&
         lda * esz < (1ull << 31) && ldw * esz < (1ull << 31);
}

// Forms of the kernel: waves, row tiles, column tiles, steps held, waves per SIMD.  An idle row tile costs the bf16 mode 2-4 %
// where it is one of three (its lanes all ask for row M - 1) and 5-18 % where it is one or two of four (registers, waves in
// flight): 24 rows in forms of 2 / 4 row tiles, four column tiles each, width 2048 QKV + FC1 14.8 / 17.7 us, 4096 48.8 / 53.5.
// The last form divides K over eight waves (fr_form).
#define RLHF_FR_FORMS(X)                                                                                          \
  X(0, 4, 1, 2, 4, 4) X(1, 4, 1, 4, 3, 3) X(2, 4, 1, 5, 4, 2) X(3, 4, 2, 2, 3, 3) X(4, 4, 2, 4, 2, 3)            \
  X(5, 4, 3, 2, 3, 2) X(6, 4, 3, 4, 2, 2) X(7, 4, 3, 5, 2, 2) X(8, 4, 4, 2, 3, 2) X(9, 4, 4, 4, 2, 2)            \
  X(10, 4, 4, 5, 2, 1) X(11, 4, 4, 8, 2, 1) X(12, 8, 1, 2, 4, 4)
#define RLHF_FR_ENTRY(ID, WV, MT, CT, PF, OCC) {MT, CT, OCC},
struct FrForm {
  int mt, ct, occ;
};
static const FrForm kForms[] = {RLHF_FR_FORMS(RLHF_FR_ENTRY)};
#undef RLHF_FR_ENTRY
constexpr int kEightWaves = 12;

// How a product is cut: 16 * ct columns per block, and K over ks blocks.  A CU can have about 32 KB of loads in flight (its
// L1), for which a block's weights, ct column tiles wide, compete with its rows of A, mt tiles; and the launch lasts as
// long as the CU with the most blocks.  So what counts is a block's steps times tiles, plus its sum over the waves
// (ct * mt), times the rounds of 256 blocks; the blocks of a further round share the CU with the first's, the more so the
// fewer steps they have.  Five column tiles for the 1120 of QKV + FC1 at width 2560 are 224 blocks, one round, where two
// are 560.  Fitted to a sweep of widths 512-4096 and 1-256 rows (dec_driver, cold).  us by column tiles (* the one taken):
//   QKV + FC1       width  768:  1 row   5.1*/ 6.2 /  8.4        32 rows  4.9*/  7.0 /  9.5    64 rows  6.2*/  9.2 / 10.7 / 15.4    (2 / 4 / 5 / 8)
//                         1536:  1 row  10.0 / 9.5*/ 11.6        32 rows 12.0 / 11.4*/ 13.7    64 rows 15.1*/ 15.3 / 17.1 / 24.7
//                         2048:  1 row  13.4 / 13.4*/ 14.9       32 rows 16.7 / 15.4*/ 18.0    64 rows 21.8 / 20.1*/ 22.1 / 30.4
//                         2560:  1 row  24.2 / 27.4 / 20.5*      32 rows 29.4 / 33.0 / 24.4*   64 rows 37.3 / 40.1 / 28.4*/ 38.6
//                         4096:  1 row  45.6 / 45.7*/ 51.9       32 rows 56.7 / 51.4*/ 58.2    64 rows 72.4 / 60.6 / 68.2 / 55.5*
//   out-proj + FC2        1152:  1 row   6.5 /  5.4*/  7.3                                                                     (K in 8)
//                         2048:  1 row   8.3*/  9.3 /  9.1       32 rows  9.5*/  9.9 / 11.3    64 rows 12.5 / 12.5*/ 13.7 / 18.7
//                         2560:  1 row  14.6 / 16.8 / 13.3*      32 rows 17.9 / 19.5 / 15.5*   64 rows 23.0 / 24.6 / 17.7*/ 23.2
//                         4096:  1 row  31.5 / 30.0*/ 34.0       32 rows 39.1 / 34.4*/ 39.5    64 rows 50.5 / 41.4 / 47.2 / 38.2*
//   LM head                768:  1 row  17.8*/ 17.3 / 19.1       32 rows 20.6 / 21.5 / 20.8*   64 rows 26.8 / 26.3*/ 30.7 / 29.6
//                         2560:  1 row  53.2 / 53.4 / 51.5 (eight waves 48.5*)                 64 rows 83.9 / 76.9 / 73.3 / 71.2*
static double fr_cost(const FrForm& f, int rows, int blocks, double steps) {
  const int row_tiles = std::min((rows + 15) / 16, 4);
  const double further = f.occ > 1 ? 0.74 * steps / (steps + 6) : 0.8;
  return (1 + further * ((blocks + 255) / 256 - 1)) * (steps * (f.ct + 0.7 * row_tiles) + 1.5 * f.ct * row_tiles);
}
// The form for products of n_a and n_b (0: none) columns and `steps` steps over `rows` rows, K cut ks ways; the least cost
// in *cost.
static int fr_form(int dtype, int n_a, int n_b, int rows, int steps, int ks, size_t ldw_bytes, double* cost) {
  const int tiles = std::min((rows + 15) / 16, 4);
  auto blocks = [&](const FrForm& f) {
    const int c = 16 * f.ct;
    return ((n_a + c - 1) / c + (n_b + c - 1) / c) * ks * ((rows + 16 * f.mt - 1) / (16 * f.mt));
  };
  auto takes = [&](const FrForm& f) {
    if (f.mt < tiles) return false;
    if (f.ct > 2 && 16 * (size_t)f.ct * ldw_bytes >= ((size_t)1 << 32)) return false;  // a lane's offset within the block's rows
    // fp32: the matrix instructions of an idle row tile take as long as any other's, eight times as many as in bf16 (an LM head
    // of 24 rows in forms of 2 x 2 / 3 x 5 tiles: width 512 30 / 45 us, 768 46 / 62); and 3 x 5 loses to 3 x 2 and 3 x 4 at all
    // four widths measured (40 rows, 512: 45.9 / 41.0).
    return dtype != 0 || (f.mt == tiles && !(f.mt == 3 && f.ct == 5));
  };
  int best = -1, done = 0;  // done: column tiles with a form already (the first that holds the rows has the fewest row tiles)
  for (int i = 0; i < kEightWaves; ++i) {
    const FrForm& f = kForms[i];
    if (!takes(f) || (done >> f.ct & 1)) continue;
    done |= 1 << f.ct;
    const double t = fr_cost(f, rows, blocks(f), (double)steps / ks);
    if (best < 0 || t < *cost) {
      best = i;
      *cost = t;
    }
  }
  // A second round that is not full costs more than the average of further ones: a wider form that does with one round, on
  // half of the CUs or more, is up to 20 % faster (1 to 16 rows, two / four column tiles, us: width 1152 out-projection + FC2
  // 6.5 / 5.4, 1536 6.9 / 6.3 and QKV + FC1 10.0 / 9.5, 2304 16.7 / 15.0; 1920 out-projection + FC2 7.8 / 7.9), but not
  // where two full rounds are against one full (2048 out-projection + FC2 8.3 / 9.3) or the rows are 49 and more.
  if (rows <= 48 && blocks(kForms[best]) > 256 && blocks(kForms[best]) < 512) {
    int one = -1;
    double one_t = 0;
    for (int i = 0; i < kEightWaves; ++i) {
      const FrForm& f = kForms[i];
      if (f.mt != tiles || f.ct <= kForms[best].ct || !takes(f) || blocks(f) > 256 || blocks(f) < 128) continue;
      const double t = fr_cost(f, rows, blocks(f), (double)steps / ks);
      if (one < 0 || t < one_t) one = i, one_t = t;
    }
    if (one >= 0) best = one;
  }
  // An LM head of few rows is weights alone, and eight waves keep more of them in flight where each has four to seven steps
  // and rows do not start at one multiple of 4 KB each, which all fall on the same memory channels.  One row, two or five
  // column tiles / eight waves, us: width 2176 41.7 / 39.8, 2560 51.5 / 48.5, 3072 62.6 / 56.2, 3584 67.9 / 64.8; but 1536
  // 29.5 / 32.2, 2048 37.7 / 40.3, 3840 73.0 / 74.7, 4096 75.0 / 96.4.  Sixteen rows: 5 column tiles win where the cost
  // takes them (2560 54.3 / 55.9), eight waves against two column tiles (2048 45.4 / 44.2, 2432 54.3 / 51.5).
  if (rows <= 16 && ks == 1 && blocks(kForms[kEightWaves]) > 1024 && steps >= 32 && steps < 58 &&
      (rows > 8 ? kForms[best].ct == 2 : ldw_bytes % 4096 != 0))
    best = kEightWaves;
  return best;
}
// The split of a product left as slabs: the same for any number of rows, its consumer adds that many.  At least seven
// steps of 128 bytes to a block; and no step from one round to a second that is not full: out-projection + FC2 of widths 3136 to
// 4032 with K in 4 / 8 (196 to 252 blocks / twice as many), us: 3328 1 row 21.1 / 22.1, 32 rows 24.6 / 26.1, 64 rows 30.5 / 32.1;
// 3840 27.2 / 27.2, 30.5 / 32.9, 37.1 / 36.5; where both are full (4096), 30.8 / 30.0, 33.4 / 34.4, 40.0 / 38.2.
int few_rows_splits(int N, int steps) {
  int best = 1, best_blocks = 0;
  double best_t = 0;
  for (int ks = 1; ks <= 8 && (ks == 1 || steps / ks >= 7); ks *= 2) {
    double t = 0;
    const int c = 16 * kForms[fr_form(1, N, 0, 32, steps, ks, 0, &t)].ct, blocks = (N + c - 1) / c * ks;
    const bool partial = best_blocks <= 256 && blocks > 256 && blocks < 512;
    if (ks == 1 || (t < best_t * 0.95 && !partial)) best = ks, best_t = t, best_blocks = blocks;
  }
  return best;
}

template <typename T, bool TWO>
static void fr_launch(const FrArgs& args, int form, int blocks, hipStream_t s) {
  const int M = args.M_max;
#define RLHF_FR(ID, WV, MT, CT, PF, OCC)                                                                        \
  case ID:                                                                                                      \
    hipLaunchKernelGGL((few_rows_kernel<T, WV, MT, CT, PF, OCC, TWO>),                                          \
                       dim3(blocks, (M + 16 * MT - 1) / (16 * MT)), dim3(64 * WV), 0, s, args);                 \
    break;
  switch (form) { RLHF_FR_FORMS(RLHF_FR) }
#undef RLHF_FR
}

hipError_t launch_few_rows(int dtype, FewRowsArgs& args, int n_prods, hipStream_t s) {
  int blocks = 0, steps = 0;
  bool two = false;
  const int ks = n_prods == 1 && args.p[0].epilogue == EPI_F32 ? args.p[0].ksplit : 1;
  size_t ldw_bytes = 0;
  for (int i = 0; i < n_prods; ++i) {
    steps = std::max(steps, args.p[i].seg[0].steps + args.p[i].seg[1].steps);
    for (const FewRowsSeg& g : args.p[i].seg) ldw_bytes = std::max(ldw_bytes, (size_t)g.ldw * (dtype == 0 ? 4 : 2));
  }
  double cost = 0;
  const int form = fr_form(dtype, args.p[0].N, n_prods > 1 ? args.p[1].N : 0, args.M_max, steps, ks, ldw_bytes, &cost);
  const int c = 16 * kForms[form].ct;
  const uint32_t esz = dtype == 0 ? 4 : 2;
  FrArgs f = {};
  for (int i = 0; i < n_prods; ++i) {
    FewRowsProd& p = args.p[i];
    if (p.epilogue != EPI_F32) p.ksplit = 1;
    blocks += ((p.N + c - 1) / c) * p.ksplit;
    two = two || p.seg[1].steps > 0;
    if (i == 0) f.blocks0 = blocks;
    FrProd& d = f.p[i];
    d.W = (fr_in_t)p.seg[0].W; d.A = (fr_in_t)p.seg[0].A;
    d.W1 = (fr_in_t)p.seg[1].W; d.A1 = (fr_in_t)p.seg[1].A;
    d.bias = (fr_in_t)(p.epilogue == EPI_F32 ? nullptr : p.bias);
    d.out = (FR_GLOBAL char*)p.out;
    d.ldw = (uint32_t)p.seg[0].ldw * esz; d.ldw1 = (uint32_t)p.seg[1].ldw * esz;
    d.steps0 = p.seg[0].steps;
    d.steps = p.seg[0].steps + p.seg[1].steps;
    d.per_block = (d.steps + p.ksplit - 1) / p.ksplit;
    while ((1 << d.ks_shift) < p.ksplit) ++d.ks_shift;  // (a power of two)
    d.a_tile = p.seg[0].a_tile; d.a_row = p.seg[0].a_row; d.a_half = p.seg[0].a_half; d.a_q = p.seg[0].a_q;
    d.a_step = p.seg[0].a_step;
    if (p.seg[1].steps > 0 && (p.seg[1].a_tile != d.a_tile || p.seg[1].a_row != d.a_row || p.seg[1].a_half != d.a_half ||
                               p.seg[1].a_q != d.a_q || p.seg[1].a_step != d.a_step))
      return hipErrorInvalidValue;  // both segments of A lie in one operand
    d.N = p.N; d.ldo = p.ldo; d.epilogue = p.epilogue; d.packed_K = p.packed_K; d.packed_k0 = p.packed_k0;
    d.bias_vec = (p.N & 3) == 0 && ((uintptr_t)p.bias & (4 * esz - 1)) == 0;
    if (p.slab >= ((size_t)1 << 32) || (1 << d.ks_shift) != p.ksplit) return hipErrorInvalidValue;
    d.slab = (uint32_t)p.slab;
  }
  f.M_max = args.M_max;
  f.M_sub = args.M_sub;
  f.M_dev = args.M_dev;
  if (dtype == 0) {
    if (two) fr_launch<float, true>(f, form, blocks, s);
    else fr_launch<float, false>(f, form, blocks, s);
  } else {
    if (two) return hipErrorInvalidValue;  // fp16 matrices that are added up lie side by side
    fr_launch<half_t, false>(f, form, blocks, s);
  }
  return hipGetLastError();
}

void fr_seg(int dtype, FewRowsSeg& g, const void* A, const void* W, int K, int lda, int ldw) {
  g.A = A;
  g.W = W;
  g.steps = K / fr_step(dtype);
  g.ldw = ldw ? ldw : K;
  const uint32_t esz = dtype == 0 ? 4 : 2;
  if (lda < 0) {
    g.a_tile = 16 * (uint32_t)-lda * esz; g.a_row = 16; g.a_half = 256; g.a_q = 512; g.a_step = 2048;
  } else {
    g.a_row = (uint32_t)(lda ? lda : K) * esz; g.a_tile = 16 * g.a_row; g.a_half = 16; g.a_q = 32; g.a_step = 128;
  }
}

hipError_t launch_few_rows_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  FewRowsArgs args;
  FewRowsProd& p = args.p[0];
  fr_seg(dtype, p.seg[0], a.A, a.W, a.K, a.lda, a.ldw);
  p.bias = a.bias;
  p.out = a.out;
  p.N = a.N;
  p.ldo = a.ldo;
  p.epilogue = a.epilogue;
  args.M_max = a.M_max;
  args.M_dev = a.M_dev;
  args.M_sub = a.M_sub;
  return launch_few_rows(dtype, args, 1, s);
}

}  // namespace rlhf
