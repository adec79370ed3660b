// Shared device helpers and the launcher declarations of the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

namespace rlhf {

// ------------------------------------------------------------------------------------------------
// Element types.  bf16_t: the storage type of a bf16 model's weights (raw 16-bit patterns).
// half_t: the type of activations, K/V cache and matrix-core operands in bf16 mode.  Both matrix
// operand types run at the same MFMA rate and occupy the same bytes; fp16's 11-bit significand
// keeps the activation rounding error 8x below bf16's, which the parity bar of this library needs,
// and every bf16 weight converts to fp16 exactly inside fp16's normal range.  Accumulation, the
// residual stream, LayerNorm statistics, softmax and the sampler are always fp32.
// ------------------------------------------------------------------------------------------------
struct bf16_t {
  uint16_t bits;
};
typedef _Float16 half_t;

struct ModeF32 {  // fp32 check mode
  typedef float W;  // weights as stored by the caller
  typedef float A;  // activations and GEMM operands
};
struct ModeBF16 {  // bf16 weights, fp16 operands
  typedef bf16_t W;
  typedef half_t A;
};

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x.bits) << 16); }
__device__ __forceinline__ float to_f32(half_t x) { return (float)x; }

// round-to-nearest-even fp32 -> bf16 (inputs are finite in this library; NaN stays NaN-ish)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
template <typename T>
__device__ __forceinline__ T from_f32(float f);
template <>
__device__ __forceinline__ float from_f32<float>(float f) {
  return f;
}
template <>
__device__ __forceinline__ bf16_t from_f32<bf16_t>(float f) {
  bf16_t r;
  r.bits = f32_to_bf16_bits(f);
  return r;
}
template <>
__device__ __forceinline__ half_t from_f32<half_t>(float f) {  // round to nearest even, saturating
  return (half_t)fminf(fmaxf(f, -65504.0f), 65504.0f);
}

// Exchanges between the lanes of a wave as register moves (DPP within 16 lanes, permlane swaps between them; all lanes take
// part).  __shfl_xor goes through the LDS pipe, a hundred cycles of latency a step, which is what a LayerNorm row or a
// softmax waits for: a 64-lane sum of six of them is six dependent round trips.
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ int dpp_mov(int v, int old = 0) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xf, BANKS, false);
}
// lane i: the value of lane i ^ O
template <int O>
__device__ __forceinline__ int lane_xor(int v) {
  static_assert(O == 1 || O == 2 || O == 4 || O == 8 || O == 16 || O == 32, "one bit");
  if constexpr (O == 1) return dpp_mov<0xB1>(v);  // quad_perm 1,0,3,2
  if constexpr (O == 2) return dpp_mov<0x4E>(v);  // quad_perm 2,3,0,1
  if constexpr (O == 4) return dpp_mov<0x114, 0xA>(v, dpp_mov<0x104, 0x5>(v));  // shifts by 4 in a row of 16, per bank
  if constexpr (O == 8) return dpp_mov<0x128>(v);  // rotation of a row by 8
  const bool upper = (threadIdx.x & O) != 0;  // (blocks are whole waves)
  if constexpr (O == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return (int)(upper ? p[0] : p[1]);
  }
  const auto p = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return (int)(upper ? p[0] : p[1]);
}
template <int O>
__device__ __forceinline__ float lane_xor(float v) {
  return __int_as_float(lane_xor<O>(__float_as_int(v)));
}
// op over all lanes, in all lanes: the tree that exchanges with lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 in this order (op
// commutative).  The swaps leave both partners' values in either lane, and after the steps before it a value repeats
// every 8, 4 or 2 lanes, so that a rotation of a row is the same exchange.
template <typename OP>
__device__ __forceinline__ float wave_fold(float v, OP op) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(q[0]), __uint_as_float(q[1]));
  v = op(v, __int_as_float(dpp_mov<0x128>(__float_as_int(v))));
  v = op(v, __int_as_float(dpp_mov<0x124>(__float_as_int(v))));
  v = op(v, __int_as_float(dpp_mov<0x122>(__float_as_int(v))));
  return op(v, __int_as_float(dpp_mov<0x121>(__float_as_int(v))));
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_fold(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_fold(v, [](float a, float b) { return fmaxf(a, b); });
}
// op with lane ^ 32, in both lanes
template <typename OP>
__device__ __forceinline__ float half_fold(float v, OP op) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  return half_fold(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float half_max(float v) {
  return half_fold(v, [](float a, float b) { return fmaxf(a, b); });
}

// One tile load of a wave, global memory straight to LDS: lane i's 16 bytes at base + off go to the LDS address lds + 16 i
// (base and lds the same in all lanes).  Assembly without destination registers, for kernels that count their own waits: the
// compiler does not know that such a load is under way, so whoever reads what it brings waits for it (s_waitcnt vmcnt) first.
// The address travels in m0, which no clobber list may name (the register is reserved) and which the compiler sets for direct
// loads of its own, once for several where the address is the same: it is put back.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off, uint32_t lds) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
               : "=&s"(m0)
               : "s"(lds), "v"(off), "s"(base)
               : "memory");
}

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// 1 / (1 + 2^t), the division correctly rounded.  The compiler's division is eleven instructions, half of the GELU below,
// and in the FC1 product's epilogue nothing hides them; the hardware reciprocal (1 ulp) with one correction step by FMA is
// three, and gives the same bits (compared for every float from 1 to 2^126).  t is capped at 127.5, which keeps the step
// away from infinities; beyond 126 the reciprocal is a denormal number, which the instruction flushes, so that the result is
// the 0 that 1 / infinity is: with the smallest normal number instead, -3e38 (a bias, say) times it would be -3.5.
__device__ __forceinline__ float recip_rn_sigmoid(float t) {
  const float y = 1.0f + __builtin_amdgcn_exp2f(fminf(t, 127.5f));
  const float r = __builtin_amdgcn_rcpf(y);
  return fmaf(fmaf(-y, r, 1.0f), r, r);
}

// GELU for the fp16 outputs of products of many rows: x * Phi(x) with Phi(x) ~ 1 / (1 + exp(-x * (c1 + c3 x^2 + c5 x^4))), the
// coefficients fitted to the erf form over [-9, 9]: absolute error below 2.6e-5 everywhere (the
// fp16 result itself is rounded to 2^-11 relative), one exp and one reciprocal per element.  x^2 is
// capped at 64: beyond |x| = 8 the polynomial would bend back, and the sigmoid is saturated there.
// The constants carry the factor -log2(e) of the base-2 exponential.
__device__ __forceinline__ float gelu_f16out(float x) {
  const float s = fminf(x * x, 64.0f);
  float p = fmaf(1.01426504e-3f, s, -1.06775735e-1f);
  p = fmaf(p, s, -2.30112140f);
  return x * recip_rn_sigmoid(x * p);
}

// ------------------------------------------------------------------------------------------------
// Launchers (host).  dtype: 0 = ModeF32, 1 = ModeBF16.  All enqueue on `s` and return the
// launch status.  "n_rows_dev", where present, points to the device-resident row count; the grid
// is sized for the host-side upper bound and surplus blocks exit.
// ------------------------------------------------------------------------------------------------
enum Epilogue {
  EPI_BIAS = 0,         // out[T]   = acc + bias
  EPI_BIAS_GELU = 1,    // out[T]   = GELU(acc + bias): gelu_erf, in the fp16 products of many rows gelu_f16out
  EPI_BIAS_RESADD = 2,  // out[f32] += acc + bias      (residual stream update, in place)
  EPI_F32 = 3,          // out[f32] = acc              (logits)
  EPI_LSE = 4,          // nothing stored but per-row softmax statistics of acc/T (scoring LM head)
  EPI_QKV = 5,          // acc + bias with the rotary turn applied, q stored as rows, K and V into the cache
  EPI_BIAS_GELU_ERF = 6 // out[T]   = gelu_erf(acc + bias); large-M fp16 kernel only (decode)
};

// EPI_LSE: the product is a [rows, vocab] logits matrix that is never stored.  Each part p (the columns of
// one wave of a tile; gemm_lse_parts() of them per row)
// of packed row t leaves max_v z and sum_v exp(z - max) (z = logit / temperature) in pmax/psum
// [p * stride + t]; the part that holds the row's target token (the next token of the same
// sequence) also leaves its z in ztgt[t].  launch_lse_combine turns these into log-probabilities.
struct LseArgs {
  const int* tok;     // [rows] packed token ids
  const int* pos;     // [rows] packed positions (pos[t+1] == pos[t] + 1 <=> same sequence)
  const int* T_dev;   // number of packed rows
  float inv_temperature;
  float* pmax;
  float* psum;
  float* ztgt;
  int stride;         // rows_max
  int vocab;
  // Rows that are a selection of the packed rows (launch_select_rows): tgt[j] is row j's target token (-1: none)
  // and replaces the tok / pos test; dst[j] is the packed row it stands for.
  const int* tgt = nullptr;
  const int* dst = nullptr;
  const float* val_in = nullptr;  // with dst: per-row values to scatter, val_out[dst[j]] = val_in[j]
  float* val_out = nullptr;
};
// lp_packed[t + 1] = ztgt[t] - logsumexp over the nparts parts, for every t whose successor is in
// the same sequence (with a selection: lp_packed[dst[j] + 1] for every row j with a target).
hipError_t launch_lse_combine(const LseArgs& a, int rows_max, int nparts, float* lp_packed, hipStream_t s);
// The rows of a packed batch from padded column first_col - 1 on (what predicts the tokens at columns >=
// first_col): sel[j] = their packed row, sequence by sequence, j < *n_sel; tgt[j] = the token the row predicts
// (-1 for a sequence's last row).  Entries n_sel .. rows_max-1 are filled with row 0 / -1, so that a gather over
// rows_max entries stays in bounds.  off [B + 1] is scratch (the selection's offsets per sequence).  One block.
hipError_t launch_select_rows(int first_col, int B, const int* start, const int* len, const int* cu, const int* tok,
                              int rows_max, int* sel, int* tgt, int* n_sel, int* off, hipStream_t s);
// Per-row scalars of the selected rows: tgt_out[j] = tgt[sel[j]], a_out[j] = a[sel[j]], b_out[j] = b[sel[j]]
// for j < *n_sel; (-1, 0, 0) for the entries up to rows.  b / b_out may be null.
hipError_t launch_gather_row_scalars(const int* sel, const int* n_sel, int rows, const int* tgt, const float* a,
                                     const float* b, int* tgt_out, float* a_out, float* b_out, hipStream_t s);
// out row sel[j] = in row j for j < *n_sel (distinct rows of row_bytes, a multiple of 16).
hipError_t launch_scatter_rows(const void* in, const int* sel, const int* n_sel, int rows, size_t row_bytes, void* out,
                               hipStream_t s);
// out row r (out_stride bytes apart) = the first row_bytes of in row src[r] (in_stride bytes apart).
hipError_t launch_gather_rows_strided(const void* in, size_t in_stride, const int* src, int rows, size_t row_bytes,
                                      void* out, size_t out_stride, hipStream_t s);
// True when launch_gemm would take EPI_LSE for these arguments (large-M fp16 kernel only).
// EPI_QKV: the product is the [rows, 3*d] QKV matrix in sections q | k | v with the rotary pairs of a
// head in neighbouring columns.  The epilogue adds the bias, turns the pairs by the row's position,
// rounds to fp16 and stores q to q[row, d] and the K / V heads to the cache slot of (sequence, head,
// position): what the product followed by the stand-alone rotary kernel leaves, without the
// [rows, 3*d] intermediate.  Large-M fp16 kernel only.
// Cache slots of a packed row: head h's K (and V) row is slot x + h * y (slots of head_dim elements).
struct __align__(8) KvSlot {
  uint32_t x, y;
};
struct QkvArgs {
  const int* pos;      // [rows] position of a packed row (+ pos_add); rows are indexed from the start of the
                       // packed batch: a launch over a row chunk (GemmArgs::M_sub) adds its offset
  const KvSlot* slots; // [rows] where a packed row's K and V go (+ pos_add slots)
  const float* cos_t;  // [positions][r/2]
  const float* sin_t;
  void* q;             // [rows, d] fp16
  void* kc;            // K cache, V cache (fp16)
  void* vc;
  int pos_add, H, hd, r;
};
struct GemmArgs;
bool gemm_takes_qkv(int dtype, const GemmArgs& a, int H, int hd, int r);
bool gemm_takes_lse(int dtype, const GemmArgs& a);
bool gemm_takes_k_major(int dtype, const GemmArgs& a);
int gemm_lse_parts(int n_cols);

struct GemmArgs {
  const void* A;      // [M, K] activations, row-major, Mode::A
  const void* W;      // [N, K] weight, row-major, Mode::A (bf16 weights are converted at create)
  const void* bias;   // [N] Mode::W or nullptr
  void* out;          // [M, ldo] (Mode::A or float by epilogue)
  int M_max;          // host upper bound of M
  const int* M_dev;   // device row count or nullptr (then M = M_max)
  int M_sub = 0;      // with M_dev: M = min(M_max, *M_dev - M_sub)  (row chunk starting at M_sub)
  int N, K, ldo;
  int epilogue;
  void* splitk_ws = nullptr;   // fp32 scratch for split-K partial sums (decode-sized M), or null (fp16, up to 64 rows:
                               // with it the split-K kernels take the product, without it the few-rows kernel)
  size_t splitk_ws_bytes = 0;
  int phase = 0;               // split-K only: 0 = GEMM + reduce, 1 = partial sums only, 2 = reduce only
  const struct LseArgs* lse = nullptr;  // EPI_LSE only
  const struct QkvArgs* qkv = nullptr;  // EPI_QKV only
  int lda = 0, ldw = 0;        // row strides of A and W in elements (0: K); fp16 kernels and the few-rows kernel
  const void* bias2 = nullptr; // second bias added like the first; EPI_BIAS_RESADD of the large-M fp16 kernel only
  const float* res = nullptr;  // EPI_BIAS_RESADD of the large-M fp16 kernel (gemm_takes_bias2): what the product is added to,
                               // rows of ldo (null: out itself)
  int max_split = 0;           // few-rows kernel: cap on the K split (0: as many as cover the chip)
  bool k_major = false;        // operands given K-major: A is [K, M_max], W is [K, N], row-major, lda / ldw their row
                               // strides (0: M_max / N); out = A^T W, fp32 (EPI_F32), large-M fp16 kernel only: ask
                               // gemm_takes_k_major first
  bool long_k = false;         // large-M kernel, fp32 output, no bias: K may be cut into slices whose fp32 slabs (in
                               // splitk_ws) are then summed in slice order -- for products with few output tiles and
                               // a very long K (weight gradients)
  bool small_footprint = false;  // few rows: stay on the staged tile kernel (24 KB of LDS, 4 blocks per CU), whose
                                 // blocks fit next to another kernel's on a CU; the weight-streaming kernel takes a
                                 // whole CU per block
  bool large_tile = false;     // take the large-M kernel up to 512 rows too (its smaller tiles; the launch has the chip to
                               // itself).  With splitk_ws K is cut into gemm_large_slices(a) slices, whose fp32 slabs
                               // [M_max, N] stay there for the consumer to add (EPI_F32) or are added to out by a second
                               // launch (EPI_BIAS_RESADD)
};
int gemm_large_slices(const GemmArgs& a);
bool gemm_takes_large(int dtype, const GemmArgs& a);
// The few-rows (decode) kernel of gemm_skinny.hip: whether it takes these arguments, the K split it would use,
// and the launch itself (ks > 1: fp32 partial slabs into a.splitk_ws; ks == 1: epilogue in the kernel).
bool gemm_skinny_takes(int dtype, const GemmArgs& a);
int gemm_skinny_splitk(const GemmArgs& a);
void launch_gemm_skinny(const GemmArgs& a, int ks, hipStream_t s);
// Products of few rows (few_rows.hip): one launch runs one or two of them over the same M rows.
constexpr int kFewRows = 64;  // most rows of a product by itself in bf16 mode, and the rows of one tile
// Packed activations: what a lane of the matrix instruction reads (16 bytes of a row) next to what its neighbour reads:
// [rows / 16][K in 16-byte chunks][16 rows][16 bytes], so that a wave's load of 16 rows is contiguous.  Element index:
template <typename T>
__device__ __forceinline__ size_t packed_index(int m, int k, int K) {
  constexpr int E = 16 / (int)sizeof(T);
  return ((size_t)(m >> 4) * (K / E) + k / E) * (16 * E) + (m & 15) * E + k % E;
}
struct FewRowsSeg {           // K = steps * 128 bytes of every row of A and W
  const void* A = nullptr;
  const void* W = nullptr;
  int steps = 0, ldw = 0;
  // byte strides of A: between 16-row tiles and rows of a tile, between a lane group's two chunks of a step, between
  // lane groups, between steps
  uint32_t a_tile = 0, a_row = 0, a_half = 0, a_q = 0, a_step = 0;
};
struct FewRowsProd {
  FewRowsSeg seg[2];          // K runs over seg[0], then (fp32 mode) over seg[1]
  const void* bias = nullptr;
  void* out = nullptr;
  int N = 0, ldo = 0, epilogue = 0;
  int packed_K = 0, packed_k0 = 0;  // packed_K > 0 (EPI_BIAS, EPI_BIAS_GELU): out is a packed operand of packed_K
                                    // columns, this product its columns from packed_k0 on
  int ksplit = 1;             // EPI_F32: K cut over this many blocks, block z writing slab z (`slab` floats each)
  size_t slab = 0;
};
struct FewRowsArgs {
  FewRowsProd p[2];
  int M_max = 0, M_sub = 0;
  const int* M_dev = nullptr;
};
bool few_rows_takes(int dtype, const GemmArgs& a);
int few_rows_splits(int N, int steps);  // the ksplit of a product left as slabs (a power of two up to 8)
// lda 0: K; lda < 0: A is packed with -lda columns in all (A points at its first column of this segment).
void fr_seg(int dtype, FewRowsSeg& g, const void* A, const void* W, int K, int lda, int ldw);
hipError_t launch_few_rows(int dtype, FewRowsArgs& args, int n_prods, hipStream_t s);
hipError_t launch_few_rows_gemm(int dtype, const GemmArgs& a, hipStream_t s);
// True when launch_gemm would route these arguments to the kernel that honours bias2.
bool gemm_takes_bias2(int dtype, const GemmArgs& a);
// > 1 when launch_gemm would take the split-K path for these arguments.
int gemm_splitk_factor(int dtype, const GemmArgs& a);
hipError_t launch_gemm(int dtype, const GemmArgs& a, hipStream_t s);

// Row metadata of a packed batch -------------------------------------------------------------------
// mask [B, L] (1 = real) -> start[b], len[b]; then cu[b] = sum_{b'<b} len, kvoff[b] = sum_{b'<b}
// (len + kv_extra), total[0] = cu[B], total[1] = kvoff[B].  cap: the rows that the caller's buffers hold; tokens past it are
// left out as if the mask ended there.
hipError_t launch_row_spans(const uint8_t* mask, int B, int L, int kv_extra, int* start, int* len, int* cu,
                            int* kvoff, int* total, hipStream_t s, int cap = INT_MAX);
// Packed row t = cu[b] + i for i < len[b]: pos[t] = i, rowid[t] = b, tok[t] = tokens[b, start[b]+i],
// x[t, :] = embed[tok[t], :]; slots[t] = the row's place in a K/V cache whose sequence b starts at slot kvoff[b] * H and
// holds len[b] + kv_extra rows per head.
hipError_t launch_pack_embed(int dtype, const int32_t* tokens, int B, int L, const int* start, const int* len,
                             const int* cu, const void* embed, int d, int vocab, int* pos, int* rowid, int* tok,
                             float* x, const int* kvoff, int H, int kv_extra, KvSlot* slots, hipStream_t s);
// Cache slots of the first token after every sequence (decode pass t stores t slots further).
hipError_t launch_decode_slots(int B, const int* len, const int* kvoff, int H, int kv_extra, KvSlot* slots, hipStream_t s);
hipError_t launch_gather_rows(const void* in, const int* src, int src_add, int rows, size_t row_bytes, void* out,
                              hipStream_t s);

// LayerNorm of fp32 rows; two affine outputs from one set of statistics (g2 may be null -> one).
hipError_t launch_layernorm(int dtype, const float* x, int rows_max, const int* rows_dev, int d, float eps,
                            const void* g1, const void* b1, void* out1, const void* g2, const void* b2,
                            void* out2, hipStream_t s);
// Two split-K products (fp32 partial slabs of `slab` floats each, row-major [rows, d]) whose reduction
// into the residual stream is still pending: x <- (x + (sum_z A_z + bias_a)) + (sum_z B_z + bias_b).
// (ks_b == 0: one product, of both biases).
struct PendingResidual {
  const float* part_a = nullptr;
  const float* part_b = nullptr;
  const void* bias_a = nullptr;  // bf16 [d]
  const void* bias_b = nullptr;
  int ks_a = 0, ks_b = 0;
  size_t slab = 0;
};
bool layernorm_pending_supported(int dtype, int rows_max, int d);
// LayerNorm as above, after folding the pending products into x (written back in place).
hipError_t launch_layernorm_pending(float* x, int rows_max, const int* rows_dev, int d, float eps, const void* g1,
                                    const void* b1, void* out1, const void* g2, const void* b2, void* out2,
                                    const PendingResidual& pend, hipStream_t s);
// Final LayerNorm of selected rows: row r reads x[src[r]] (src may be null: identity), optionally
// also the value head val[r] = w_v . h + b_v.
hipError_t launch_final_ln(int dtype, const float* x, const int* src, int src_add, int rows_max,
                           const int* rows_dev, int d, float eps, const void* g, const void* b, void* out,
                           const void* value_w, float value_b, float* val, hipStream_t s);

// K/V layout: sequence b owns the slab of slots [kvoff[b]*H, kvoff[b+1]*H); inside it head h has
// len[b] + kv_extra consecutive rows of hd elements (kv_extra = room for generated tokens), so one
// (sequence, head) pair is one contiguous run and a sequence's heads are neighbours.
// Rotary on q,k (first r dims of each head) + K/V store.  qkv [rows, 3d] -> q [rows, d] and
// kc/vc at row pos[t] + pos_add of (sequence rowid[t], head h).  rowid may be null (row t is
// sequence t).  cos/sin tables are [max_pos][r/2].
hipError_t launch_rope_kv(int dtype, const void* qkv, int rows_max, const int* rows_dev, const int* pos,
                          int pos_add, const int* rowid, const int* kvoff, const int* len, int H, int hd, int r,
                          const float* cos_t, const float* sin_t, void* q, void* kc, void* vc,
                          long kv_extra, hipStream_t s);

// Same, one row per sequence, with the qkv row formed from the fp32 partial slabs of a split-K
// product (`slab` floats each, row-major [rows, 3*H*hd]) plus bias instead of being read.
bool rope_kv_splitk_supported(int dtype, int H, int hd, int r);
hipError_t launch_rope_kv_splitk(const float* part, int ksplit, size_t slab, const void* bias, int rows_max,
                                 const int* rows_dev, const int* pos, int pos_add, const int* rowid,
                                 const int* kvoff, const int* len, int H, int hd, int r, const float* cos_t,
                                 const float* sin_t, void* q, void* kc, void* vc, long kv_extra, hipStream_t s);

// Causal attention over packed sequences (prefill / scoring).  q [T, H*hd]; kc/vc [H][*][hd] with
// sequence b's keys at slots kvoff[b] .. kvoff[b]+len[b]; out [T, H*hd].
hipError_t launch_attn_prefill(int dtype, const void* q, const void* kc, const void* vc, long kv_extra,
                               int B, int Lmax, const int* len, const int* cu, const int* kvoff, int H, int hd,
                               void* out, int out_ld, hipStream_t s);
// Decode attention: one query row per sequence against ctx = len[b] + ctx_add cached keys.
hipError_t launch_attn_decode(int dtype, const void* q, const void* kc, const void* vc, long kv_extra,
                              int B, const int* len, int ctx_add, int ctx_max, const int* kvoff, int H, int hd,
                              void* out, hipStream_t s, int out_ld = 0);  // out_ld: row stride of out (0: H * hd)

// The decode pass of few sequences (decode.hip).
// x <- x + (sum of ks <= 8 slabs) + bias_a + bias_b (ks = 0: x as it is), then LayerNorm with one or two affine outputs
// (out2 null: one); x is written back if write_x.  d a multiple of 4 up to 4096, ks a power of two; the outputs are
// packed operands (packed_index).
bool ln_decode_supported(int d);
hipError_t launch_ln_decode(int dtype, float* x, int rows, int d, float eps, const void* g1, const void* b1, void* out1,
                            const void* g2, const void* b2, void* out2, const float* part, int ks, size_t slab,
                            const void* bias_a, const void* bias_b, bool write_x, hipStream_t s);
// Decode attention from the QKV product's rows [B, 3*H*hd]: rotary turn of q and k at position len[b] + step, K / V
// store at that row of the cache, attention over rows 0 .. len[b] + step into the first
// H*hd columns of the packed operand `out` of out_cols columns.
bool attn_decode_rope_supported(int hd, int r);
hipError_t launch_attn_decode_rope(int dtype, const void* qkv, void* kc, void* vc, long kv_extra, int B, const int* len,
                                   int step, int ctx_max, const int* kvoff, int H, int hd, int r, const float* cos_t,
                                   const float* sin_t, void* out, int out_cols, hipStream_t s);

// Sampler: one step for every row from fp32 logits [B, V].
struct SampleArgs {
  const float* logits;
  int B, V, Lq, N, step;
  uint64_t seed, seq_base;
  float temperature;
  int eos_id, pad_id;
  const int* len;       // true query lengths (0 = all-pad row)
  int* finished;        // [B] state, initialised at step 0
  int32_t* out_tokens;  // [B, Lq+N]
  float* out_logprobs;  // [B, N]
  int32_t* out_lengths; // [B]
  uint8_t* out_mask;    // [B, Lq+N] or null
  void* parts;          // scratch: sampler_scratch_bytes(B, V)
};
size_t sampler_scratch_bytes(int B, int V);
// x (null after the last step): row b receives the embedding of the token sampled for row b, the next pass's input.
hipError_t launch_sampler(const SampleArgs& a, int dtype, const void* embed, int d, float* x, hipStream_t s);
hipError_t launch_copy_queries(const int32_t* queries, const uint8_t* pad_mask, int B, int Lq, int N, int pad_id,
                               int32_t* out_tokens, uint8_t* out_mask, hipStream_t s);

// Scoring: log softmax(logits[t]/T)[tok[t+1]] for packed rows t0 .. t0+rows of a logits chunk;
// result goes to lp_packed[t+1] when t+1 belongs to the same sequence.
hipError_t launch_lse_gather(const float* logits, int rows_max, int t0, const int* T_dev, int V,
                             float temperature, const int* tok, const int* pos, float* lp_packed,
                             hipStream_t s);
// Packed -> padded [B, L] outputs with zeros at masked slots; logprob of a row's first token is 0.
// val_bias_dev: optional device scalar added to every real position's value (a value-head bias that lives on the
// device because an optimizer updates it there).
// first_col: log-probs of columns before it and values of columns before first_col - 1 are written as 0.
hipError_t launch_unpack_scores(const float* lp_packed, const float* val_packed, int B, int L, const int* start,
                                const int* len, const int* cu, float* out_lp, float* out_val, hipStream_t s,
                                const float* val_bias_dev = nullptr, int first_col = 0);
// Gather helper for the debug entry point: idx[i] = cu[b_i] + (col_i - start[b_i]).
hipError_t launch_rows_to_packed(const int32_t* rows_bt, int n, const int* start, const int* cu, int* idx,
                                 hipStream_t s);

// PPO signals (reward assembly, advantage estimation, whitening); see ppo_signals.hip.
hipError_t launch_ppo_rewards(const float* lp, const float* ref_full, const float* rm_full, const int* tokens, int B,
                              int Lq, int N, int eos_id, int pad_id, float beta, float miss, float* rewards,
                              float* scores, float* kl, int* kept, hipStream_t s);
hipError_t launch_ppo_gae(const float* rewards, const float* values, long vstride, const int* kept, int B, int N,
                          float gamma, float lam, float* adv, float* ret, hipStream_t s);
hipError_t launch_ppo_whiten(const float* x, const int* kept, int B, int N, int shift_mean, float* out,
                             hipStream_t s);
hipError_t launch_ppo_loss(const float* lp, const float* lp0, const float* adv, const float* v, const float* v0,
                           const float* ret, const int* kept, int B, int N, float eps, float eps_v, float c1,
                           float* d_lp, float* d_v, float* stats, hipStream_t s);
// The PPO update's glue between the padded [B, L] outputs of a forward pass and the packed rows of the backward
// pass.  Slices: new_lp[b, j] = lp_full[b, Lq + j], new_v[b, j] = val_full[b, Lq - 1 + j] (j < N).
hipError_t launch_ppo_slice(const float* lp_full, const float* val_full, int B, int L, int Lq, int N, float* new_lp,
                            float* new_v, hipStream_t s);
// Packed row cu[b] + i holds token (b, c = start[b] + i); it predicts token (b, c + 1):
//   targets = that token if it is real, else -1;  gl = d_lp[b, c + 1 - Lq] if that is a response position, else 0;
//   gv = d_v[b, c - (Lq - 1)] if 0 <= c - (Lq - 1) < N, else 0.
hipError_t launch_ppo_pack_grads(const int32_t* tokens, int B, int L, int Lq, int N, const int* start, const int* len,
                                 const int* cu, const float* d_lp, const float* d_v, int32_t* targets, float* gl,
                                 float* gv, hipStream_t s);
// Optimizer step (optimizer.hip).
struct AdamwTensor {  // p, g, m, v fp32, 16-byte aligned; p_bf16 (8-byte aligned) may be null
  float* p;
  const float* g;
  float *m, *v;
  uint16_t* p_bf16;
  size_t n;
};
// decay = 1 - lr * weight_decay; omb1 = 1 - beta1; omb2 = 1 - beta2; step_size = lr / (1 - beta1^t);
// inv_sqrt_bias2 = 1 / sqrt(1 - beta2^t): formed once on the host in double (1 - 0.999 in fp32 would
// already be off by 1.3e-5 relative).
struct AdamwScalars {
  float decay, beta1, omb1, beta2, omb2, step_size, inv_sqrt_bias2, eps, grad_scale;
};
constexpr int kAdamwTensors = 32;  // per launch: 1.8 KB of kernel arguments; a power of two
hipError_t launch_adamw(const AdamwTensor* ts, int count, const AdamwScalars& c, hipStream_t s);

// bf16 -> fp16 conversion of a weight matrix (exact within fp16's normal range).
// ---- backward through the output heads (head_backward.hip); dtype 0: float operands, 1: fp16 ----
// dst[c][r] = src[r][c] (r < R, c < C); dst columns R .. R_pad-1 are zeroed.
hipError_t launch_transpose_pad(int dtype, const void* src, size_t ld_src, void* dst, size_t ld_dst, int R, int C,
                                int R_pad, hipStream_t s);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);  // bytes: a multiple of 4
struct ZeroSpans {  // bytes: multiples of 4
  void* p[4];
  size_t bytes[4];
  int count = 0;
  void add(void* at, size_t b) { p[count] = at, bytes[count++] = b; }
};
hipError_t launch_fill_zero_spans(const ZeroSpans& z, hipStream_t s);
// dz[r][v] = gl[r] * scale * inv_temp * (onehot(targets[r])[v] - softmax(logits[r] * inv_temp)[v]) for r < rows with
// a target; zero for rows without one, rows rows .. rows_pad-1 and columns V .. V_pad-1.
hipError_t launch_softmax_grad(int dtype, const float* logits, int V, int V_pad, const int* targets, const float* gl,
                               int rows, int rows_pad, float inv_temp, float scale, void* dz, hipStream_t s);
// dy = dhl + gv * scale * value_w; dx = LayerNorm input gradient of dy; d_g = sum_t dy * xhat, d_b = sum_t dy,
// d_wv = sum_t gv * scale * h, d_bv = scale * sum_t gv.  stats [T, 2] and part [splits, 3, d] are scratch.
// LayerNorm backward of a layer (no value-head term) in one pass: dx, d_g = sum_t dy * xhat, d_b = sum_t dy.
// bf16 parameters, d a multiple of 256 up to 4096; part: ln_backward_rows_scratch_floats(T, d) floats of scratch.
bool ln_backward_rows_supported(int dtype, int d);
size_t ln_backward_rows_scratch_floats(int T, int d);
// base (optional): dx = base + the LayerNorm input gradient (rows of d floats like dx).
hipError_t launch_ln_backward_rows(const float* x, const float* dy, const void* g, int T, int d, float eps, float* dx,
                                   float* part, float* d_g, float* d_b, hipStream_t s, const float* base = nullptr);
// The two LayerNorms of one input together: dx = (base + the gradient of a.dy) + that of b.dy; twice the scratch; widths up
// to 1536 (a row of four arrays and four rows of sums in a wave's registers).
bool ln_backward_pair_supported(int dtype, int d);
struct LnTerm {
  const float* dy;
  const void* g;
  float *d_g, *d_b;
};
hipError_t launch_ln_backward_pair(const float* x, const LnTerm& a, const LnTerm& b, int T, int d, float eps, float* dx,
                                   float* part, hipStream_t s, const float* base);
// sums[c] = sum_r a[r][c] of a float [R, C] matrix (C a multiple of 4) and out_f16 = its fp16 copy, in one pass;
// part: [splits][C] floats of scratch.
hipError_t launch_convert_colsum(const float* a, int R, int C, float* part, int splits, float* sums, void* out_f16,
                                 hipStream_t s);
hipError_t launch_head_ln_backward(int dtype, const float* x, const float* dhl, const float* gv, float scale,
                                   const void* value_w, const void* g, const void* b, int T, int d, float eps,
                                   float* dx, float* stats, float* part, int splits, float* d_g, float* d_b,
                                   float* d_wv, float* d_bv, hipStream_t s);

// Element-wise pieces of a layer's backward pass (dtype 0: float activations, 1: fp16).
hipError_t launch_gelu(int dtype, const void* u, void* f, size_t n, hipStream_t s);            // f = gelu(u)
// the same on fp16 rows with strides (elements; cols and strides multiples of 8, 16-byte aligned bases)
hipError_t launch_gelu_rows_f16(const void* u, size_t ld_u, void* f, size_t ld_f, int rows, int cols, hipStream_t s);
hipError_t launch_gelu_backward(int dtype, const void* u, void* df, size_t n, hipStream_t s);  // df *= gelu'(u)
// the same on an fp16 [R, C] matrix together with the column sums of the result (sums[c]; part: [splits][C] scratch) and
// f = gelu(u)
bool gelu_backward_colsum_supported(int dtype, const void* u, const void* df, const void* f, int C);
hipError_t launch_gelu_backward_colsum(const void* u, void* df, void* f, int R, int C, float* part, int splits,
                                       float* sums, hipStream_t s);
hipError_t launch_convert_from_f32(int dtype, const float* src, void* dst, size_t n, hipStream_t s);
// out[c] = sum_r a[r][c] over a contiguous [R, C] matrix (elem 0: float, 1: fp16); part: [splits][C] scratch.
hipError_t launch_colsum(int elem, const void* a, int R, int C, float* part, int splits, float* out, hipStream_t s);

// Backward of packed causal attention (attention_backward.hip): q, k, v, g = dO and the outputs dq, dk, dv are
// [T, H*hd] row-major in float (dtype 0) or fp16 (1); cu [B+1] packed-row offsets of the sequences;
// lse, delta: [T*H] floats of scratch.  hd a multiple of 4 (float) or 8 (fp16); sequences of at most max_len rows.
hipError_t launch_attention_backward(int dtype, const void* q, const void* k, const void* v, const void* g,
                                     const int* cu, int B, int Tn, int H, int hd, int max_len, float* lse,
                                     float* delta, void* dq, void* dk, void* dv, hipStream_t s, size_t ld_qkv = 0,
                                     size_t ld_g = 0, size_t ld_out = 0, void* o = nullptr, size_t ld_o = 0,
                                     bool kv_cache = false, int rot = 0, const float* cos_t = nullptr,
                                     const float* sin_t = nullptr);
// (row strides in elements: ld_qkv of q, k, v; ld_g of g; ld_out of dq, dk, dv; 0 = H*hd.  o: optional forward
// output O = P V, [T, ld_o].  kv_cache: k and v are a layer's K / V cache as the forward pass of a packed batch
// leaves it -- sequence b's slab starts at slot cu[b] * H, head h of it holds the sequence's rows consecutively --
// and ld_qkv is q's stride alone.  rot: the rotary turn of the first rot dims is taken back from dq and dk as they are
// stored, in the reordered pair layout, as launch_rope_inplace would.  Both only where attention_backward_takes_cache
// says so.)
bool attention_backward_takes_cache(int dtype, int hd);

// Rotary turn, in place, of the q and k sections of a [T, 3*d] matrix (row stride ld) by each row's position in
// its sequence; backward != 0 applies the transpose (turn by the negative angle).  dtype 1 uses the reordered
// pair layout (2i, 2i+1) of the fp16 path, dtype 0 the pairs (i, i + r/2).
hipError_t launch_rope_inplace(int dtype, void* qkv, size_t ld, const int* cu, int B, int Tn, int H, int hd, int r,
                               const float* cos_t, const float* sin_t, int backward, hipStream_t s);
// Rows of a [3*d, C] fp32 matrix from the fp16 path's reordered W_qkv row order back to the caller's.
hipError_t launch_qkv_rows_to_caller_order(const float* in, float* out, int d, int hd, int r, int C, hipStream_t s);

// out[v][:] = sum over packed rows t with tok[t] == v of dx[t][:], in increasing t; out is [V, d], d <= 8192; scratch:
// embed_backward_scratch_bytes(V).
size_t embed_backward_scratch_bytes(int V);
hipError_t launch_embed_backward(const int* tok, const float* dx, int T, int d, int V, void* scratch, float* out,
                                 hipStream_t s);
hipError_t launch_add3(const float* a, const float* b, const float* c, float* out, size_t n, hipStream_t s);  // (a+b)+c

hipError_t launch_bf16_to_f16(const void* src, void* dst, size_t n, hipStream_t s);
// Same for a [rows, cols] matrix written with row stride dst_ld (elements).
// fp16 copy of W_qkv and a bf16 copy of its bias with the rotary dims of every q and k head
// reordered pairwise ((i, i + r/2) -> (2i, 2i + 1)): the layout every fp16 rotary kernel assumes.
hipError_t launch_qkv_weights_f16(const void* w, const void* b, void* w16, void* b_out, int d, int hd, int r,
                                  hipStream_t s);
hipError_t launch_bf16_to_f16_2d(const void* src, void* dst, size_t rows, size_t cols, size_t dst_ld, hipStream_t s);

}  // namespace rlhf
