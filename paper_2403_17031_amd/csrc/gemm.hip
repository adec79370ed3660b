// C[M,N] = A[M,K] * W[N,K]^T (+ bias, + epilogue).  Both operands are K-contiguous, which is the
// natural operand order of the CDNA matrix cores: every lane loads 8 consecutive K elements of one
// row of A and of one row of W.
//
//  * bf16 mode (fp16 operands), many rows: v_mfma_f32_32x32x16_f16, 256x256 block tile, 8 waves
//    (2x4) of 128x64, K step 64 (a tile row is one full 128-byte line), two 64 KB LDS stages
//    filled directly from global memory, XOR-swizzled 16-byte chunks (conflict-free ds_read_b128).
//    One block per CU takes tile after tile, in rounds in which the 32 tiles of an XCD are neighbours
//    and share A and W panels in its L2; what is left for a last round is cut smaller.
//    Up to 512 rows where the caller says so (GemmArgs::large_tile: prefill, scoring, decode of many sequences) its smaller
//    tiles alone; other products of few rows: 128x64 tiles staged through registers, split over K (weights streamed in
//    gemm_skinny.hip and few_rows.hip).
//  * fp32: plain FMA tile kernel (check mode only; not tuned).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rlhf {

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

template <int EPI, typename T>
__device__ __forceinline__ void epilogue_store(void* out, size_t idx, float acc, float bias) {
  if (EPI == EPI_BIAS) {
    ((T*)out)[idx] = from_f32<T>(acc + bias);
  } else if (EPI == EPI_BIAS_GELU) {
    ((T*)out)[idx] = from_f32<T>(gelu_erf(acc + bias));
  } else if (EPI == EPI_BIAS_RESADD) {
    ((float*)out)[idx] += acc + bias;
  } else {
    ((float*)out)[idx] = acc;
  }
}

// =================================================================================================
// fp16-operand MFMA kernel
// =================================================================================================
constexpr int TK = 64;
constexpr int GROUP_M = 4;  // m-tiles per scheduling group

// LDS position (in halfs) of logical 16-byte chunk c (0..7) of tile row r (A rows first, then W
// rows): rows are 128 B apart; the chunk index is XORed with bits 1..3 of the row so that 16
// consecutive rows reading the same logical chunk hit 16 different 16-byte bank groups.
__device__ __forceinline__ int lds_pos(int r, int c) { return r * TK + ((c ^ ((r >> 1) & 7)) << 3); }

// MT x NT: 32x32 accumulator tiles per wave along M and N; the block is 2x2 waves.
// PF: k-steps of global loads kept in flight in registers; OCC: blocks per CU the register
// allocation is sized for.
template <int EPI, int MT, int NT, int PF, int OCC>
__global__ void __launch_bounds__(256, OCC)
    gemm_f16_kernel(const half_t* __restrict__ A, const half_t* __restrict__ W, const bf16_t* __restrict__ bias,
                    void* __restrict__ out, int M_max, const int* __restrict__ M_dev, int M_sub, int N, int K,
                    int ldo, int nb_m, int nb_n, int ksplit, int lda, int ldw) {
  constexpr int TM = 64 * MT, TN = 64 * NT;
  constexpr int NLD = (TM + TN) / 32;  // 16-byte chunks per thread per k-step
  constexpr int NLD_A = TM / 32;
  __shared__ __attribute__((aligned(16))) uint16_t lds[(TM + TN) * TK];
  const int M = M_dev ? min(M_max, *M_dev - M_sub) : M_max;

  // ---- tile assignment: workgroup w runs on XCD w % 8; give each XCD a contiguous run of tiles,
  //      ordered so that consecutive tiles walk GROUP_M m-tiles for each n-tile.
  //      The split uses the device-side row count, so that tiles past it do not leave XCDs idle.
  nb_m = min(nb_m, (M + TM - 1) / TM);
  const int total = nb_m * nb_n;
  const int per_xcd = (total + 7) >> 3;
  if ((int)(blockIdx.x >> 3) >= per_xcd) return;
  const int lt = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lt >= total) return;
  const int group_sz = GROUP_M * nb_n;
  const int grp = lt / group_sz, rem = lt - grp * group_sz;
  const int gm = min(GROUP_M, nb_m - grp * GROUP_M);
  const int tm = grp * GROUP_M + rem % gm, tn = rem / gm;
  const int m0 = tm * TM, n0 = tn * TN;
  if (m0 >= M) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (32 * MT), wn = (wave & 1) * (32 * NT);

  // ---- global -> register staging: a row of the tile is one full 128-byte line, read by 8
  //      consecutive lanes; thread handles rows ld_r + 32*i (A rows first, then W rows)
  const int ld_r = tid >> 3, ld_c = tid & 7;
  // element offset of this thread's chunk i from A (i < NLD_A) or W, recomputed per use: keeping
  // NLD offsets live would push the kernel past 256 registers and into scratch
  auto goff = [&](int i) -> uint32_t {
    const int r = ld_r + 32 * (i < NLD_A ? i : i - NLD_A);
    return (uint32_t)((i < NLD_A ? min(m0 + r, M - 1) * lda : min(n0 + r, N - 1) * ldw) + ld_c * 8);
  };
  const int st_off = lds_pos(ld_r, ld_c);  // + 32*i rows: (r>>1)&7 is unchanged by adding 32*i
  u32x4_t stage[PF][NLD];
  // Full K tiles load unconditionally (a select on the loaded value would force the wave to wait
  // for the data right away); only a ragged last tile takes the guarded form.
  auto load_global = [&](int set, int k0) {
    if (k0 + TK <= K) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) stage[set][i] = *(const u32x4_t*)((i < NLD_A ? A : W) + goff(i) + k0);
    } else {
      const bool kok = k0 + ld_c * 8 < K;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        u32x4_t z = {0, 0, 0, 0};
        if (kok) z = *(const u32x4_t*)((i < NLD_A ? A : W) + goff(i) + k0);
        stage[set][i] = z;
      }
    }
  };
  auto store_lds = [&](int set) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) *(u32x4_t*)(lds + st_off + 32 * i * TK) = stage[set][i];
  };

  // ---- fragment addressing: lane reads row (lane & 31) of a 32-row fragment, logical chunk
  //      2*ks + (lane >> 5); the swizzle key depends on (lane & 31) >> 1 only.
  const int key = ((lane & 31) >> 1) & 7;
  const int fr = (lane & 31) * TK;
  const int a_off = wm * TK + fr, w_off = (TM + wn) * TK + fr;

  f32x16_t acc[NT][MT];  // [j over N][i over M]
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;

  // split-K: block z = blockIdx.y owns k-steps [kt0, nk); its fp32 partial sums go to slab z of
  // `out` ([ksplit][M_max][ldo]) and a second kernel adds the slabs in a fixed order
  const int nk_all = (K + TK - 1) / TK;
  const int per_split = (nk_all + ksplit - 1) / ksplit;
  const int kt0 = blockIdx.y * per_split;
  const int nk = min(nk_all, kt0 + per_split);
  if (ksplit > 1) out = (float*)out + (size_t)blockIdx.y * M_max * ldo;
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (kt0 + p < nk) load_global(p, (kt0 + p) * TK);
  for (int kt = kt0; kt < nk; kt += PF) {
#pragma unroll
   for (int p = 0; p < PF; ++p) {
    if (kt + p >= nk) break;
    store_lds(p);
    __syncthreads();
    if (kt + p + PF < nk) load_global(p, (kt + p + PF) * TK);  // in flight for PF k-steps of math
    // Fragments are double-buffered by hand and the scheduler is fenced, so that the LDS reads of
    // sub-step ks+1 are in flight while the matrix instructions of sub-step ks issue (left alone,
    // the compiler re-reads into one register quad and waits before every few MFMAs).
    constexpr int FB = (MT * NT > 8) ? 2 : 1;  // fragment buffers: two when one wave owns the SIMD
    f16x8_t fa[FB][MT], fw[FB][NT];
    auto load_frags = [&](int buf, int ks) {
      const int ch = ((2 * ks + (lane >> 5)) ^ key) << 3;
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[buf][i] = *(const f16x8_t*)(lds + a_off + i * 32 * TK + ch);
#pragma unroll
      for (int j = 0; j < NT; ++j) fw[buf][j] = *(const f16x8_t*)(lds + w_off + j * 32 * TK + ch);
    };
    if (FB == 2) load_frags(0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (FB == 2) {
        if (ks < 3) load_frags((ks + 1) & 1, ks + 1);
      } else {
        load_frags(0, ks);
      }
      __builtin_amdgcn_sched_barrier(0);
      // weights as the first operand: accumulator element e of a lane is then
      // (n = 8*(e/4) + 4*(lane/32) + e%4, m = lane%32), i.e. 4 consecutive output columns per lane
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[ks & (FB - 1)][j], fa[ks & (FB - 1)][i], acc[j][i],
                                                             0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
   }
  }

  // ---- epilogue
  const bool vec_ok = (ldo & 3) == 0;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int nb = n0 + wn + 32 * j + 8 * g + 4 * (lane >> 5);
      if (nb >= N) continue;
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (EPI != EPI_F32 && bias) {
#pragma unroll
        for (int u = 0; u < 4; ++u) bv[u] = (nb + u < N) ? to_f32(bias[nb + u]) : 0.f;
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int row = m0 + wm + 32 * i + (lane & 31);
        if (row >= M) continue;
        const size_t o = (size_t)row * ldo + nb;
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = acc[j][i][4 * g + u] + bv[u];
        if (vec_ok && nb + 4 <= N) {
          if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
            f16x4_t h;
#pragma unroll
            for (int u = 0; u < 4; ++u) h[u] = from_f32<half_t>(EPI == EPI_BIAS_GELU ? gelu_f16out(v[u]) : v[u]);
            *(f16x4_t*)((half_t*)out + o) = h;
          } else if (EPI == EPI_BIAS_RESADD) {
            f32x4_t x = *(f32x4_t*)((float*)out + o);
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] += v[u];
            *(f32x4_t*)((float*)out + o) = x;
          } else {
            f32x4_t x = {v[0], v[1], v[2], v[3]};
            *(f32x4_t*)((float*)out + o) = x;
          }
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (nb + u < N) epilogue_store<EPI, half_t>(out, o + u, acc[j][i][4 * g + u], bv[u]);
        }
      }
    }
  }
}

// =================================================================================================
// fp32 check-mode kernel: 64x64 tile, 256 threads, 4x4 outputs per thread, K step 16.
// =================================================================================================
template <int EPI>
__global__ void __launch_bounds__(256)
    gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias,
                    void* __restrict__ out, int M_max, const int* __restrict__ M_dev, int M_sub, int N, int K, int ldo) {
  __shared__ float As[16][64 + 4], Ws[16][64 + 4];
  const int M = M_dev ? min(M_max, *M_dev - M_sub) : M_max;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  const int tid = threadIdx.x;
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  const int ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    const int ar = min(m0 + lr, M - 1), wr = min(n0 + lr, N - 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + lk + e;
      As[lk + e][lr] = k < K ? A[(size_t)ar * K + k] : 0.f;
      Ws[lk + e][lr] = k < K ? W[(size_t)wr * K + k] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = As[k][ty * 4 + i];
        w[i] = Ws[k][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + ty * 4 + i;
    if (row >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + tx * 4 + j;
      if (col >= N) continue;
      const float bv = (EPI != EPI_F32 && bias) ? bias[col] : 0.f;
      epilogue_store<EPI, float>(out, (size_t)row * ldo + col, acc[i][j], bv);
    }
  }
}

// =================================================================================================
// Large-M kernel: 256x256 block tile, one block per CU, 8 waves of 128x64 (two per SIMD: what one wave
// cannot overlap the SIMD's other wave fills; measured 8-10 % faster than 4 waves of 128x128).  Tiles go global -> LDS
// directly (global_load_lds, 16 bytes per lane: a wave instruction fills 1 KB; no staging registers, no ds_write) into
// TWO 64 KB stages of K depth 64.
// The depth is what matters: a tile row is then one full 128-byte line per stage.  With half
// lines (K depth 32, more and smaller stages) every line was requested twice from L2, one half per
// k-step, and the matrix cores waited on that request stream; fetching whole lines removed the
// stall, and a lookahead of one stage proved as good as three.  One raw s_barrier per stage with
// an explicit s_waitcnt; the tile loads and fragment reads of a stage are dealt out one at a time
// between the matrix instructions (scheduling fences
// keep the order), so each issues in the shadow of a matrix instruction.  Each lane picks its
// global chunk so that the linear LDS image is the XOR-swizzled layout the fragment reads expect
// (conflict-free ds_read_b128).
//
// The launch is persistent: one block per CU walks its share of the tiles, and the last two stages of a tile issue the
// loads of the next tile's first two, so that its start-up (index arithmetic, two cold loads) runs under the epilogue,
// which has 32 KB of LDS of its own.  A round is 256 neighbouring tiles, 32 in a row on each XCD (they share panels in its
// L2).  (One block per tile and an eighth of all tiles per XCD put 33 tiles on 32 CUs whenever the count was a little above
// a multiple of 256, or 35 in the K-sliced form: a whole extra round.)  gemm_driver, us, one block per tile / this: 22,200
// rows of width 768 QKV 118 / 97, FC1 180 / 132, out-projection + FC2 190 / 150, K-major 159 / 110; 83,373 rows of width
// 2560 3381 / 3280, 4511 / 4240, 5203 / 5065; 21,504 of 4096 2041 / 1970, 2709 / 2572, 3410 / 3186 (FC1's with a fifth less
// GELU arithmetic, and about 2 % of each between runs).
//
// What is left over after the whole rounds is cut into 128x128 tiles if that fills at most two shorter rounds (K-major one:
// its transposing reads make a quarter tile cost half of a whole one), and into 64x128 tiles where those are one round; the
// sums of an output element are formed in the same order whatever the cut.  Such a tile has little matrix work per stage,
// so its loads go through a ring of four stages with three under way: with two stages (of twice the depth, the second
// requested when the first had landed) it waited for every one of them.  us, two stages and quarter tiles / the ring and
// both sizes: 22,272 rows of 768 out-projection + FC2 148 / 137, the gradients' fp32 products 87 / 82 and 112 / 105; 3,456
// rows 39 / 31, 23 / 20, 29 / 24; 1,000 rows 35 / 22, 19.5 / 12.4, 26 / 16; 600 rows of 2560 104 / 63, 64 / 41, 82 / 53; 2,200
// rows 222 / 183, 134 / 111, 176 / 144; 2,500 of 2048 178 / 148; K-major 768 x 768 over 3,456 rows 31 / 15; where whole
// rounds are most of the work 1 to 2 %.
// =================================================================================================
#define RLHF_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define RLHF_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
constexpr int kCUs = 256;                   // CUs of the chip = blocks of a launch (a multiple of its 8 XCDs)
constexpr int DK = 64;                      // K depth of one stage: 128 bytes per tile row
constexpr int DOP = 256 * DK;               // halfs per stage and operand (32 KB)
constexpr int EPW = 2048;                   // halfs of epilogue LDS per wave (4 KB)

struct DmaArgs {
  const half_t *A, *W;
  const bf16_t *bias, *bias2;
  void* out;
  const float* res;     // EPI_BIAS_RESADD: what the product is added to
  const int* M_dev;
  int M_max, M_sub, N, K, ldo, lda, ldw;
  int slices, k_slice;  // K cut into `slices` ranges of k_slice; slice z writes its fp32 result to slab z of out
  size_t slab;
};

// The epilogue of one wave: its 32 * MT rows x 64 columns from (row0, col0) on, accumulators in acc.  In the accumulator
// layout a lane owns 4 consecutive columns of ONE row (n = 32*j + 8*g + 4*hf + u, m = 32*i + l32), so a direct store
// would touch 32 rows with 8-16 bytes each -- partial-line writes that the memory system handles an order of magnitude
// slower than full lines.  The wave therefore transposes 32 rows at a time through its own 4 KB of LDS (ep; XOR-swizzled
// by row) and stores 16 bytes per lane, 8 lanes per 128-byte row segment.  Waves need not wait for each other.
// bv: the bias of the lane's columns (bf16 pairs), loaded ahead; prow: the positions of its rows (EPI_QKV).
#define RLHF_WAVE_LDS_FENCE()                  \
  __builtin_amdgcn_sched_barrier(0);           \
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); \
  __builtin_amdgcn_wave_barrier();             \
  __builtin_amdgcn_sched_barrier(0);
template <int EPI, int MT>
__device__ __forceinline__ void dma_epilogue(const DmaArgs& g, const LseArgs& lse, const QkvArgs& qk, void* out,
                                             const f32x16_t (&acc)[2][MT], int row0, int col0, int M, uint16_t* ep,
                                             int lane, const u32x2_t (&bv)[2][4], const u32x2_t (&bv2)[2][4],
                                             const int (&prow)[MT]) {
  constexpr int NT = 2;
  // (opaque, so that what is derived from it is formed here, per tile, and not kept in registers through the main loop)
  asm volatile("" : "+v"(lane));
  const int l32 = lane & 31, hf = lane >> 5;
  const int N = g.N, ldo = g.ldo;
  if constexpr (EPI == EPI_LSE) {
    // ---- scoring LM head: the logits stay in the accumulators.  A lane holds, for each of its rows (32*i + l32), half
    //      of the wave's 64 columns (the other half is in lane ^ 32): running max and sum of exp over them, combined
    //      across the two half-waves, plus the target token's z if its column is among this lane's.
    const int part = col0 >> 6;
    const int T = *lse.T_dev;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int tr = g.M_sub + row0 + 32 * i + l32;  // packed row
      const bool row_ok = row0 + 32 * i + l32 < M;
      int tcol = -1;  // target column relative to this wave's first column, or out of range
      if (lse.tgt) {
        const int tg = row_ok && tr < T ? lse.tgt[tr] : -1;
        if (tg >= 0) tcol = tg - col0;
      } else if (row_ok && tr + 1 < T && lse.pos[tr + 1] == lse.pos[tr] + 1) {
        tcol = lse.tok[tr + 1] - col0;
      }
      // the target's logit is this lane's if its column falls into one of the lane's groups of four
      const bool has_t = tcol >= 0 && tcol < 64 && ((tcol >> 2) & 1) == hf;
      int lim = N - col0;  // columns of this wave that exist (kept opaque: 32 masks would otherwise be held in registers)
      asm volatile("" : "+s"(lim));
      float m = -INFINITY, zt = 0.f;
      float z[NT][16];
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int col = 32 * j + 8 * (e >> 2) + 4 * hf + (e & 3);
          float v = acc[j][i][e] * lse.inv_temperature;
          if (col >= lim) v = -INFINITY;
          zt = col == tcol ? v : zt;
          z[j][e] = v;
          m = fmaxf(m, v);
        }
      m = half_max(m);
      float sum = 0.f;
      if (m > -INFINITY) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) sum += __expf(z[j][e] - m);
      }
      sum = half_sum(sum);
      if (row_ok) {
        if (hf == 0) {
          lse.pmax[(size_t)part * lse.stride + tr] = m;
          lse.psum[(size_t)part * lse.stride + tr] = sum;
        }
        if (has_t) lse.ztgt[tr] = zt;
      }
    }
  } else {
    f32x4_t bias_v[NT][4];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bias_v[j][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (EPI != EPI_F32) {
          const u32x2_t raw = bv[j][q];
          bias_v[j][q] = f32x4_t{__uint_as_float(raw[0] << 16), __uint_as_float(raw[0] & 0xFFFF0000u),
                                 __uint_as_float(raw[1] << 16), __uint_as_float(raw[1] & 0xFFFF0000u)};
        }
        if (EPI == EPI_BIAS_RESADD) {
          const u32x2_t raw = bv2[j][q];
          bias_v[j][q][0] += __uint_as_float(raw[0] << 16);
          bias_v[j][q][1] += __uint_as_float(raw[0] & 0xFFFF0000u);
          bias_v[j][q][2] += __uint_as_float(raw[1] << 16);
          bias_v[j][q][3] += __uint_as_float(raw[1] & 0xFFFF0000u);
        }
      }
    const int rd_row = lane >> 3, rd_c = lane & 7;  // on the way out: row within a group of 8, 16-byte chunk of the row
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_ERF || EPI == EPI_QKV) {
      // EPI_QKV: for each of the lane's eight 4-column groups the index of its first rotary angle (-1: the group is not
      // rotary).  A group is two whole pairs.
      const int qd = qk.H * qk.hd;
      int ang[NT][4];
      if (EPI == EPI_QKV) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = col0 + 32 * j + 8 * q + 4 * hf;
            const int sec = c >= 2 * qd ? 2 : (c >= qd ? 1 : 0);
            const int e = (c - sec * qd) % qk.hd;
            ang[j][q] = (sec < 2 && e < qk.r && c < N) ? (e >> 1) : -1;
          }
      }
      const int gcol = col0 + rd_c * 8;
      const int ld = EPI == EPI_QKV ? qd : ldo;  // row stride of what is stored as rows
      char* const ob = EPI == EPI_QKV ? (char*)((half_t*)qk.q + (size_t)(g.M_sub + row0) * ld + col0)
                                      : (char*)((half_t*)out + (size_t)row0 * ld + col0);
      const uint32_t lo = 2u * (uint32_t)(rd_row * ld + rd_c * 8);
      // this lane's 16-byte chunk lies in one head of one section (head_dim is a multiple of 8)
      const int sec = EPI == EPI_QKV ? (gcol >= 2 * qd ? 2 : (gcol >= qd ? 1 : 0)) : 0;
      const int hh = EPI == EPI_QKV ? (gcol - sec * qd) / qk.hd : 0, e0 = gcol - sec * qd - hh * qk.hd;
      half_t* const cache = (half_t*)(sec == 1 ? qk.kc : qk.vc);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        KvSlot slot[4];
        if (EPI == EPI_QKV && sec > 0) {
#pragma unroll
          for (int it = 0; it < 4; ++it) slot[it] = qk.slots[g.M_sub + min(row0 + 32 * i + 8 * it + rd_row, M - 1)];
        }
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f16x4_t h;
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = acc[j][i][4 * q + u] + bias_v[j][q][u];
            if (EPI == EPI_QKV) {
              if (ang[j][q] >= 0) {
                // the stand-alone kernel turns values already rounded to fp16: keep that order of roundings
                const f32x2_t co = *(const f32x2_t*)(qk.cos_t + prow[i] + ang[j][q]);
                const f32x2_t si = *(const f32x2_t*)(qk.sin_t + prow[i] + ang[j][q]);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                  const float lo = (float)from_f32<half_t>(v[2 * u]), hi = (float)from_f32<half_t>(v[2 * u + 1]);
                  v[2 * u] = lo * co[u] - hi * si[u];
                  v[2 * u + 1] = hi * co[u] + lo * si[u];
                }
              }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              h[u] = from_f32<half_t>(EPI == EPI_BIAS_GELU ? gelu_f16out(v[u]) : EPI == EPI_BIAS_GELU_ERF ? gelu_erf(v[u]) : v[u]);
            *(f16x4_t*)(ep + l32 * 64 + (((4 * j + q) ^ (l32 & 7)) << 3) + 4 * hf) = h;
          }
        RLHF_WAVE_LDS_FENCE();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = 8 * it + rd_row, grow = row0 + 32 * i + row;
          const u32x4_t v = *(const u32x4_t*)(ep + row * 64 + ((rd_c ^ (row & 7)) << 3));
          if (grow < M && gcol < N) {
            if (EPI == EPI_QKV && sec != 0)
              *(u32x4_t*)(cache + ((size_t)slot[it].x + qk.pos_add + (size_t)hh * slot[it].y) * qk.hd + e0) = v;
            else
              *(u32x4_t*)(ob + (size_t)(32 * i + 8 * it) * ld * 2 + lo) = v;
          }
        }
        RLHF_WAVE_LDS_FENCE();
      }
    } else {
      // fp32 results: 32 rows x 32 columns per pass; the residual rows are requested two passes ahead (more do not fit the
      // registers beside the accumulators)
      float* const epf = (float*)ep;
      char* const ob = (char*)((float*)out + (size_t)row0 * ldo + col0);
      const char* const rb = EPI == EPI_BIAS_RESADD ? (const char*)(g.res + (size_t)row0 * ldo + col0) : nullptr;
      const uint32_t lo = 4u * (uint32_t)(rd_row * ldo + rd_c * 4);
      f32x4_t xv[3][4];
      auto fetch = [&](int p) {
        const int i = p / NT, j = p % NT;
#pragma unroll
        for (int it = 0; it < 4; ++it)
          if (row0 + 32 * i + 8 * it + rd_row < M && col0 + 32 * j + 4 * rd_c < N)
            xv[p % 3][it] = *(const f32x4_t*)(rb + ((size_t)(32 * i + 8 * it) * ldo + 32 * j) * 4 + lo);
      };
      if (EPI == EPI_BIAS_RESADD) {
        fetch(0);
        fetch(1);
      }
#pragma unroll
      for (int p = 0; p < MT * NT; ++p) {
        const int i = p / NT, j = p % NT;
        if (EPI == EPI_BIAS_RESADD && p + 2 < MT * NT) fetch(p + 2);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16_t& a = acc[j][i];
          const f32x4_t v = {a[4 * q] + bias_v[j][q][0], a[4 * q + 1] + bias_v[j][q][1],
                             a[4 * q + 2] + bias_v[j][q][2], a[4 * q + 3] + bias_v[j][q][3]};
          *(f32x4_t*)(epf + l32 * 32 + (((2 * q + hf) ^ (l32 & 7)) << 2)) = v;
        }
        RLHF_WAVE_LDS_FENCE();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = 8 * it + rd_row;
          f32x4_t v = *(const f32x4_t*)(epf + row * 32 + ((rd_c ^ (row & 7)) << 2));
          if (row0 + 32 * i + row < M && col0 + 32 * j + 4 * rd_c < N) {
            if (EPI == EPI_BIAS_RESADD) v += xv[p % 3][it];
            *(f32x4_t*)(ob + ((size_t)(32 * i + 8 * it) * ldo + 32 * j) * 4 + lo) = v;
          }
        }
        RLHF_WAVE_LDS_FENCE();
      }
    }
  }
}

// Bias of a lane's columns from col0 on: eight 8-byte loads (N is a multiple of 8 here and every column group starts at a
// multiple of 4, so a group is inside or outside as a whole).
__device__ __forceinline__ void dma_load_bias(const bf16_t* bias, int col0, int N, int hf, u32x2_t (&bv)[2][4]) {
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int nb = col0 + 32 * j + 8 * q + 4 * hf;
      bv[j][q] = u32x2_t{0, 0};
      if (bias && nb < N) bv[j][q] = *(const u32x2_t*)(bias + nb);
    }
}

// KMAJ: both operands are given K-major -- A as [K, M] and W as [K, N], row-major, lda / ldw their row strides
// (the weight-gradient products of a backward pass: out = A^T W over the batch's rows, no transposed copies).  A stage
// then holds 64 k-rows of 512 bytes per operand, and a matrix-instruction operand slice (8 consecutive k of one
// column) comes from two transposing LDS reads (ds_read_b64_tr_b16: within a group of 16 lanes, lane i receives the
// (i mod 4)-th element of the 8-byte items addressed by lanes i/4, i/4+4, i/4+8, i/4+12; with lane r pointing at row
// k + r/4, columns 4(r mod 4).. of the tile, lane i gets column i of rows k .. k+3).  16-byte chunk c of k-row k sits at
// chunk c ^ 2(k mod 4) of the row, so that the four rows one group reads fall into four different 32-byte bank groups.
template <int EPI, bool KMAJ>
__global__ void __launch_bounds__(512, 1) gemm_f16_dma_kernel(DmaArgs g, LseArgs lse, QkvArgs qk) {
  constexpr int TM = 256, TN = 256, MT = 4, NT = 2;
  constexpr int NLD = 4;        // tile loads per wave, stage and operand
  constexpr int NMF = MT * NT;  // matrix instructions per wave per sub-step
  // stage s of the big tile: A rows in la<s>, W rows in lw<s> (separate variables, so that a read of one does not wait for
  // the loads into another); the smaller tiles use them as a ring of four stages
  __shared__ __attribute__((aligned(16))) uint16_t la0[DOP];
  __shared__ __attribute__((aligned(16))) uint16_t lw0[DOP];
  __shared__ __attribute__((aligned(16))) uint16_t la1[DOP];
  __shared__ __attribute__((aligned(16))) uint16_t lw1[DOP];
  __shared__ __attribute__((aligned(16))) uint16_t lep[8 * EPW];
  const int M = g.M_dev ? min(g.M_max, *g.M_dev - g.M_sub) : g.M_max;
  const int N = g.N;
  const int nb_m = (M + TM - 1) / TM, nb_n = (N + TN - 1) / TN;
  const int tiles = max(nb_m, 0) * nb_n, items = tiles * g.slices;
  const int G = gridDim.x, P = G >> 3;
  const int xcd = blockIdx.x & 7, slot_x = blockIdx.x >> 3;
  const int full = items / G, rem = items - full * G;
  const bool cut = (KMAJ ? 4 : 2) * rem <= G;  // the rest in smaller tiles
  // whole tiles of this block: `full` rounds, and one more if the rest is not cut and reaches it
  const int per_x = (rem + 7) >> 3;
  const int rest = full * G + xcd * per_x + slot_x;
  const int mine = full + (!cut && slot_x < per_x && rest < items ? 1 : 0);
  auto item_at = [&](int it) { return it < full ? it * G + xcd * P + slot_x : rest; };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps LDS bases in SGPRs
  const int l32 = lane & 31, hf = lane >> 5;
  const int key = (l32 >> 1) & 7;
  uint16_t* const ep = lep + wave * EPW;

  // tile t of the current row count: consecutive tiles walk GROUP_M m-tiles for each n-tile
  auto tile_pos = [&](int lt, int& m0, int& n0) {
    const int group_sz = GROUP_M * nb_n;
    const int grp = lt / group_sz, r = lt - grp * group_sz;
    const int gm = min(GROUP_M, nb_m - grp * GROUP_M);
    m0 = (grp * GROUP_M + r % gm) * TM;
    n0 = (r / gm) * TN;
  };

  {
    const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
    // the tile's first rows (wave-uniform), and this lane's chunks as byte offsets from there: A rows, then W rows
    const char *gA = nullptr, *gW = nullptr;
    uint32_t goff[2 * NLD];
    int m0 = 0, n0 = 0, nk = 0;
    void* out = g.out;
    // ---- direct loads: a stage row is 128 B (8 chunks); wave-load j (= NLD*wave + i) of an operand fills its rows
    //      8j .. 8j+7; lane l lands at row 8j + l/8, physical chunk l%8, and therefore fetches logical chunk
    //      (l%8) ^ ((row>>1)&7).  KMAJ: wave-load j covers k-rows 2j, 2j+1; lane l lands at k-row 2j + l/32, physical
    //      chunk l%32, and fetches logical chunk (l%32) ^ 2(k-row mod 4); columns past the operand's width re-read its
    //      last chunk (those output columns are never stored).
    auto set_item = [&](int item, int& m, int& n, int& kk, void*& o) {
      int lane = tid & 63;  // (opaque: see dma_epilogue)
      asm volatile("" : "+v"(lane));
      const int z = KMAJ || g.slices > 1 ? item / tiles : 0;
      tile_pos(item - z * tiles, m, n);
      const int kb = z * g.k_slice;
      kk = (g.k_slice > 0 ? min(g.k_slice, g.K - kb) : g.K) / DK;
      gA = (const char*)(g.A + (KMAJ ? (size_t)kb * g.lda + m : (size_t)m * g.lda + kb));
      gW = (const char*)(g.W + (KMAJ ? (size_t)kb * g.ldw + n : (size_t)n * g.ldw + kb));
      o = g.slices > 1 ? (void*)((float*)g.out + (size_t)z * g.slab) : g.out;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        if (KMAJ) {
          const int krow = 2 * (NLD * wave + i) + (lane >> 5);
          const int c = ((lane & 31) ^ (2 * (krow & 3))) * 8;
          goff[i] = 2u * (uint32_t)(krow * g.lda + min(c, M - 8 - m));
          goff[NLD + i] = 2u * (uint32_t)(krow * g.ldw + min(c, N - 8 - n));
        } else {
          const int row = 8 * (NLD * wave + i) + (lane >> 3);
          const int c = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
          goff[i] = 2u * (uint32_t)(min(row, M - 1 - m) * g.lda + c);
          goff[NLD + i] = 2u * (uint32_t)(min(row, N - 1 - n) * g.ldw + c);
        }
      }
    };
    // (the uniform part of the address is kept opaque per stage: scalar base + 32-bit lane offset, no 64-bit vector adds)
    auto k_base = [&](int k0, const char*& pa, const char*& pw) {
      pa = gA + 2 * (KMAJ ? (size_t)k0 * g.lda : (size_t)k0);
      pw = gW + 2 * (KMAJ ? (size_t)k0 * g.ldw : (size_t)k0);
      asm volatile("" : "+s"(pa), "+s"(pw));
    };
    auto load_one = [&](uint16_t* la, uint16_t* lw, const char* pa, const char* pw, int i) {
      uint32_t o = goff[i];
      asm volatile("" : "+v"(o));
      if (i < NLD)
        __builtin_amdgcn_global_load_lds(RLHF_GLOBAL_PTR(pa + o), RLHF_LDS_PTR(la + 8 * (NLD * wave + i) * DK), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds(RLHF_GLOBAL_PTR(pw + o), RLHF_LDS_PTR(lw + 8 * (NLD * wave + i - NLD) * DK),
                                         16, 0, 0);
    };

    const int a_off = (wm + l32) * DK, w_off = (wn + l32) * DK;
    // sub-step s (16 of the 64 k of a stage) reads logical chunks 2s and 2s+1: one per half-wave
    // KMAJ: sub-step s reads k-rows 16s + 8hf .. +7 (256 halfs per row); the column part of a lane's address, with
    // the row swizzle, is fixed per fragment
    const int ch0 = KMAJ ? (0 + 8 * hf) * 256 : ((0 + hf) ^ key) << 3, ch1 = KMAJ ? (16 + 8 * hf) * 256 : ((2 + hf) ^ key) << 3,
              ch2 = KMAJ ? (32 + 8 * hf) * 256 : ((4 + hf) ^ key) << 3, ch3 = KMAJ ? (48 + 8 * hf) * 256 : ((6 + hf) ^ key) << 3;
    int koff[MT + NT];
    if (KMAJ) {
      const int r = lane & 15, gsel = (lane >> 4) & 1;
#pragma unroll
      for (int q = 0; q < MT + NT; ++q) {
        const int colb = (q < MT ? wm + 32 * q : wn + 32 * (q - MT)) + 16 * gsel;  // first column of the group's 16
        const int chunk = ((colb >> 3) + ((r & 3) >> 1)) ^ (2 * ((r >> 2) & 3));
        koff[q] = (r >> 2) * 256 + chunk * 8 + (r & 1) * 4;
      }
    }

    f32x16_t acc[NT][MT];
    // fragment buffers, used alternately by the four sub-steps of a stage.  Weights are the first
    // matrix operand: accumulator element e of a lane is then (n = 8*(e/4) + 4*(lane/32) + e%4,
    // m = lane%32), i.e. 4 consecutive output columns per lane
    f16x8_t fa0[MT], fw0[NT], fa1[MT], fw1[NT];
    auto frag_one = [&](const uint16_t* la, const uint16_t* lw, int ch, int q, f16x8_t* fa, f16x8_t* fw) {
      const uint16_t* ls = q < MT ? la : lw;
      f16x8_t v;
      if (KMAJ) {
        typedef __attribute__((ext_vector_type(4))) short s16x4_t;
        typedef __attribute__((ext_vector_type(8))) short s16x8_t;
        typedef __attribute__((address_space(3))) s16x4_t* lds4_t;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(ls + koff[q] + ch));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(ls + koff[q] + ch + 4 * 256));
        const s16x8_t b = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        v = __builtin_bit_cast(f16x8_t, b);
      } else {
        v = *(const f16x8_t*)(ls + (q < MT ? a_off + q * 32 * DK : w_off + (q - MT) * 32 * DK) + ch);
      }
      if (q < MT) fa[q] = v;
      else fw[q - MT] = v;
    };
  // NMF matrix instructions on (FA, FW); after the n-th, fragment read n (n < MT + NT) of the next
  // sub-step from (LA, LW, CH) into (GA, GW) and, if LOAD, tile load n of the stage at (pa, pw)
#define RLHF_SUB(FA, FW, LA, LW, CH, GA, GW, LOAD, SA, SW)                                         \
  _Pragma("unroll") for (int n = 0; n < NMF; ++n) {                                               \
    const int mi = ((n >> 2) & 1) ? 3 - (n & 3) : (n & 3); /* serpentine: one operand changes at a time */ \
    acc[n >> 2][mi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(FW[n >> 2], FA[mi],                  \
                                                             acc[n >> 2][mi], 0, 0, 0);           \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    if (n < MT + NT) frag_one(LA, LW, CH, n, GA, GW);                                             \
    if (LOAD && n < 2 * NLD) load_one(SA, SW, pa, pw, n);                                         \
    __builtin_amdgcn_sched_barrier(0);                                                            \
  }
  // vmcnt(0) lgkmcnt(0) + barrier: every wave's tile loads have landed and every wave has finished
  // reading the current stage
#define RLHF_WAIT_BARRIER()                      \
  __builtin_amdgcn_sched_barrier(0);             \
  asm volatile("" ::: "memory");                 \
  __builtin_amdgcn_s_waitcnt(0x0070);            \
  __builtin_amdgcn_s_barrier();                  \
  asm volatile("" ::: "memory");                 \
  __builtin_amdgcn_sched_barrier(0);
  // The same after an epilogue, which stored at least kStores times if the whole tile exists: memory operations complete in
  // order, so the loads that are waited for, issued before it, have landed when at most that many are under way, and the
  // stores need not have (1 to 2 % of products of several rounds)
#define RLHF_WAIT_BARRIER_FIRST()                \
  __builtin_amdgcn_sched_barrier(0);             \
  asm volatile("" ::: "memory");                 \
  if (pending) __builtin_amdgcn_s_waitcnt(kStores == 16 ? 0x4070 : 0x8070); /* vmcnt(16), (32) */ \
  else __builtin_amdgcn_s_waitcnt(0x0070);       \
  pending = false;                               \
  __builtin_amdgcn_s_barrier();                  \
  asm volatile("" ::: "memory");                 \
  __builtin_amdgcn_sched_barrier(0);
  // One stage (K depth 64).  The first three sub-steps read their successors' fragments from the stage itself (CA, CW).
  // After the barrier it is free and (OA, OW) holds the next stage: the last sub-step reads the next
  // stage's first fragments from there and issues the loads at K offset KL into (CA, CW), so a
  // load has a whole stage of matrix work to land.
#define RLHF_STAGE(CA, CW, OA, OW, KL, WAIT)                                                      \
  {                                                                                               \
    const char *pa, *pw;                                                                          \
    k_base(KL, pa, pw);                                                                           \
    RLHF_SUB(fa0, fw0, CA, CW, ch1, fa1, fw1, false, CA, CW)                                      \
    RLHF_SUB(fa1, fw1, CA, CW, ch2, fa0, fw0, false, CA, CW)                                      \
    RLHF_SUB(fa0, fw0, CA, CW, ch3, fa1, fw1, false, CA, CW)                                      \
    WAIT()                                                                                        \
    RLHF_SUB(fa1, fw1, OA, OW, ch0, fa0, fw0, true, CA, CW)                                       \
  }
    if (mine > 0) {
      set_item(item_at(0), m0, n0, nk, out);
      const char *pa, *pw;
      k_base(0, pa, pw);
#pragma unroll
      for (int i = 0; i < 2 * NLD; ++i) load_one(la0, lw0, pa, pw, i);
      k_base(DK, pa, pw);
#pragma unroll
      for (int i = 0; i < 2 * NLD; ++i) load_one(la1, lw1, pa, pw, i);
      RLHF_WAIT_BARRIER()
    }
    constexpr int kStores = EPI == EPI_F32 || EPI == EPI_BIAS_RESADD ? 32 : 16;
    bool pending = false;
    for (int it = 0; it < mine; ++it) {
      // here stage 0 of this tile is in LDS for every wave, and its stage 1 has been requested
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;
#pragma unroll
      for (int q = 0; q < MT + NT; ++q) frag_one(la0, lw0, ch0, q, fa0, fw0);
      // K is a multiple of 2*DK here (the launcher routes other shapes to the staged kernel)
      for (int kt = 0; kt + 2 < nk; kt += 2) {
        RLHF_STAGE(la0, lw0, la1, lw1, (kt + 2) * DK, RLHF_WAIT_BARRIER_FIRST)
        RLHF_STAGE(la1, lw1, la0, lw0, (kt + 3) * DK, RLHF_WAIT_BARRIER)
      }
      // The last two stages request the first two of the block's next tile; after its last tile they re-issue a stage
      // that nobody reads.
      const int cm0 = m0, cn0 = n0;
      void* const cout = out;
      int kl0 = (nk - 1) * DK, kl1 = kl0;
      if (it + 1 < mine) {
        set_item(item_at(it + 1), m0, n0, nk, out);
        kl0 = 0;
        kl1 = DK;
      }
      u32x2_t bv[2][4], bv2[2][4];
      int prow[MT];
      if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_ERF || EPI == EPI_QKV)
        dma_load_bias(g.bias, cn0 + wn, N, hf, bv);
      if (EPI == EPI_QKV) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
          prow[i] = (qk.pos[g.M_sub + min(cm0 + wm + 32 * i + l32, M - 1)] + qk.pos_add) * (qk.r >> 1);
      }
      RLHF_STAGE(la0, lw0, la1, lw1, kl0, RLHF_WAIT_BARRIER)
      RLHF_STAGE(la1, lw1, la0, lw0, kl1, RLHF_WAIT_BARRIER)
      if (EPI == EPI_BIAS_RESADD) {  // (two biases do not fit the registers beside the main loop's)
        dma_load_bias(g.bias, cn0 + wn, N, hf, bv);
        dma_load_bias(g.bias2, cn0 + wn, N, hf, bv2);
      }
      dma_epilogue<EPI, MT>(g, lse, qk, cout, acc, cm0 + wm, cn0 + wn, M, ep, lane, bv, bv2, prow);
      pending = !KMAJ && EPI != EPI_LSE && cm0 + TM <= M && cn0 + TN <= N;
    }
#undef RLHF_STAGE
#undef RLHF_SUB
  }

  // ---- the rest: PM x 128 tiles, PM / 16 waves (PM / 32 x 2) of 32x64, a ring of four stages of K depth 64 (A rows, then W
  //      rows; KMAJ: 64 k-rows of 2 PM and of 256 bytes).  A tile's matrix work is short against the way of its loads
  //      (8 matrix instructions per wave and stage), so three stages are under way while one is used.  PM = 64 (half of the
  //      waves only load) where that still is one round: half the matrix work per stage.
  if (!cut || rem == 0) return;
  auto run_rest = [&](auto pm) {
    constexpr int PM = decltype(pm)::value, PER = 512 / PM;  // pieces per whole tile
    constexpr int NLA = PM / 64, NL = NLA + 2;               // tile loads per wave and stage: A, then W
    const int n_sub = PER * rem, per_sx = (n_sub + 7) >> 3;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 64;
    constexpr int AOP = PM * DK;  // halfs of a stage's A part
    const bool works = PM == 128 || wave < PM / 16;
    uint16_t* const slots[4] = {la0, lw0, la1, lw1};
    int koff[3] = {0, 0, 0};
    if (KMAJ) {
      const int r = lane & 15, gsel = (lane >> 4) & 1;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int colb = (q < 1 ? wm : wn + 32 * (q - 1)) + 16 * gsel;
        const int chunk = ((colb >> 3) + ((r & 3) >> 1)) ^ (2 * ((r >> 2) & 3));
        koff[q] = (q < 1 ? 0 : AOP) + (8 * hf + (r >> 2)) * (q < 1 ? PM : 128) + chunk * 8 + (r & 1) * 4;
      }
    }
    for (int j = slot_x; j < per_sx; j += P) {
      const int st = xcd * per_sx + j;
      if (st >= n_sub) break;
      int m0, n0;
      const int item = full * G + st / PER, z = KMAJ || g.slices > 1 ? item / tiles : 0;
      tile_pos(item - z * tiles, m0, n0);
      m0 += PM * ((st % PER) >> 1);
      n0 += 128 * (st & 1);
      if (m0 >= M || (EPI != EPI_LSE && n0 >= N)) continue;  // (EPI_LSE: columns past N leave empty parts)
      const int nw = min(n0, KMAJ ? N - 8 : N - 1);  // (first W row, KMAJ: column, to read)
      const int kb = z * g.k_slice, nk = (g.k_slice > 0 ? min(g.k_slice, g.K - kb) : g.K) / DK;
      // wave-load i of an operand's `per` per wave: rows 8(per*wave + i) .. +7, 8 lanes per row; KMAJ: as many k-rows as 64
      // chunks of 16 bytes are (see set_item for the chunks)
      uint32_t goff[NL];
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        const bool w = q >= NLA;
        const int j = w ? 2 * wave + q - NLA : NLA * wave + q;
        if (KMAJ) {
          const int lanes = w ? 16 : PM / 8, krow = 64 / lanes * j + lane / lanes;
          const int c = ((lane & (lanes - 1)) ^ (2 * (krow & 3))) * 8;
          goff[q] = 2u * (uint32_t)(krow * (w ? g.ldw : g.lda) + (w ? min(c, N - 8 - nw) : min(c, M - 8 - m0)));
        } else {
          const int row = 8 * j + (lane >> 3);
          const int c = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
          goff[q] = 2u * (uint32_t)((w ? (min(n0 + row, N - 1) - nw) * g.ldw : min(row, M - 1 - m0) * g.lda) + c);
        }
      }
      const char* const gA = (const char*)(g.A + (KMAJ ? (size_t)kb * g.lda + m0 : (size_t)m0 * g.lda + kb));
      const char* const gW = (const char*)(g.W + (KMAJ ? (size_t)kb * g.ldw + nw : (size_t)nw * g.ldw + kb));
      void* const out = g.slices > 1 ? (void*)((float*)g.out + (size_t)z * g.slab) : g.out;
      // The ring's loads are load_to_lds, because the compiler, which cannot tell the ring's stages apart, would wait for
      // all of them at every fragment read.  What orders them is the counted wait before the barrier.
      auto load_one = [&](uint16_t* slot, int kt, int i) {
        const size_t k0 = (size_t)min(kt, nk - 1) * DK;
        const char* const p = i < NLA ? gA + 2 * (KMAJ ? k0 * g.lda : k0) : gW + 2 * (KMAJ ? k0 * g.ldw : k0);
        const int at = i < NLA ? 8 * (NLA * wave + i) * DK : AOP + 8 * (2 * wave + i - NLA) * DK;
        const uint32_t dst = (uint32_t)(uintptr_t)RLHF_LDS_PTR(slot + at);
        load_to_lds(p, goff[i], dst);
      };
      f16x8_t fa[2], fw[2][2];
      auto frag = [&](const uint16_t* slot, int ks, int buf) {
        if (KMAJ) {
          typedef __attribute__((ext_vector_type(4))) short s16x4_t;
          typedef __attribute__((ext_vector_type(8))) short s16x8_t;
          typedef __attribute__((address_space(3))) s16x4_t* lds4_t;
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const int row = q < 1 ? PM : 128;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(slot + koff[q] + 16 * ks * row));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(slot + koff[q] + (16 * ks + 4) * row));
            const s16x8_t b = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            (q < 1 ? fa[buf] : fw[buf][q - 1]) = __builtin_bit_cast(f16x8_t, b);
          }
        } else {
          const int ch = ((2 * ks + hf) ^ key) << 3;
          fa[buf] = *(const f16x8_t*)(slot + (wm + l32) * DK + ch);
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) fw[buf][jj] = *(const f16x8_t*)(slot + AOP + (wn + 32 * jj + l32) * DK + ch);
        }
      };
      f32x16_t acc[2][1];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[jj][0][e] = 0.f;
      auto mul = [&](int buf) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
          acc[jj][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[buf][jj], fa[buf], acc[jj][0], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      // at most N tile loads of the wave still under way (NL per stage), its fragment reads done, and every wave there
#define RLHF_RING_BARRIER(N)                  \
  __builtin_amdgcn_sched_barrier(0);          \
  asm volatile("" ::: "memory");              \
  __builtin_amdgcn_s_waitcnt(0x0070 | (N));   \
  __builtin_amdgcn_s_barrier();               \
  asm volatile("" ::: "memory");              \
  __builtin_amdgcn_sched_barrier(0);
      RLHF_WAIT_BARRIER()  // every wave is done with the stages
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < NL; ++i) load_one(slots[u], u, i);
      RLHF_RING_BARRIER(3 * NL)
      auto stages = [&](auto multiplies) {
        constexpr bool MUL = decltype(multiplies)::value;
        if (MUL) frag(slots[0], 0, 0);
        for (int kt = 0; kt < nk; kt += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (kt + u >= nk) break;
            uint16_t *const cur = slots[u], *const nxt = slots[(u + 1) & 3];
            if (MUL) {
              frag(cur, 1, 1);
              mul(0);
              frag(cur, 2, 0);
              mul(1);
              frag(cur, 3, 1);
              mul(0);
            }
            // the next stage is there for every wave, and every wave has read the last of this one: its place is free
            RLHF_RING_BARRIER(2 * NL)
#pragma unroll
            for (int i = 0; i < NL; ++i) load_one(cur, kt + u + 4, i);
            if (MUL) {
              frag(nxt, 0, 0);
              mul(1);
            }
          }
        }
      };
      if (works) stages(std::true_type{});
      else stages(std::false_type{});
#undef RLHF_RING_BARRIER
      if (!works) continue;
      u32x2_t bv[2][4], bv2[2][4];
      int prow[1];
      if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_ERF || EPI == EPI_BIAS_RESADD || EPI == EPI_QKV)
        dma_load_bias(g.bias, n0 + wn, N, hf, bv);
      if (EPI == EPI_BIAS_RESADD) dma_load_bias(g.bias2, n0 + wn, N, hf, bv2);
      if (EPI == EPI_QKV) prow[0] = (qk.pos[g.M_sub + min(m0 + wm + l32, M - 1)] + qk.pos_add) * (qk.r >> 1);
      dma_epilogue<EPI, 1>(g, lse, qk, out, acc, m0 + wm, n0 + wn, M, ep, lane, bv, bv2, prow);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the last tile's surplus loads)
  };
  if (8 * rem <= G) run_rest(std::integral_constant<int, 64>{});
  else run_rest(std::integral_constant<int, 128>{});
#undef RLHF_WAIT_BARRIER
}
#undef RLHF_WAVE_LDS_FENCE

template <int EPI>
static void launch_f16_dma(const GemmArgs& a, hipStream_t s, int k_slices = 1, int k_slice = 0) {
  const bool split = k_slices > 1;
  DmaArgs g;
  g.A = (const half_t*)a.A;
  g.W = (const half_t*)a.W;
  g.bias = (const bf16_t*)a.bias;
  g.bias2 = (const bf16_t*)a.bias2;
  g.out = split ? a.splitk_ws : a.out;
  g.res = a.res ? a.res : (const float*)a.out;
  g.M_dev = a.M_dev;
  g.M_max = a.M_max; g.M_sub = a.M_sub; g.N = a.N; g.K = a.K;
  g.ldo = split ? a.N : a.ldo;
  g.slices = split ? k_slices : 1;
  g.k_slice = split ? k_slice : 0;
  g.slab = split ? (size_t)a.M_max * a.N : (size_t)0;
  const dim3 grid(kCUs), block(512);
  if constexpr (EPI == EPI_F32) {
    if (a.k_major) {
      g.lda = a.lda ? a.lda : a.M_max;
      g.ldw = a.ldw ? a.ldw : a.N;
      hipLaunchKernelGGL((gemm_f16_dma_kernel<EPI_F32, true>), grid, block, 0, s, g, LseArgs{}, QkvArgs{});
      return;
    }
  }
  g.lda = a.lda ? a.lda : a.K;
  g.ldw = a.ldw ? a.ldw : a.K;
  hipLaunchKernelGGL((gemm_f16_dma_kernel<EPI, false>), grid, block, 0, s, g, a.lse ? *a.lse : LseArgs{},
                     a.qkv ? *a.qkv : QkvArgs{});
}

#ifndef RLHF_GEMM_DMA
#define RLHF_GEMM_DMA 1
#endif
#ifndef RLHF_GEMM_MT
#define RLHF_GEMM_MT 2
#define RLHF_GEMM_NT 4
#define RLHF_GEMM_PF 1
#define RLHF_GEMM_OCC 2
#endif
#ifndef RLHF_GEMM_SKINNY
#define RLHF_GEMM_SKINNY 1
#endif
#ifndef RLHF_DEC_PF
#define RLHF_DEC_PF 1
#define RLHF_DEC_OCC 4
#endif

template <int EPI, int MT, int NT, int PF, int OCC>
static void launch_f16(const GemmArgs& a, hipStream_t s, void* out, int ksplit) {
  const int nb_m = (a.M_max + 64 * MT - 1) / (64 * MT), nb_n = (a.N + 64 * NT - 1) / (64 * NT);
  const int per_xcd = (nb_m * nb_n + 7) / 8;
  hipLaunchKernelGGL((gemm_f16_kernel<EPI, MT, NT, PF, OCC>), dim3(per_xcd * 8, ksplit), dim3(256), 0, s,
                     (const half_t*)a.A, (const half_t*)a.W, (const bf16_t*)a.bias, out, a.M_max, a.M_dev, a.M_sub,
                     a.N, a.K, a.ldo, nb_m, nb_n, ksplit, a.lda ? a.lda : a.K, a.ldw ? a.ldw : a.K);
}

// out = epilogue(sum_z partial[z] + bias (+ bias2)), slabs added in index order: deterministic.  M_dev: the device-side row
// count, where the slabs' rows beyond it are not written.
template <int EPI>
__global__ void __launch_bounds__(256)
    splitk_reduce_kernel(const float* __restrict__ part, int ksplit, size_t slab, const bf16_t* __restrict__ bias,
                         void* __restrict__ out, int M, int N, int ldo, const bf16_t* __restrict__ bias2 = nullptr,
                         const int* __restrict__ M_dev = nullptr) {
  if (M_dev) M = min(M, *M_dev);
  const size_t i4 = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 >= (size_t)M * ldo) return;
  const int col = (int)(i4 % ldo);
  if (col >= N) return;
  f32x4_t v = *(const f32x4_t*)(part + i4);
  for (int z = 1; z < ksplit; ++z) v += *(const f32x4_t*)(part + z * slab + i4);
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (col + u < N)
      epilogue_store<EPI, half_t>(out, i4 + u, v[u], ((EPI != EPI_F32 && bias) ? to_f32(bias[col + u]) : 0.f) +
                                                         ((EPI != EPI_F32 && bias2) ? to_f32(bias2[col + u]) : 0.f));
}

// Split factor of the few-rows path (1 = not split).  Few rows (decode): the chip is filled by small
// N tiles and by splitting K, so that every CU holds several short k-loops in flight; partial sums
// go through the caller's fp32 scratch.
int gemm_splitk_factor(int dtype, const GemmArgs& a) {
  if (few_rows_takes(dtype, a)) return 1;  // sums over K inside a block
  if (RLHF_GEMM_SKINNY && gemm_skinny_takes(dtype, a)) return gemm_skinny_splitk(a);
  if (dtype != 1 || a.M_max > 512 || !a.splitk_ws || (a.ldo & 3) != 0) return 1;
  const int tiles = ((a.M_max + 127) / 128) * ((a.N + 63) / 64);
  const int nk = (a.K + TK - 1) / TK;
  // Measured on the decode layer of the 2.8B shape (batch 256, next to the attention kernel of the
  // same layer): a product whose tiles already cover the 256 CUs is fastest unsplit; otherwise K is
  // split while that leaves at least 16 k-steps per block and at most 640 blocks -- beyond that the
  // fp32 partial sums (written, then read by the reduction) outweigh the extra parallelism.
  if (tiles >= 256) return 1;
  int ksplit = 1;
  while (ksplit < 16 && tiles * ksplit * 2 <= 640 && nk / (ksplit * 2) >= 16) ksplit *= 2;
  if ((size_t)ksplit * a.M_max * a.ldo * sizeof(float) > a.splitk_ws_bytes) return 1;
  return ksplit;
}

// Shapes the large-M kernel takes: K a multiple of two stages, 16-byte aligned rows, 32-bit offsets.
static bool takes_dma(const GemmArgs& a) {
  if (a.k_major) {  // [K, M] and [K, N] operands, fp32 output: whole 16-byte chunks per operand row, 32-bit offsets
    const size_t lda = a.lda ? a.lda : a.M_max, ldw = a.ldw ? a.ldw : a.N;
    return RLHF_GEMM_DMA && a.epilogue == EPI_F32 && !a.M_dev && !a.bias && !a.bias2 && a.M_max > 512 && a.N >= 8 &&
           (a.M_max % 8) == 0 && (a.N % 8) == 0 && (a.K % (2 * DK)) == 0 && (a.ldo % 8) == 0 && (lda % 8) == 0 &&
           (ldw % 8) == 0 && (size_t)a.K * std::max(lda, ldw) < (1ull << 32);
  }
  const size_t lda = a.lda ? a.lda : a.K, ldw = a.ldw ? a.ldw : a.K;
  return RLHF_GEMM_DMA && (a.M_max > 512 || a.large_tile) && (a.K % (2 * DK)) == 0 && (a.N % 8) == 0 && (a.ldo % 8) == 0 &&
         (lda % 8) == 0 && (ldw % 8) == 0 && std::max((size_t)a.M_max * lda, (size_t)a.N * ldw) < (1ull << 32);
}
// K slices of a large-M product with few output tiles and a long K (GemmArgs::long_k: the weight-gradient
// products of a backward pass, K = the batch's rows): the slice count (at most 8, each slice a whole number of
// stage pairs, the fp32 slabs fitting the caller's scratch) that minimises rounds of 256 whole tiles times slice length.  It
// knows nothing of the smaller tiles that the kernel cuts a K-major rest of up to a quarter round into (768 x 768 over 22,272
// rows: eight slices, 72 whole tiles, where seven would be 252 quarter tiles); another count is another order of sums.
static int dma_k_slices(const GemmArgs& a, int* k_slice) {
  *k_slice = 0;
  if (!a.long_k || !a.splitk_ws || a.M_dev || a.bias || a.bias2 || a.ldo != a.N ||
      (a.epilogue != EPI_F32 && a.epilogue != EPI_BIAS_RESADD))
    return 1;
  const int tiles = ((a.M_max + 255) / 256) * ((a.N + 255) / 256), pairs = a.K / (2 * DK);
  int best = 1, best_q = pairs;
  double best_t = (double)((tiles + 255) / 256) * pairs;
  for (int sp = 2; sp <= 8; ++sp) {
    const int q = (pairs + sp - 1) / sp, n = (pairs + q - 1) / q;  // n non-empty slices of q stage pairs
    if (q < 8 || (size_t)n * a.M_max * a.N * sizeof(float) > a.splitk_ws_bytes) continue;
    const double t = (double)((tiles * n + 255) / 256) * q;
    if (t < best_t * 0.97) { best_t = t; best = n; best_q = q; }
  }
  *k_slice = best_q * 2 * DK;
  return best;
}
// The residual epilogue alone reads a second bias (the others request theirs ahead, under the main loop, where a second
// one does not fit the registers).
bool gemm_takes_bias2(int dtype, const GemmArgs& a) {
  return dtype == 1 && a.epilogue == EPI_BIAS_RESADD && takes_dma(a);
}
bool gemm_takes_large(int dtype, const GemmArgs& a) { return dtype == 1 && takes_dma(a); }
// K slices of a large_tile product with scratch, as many as minimise the length of a slice's stages
// (about 0.24 us each in the 64x128 tiles, 0.36 in the 128x128, one round of them; two rounds of 128x128 are charged as one of
// whole tiles) plus what the slabs cost to write and to read again.  Fitted at 256 rows with the weights in the caches, us
// with 1 / 2 / 3 / 4 / 6 / 8 slices: out-projection and FC2 of width 2560 as one product (K = 12,800) 55 / 31 / 25 / 25 / 22 / 29,
// of 2048 45 / 25 / 20 / 17 / 18 / 17, of 4096 83 / 52 / 48 / 46 / 52 / 49.  A decode pass finds the weights cold, and the count
// taken (the last) still is the fastest of those the rule weighs: width 768 256 rows 1 / 2 / 3 / 4 / 6 slices 31 / 18 / 14 / 12 /
// 10, 512 rows 1 / 2 / 5 30 / 18 / 11; 1024 65 rows 1 / 4 / 8 33 / 12 / 9; 2048 256 rows 1 / 2 / 4 74 / 40 / 25; 2560 128 rows 1 /
// 3 / 6 92 / 37 / 29, 256 90 / 39 / 32, 512 1 / 2 / 3 89 / 65 / 51; 4096 256 rows 1 / 2 / 4 141 / 82 / 63, 512 1 / 2 145 / 108.
// The residual form adds the launch that sums them.
int gemm_large_slices(const GemmArgs& a) {
  const int tiles = ((a.M_max + 255) / 256) * ((a.N + 255) / 256), pairs = a.K / (2 * DK);
  int best = 1;
  double best_t = 1e30;
  for (int n = 1; n <= 16 && n <= pairs; ++n) {
    const int q = (pairs + n - 1) / n;
    if ((pairs + q - 1) / q != n || (n > 1 && (size_t)n * a.M_max * a.N * sizeof(float) > a.splitk_ws_bytes)) continue;
    const double stage = 8 * tiles * n <= kCUs ? 0.24 : 4 * tiles * n <= kCUs ? 0.36 : 1.5 * ((tiles * n + kCUs - 1) / kCUs);
    const double t = 2 * q * stage + (double)n * a.M_max * a.N * 8 / 5e6 + (a.epilogue == EPI_F32 || n == 1 ? 0.0 : 6.0);
    if (t < best_t) { best_t = t; best = n; }
  }
  return best;
}
bool gemm_takes_k_major(int dtype, const GemmArgs& a) { return dtype == 1 && a.k_major && takes_dma(a); }
bool gemm_takes_lse(int dtype, const GemmArgs& a) { return dtype == 1 && takes_dma(a); }
// EPI_QKV: 16-byte chunks must not straddle heads, a lane's 4-column group must be whole pairs, and the
// cos / sin pairs are read as aligned 8-byte words.
bool gemm_takes_qkv(int dtype, const GemmArgs& a, int H, int hd, int r) {
  return dtype == 1 && takes_dma(a) && H > 0 && hd > 0 && (hd % 8) == 0 && (r % 4) == 0 && r <= hd &&
         a.N == 3 * H * hd && a.bias != nullptr;
}
// Parts (column groups with their own max / sum-exp) the log-sum-exp epilogue leaves per row: one per wave
// column of every 256-column tile.
int gemm_lse_parts(int n_cols) { return 4 * ((n_cols + 255) / 256); }

template <int EPI>
static void launch_epi(int dtype, const GemmArgs& a, hipStream_t s) {
  if (dtype == 0) {
    dim3 grid((a.N + 63) / 64, (a.M_max + 63) / 64);
    hipLaunchKernelGGL(gemm_f32_kernel<EPI>, grid, dim3(256), 0, s, (const float*)a.A, (const float*)a.W,
                       (const float*)a.bias, a.out, a.M_max, a.M_dev, a.M_sub, a.N, a.K, a.ldo);
  } else {
    if (a.large_tile && !a.long_k && takes_dma(a)) {
      if constexpr (EPI == EPI_F32 || EPI == EPI_BIAS_RESADD) {
        const int n = a.splitk_ws ? gemm_large_slices(a) : 1, pairs = a.K / (2 * DK);
        if (a.splitk_ws && (EPI == EPI_F32 || (n > 1 && a.ldo == a.N && a.M_sub == 0))) {
          GemmArgs b = a;
          b.out = a.splitk_ws;
          b.ldo = a.N;
          launch_f16_dma<EPI_F32>(b, s, n, (pairs + n - 1) / n * 2 * DK);
          if constexpr (EPI == EPI_BIAS_RESADD) {
            const size_t quads = ((size_t)a.M_max * a.N + 3) / 4;
            hipLaunchKernelGGL(splitk_reduce_kernel<EPI>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s,
                               (const float*)a.splitk_ws, n, (size_t)a.M_max * a.N, (const bf16_t*)a.bias, a.out, a.M_max,
                               a.N, a.ldo, (const bf16_t*)a.bias2, a.M_dev);
          }
          return;
        }
      }
      launch_f16_dma<EPI>(a, s);
      return;
    }
    // Few rows (decode): the chip is filled by small N tiles and by splitting K, so that every CU
    // holds several short k-loops in flight; partial sums go through the caller's fp32 scratch.
    const int ksplit = gemm_splitk_factor(dtype, a);
    const bool skinny = RLHF_GEMM_SKINNY && gemm_skinny_takes(dtype, a);
    if (skinny && ksplit == 1) {
      launch_gemm_skinny(a, 1, s);
      return;
    }
    if (ksplit > 1) {
      if (a.phase != 2) {
        if (skinny) launch_gemm_skinny(a, ksplit, s);
        else launch_f16<EPI_F32, 2, 1, RLHF_DEC_PF, RLHF_DEC_OCC>(a, s, a.splitk_ws, ksplit);
      }
      if (a.phase != 1) {
        const size_t n4 = ((size_t)a.M_max * a.ldo + 3) / 4;
        hipLaunchKernelGGL(splitk_reduce_kernel<EPI>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                           (const float*)a.splitk_ws, ksplit, (size_t)a.M_max * a.ldo, (const bf16_t*)a.bias, a.out,
                           a.M_max, a.N, a.ldo);
      }
      return;
    }
    if (a.M_max <= 512)
      launch_f16<EPI, 2, 1, RLHF_DEC_PF, RLHF_DEC_OCC>(a, s, a.out, 1);
    else if (takes_dma(a)) {
      int k_slice = 0;
      const int n = dma_k_slices(a, &k_slice);
      if constexpr (EPI == EPI_F32 || EPI == EPI_BIAS_RESADD) {
        if (n > 1) {  // fp32 slabs, then their sum in slab order into (or, residual form, onto) the output
          launch_f16_dma<EPI_F32>(a, s, n, k_slice);
          const size_t quads = ((size_t)a.M_max * a.ldo + 3) / 4;
          hipLaunchKernelGGL((splitk_reduce_kernel<EPI>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s,
                             (const float*)a.splitk_ws, n, (size_t)a.M_max * a.N, (const bf16_t*)nullptr, a.out,
                             a.M_max, a.N, a.ldo);
          return;
        }
      }
      launch_f16_dma<EPI>(a, s);
    }
    else
      launch_f16<EPI, RLHF_GEMM_MT, RLHF_GEMM_NT, RLHF_GEMM_PF, RLHF_GEMM_OCC>(a, s, a.out, 1);
  }
}

hipError_t launch_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.M_max <= 0) return hipSuccess;
  if (dtype == 1 && (a.K % 8) != 0) return hipErrorInvalidValue;
  if (dtype != 1 && (a.bias2 || ((a.lda || a.ldw) && !few_rows_takes(dtype, a)))) return hipErrorInvalidValue;
  if ((a.bias2 || a.res) && !gemm_takes_bias2(dtype, a)) return hipErrorInvalidValue;
  if (a.res && (a.splitk_ws || a.long_k)) return hipErrorInvalidValue;
  if (a.k_major && !gemm_takes_k_major(dtype, a)) return hipErrorInvalidValue;
  if (few_rows_takes(dtype, a)) return launch_few_rows_gemm(dtype, a, s);
  switch (a.epilogue) {
    case EPI_BIAS: launch_epi<EPI_BIAS>(dtype, a, s); break;
    case EPI_BIAS_GELU: launch_epi<EPI_BIAS_GELU>(dtype, a, s); break;
    case EPI_BIAS_RESADD: launch_epi<EPI_BIAS_RESADD>(dtype, a, s); break;
    case EPI_F32: launch_epi<EPI_F32>(dtype, a, s); break;
    case EPI_LSE:
      if (!a.lse || !gemm_takes_lse(dtype, a)) return hipErrorInvalidValue;
      launch_f16_dma<EPI_LSE>(a, s);
      break;
    case EPI_BIAS_GELU_ERF:
      if (!gemm_takes_large(dtype, a)) return hipErrorInvalidValue;
      launch_f16_dma<EPI_BIAS_GELU_ERF>(a, s);
      break;
    case EPI_QKV:
      if (!a.qkv || !gemm_takes_qkv(dtype, a, a.qkv->H, a.qkv->hd, a.qkv->r)) return hipErrorInvalidValue;
      launch_f16_dma<EPI_QKV>(a, s);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rlhf
