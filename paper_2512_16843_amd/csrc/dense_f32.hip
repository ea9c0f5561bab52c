// The fp32 linear layers and the fp32 attention of the miss path, on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: 64 flops per clock and SIMD, twice what plain vector FMAs reach here).
//
// One instruction shape for every tiling, and one order of k (see below): the bits of a row do not depend on how many
// rows are computed with it.
//
// Fragment layout of the 16x16x4 instruction, per lane l of 64:
//   A operand: row  (l % 16), k = l / 16      B operand: col (l % 16), k = l / 16
//   C/D:       col  (l % 16); register r (0..3) is row (l / 16) * 4 + r
// A lane fetches four consecutive k at once (16 bytes at k = 16 i + 4 (l / 16)) and feeds one of them to each of four
// instructions, so instruction j of a group of 16 k multiplies k = j, 4 + j, 8 + j, 12 + j: the k index is a free
// permutation as long as both operands use the same one.
#include <algorithm>
#include "common.h"
#include "gemm.h"

namespace llmc {
namespace {


// ---- linear layers -------------------------------------------------------------------------------
// BM x BN block of 4 wavefronts (2 x 2), k in steps of 32 (128-byte tile rows) through a ring of STAGES tiles filled
// by direct global -> LDS loads, 16-byte chunks XOR-swizzled by half the row number as in the bf16 kernel.  The
// weights are the M side of the instruction, so a lane holds four consecutive output columns of one token and bias,
// residual and output move as 16-byte vectors straight from registers.
template <int BM_, int BN_, int STAGES_>
struct F32Cfg {
  static constexpr int BM = BM_, BN = BN_, BK = 32, STAGES = STAGES_, NW = 4;
  static constexpr int FM = BM / 2 / 16, FN = BN / 2 / 16;
  static constexpr int A_INSTR = BM / 8 / NW, B_INSTR = BN / 8 / NW, L = A_INSTR + B_INSTR;
  static constexpr int STAGE = (BM + BN) * BK;                      // floats
  static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE * 4;
  static_assert(BM % 32 == 0 && BN % 32 == 0 && (STAGES - 2) * L <= 15, "tiling");
};
// 32 KiB either way: the launch's four workgroups per compute unit (kF32MaxGrid) are resident together and hide each
// other's waits.  Deeper rings (48 KiB, of which three fit, and 40 KiB) are 2-8 % slower from 512 to 4096 rows, a
// three-stage small ring 5 % at 128 rows.
typedef F32Cfg<64, 64, 2> F32Wide;
typedef F32Cfg<32, 32, 4> F32Small;

// At most this many 64 x 64 tiles: the launch is cut into 32 x 32 tiles.  A 64 x 64 tile keeps its SIMDs busy four times
// as long, so with up to two and a half tiles per compute unit the last round of them leaves much of the chip idle;
// beyond that the wide tiles' halved operand traffic wins.  The four linear layers of a 768-wide block, small / wide: 62 / 124 us
// at 128 rows, 106 / 152 at 512, 156 (the line) / 183 at 1024; 589 (all below 1024 tiles small) / 514 at 4096, where
// they reach 113 TFLOP/s.  (512 rows: 96 since a step's fragments are read behind the multiplies of the step before.)
constexpr int kF32SmallTiles = 640;
constexpr int kF32MaxGrid = 1024;        // four workgroups for each of 256 compute units

template <class C>
__device__ __forceinline__ void f32_tiles(const GemmArgs& g, int M, float* lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_n = (g.N + C::BN - 1) / C::BN;
  const int total = ((M + C::BM - 1) / C::BM) * tiles_n;
  const float* A = (const float*)g.A;
  const float* W = (const float*)g.W;
  const float* bias = (const float*)g.bias;
  const float* resid = (const float*)g.resid;
  float* out = (float*)g.out;
  const int nk = g.K / C::BK;
  // every XCD walks its own eighth of the row-major tile list (gridDim.x % 8 == 0)
  const int xcd = blockIdx.x & 7, per_xcd = (total + 7) >> 3;
  for (int it = blockIdx.x >> 3; it < per_xcd; it += gridDim.x >> 3) {
    const int tile = xcd * per_xcd + it;
    if (tile >= total) break;
    const int m0 = (tile / tiles_n) * C::BM, n0 = (tile % tiles_n) * C::BN;
    const float* a_ptr[C::A_INSTR];
    const float* w_ptr[C::B_INSTR];
#pragma unroll
    for (int j = 0; j < C::A_INSTR; ++j) {
      const int row = (j * C::NW + wave) * 8 + (lane >> 3);
      const int r = min(m0 + row, M - 1);
      a_ptr[j] = A + map_row(g.a_rows, r, g.S) * g.lda + (((lane & 7) ^ ((row >> 1) & 7)) * 4);
    }
#pragma unroll
    for (int j = 0; j < C::B_INSTR; ++j) {
      const int row = (j * C::NW + wave) * 8 + (lane >> 3);
      const int r = min(n0 + row, g.N - 1);
      w_ptr[j] = W + (size_t)r * g.K + (((lane & 7) ^ ((row >> 1) & 7)) * 4);
    }
    auto issue = [&](int kt) {
      float* st = lds + (kt % C::STAGES) * C::STAGE;
#pragma unroll
      for (int j = 0; j < C::A_INSTR; ++j)
        __builtin_amdgcn_global_load_lds(LLMC_GPTR(a_ptr[j] + kt * C::BK), LLMC_LPTR(st + (j * C::NW + wave) * 8 * C::BK),
                                         16, 0, 0);
#pragma unroll
      for (int j = 0; j < C::B_INSTR; ++j)
        __builtin_amdgcn_global_load_lds(LLMC_GPTR(w_ptr[j] + kt * C::BK),
                                         LLMC_LPTR(st + C::BM * C::BK + (j * C::NW + wave) * 8 * C::BK), 16, 0, 0);
    };
    f32x4_t acc[C::FM][C::FN];
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int j = 0; j < C::FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int a_row = (wm * (C::BM / 2) + (lane & 15)) * C::BK;
    const int w_row = C::BM * C::BK + (wn * (C::BN / 2) + (lane & 15)) * C::BK;
#pragma unroll
    for (int s = 0; s < C::STAGES - 1; ++s)
      if (s < nk) issue(s);
    // The fragments of step kt are read behind the multiplies of step kt - 1 that free their registers, so the matrix
    // pipe has work across the barrier (zeros before the first step).  Against reading and multiplying in turn, a
    // 12-layer stack of a 768-wide block at 512 computed rows: 2078 -> 1977 us, 8 of the 105 us of its layers' products.
    f32x4_t fa[2][C::FM], fw[2][C::FN];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < C::FM; ++i) fa[ks][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < C::FN; ++j) fw[ks][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    auto multiply = [&](int ks) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
          for (int j = 0; j < C::FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[ks][j][e], fa[ks][i][e], acc[i][j], 0, 0, 0);
    };
    for (int kt = 0; kt < nk; ++kt) {
      // this wavefront's loads of step kt have landed; at the end of the tile nothing is left to overlap with
      if (nk - 1 - kt >= C::STAGES - 2) LLMC_WAIT_VM((C::STAGES - 2) * C::L);
      else LLMC_WAIT_VM(0);
      LLMC_WAIT_LGKM(0);              // ... and so have its fragments of the step before, whose stage is loaded next
      dma::barrier();
      if (kt + C::STAGES - 1 < nk) issue(kt + C::STAGES - 1);
      const float* st = lds + (kt % C::STAGES) * C::STAGE;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        multiply(ks);
        const int sw = (((ks * 4 + (lane >> 4)) ^ ((lane >> 1) & 7)) * 4);
#pragma unroll
        for (int i = 0; i < C::FM; ++i) fa[ks][i] = *reinterpret_cast<const f32x4_t*>(st + a_row + i * 16 * C::BK + sw);
#pragma unroll
        for (int j = 0; j < C::FN; ++j) fw[ks][j] = *reinterpret_cast<const f32x4_t*>(st + w_row + j * 16 * C::BK + sw);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    multiply(0);
    multiply(1);
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
      const int m = m0 + wm * (C::BM / 2) + i * 16 + (lane & 15);
      if (m < M) {
        const int64_t ro = map_row(g.o_rows, m, g.S) * g.ldo;
        const int64_t rr = resid ? map_row(g.r_rows, m, g.S) * g.ldr : 0;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
          const int n = n0 + wn * (C::BN / 2) + j * 16 + (lane >> 4) * 4;
          if (n >= g.N) continue;
          f32x4_t v = acc[i][j];
          if (bias) v += *reinterpret_cast<const f32x4_t*>(bias + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], g.act);
          if (resid) v += *reinterpret_cast<const f32x4_t*>(resid + rr + n);
          *reinterpret_cast<f32x4_t*>(out + ro + n) = v;
        }
      }
    }
    dma::barrier();      // every wavefront has read its last fragments before the next tile's first loads land
  }
}

__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int n_seq = g.count ? min(*g.count, g.max_seqs) : g.max_seqs;
  const int M = n_seq * g.S;
  const int wide = ((M + F32Wide::BM - 1) / F32Wide::BM) * ((g.N + F32Wide::BN - 1) / F32Wide::BN);
  if (wide <= kF32SmallTiles) f32_tiles<F32Small>(g, M, lds_f32);
  else f32_tiles<F32Wide>(g, M, lds_f32);
}

// ---- attention -----------------------------------------------------------------------------------
// A workgroup of 4 wavefronts owns 64 queries of one (sequence, head), 16 per wavefront, and walks the keys in tiles
// of 32 with an online softmax.  Both products are computed transposed (S^T = K Q^T, O^T = V^T P^T) so that a lane
// holds one query column and the probabilities feed the second product from registers: register r of S^T is key
// (l / 16) * 4 + r, which is the k that the lane supplies to instruction r of the second product.
// Bound by the matrix instructions (2048 of about 2600 clocks per tile and wavefront) once the chip is full: 16 sequences
// of 1024 tokens, 12 heads, 477 us = 108 TFLOP/s, causal 265 us; with 4 sequences of 128 tokens (96 workgroups, four
// tiles each) it is latency, 10 us.  The kernel it replaces, one thread per query, took 83 us there.
struct AttnF32 {
  static constexpr int DH = 64, KT = 32, QB = 64;
  static constexpr int STRIDE = 68;       // floats per LDS row: 16 rows of 16-byte reads, and rows 4 apart of 4-byte reads, fall on distinct banks
};

template <bool CAUSAL>
__global__ __launch_bounds__(256) void attention_f32_kernel(const float* __restrict__ qkv, float* __restrict__ ctx, int S,
                                                            int d, int n_heads, float scale_log2e, const int32_t* count,
                                                            int max_seqs) {
  using C = AttnF32;
  __shared__ __attribute__((aligned(16))) float sK[2][C::KT * C::STRIDE];
  __shared__ __attribute__((aligned(16))) float sV[2][C::KT * C::STRIDE];
  const int n_seq = count ? min(*count, max_seqs) : max_seqs;
  const int n_qb = (S + C::QB - 1) / C::QB;
  const int total = n_seq * n_heads * n_qb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, quad = lane >> 4;
  const size_t ld = 3 * (size_t)d;
  // staging role: keys tid / 16 and tid / 16 + 16, dh chunk of four
  const int st_key = tid >> 4, st_c = (tid & 15) * 4;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    // causal: all blocks with the most keys first, then the next shorter ones, so that the workgroups' shares even out
    const int sh = item % (n_seq * n_heads), qb = n_qb - 1 - item / (n_seq * n_heads);
    const int head = sh % n_heads, seq = sh / n_heads;
    const int q0 = qb * C::QB;
    const float* base = qkv + (size_t)seq * S * ld + head * C::DH;
    const int kv_end = CAUSAL ? min(S, q0 + C::QB) : S;
    const int n_tiles = (kv_end + C::KT - 1) / C::KT;
    const int q_lane = q0 + wave * 16 + l16;
    const int q_clamped = min(q_lane, S - 1);
    f32x4_t fq[4];                                   // Q as the B operand: column l % 16, dh = 16 i + 4 quad ..
#pragma unroll
    for (int i = 0; i < 4; ++i)
      fq[i] = *reinterpret_cast<const f32x4_t*>(base + (size_t)q_clamped * ld + i * 16 + quad * 4);
    f32x4_t o[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) o[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    f32x4_t rk[2], rv[2];
    auto load = [&](int t) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int kr = min(t * C::KT + st_key + u * 16, S - 1);
        rk[u] = *reinterpret_cast<const f32x4_t*>(base + (size_t)kr * ld + d + st_c);
        rv[u] = *reinterpret_cast<const f32x4_t*>(base + (size_t)kr * ld + 2 * d + st_c);
      }
    };
    auto store = [&](int buf) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        *reinterpret_cast<f32x4_t*>(&sK[buf][(st_key + u * 16) * C::STRIDE + st_c]) = rk[u];
        *reinterpret_cast<f32x4_t*>(&sV[buf][(st_key + u * 16) * C::STRIDE + st_c]) = rv[u];
      }
    };
    __syncthreads();                                 // the previous item's readers are done with both buffers
    load(0);
    store(0);
    __syncthreads();
    for (int t = 0; t < n_tiles; ++t) {
      const int buf = t & 1, kv0 = t * C::KT;
      if (t + 1 < n_tiles) load(t + 1);
      // a tile wholly behind this wavefront's queries contributes nothing
      if (!(CAUSAL && kv0 > q0 + wave * 16 + 15)) {
        f32x4_t s[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f32x4_t fk[2];
#pragma unroll
          for (int f = 0; f < 2; ++f)
            fk[f] = *reinterpret_cast<const f32x4_t*>(&sK[buf][(f * 16 + l16) * C::STRIDE + i * 16 + quad * 4]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int f = 0; f < 2; ++f) s[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(fk[f][e], fq[i][e], s[f], 0, 0, 0);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int kv = kv0 + f * 16 + quad * 4 + r;
            s[f][r] = (kv >= S || (CAUSAL && kv > q_lane)) ? -INFINITY : s[f][r] * scale_log2e;
            mx = fmaxf(mx, s[f][r]);
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        // Key 0 is visible to every query, but its score may have overflowed to -inf, like all others so far: such a
        // query keeps its zeros (of l_run and o) until a tile brings a score that has not.
        const bool none = m_new == -INFINITY;
        const bool any_none = __ballot(none) != 0;
        const float m_sub = none ? 0.f : m_new;
        const float corr = __builtin_amdgcn_exp2f(m_run - m_sub);
        m_run = m_new;
        l_run *= corr;
#pragma unroll
        for (int f = 0; f < 4; ++f) o[f] *= corr;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s[f][r] = __builtin_amdgcn_exp2f(s[f][r] - m_sub);
            l_run += s[f][r];
          }
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float* vp = &sV[buf][(f * 16 + quad * 4 + r) * C::STRIDE + l16];
#pragma unroll
            for (int h = 0; h < 4; ++h)
              o[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(vp[h * 16], s[f][r], o[h], 0, 0, 0);
          }
        if (any_none && none) {                      // whatever the tile holds: not-a-numbers among its scores, infinite values
          l_run = 0.f;
#pragma unroll
          for (int h = 0; h < 4; ++h) o[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
      }
      if (t + 1 < n_tiles) store(buf ^ 1);
      __syncthreads();
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    const float inv = 1.0f / l_run;
    if (q_lane < S) {
      float* dst = ctx + ((size_t)seq * S + q_lane) * d + head * C::DH + quad * 4;
#pragma unroll
      for (int h = 0; h < 4; ++h) *reinterpret_cast<f32x4_t*>(dst + h * 16) = o[h] * inv;
    }
  }
}

}  // namespace

llmc_status_t launch_gemm_f32(const GemmArgs& g, hipStream_t st) {
  static std::atomic<bool> lds_set[64];
  const size_t lds = std::max(F32Wide::LDS_BYTES, F32Small::LDS_BYTES);
  LLMC_TRY(ensure_dynamic_lds((const void*)gemm_f32_mfma_kernel, lds, lds_set));
  // the grid covers the smaller tiling, which the kernel takes when the rows it finds on the device are few
  const int64_t tiles = (int64_t)((g.max_seqs * g.S + F32Small::BM - 1) / F32Small::BM) * ((g.N + F32Small::BN - 1) / F32Small::BN);
  const int grid = (int)std::min<int64_t>((tiles + 7) & ~7ll, kF32MaxGrid);
  ProfScope ps_("gemm_f32_kernel", st);
  LLMC_KERNEL_GGL(gemm_f32_mfma_kernel, dim3(grid), dim3(256), lds, st, g);
  LLMC_LAUNCH_CHECK("gemm_f32");
  return LLMC_OK;
}

llmc_status_t launch_attention_f32(const void* qkv, void* ctx, int S, int d, int n_heads, bool causal, const int32_t* count,
                                   int max_seqs, hipStream_t st) {
  if (d != n_heads * AttnF32::DH) return LLMC_ERR_SHAPE;
  const float scale_log2e = (1.0f / sqrtf((float)AttnF32::DH)) * 1.4426950408889634f;
  const int64_t items = (int64_t)((S + AttnF32::QB - 1) / AttnF32::QB) * n_heads * max_seqs;
  const dim3 grid((unsigned)std::min<int64_t>(items, 1024));
  ProfScope ps_("attention_kernel", st);
  if (causal)
    LLMC_KERNEL_GGL(attention_f32_kernel<true>, grid, dim3(256), 0, st, (const float*)qkv, (float*)ctx, S, d, n_heads,
                    scale_log2e, count, max_seqs);
  else
    LLMC_KERNEL_GGL(attention_f32_kernel<false>, grid, dim3(256), 0, st, (const float*)qkv, (float*)ctx, S, d, n_heads,
                    scale_log2e, count, max_seqs);
  LLMC_LAUNCH_CHECK("attention_f32");
  return LLMC_OK;
}

}  // namespace llmc
