// The fp32 linear layers of the miss path, on the fp32 matrix instructions
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
// 32 KiB either way, so that five workgroups share a compute unit and hide each other's waits: deeper rings (48 and
// 40 KiB, three workgroups) are 2-8 % slower from 512 to 4096 rows, a three-stage small ring 5 % at 128 rows.
typedef F32Cfg<64, 64, 2> F32Wide;
typedef F32Cfg<32, 32, 4> F32Small;

// At most this many 64 x 64 tiles: the launch is cut into 32 x 32 tiles.  A 64 x 64 tile keeps its SIMDs busy four times
// as long, so with two tiles or fewer per compute unit the last round of them leaves much of the chip idle; beyond
// that the wide tiles' halved operand traffic wins.  The four linear layers of a 768-wide block, small / wide: 62 / 124 us
// at 128 rows, 106 / 152 at 512, 156 (the line) / 183 at 1024; 589 (all below 1024 tiles small) / 514 at 4096, where
// they reach 113 TFLOP/s.
constexpr int kF32SmallTiles = 640;
constexpr int kF32MaxGrid = 1024;

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
    for (int kt = 0; kt < nk; ++kt) {
      // this wavefront's loads of step kt have landed; at the end of the tile nothing is left to overlap with
      if (nk - 1 - kt >= C::STAGES - 2) LLMC_WAIT_VM((C::STAGES - 2) * C::L);
      else LLMC_WAIT_VM(0);
      dma::barrier();
      if (kt + C::STAGES - 1 < nk) issue(kt + C::STAGES - 1);
      const float* st = lds + (kt % C::STAGES) * C::STAGE;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int sw = (((ks * 4 + (lane >> 4)) ^ ((lane >> 1) & 7)) * 4);
        f32x4_t fa[C::FM], fw[C::FN];
#pragma unroll
        for (int i = 0; i < C::FM; ++i) fa[i] = *reinterpret_cast<const f32x4_t*>(st + a_row + i * 16 * C::BK + sw);
#pragma unroll
        for (int j = 0; j < C::FN; ++j) fw[j] = *reinterpret_cast<const f32x4_t*>(st + w_row + j * 16 * C::BK + sw);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[j][e], fa[i][e], acc[i][j], 0, 0, 0);
      }
    }
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

}  // namespace llmc
