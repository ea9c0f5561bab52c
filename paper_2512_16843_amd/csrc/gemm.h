// Linear layer  out = act(A * W^T + bias) (+ residual)  on the bf16 matrix cores, with the
// row gather / scatter of the miss path fused into operand loads and the epilogue.
#pragma once
#include <type_traits>
#include "common.h"
#include "gemm_rule.h"
#include "mma.h"

namespace llmc {

// compact token -> row of a [B*S, *] array through an optional sequence list
__device__ __forceinline__ int64_t map_row(const int32_t* rows, int r, int S) {
  if (!rows) return r;
  const int q = r / S;
  return (int64_t)rows[q] * S + (r - q * S);
}
// The same with the division as a multiplication by row_magic(S) = floor(2^61 / S) + 1: exact for r < 2^31, S <= 2^30 (the
// quotient comes out too large by at most r / 2^61, less than 1 / S).  Five instructions for about thirty: a tile's
// addresses and its epilogue take a dozen of them, and a small launch runs through its code once, from a cold cache.
inline uint64_t row_magic(int S) { return (1ull << 61) / (uint64_t)S + 1; }
__device__ __forceinline__ int64_t map_row(const int32_t* rows, int r, int S, uint64_t magic) {
  if (!rows) return r;
  const uint64_t t = (uint64_t)(uint32_t)r * (uint32_t)(magic >> 32) + __umulhi((uint32_t)r, (uint32_t)magic);
  const int q = (int)(t >> 29);
  return (int64_t)rows[q] * S + (r - q * S);
}

// erf by the five-term rational approximation of Abramowitz & Stegun 7.1.26
// (absolute error below 1.5e-7), with the hardware reciprocal and exponential
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __expf(-ax * ax);
  const float r = fmaf(-p * t, e, 1.0f);
  return copysignf(r, x);
}
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_tanh(float x) {
  const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
  // tanh(u) = 1 - 2 / (1 + e^{2u}); e^{2u} = inf gives 1, 0 gives -1
  const float th = 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __expf(2.0f * u));
  return 0.5f * x * (1.0f + th);
}

struct GemmArgs {
  const void* A; int lda;          // [rows, K]
  const void* W;                   // [N, K]
  const void* bias;                // [N] or null
  const void* resid; int ldr;      // [rows, N] or null
  void* out; int ldo;              // [rows, N]
  int N, K, S;
  const int32_t* count;            // device: number of sequences; null = max_seqs
  int max_seqs;
  uint64_t s_magic;                // row_magic(S), of the bf16 form
  const void* ahead[3];            // bf16 form: weights of the launches that follow (or null) ...
  uint32_t ahead_bytes[3];         // ... and their sizes, multiples of 16
  const int32_t* a_rows;           // sequence list applied to A rows, or null
  const int32_t* r_rows;           // ... to residual rows
  const int32_t* o_rows;           // ... to output rows
  int act;                         // 0 none, 1 GELU erf, 2 GELU tanh
};

// What a workgroup without a tile reads of the weights that follow: four rounds of 16 KiB, about as long as the tiles of a
// small launch take.  Without the limit the 44 workgroups that 788 rows of a 768-wide block leave over read for 16 us beside
// tiles of 8.
constexpr uint32_t kGemmTouchBytes = 64 * 1024;
// by the workgroups (of 256 threads) from number `busy` on
__device__ __forceinline__ void gemm_read_ahead(const GemmArgs& g, int busy) {
  const int n = gridDim.x - busy;
  uint32_t left = (uint32_t)n * kGemmTouchBytes;
  for (int i = 0; i < 3; ++i) {
    const uint32_t bytes = min(g.ahead_bytes[i], left);
    touch(g.ahead[i], bytes, blockIdx.x - busy, n, 256);
    left -= bytes;
  }
}

// the fp32 form (dense_f32.hip)
llmc_status_t launch_gemm_f32(const GemmArgs& g, hipStream_t st);

__device__ __forceinline__ float apply_act(float v, int act) {
  if (act == 1) return gelu_erf(v);
  if (act == 2) return gelu_tanh(v);
  return v;
}

// ---- bf16 GEMM on the matrix cores -------------------------------------------------------
// Workgroups of four wavefronts, two to a compute unit (80 KiB of LDS each), that walk the tiles of a launch.  The product
// is formed transposed (rows of W are the rows of the matrix instruction's result), so a lane holds outputs of ONE row of
// `out` and the epilogue needs no LDS.  Every tiling accumulates an output element over k in ascending order with the
// same instruction, so the bits of a row do not depend on how many rows are computed with it.
//
// What bounds it: partly power, inferred from the clock (a loop of nothing but these matrix instructions on such values runs
// at 1650 TFLOP/s and 1.7 GHz; with the fragment reads from LDS it reaches 1400, with the loads as well 950 to 1100).  Not it
// alone: counters at 24,576 rows show the matrix pipe 35, 35 and 43 % busy (QKV, both feed-forward layers) at 2.1 to 2.3 GHz
// and wavefronts waiting 40 to 52 % of their cycles.  So bytes per flop count on every level even where their latency is
// hidden: a wavefront owns 64 x 96 outputs (64 x 32 before: 1.8 times the bytes read from LDS), a compute unit two tiles of
// 128 x 192.  Then the epilogue, which only the other workgroup's main loop covers: an activation chosen at compile time (the
// layer with GELU over 24,576 x 3072 outputs, all of it: 171 -> 155 us).
// The four layers of a 768-wide block (microseconds, one run): eight wavefronts of 64 x 32 on 128 x 128 tiles / now: 32,768
// rows 639 / 563, 24,576 rows 481 / 420, 10,240 rows 206 / 189, 8192 rows 182 / 165, 4096 rows 105 / 105, 2048 rows 69 / 64,
// 788 rows 47 / 40, 128 rows 30 / 29; 4096 rows of 1024: 154 / 148.  Slower than those eight wavefronts: shallow products of
// many rows, where the epilogue of four wavefronts has less behind it to hide (128 wide: 24,576 rows 43 / 46, 32,768 rows
// 50 / 53; 64 wide, 6144 rows and more, and 256 wide, 10,240 rows and more: 2 to 4 %).
// Timed and not taken at 24,576 and 32,768 rows: 256 x 256 tiles with eight wavefronts of 128 x 64 and one workgroup to a
// compute unit (within 2 % over 32,768 rows of 1024, where the tile count divides by 256, 20 to 60 % more elsewhere); steps of
// 32 columns with three to five stages (64-byte rows of a panel: 7 to 20 % more); a third stage for A (4 % more).

// what follows the product: 0 nothing, 1 GELU (erf), 2 GELU (tanh), 3 the residual is added
constexpr int kEpiPlain = 0, kEpiGeluErf = 1, kEpiGeluTanh = 2, kEpiResidual = 3;

template <int EPI>
__device__ __forceinline__ float gemm_act(float v) {
  return EPI == kEpiGeluErf ? gelu_erf(v) : EPI == kEpiGeluTanh ? gelu_tanh(v) : v;
}

// One 32 x 32 fragment of the transposed product, in registers, finished: v[p][0..7] are eight consecutive columns of row
// p * 16 + lane % 16, at column 16 * (row of 16 lanes % 2) + 8 * (row of 16 lanes / 2) of the fragment, so four lanes
// cover 64 consecutive bytes of an output row.  Two exchanges of lane halves do it.
__device__ __forceinline__ int epi_col(int lane) { return (lane >> 4 & 1) * 16 + (lane >> 5) * 8; }
__device__ __forceinline__ void epi_rows(const f32x16_t& acc, float (&v)[2][8]) {
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[8 * p + e]), __float_as_uint(acc[8 * p + 4 + e]),
                                                      false, false);
      v[p][e] = __uint_as_float(s[0]);
      v[p][4 + e] = __uint_as_float(s[1]);
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0][e]), __float_as_uint(v[1][e]), false, false);
    v[0][e] = __uint_as_float(s[0]);
    v[1][e] = __uint_as_float(s[1]);
  }
}
// bias, activation and residual of eight columns, packed
template <int EPI>
__device__ __forceinline__ uint4 epi_finish(float (&v)[8], uint4 bias, uint4 resid) {
  const uint32_t bw[4] = {bias.x, bias.y, bias.z, bias.w}, rw[4] = {resid.x, resid.y, resid.z, resid.w};
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo = gemm_act<EPI>(v[2 * e] + __uint_as_float(bw[e] << 16));
    float hi = gemm_act<EPI>(v[2 * e + 1] + __uint_as_float(bw[e] & 0xFFFF0000u));
    if (EPI == kEpiResidual) {
      lo += __uint_as_float(rw[e] << 16);
      hi += __uint_as_float(rw[e] & 0xFFFF0000u);
    }
    o[e] = f32x2_to_bf16x2(lo, hi);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// LDS stage of a 64-column step: BM rows of A, then BN rows of W, 128 bytes each; the eight 16-byte chunks of row r lie
// XOR-swizzled by r / 2 (see mma.h).  A wavefront's load fetches eight rows, `gemm_chunk` is the lane's element offset.
__device__ __forceinline__ int gemm_chunk(int tr, int lane) { return ((lane & 7) ^ ((tr >> 1) & 7)) * 8; }
// element offset of a lane's fragment chunk of 16-column sub-step ks within its row
__device__ __forceinline__ int gemm_slot(int ks, int lane) { return ((ks * 2 + (lane >> 5)) ^ ((lane >> 1) & 7)) * 8; }

// ---- many rows -------------------------------------------------------------------------------------------
// 2 x 2 wavefronts, each (BM / 2) x (BN / 2) outputs, and a ring of two 64-column stages that runs on across the tiles of a
// workgroup: the loads of the next tile start two steps before this one ends.  The refill of a stage is issued behind the
// first two multiplies after the barrier, not in front of them (10 % of the loop's time).
template <int BM_, int BN_>
struct GemmRing {
  static constexpr int BM = BM_, BN = BN_, BK = 64, NW = 4;
  static constexpr int FM = BM / 64, FN = BN / 64;                 // 32 x 32 fragments of a wavefront
  static constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;         // its loads of a stage
  static constexpr int STAGE = (BM + BN) * BK;
  static constexpr size_t LDS_BYTES = 2ull * STAGE * 2;
  static_assert(BM % 64 == 0 && BN % 64 == 0 && FM * FN >= 2, "fragments");
};

template <class C, int EPI>
__device__ __forceinline__ void gemm_ring_tiles(const GemmArgs& g, int M, uint16_t* lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_n = (g.N + C::BN - 1) / C::BN, tiles_m = (M + C::BM - 1) / C::BM, total = tiles_m * tiles_n;
  const uint16_t* A = (const uint16_t*)g.A;
  const uint16_t* W = (const uint16_t*)g.W;
  const uint16_t* bias = (const uint16_t*)g.bias;
  const uint16_t* resid = (const uint16_t*)g.resid;
  uint16_t* out = (uint16_t*)g.out;
  const int nk = g.K / C::BK;
  // Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  XCD x walks the x-th eighth of the tile
  // list, so that neighbouring tiles share their operand panels there: row by row for narrow outputs; wide outputs down
  // eight row blocks before the list moves one column tile on.  Where the column tiles divide by eight, plain striding
  // gives every XCD its own eighth of the columns instead: its L2 keeps those rows of W and only A streams.
  // Each order forced on both tilings, blocks 64 to 2048 wide, geometric means over 2048 to 32,768 rows, against row by row:
  // up to 8 column tiles grouped 0.98 to 1.04, strided 0.99 to 1.09 (two steps of k: 0.95 to 1.05); more, not divisible by
  // eight, grouped 0.95 to 1.02, strided 0.95 to 1.09; divisible, strided / grouped 1.02 / 1.00 (128 x 192 tiles, 3072
  // columns, K = 768), 1.00 / 0.97 (K = 1024), 0.95 / 0.99 (4608), 0.90 / 0.93 (6144), 0.93 / 0.95 (128 x 128, 4096), 0.98 /
  // 0.94 (2048, K = 8192).  The rule is within 5 % of the best order in all of them, mostly within 2, which is what two runs
  // differ by.
  const int order = tiles_n <= 8 ? 1 : tiles_n % 8 == 0 ? 0 : 2;
  const int xcd = blockIdx.x & 7, per_xcd = (total + 7) >> 3;
  const int it_step = order ? (int)(gridDim.x >> 3) : (int)gridDim.x;
  auto locate = [&](int it, int& m, int& n) -> bool {
    if (order && it >= per_xcd) return false;
    const int tile = order ? xcd * per_xcd + it : it;
    if (tile >= total) return false;
    int tile_m = tile / tiles_n, tile_n = tile % tiles_n;
    if (order == 2) {
      const int group = tile / (8 * tiles_n), in_group = tile % (8 * tiles_n);
      const int rows_in_group = min(8, tiles_m - group * 8);
      tile_m = group * 8 + in_group % rows_in_group;
      tile_n = in_group / rows_in_group;
    }
    m = tile_m * C::BM;
    n = tile_n * C::BN;
    return true;
  };
  int it = order ? (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  int m0 = 0, n0 = 0;
  if (!locate(it, m0, n0)) return;

  // the load side: position, and this lane's addresses in the tile it stands in
  const uint16_t* a_ptr[C::LA];
  const uint16_t* b_ptr[C::LB];
  auto address = [&](int m, int n) {
#pragma unroll
    for (int j = 0; j < C::LA; ++j) {
      const int tr = (j * C::NW + wave) * 8 + (lane >> 3);
      a_ptr[j] = A + map_row(g.a_rows, min(m + tr, M - 1), g.S, g.s_magic) * g.lda + gemm_chunk(tr, lane);
    }
#pragma unroll
    for (int j = 0; j < C::LB; ++j) {
      const int tr = (j * C::NW + wave) * 8 + (lane >> 3);
      b_ptr[j] = W + (size_t)min(n + tr, g.N - 1) * g.K + gemm_chunk(tr, lane);
    }
  };
  address(m0, n0);
  int kl = 0, fill = 0;
  bool live = true;
  auto issue_b = [&]() {
    if (kl == nk) {
      int m, n;
      kl = 0;
      live = locate(it + it_step, m, n);
      if (live) address(m, n);
    }
    if (!live) return;
    uint16_t* st = lds + fill * C::STAGE + C::BM * C::BK;
#pragma unroll
    for (int j = 0; j < C::LB; ++j)
      __builtin_amdgcn_global_load_lds(LLMC_GPTR(b_ptr[j] + kl * C::BK), LLMC_LPTR(st + (j * C::NW + wave) * 512), 16, 0, 0);
  };
  auto issue_a = [&]() {
    if (!live) return;
    uint16_t* st = lds + fill * C::STAGE;
#pragma unroll
    for (int j = 0; j < C::LA; ++j)
      __builtin_amdgcn_global_load_lds(LLMC_GPTR(a_ptr[j] + kl * C::BK), LLMC_LPTR(st + (j * C::NW + wave) * 512), 16, 0, 0);
    fill ^= 1;
    ++kl;
  };

  int sw[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) sw[ks] = gemm_slot(ks, lane);
  const int a_row = (wm * (C::BM / 2) + (lane & 31)) * C::BK;
  const int b_row = (C::BM + wn * (C::BN / 2) + (lane & 31)) * C::BK;
  bf16x8_t fa[2][C::FM], fb[2][C::FN];
  int stage = 0;
  auto read = [&](int ks, int buf) {
    const uint16_t* st = lds + stage * C::STAGE + sw[ks];
#pragma unroll
    for (int i = 0; i < C::FN; ++i) fb[buf][i] = *reinterpret_cast<const bf16x8_t*>(st + b_row + i * 32 * C::BK);
#pragma unroll
    for (int j = 0; j < C::FM; ++j) fa[buf][j] = *reinterpret_cast<const bf16x8_t*>(st + a_row + j * 32 * C::BK);
  };

  // this lane's columns and rows of the epilogue; bias and the first rows of the residual are fetched two steps early
  const int col = wn * (C::BN / 2) + epi_col(lane), row = wm * (C::BM / 2) + (lane & 15);
  uint4 bq[C::FN], rq[2][C::FN];
  auto load_resid = [&](int j, int i0, int i1) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint16_t* src = resid + map_row(g.r_rows, min(m0 + row + j * 32 + p * 16, M - 1), g.S, g.s_magic) * g.ldr;
#pragma unroll
      for (int i = 0; i < C::FN; ++i)
        if (i >= i0 && i < i1) rq[p][i] = *reinterpret_cast<const uint4*>(src + min(n0 + col + i * 32, g.N - 8));
    }
  };
#pragma unroll
  for (int i = 0; i < C::FN; ++i) bq[i] = rq[0][i] = rq[1][i] = make_uint4(0, 0, 0, 0);

  issue_b(); issue_a();
  issue_b(); issue_a();                                     // nk >= 2
  LLMC_WAIT_VM(C::LA + C::LB);
  dma::barrier();
  read(0, 0);
  bool first = true;
  while (true) {
    f32x16_t acc[C::FN][C::FM];
#pragma unroll
    for (int i = 0; i < C::FN; ++i)
#pragma unroll
      for (int j = 0; j < C::FM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int c = ks & 1;
        // this sub-step's fragments were requested one sub-step ago
        __builtin_amdgcn_sched_barrier(0);
        LLMC_WAIT_LGKM(0);
        __builtin_amdgcn_sched_barrier(0);
        if (ks == 3) {
          // The step's last fragments are in registers: its stage is free once everybody stands here, and everybody's loads
          // of the next step have landed (of a tile's second step: waited for before the stores of the tile before).
          if (kt > 0 || first) LLMC_WAIT_VM(0);
          dma::barrier();
          stage ^= 1;
          read(0, c ^ 1);                                   // behind the last tile: old contents, not used
          if (kt + 2 == nk) {
            if (bias) {
#pragma unroll
              for (int i = 0; i < C::FN; ++i) bq[i] = *reinterpret_cast<const uint4*>(bias + min(n0 + col + i * 32, g.N - 8));
            }
            if (EPI == kEpiResidual) load_resid(0, 0, 2);    // a third column of fragments: registers
          }
        } else {
          read(ks + 1, c ^ 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < C::FN; ++i)
#pragma unroll
          for (int j = 0; j < C::FM; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][i], fa[c][j], acc[i][j], 0, 0, 0);
            // the loads that refill the stage are issued behind the first multiplies, not in front of them
            if (ks == 3 && i * C::FM + j < 2) {
              __builtin_amdgcn_sched_barrier(0);
              if (i * C::FM + j == 0) issue_b();
              else issue_a();
              __builtin_amdgcn_sched_barrier(0);
            }
          }
      }
    }
    first = false;
    if (EPI == kEpiResidual) load_resid(0, 2, C::FN);
    // the finished values are packed into the registers of the sums: two rows of 16-byte vectors in registers 0..7
#pragma unroll
    for (int j = 0; j < C::FM; ++j) {
#pragma unroll
      for (int i = 0; i < C::FN; ++i) {
        float v[2][8];
        epi_rows(acc[i][j], v);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const uint4 o = epi_finish<EPI>(v[p], bq[i], rq[p][i]);
          acc[i][j][4 * p] = __uint_as_float(o.x);
          acc[i][j][4 * p + 1] = __uint_as_float(o.y);
          acc[i][j][4 * p + 2] = __uint_as_float(o.z);
          acc[i][j][4 * p + 3] = __uint_as_float(o.w);
        }
        __builtin_amdgcn_sched_barrier(0);                    // one fragment at a time: registers
      }
      if (EPI == kEpiResidual && j + 1 < C::FM) load_resid(j + 1, 0, C::FN);
    }
    // This wavefront's loads of the next tile have landed before its stores go out: the next tile's first steps wait for
    // neither.
    LLMC_WAIT_VM(0);
#pragma unroll
    for (int j = 0; j < C::FM; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int m = m0 + row + j * 32 + p * 16;
        if (m < M) {
          uint16_t* dst = out + map_row(g.o_rows, m, g.S, g.s_magic) * g.ldo;
#pragma unroll
          for (int i = 0; i < C::FN; ++i) {
            const int n = n0 + col + i * 32;
            if (n < g.N)
              *reinterpret_cast<uint4*>(dst + n) =
                  make_uint4(__float_as_uint(acc[i][j][4 * p]), __float_as_uint(acc[i][j][4 * p + 1]),
                             __float_as_uint(acc[i][j][4 * p + 2]), __float_as_uint(acc[i][j][4 * p + 3]));
          }
        }
      }
    it += it_step;
    if (!locate(it, m0, n0)) return;
  }
}

// ---- fewer rows: a ring of its own per tile ----------------------------------------------------------------
// A launch with few tiles lasts as long as the latency of its loads times the steps over the steps in flight, and a
// step as long as its own fragments take to arrive from LDS.  (788 rows of a 768-wide block: 17.7 -> 12.8 us for K = 3072.)
// So: smaller tiles, more stages, and a whole step's fragments held in registers: those of step kt are read from LDS behind
// the multiplies of step kt - 1 that free theirs.
// WM x WN wavefronts multiply (they fetch PC blocks of eight rows a stage), the others only load (PL blocks).
template <int BM_, int BN_, int WM_, int WN_, int STAGES_, int PC_, int PL_>
struct GemmStep {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, BK = 64, STAGES = STAGES_, PC = PC_, PL = PL_, NW = 4;
  static constexpr int FM = BM / WM / 32, FN = BN / WN / 32, COMPUTE = WM * WN;
  static constexpr int STAGE = (BM + BN) * BK;
  static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE * 2;
  static_assert(COMPUTE * PC + (NW - COMPUTE) * PL == (BM + BN) / 8, "the blocks of a stage");
  static_assert(STAGES >= 3 && STAGES <= 6, "the waits of the loop");
};

// The k loop of one wavefront that fetches PER blocks a step and, with MUL, multiplies.
template <class C, int PER, bool MUL>
__device__ __forceinline__ void gemm_step_loop(const uint16_t* const (&src)[PER], int first_block, int nk, uint16_t* lds,
                                               int a_row, int b_row, const int (&sw)[4], f32x16_t (&acc)[C::FN][C::FM]) {
  int in = 0, rd = 0;                                        // ring stages of the next load and of the next read
  auto issue = [&](int kt) {
    uint16_t* st = lds + in * C::STAGE + first_block * 512;
    in = in + 1 == C::STAGES ? 0 : in + 1;
#pragma unroll
    for (int j = 0; j < PER; ++j)
      __builtin_amdgcn_global_load_lds(LLMC_GPTR(src[j] + kt * C::BK), LLMC_LPTR(st + j * 512), 16, 0, 0);
  };
  bf16x8_t fa[4][C::FM], fb[4][C::FN];                       // zeros until the first step has been read
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
    for (int j = 0; j < C::FM; ++j) fa[ks][j] = bf16x8_t{};
#pragma unroll
    for (int i = 0; i < C::FN; ++i) fb[ks][i] = bf16x8_t{};
  }
  auto mul = [&](int ks) {
#pragma unroll
    for (int i = 0; i < C::FN; ++i)
#pragma unroll
      for (int j = 0; j < C::FM; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][i], fa[ks][j], acc[i][j], 0, 0, 0);
  };
  // everybody's loads of this step have landed, and everybody has its fragments of the step before
  auto step = [&](int kt, bool more) {
    if (MUL) LLMC_WAIT_LGKM(0);
    dma::barrier();
    if (more) issue(kt + C::STAGES - 1);
    if (MUL) {
      const uint16_t* st = lds + rd * C::STAGE;
      rd = rd + 1 == C::STAGES ? 0 : rd + 1;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        mul(ks);
#pragma unroll
        for (int i = 0; i < C::FN; ++i) fb[ks][i] = *reinterpret_cast<const bf16x8_t*>(st + b_row + i * 32 * C::BK + sw[ks]);
#pragma unroll
        for (int j = 0; j < C::FM; ++j) fa[ks][j] = *reinterpret_cast<const bf16x8_t*>(st + a_row + j * 32 * C::BK + sw[ks]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < C::STAGES - 1; ++s)
    if (s < nk) issue(s);
  int kt = 0;
  for (; kt + C::STAGES - 1 < nk; ++kt) {
    LLMC_WAIT_VM((C::STAGES - 2) * PER);
    step(kt, true);
  }
  auto tail = [&](auto steps) {
    constexpr int ahead = decltype(steps)::value;
    if (ahead <= C::STAGES - 2 && kt == nk - 1 - ahead) {    // not for every one when nk < STAGES - 1
      LLMC_WAIT_VM(ahead * PER);
      step(kt, false);
      ++kt;
    }
  };
  tail(std::integral_constant<int, 4>());
  tail(std::integral_constant<int, 3>());
  tail(std::integral_constant<int, 2>());
  tail(std::integral_constant<int, 1>());
  tail(std::integral_constant<int, 0>());
  if (MUL) {
    LLMC_WAIT_LGKM(0);           // the last fragments are in registers before the caller's barrier hands their stage on
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) mul(ks);
  }
}

template <class C, int EPI>
__device__ __forceinline__ void gemm_step_tiles(const GemmArgs& g, int M, uint16_t* lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;            // of the multiplying wavefronts
  const int tiles_n = (g.N + C::BN - 1) / C::BN, total = ((M + C::BM - 1) / C::BM) * tiles_n;
  const uint16_t* A = (const uint16_t*)g.A;
  const uint16_t* W = (const uint16_t*)g.W;
  const uint16_t* bias = (const uint16_t*)g.bias;
  const uint16_t* resid = (const uint16_t*)g.resid;
  uint16_t* out = (uint16_t*)g.out;
  const int nk = g.K / C::BK;
  int sw[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) sw[ks] = gemm_slot(ks, lane);
  const int a_row = (wm * (C::BM / C::WM) + (lane & 31)) * C::BK;
  const int b_row = (C::BM + wn * (C::BN / C::WN) + (lane & 31)) * C::BK;
  for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
    const int m0 = (tile / tiles_n) * C::BM, n0 = (tile % tiles_n) * C::BN;
    auto source = [&](int block) -> const uint16_t* {        // blocks 0 .. BM / 8 - 1 are rows of A, the others rows of W
      const int tr = block * 8 + (lane >> 3);
      if (block < C::BM / 8) return A + map_row(g.a_rows, min(m0 + tr, M - 1), g.S, g.s_magic) * g.lda + gemm_chunk(tr, lane);
      return W + (size_t)min(n0 + tr - C::BM, g.N - 1) * g.K + gemm_chunk(tr, lane);
    };
    if (wave < C::COMPUTE) {
      const uint16_t* src[C::PC];
#pragma unroll
      for (int j = 0; j < C::PC; ++j) src[j] = source(wave * C::PC + j);
      // bias and residual are on their way before the first step: behind the last one each would cost its latency
      const int n = n0 + wn * (C::BN / C::WN) + epi_col(lane), m = m0 + wm * (C::BM / C::WM) + (lane & 15);
      uint4 bq[C::FN], rq[C::FN][C::FM][2];
#pragma unroll
      for (int i = 0; i < C::FN; ++i) {
        bq[i] = bias ? *reinterpret_cast<const uint4*>(bias + min(n + i * 32, g.N - 8)) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
#pragma unroll
          for (int p = 0; p < 2; ++p) rq[i][j][p] = make_uint4(0, 0, 0, 0);
      }
      if (EPI == kEpiResidual) {
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const uint16_t* row = resid + map_row(g.r_rows, min(m + j * 32 + p * 16, M - 1), g.S, g.s_magic) * g.ldr;
#pragma unroll
            for (int i = 0; i < C::FN; ++i) rq[i][j][p] = *reinterpret_cast<const uint4*>(row + min(n + i * 32, g.N - 8));
          }
      }
      f32x16_t acc[C::FN][C::FM];
#pragma unroll
      for (int i = 0; i < C::FN; ++i)
#pragma unroll
        for (int j = 0; j < C::FM; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      gemm_step_loop<C, C::PC, true>(src, wave * C::PC, nk, lds, a_row, b_row, sw, acc);
#pragma unroll
      for (int j = 0; j < C::FM; ++j) {
        uint16_t* dst[2];
#pragma unroll
        for (int p = 0; p < 2; ++p)
          dst[p] = out + map_row(g.o_rows, min(m + j * 32 + p * 16, M - 1), g.S, g.s_magic) * g.ldo + n;
#pragma unroll
        for (int i = 0; i < C::FN; ++i) {
          float v[2][8];
          epi_rows(acc[i][j], v);
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const uint4 o = epi_finish<EPI>(v[p], bq[i], rq[i][j][p]);
            if (m + j * 32 + p * 16 < M && n + i * 32 < g.N) *reinterpret_cast<uint4*>(dst[p] + i * 32) = o;
          }
        }
      }
    } else if constexpr (C::COMPUTE < C::NW) {
      const int b0 = C::COMPUTE * C::PC + (wave - C::COMPUTE) * C::PL;
      const uint16_t* src[C::PL];
#pragma unroll
      for (int j = 0; j < C::PL; ++j) src[j] = source(b0 + j);
      f32x16_t none[C::FN][C::FM];
      gemm_step_loop<C, C::PL, false>(src, b0, nk, lds, a_row, b_row, sw, none);
    }
    dma::barrier();               // every fragment has been read before the next tile's first loads land
  }
}

// ---- the kernel: which tiling a launch takes ----------------------------------------------------------------
typedef GemmRing<128, 192> GemmBig;                    // 80 KiB
typedef GemmRing<128, 128> GemmMid;                    // 64 KiB
typedef GemmStep<64, 128, 2, 2, 3, 6, 6> GemmLow;      // 72 KiB
typedef GemmStep<64, 64, 2, 2, 4, 4, 4> GemmTiny;      // 64 KiB
typedef GemmStep<32, 64, 1, 2, 6, 2, 4> GemmFew;       // 72 KiB
constexpr size_t kGemmLdsBytes = GemmBig::LDS_BYTES;
static_assert(GemmMid::LDS_BYTES <= kGemmLdsBytes && GemmLow::LDS_BYTES <= kGemmLdsBytes &&
              GemmTiny::LDS_BYTES <= kGemmLdsBytes && GemmFew::LDS_BYTES <= kGemmLdsBytes, "one launch serves all tilings");
template <class C, int PATH>
constexpr bool gemm_same_tile = C::BM == kGemmTileRows[PATH] && C::BN == kGemmTileCols[PATH];
static_assert(gemm_same_tile<GemmBig, kGemmBig> && gemm_same_tile<GemmMid, kGemmMid> && gemm_same_tile<GemmLow, kGemmLow> &&
              gemm_same_tile<GemmTiny, kGemmTiny> && gemm_same_tile<GemmFew, kGemmFew>, "the rule counts these tiles");

template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_bf16_dma_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_dyn[];
  const int n_seq = g.count ? min(*g.count, g.max_seqs) : g.max_seqs;
  const int M = n_seq * g.S;
  if (M <= 0) return;
  const GemmPick pick = gemm_pick(M, g.N, g.K / 64, EPI == kEpiGeluErf || EPI == kEpiGeluTanh, EPI == kEpiResidual);
  const int busy = (pick.tiles + 7) & ~7;                // workgroups beyond have no tile, in any order of the tiles
  if ((int)blockIdx.x >= busy) {
    gemm_read_ahead(g, busy);
    return;
  }
  if (pick.path == kGemmBig) gemm_ring_tiles<GemmBig, EPI>(g, M, lds_dyn);
  else if (pick.path == kGemmMid) gemm_ring_tiles<GemmMid, EPI>(g, M, lds_dyn);
  else if (pick.path == kGemmLow) gemm_step_tiles<GemmLow, EPI>(g, M, lds_dyn);
  else if (pick.path == kGemmTiny) gemm_step_tiles<GemmTiny, EPI>(g, M, lds_dyn);
  else gemm_step_tiles<GemmFew, EPI>(g, M, lds_dyn);
}

}  // namespace llmc
