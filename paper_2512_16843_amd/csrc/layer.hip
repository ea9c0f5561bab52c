// The miss path: one transformer block f_l (Section IV-A of the paper) applied to the
// sequences that found no match, named by a device-side row list and count.
//
// Rows are processed in a compact token space: compact token r belongs to list entry
// r / S and is token r % S of sequence rows[r / S].  Every kernel is launched for the
// worst case (all B sequences) and reads the real count on the device; workgroups
// beyond it exit at once, so the host never learns the number of misses.
//
// Kernels: linear layers on the bf16 matrix cores (fp32 accumulate) with bias, GELU,
// residual and row gather/scatter fused into the epilogue; LayerNorm with one wavefront per
// token (the last LayerNorm of a post-LN block also leaves the pooled chunk sums of the rows
// it writes for the next fingerprint).  The two attention kernels and the linear layers of
// fp32 runs are translation units of their own.
#include "common.h"
#include <algorithm>
#include <initializer_list>
#include <utility>
#include "gemm.h"

namespace llmc {

// Launches are sized for the worst case (every sequence a miss) but capped: workgroups walk
// their tiles / rows with a grid stride and read the real count on the device, so a layer
// with few or no misses costs a small, fixed number of idle workgroups.
constexpr int kMaxGrid = 512;

template <int EPI>
static llmc_status_t launch_gemm_bf16(const GemmArgs& args, hipStream_t st) {
  GemmArgs g = args;
  g.s_magic = row_magic(g.S);
  static std::atomic<bool> lds_set[64];
  const auto kernel = gemm_bf16_dma_kernel<EPI>;
  LLMC_TRY(ensure_dynamic_lds((const void*)kernel, kGemmLdsBytes, lds_set));
  // as many workgroups as the smallest tiles could use if every sequence were computed; the kernel reads the count
  const int64_t tiles = (((int64_t)g.max_seqs * g.S + GemmFew::BM - 1) / GemmFew::BM) * ((g.N + GemmFew::BN - 1) / GemmFew::BN);
  const int64_t grid = g.ahead[0] ? kGemmGrid : std::min<int64_t>((tiles + 7) & ~7ll, kGemmGrid);
  ProfScope ps_("gemm_bf16_kernel", st);
  LLMC_KERNEL_GGL(kernel, dim3((unsigned)grid), dim3(256), kGemmLdsBytes, st, g);
  LLMC_LAUNCH_CHECK("gemm");
  return LLMC_OK;
}

// K a multiple of 64, N of 8; an activation and a residual exclude each other
static llmc_status_t launch_gemm(const GemmArgs& g, int dtype, hipStream_t st) {
  if (dtype != LLMC_BF16) return launch_gemm_f32(g, st);
  if (g.act == 1) return launch_gemm_bf16<kEpiGeluErf>(g, st);
  if (g.act == 2) return launch_gemm_bf16<kEpiGeluTanh>(g, st);
  if (g.resid) return launch_gemm_bf16<kEpiResidual>(g, st);
  return launch_gemm_bf16<kEpiPlain>(g, st);
}

// ---- LayerNorm: one wavefront per token, two-pass statistics in fp32 -----------------------------
template <typename T, int MAXV>
__global__ __launch_bounds__(256) void layernorm_kernel(const T* __restrict__ in, int ld_in, const int32_t* in_rows,
                                                        T* __restrict__ out, int ld_out, const int32_t* out_rows,
                                                        const T* __restrict__ gamma, const T* __restrict__ beta,
                                                        float eps, int d, int S, const int32_t* count, int max_seqs) {
  constexpr int VEC = Vec16<T>::N;
  const int n_seq = count ? min(*count, max_seqs) : max_seqs;
  const int M = n_seq * S;
  const int lane = threadIdx.x & 63;
  const int nvec = d / VEC;
  for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < M; r += gridDim.x * 4) {
  const T* src = in + map_row(in_rows, r, S) * ld_in;
  float x[MAXV][VEC];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int v = lane + i * 64;
    if (v < nvec) {
      Vec16<T>::load(src + v * VEC, x[i]);
#pragma unroll
      for (int e = 0; e < VEC; ++e) s += x[i][e];
    }
  }
  const float mean = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int v = lane + i * 64;
    if (v < nvec) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float c = x[i][e] - mean;
        q += c * c;
      }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
  T* dst = out + map_row(out_rows, r, S) * ld_out;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int v = lane + i * 64;
    if (v < nvec) {
      float gv[VEC], bv[VEC], y[VEC];
      Vec16<T>::load(gamma + v * VEC, gv);
      Vec16<T>::load(beta + v * VEC, bv);
#pragma unroll
      for (int e = 0; e < VEC; ++e) y[e] = (x[i][e] - mean) * rstd * gv[e] + bv[e];
      Vec16<T>::store(dst + v * VEC, y);
    }
  }
  }
}

// ---- the block's LAST LayerNorm with the next layer's pooling folded in ---------------------------------------
// The output of a post-LayerNorm block is written by this kernel, and the next layer's fingerprint starts by
// summing exactly these rows over the tokens.  A workgroup owns one (sequence, 64-token chunk): its wavefronts
// normalise the chunk's tokens (same arithmetic as layernorm_kernel), store them, and keep the ROUNDED outputs in
// LDS; then the chunk's column sums are formed in the order of the fingerprint's pooling kernel -- token t of the
// chunk belongs to row group t % R, a group's tokens are added in ascending order starting from zero, and the
// groups are added in ascending order -- so the partial sums are the bits that kernel would produce, and the
// sequence is flagged so that the next call does not read its rows again.  grid (chunks, max_seqs).
// Bound: memory at many rows, latency of one workgroup's chain at few.  Two chunks of 768: 12.0 -> 9.1 us (an empty
// launch 2.4) with the tokens' butterflies side by side and the column sums by R x d / 8 threads that read 16 bytes
// (a thread per column read 64 tokens two bytes at a time); 24,576 tokens: 29.2 -> 24.5.
constexpr int kLnPoolThreads = 1024;
constexpr int kLnPoolChunk = 64;             // tokens per pooling chunk: must equal the fingerprint's
constexpr int kLnPoolTokPerWave = kLnPoolChunk / (kLnPoolThreads / 64);

template <typename T, int MAXV>
__global__ __launch_bounds__(kLnPoolThreads) void layernorm_pool_kernel(
    const T* __restrict__ in, int ld_in, T* __restrict__ out, int ld_out, const int32_t* __restrict__ out_rows,
    const T* __restrict__ gamma, const T* __restrict__ beta, float eps, int d, int S, const int32_t* count, int max_seqs,
    float* __restrict__ partial, int n_chunks, int R, uint8_t* __restrict__ pooled_flags) {
  constexpr int VEC = Vec16<T>::N;
  constexpr int TPW = kLnPoolTokPerWave;
  extern __shared__ __attribute__((aligned(16))) unsigned char ln_lds[];
  T* tile = reinterpret_cast<T*>(ln_lds);                 // [kLnPoolChunk][d], the outputs as stored
  const int n_seq = count ? min(*count, max_seqs) : max_seqs;
  const int q = blockIdx.y, chunk = blockIdx.x;
  if (q >= n_seq) return;
  const int seq = out_rows ? out_rows[q] : q;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nvec = d / VEC;
  const int t0 = chunk * kLnPoolChunk, t1 = min(S, t0 + kLnPoolChunk);
  // A wavefront owns TPW consecutive tokens of the chunk; all their rows are requested before the first is reduced, and
  // the tokens' butterflies run side by side.  Lanes beyond the row hold zeros (no branches: they would part the tokens).
  const int tw = t0 + wave * TPW;
  float x[TPW][MAXV][VEC];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    const int t = min(tw + u, S - 1);                     // the block's temporaries are in compact token order
    const T* src = in + ((size_t)q * S + t) * ld_in;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) Vec16<T>::load(src + min(lane + i * 64, nvec - 1) * VEC, x[u][i]);
  }
  float gv[MAXV][VEC], bv[MAXV][VEC];
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int v = min(lane + i * 64, nvec - 1);
    Vec16<T>::load(gamma + v * VEC, gv[i]);
    Vec16<T>::load(beta + v * VEC, bv[i]);
  }
  float mean[TPW], rstd[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
#pragma unroll
      for (int e = 0; e < VEC; ++e) s += lane + i * 64 < nvec ? x[u][i][e] : 0.f;
    mean[u] = s;
  }
  wave_sums(mean);
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    mean[u] /= (float)d;
    float qq = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float c = lane + i * 64 < nvec ? x[u][i][e] - mean[u] : 0.f;
        qq += c * c;
      }
    rstd[u] = qq;
  }
  wave_sums(rstd);
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    rstd[u] = 1.0f / sqrtf(rstd[u] / (float)d + eps);
    const int t = tw + u;
    if (t < t1) {
      T* dst = out + ((size_t)seq * S + t) * ld_out;
      T* keep = tile + (size_t)(t - t0) * d;
#pragma unroll
      for (int i = 0; i < MAXV; ++i) {
        const int v = lane + i * 64;
        if (v < nvec) {
          float y[VEC];
#pragma unroll
          for (int e = 0; e < VEC; ++e) y[e] = (x[u][i][e] - mean[u]) * rstd[u] * gv[i][e] + bv[i][e];
          Vec16<T>::store(dst + v * VEC, y);
          Vec16<T>::store(keep + v * VEC, y);
        }
      }
    }
  }
  __syncthreads();
  // a thread takes the tokens of one row group and VEC columns, 16 bytes a read; then a thread per column adds the groups
  float* red = reinterpret_cast<float*>(tile + (size_t)kLnPoolChunk * d);                // [R][d]
  for (int j = threadIdx.x; j < R * nvec; j += kLnPoolThreads) {
    const int r = j / nvec, c = (j - r * nvec) * VEC;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
#pragma unroll 4
    for (int t = r; t < t1 - t0; t += R) {
      float y[VEC];
      Vec16<T>::load(tile + (size_t)t * d + c, y);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += y[e];
    }
#pragma unroll
    for (int e = 0; e < VEC; e += 4)
      *reinterpret_cast<float4*>(red + (size_t)r * d + c + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
  }
  __syncthreads();
  float* po = partial + ((size_t)seq * n_chunks + chunk) * d;
  for (int c = threadIdx.x; c < d; c += kLnPoolThreads) {
    float total = red[c];
    for (int r = 1; r < R; ++r) total += red[(size_t)r * d + c];
    po[c] = total;
  }
  if (chunk == 0 && threadIdx.x == 0) pooled_flags[seq] = 2;
}

template <typename T>
static llmc_status_t launch_ln(const void* in, const int32_t* in_rows, void* out, const int32_t* out_rows,
                               const void* gamma, const void* beta, float eps, int d, int S, const int32_t* count,
                               int max_seqs, hipStream_t st) {
  constexpr int VEC = Vec16<T>::N;
  const int nvec = d / VEC;
  const unsigned blocks = (unsigned)std::min((max_seqs * S + 3) / 4, 2 * kMaxGrid);
#define LN_CASE(MV)                                                                                     \
  {                                                                                                     \
    ProfScope ps_("layernorm_kernel", st);                                                              \
    LLMC_KERNEL_GGL((layernorm_kernel<T, MV>), dim3(blocks), dim3(256), 0, st, (const T*)in, d,      \
                       in_rows, (T*)out, d, out_rows, (const T*)gamma, (const T*)beta, eps, d, S, count, \
                       max_seqs);                                                                       \
  }
  if (nvec <= 64) LN_CASE(1)
  else if (nvec <= 128) LN_CASE(2)
  else if (nvec <= 256) LN_CASE(4)
  else if (nvec <= 512) LN_CASE(8)
  else return set_error(LLMC_ERR_SHAPE, "LayerNorm width %d too large", d);
#undef LN_CASE
  LLMC_LAUNCH_CHECK("layernorm");
  return LLMC_OK;
}

// the pooling kernel's row groups for this width
template <typename T>
static int ln_pool_groups(int d) { return std::max(1, std::min(8, 1024 / (d / Vec16<T>::N))); }
// the chunk's outputs and a sum per row group and column
template <typename T>
static size_t ln_pool_lds_bytes(int d) { return (size_t)kLnPoolChunk * d * sizeof(T) + (size_t)ln_pool_groups<T>(d) * d * sizeof(float); }
// the fused form needs both in LDS; wider rows take the plain kernel and the next call pools them
template <typename T>
static bool ln_pool_fits(int d) { return (size_t)kLnPoolChunk * d * sizeof(T) <= 128 * 1024 && d / Vec16<T>::N <= 128; }

template <typename T>
static llmc_status_t launch_ln_pool(const void* in, void* out, const int32_t* out_rows, const void* gamma,
                                    const void* beta, float eps, int d, int S, const int32_t* count, int max_seqs,
                                    float* partial, uint8_t* pooled_flags, hipStream_t st) {
  constexpr int VEC = Vec16<T>::N;
  const int nvec = d / VEC;
  const int R = ln_pool_groups<T>(d);
  const int n_chunks = (S + kLnPoolChunk - 1) / kLnPoolChunk;
  const size_t lds = ln_pool_lds_bytes<T>(d);
  dim3 grid(n_chunks, max_seqs);
#define LNP_CASE(MV)                                                                                            \
  {                                                                                                             \
    static std::atomic<bool> lds_set[64];                                                                       \
    LLMC_TRY(ensure_dynamic_lds((const void*)(layernorm_pool_kernel<T, MV>), 160 * 1024, lds_set));             \
    ProfScope ps_("layernorm_kernel", st);                                                                      \
    LLMC_KERNEL_GGL((layernorm_pool_kernel<T, MV>), grid, dim3(kLnPoolThreads), lds, st, (const T*)in, d, (T*)out, \
                    d, out_rows, (const T*)gamma, (const T*)beta, eps, d, S, count, max_seqs, partial, n_chunks, R,  \
                    pooled_flags);                                                                              \
  }
  if (nvec <= 64) LNP_CASE(1)
  else LNP_CASE(2)
#undef LNP_CASE
  LLMC_LAUNCH_CHECK("layernorm_pool");
  return LLMC_OK;
}

// ---- attention (translation units of their own) ------------------------------------------------------
template <typename T>
static llmc_status_t launch_attention(const void* qkv, void* ctx, int S, int d, int n_heads, bool causal,
                                      const int32_t* count, int max_seqs, hipStream_t st) {
  if (sizeof(T) == 2) return launch_attention_bf16(qkv, ctx, S, d, n_heads, causal, count, max_seqs, st);
  return launch_attention_f32(qkv, ctx, S, d, n_heads, causal, count, max_seqs, st);
}

// ---- the block -----------------------------------------------------------------------------------
size_t layer_ws_bytes(const llmc_layer_desc_t* L, int B, int S) {
  const size_t T = (size_t)B * S, e = elem_size(L->dtype);
  return align_up(T * 3 * L->d * e, 256) + 3 * align_up(T * L->d * e, 256) + align_up(T * L->d_ff * e, 256);
}

template <typename T>
static llmc_status_t layer_t(const llmc_layer_desc_t* L, const void* h_in, void* h_out, int B, int S,
                             const int32_t* rows, const int32_t* count, void* ws, hipStream_t st,
                             float* pool_partial, uint8_t* pooled_flags) {
  const int d = L->d, dff = L->d_ff;
  const size_t Tn = (size_t)B * S, e = sizeof(T);
  char* p = (char*)ws;
  void* qkv = p; p += align_up(Tn * 3 * d * e, 256);
  void* ctx = p; p += align_up(Tn * d * e, 256);
  void* t0 = p;  p += align_up(Tn * d * e, 256);
  void* t1 = p;  p += align_up(Tn * d * e, 256);
  void* ff = p;
  const int act = L->gelu == 0 ? 1 : 2;
  GemmArgs g{};
  g.S = S; g.count = count; g.max_seqs = B;
  auto gemm = [&](const void* A, int lda, const int32_t* a_rows, const void* W, const void* bias, int N, int K,
                  int act_, const void* resid, const int32_t* r_rows, void* out, const int32_t* o_rows) {
    GemmArgs a = g;
    a.A = A; a.lda = lda; a.a_rows = a_rows; a.W = W; a.bias = bias; a.N = N; a.K = K; a.act = act_;
    a.resid = resid; a.ldr = N; a.r_rows = r_rows; a.out = out; a.ldo = N; a.o_rows = o_rows;
    return launch_gemm(a, L->dtype, st);
  };
  // Workgroups of the first two products that find no tile read the weights of those that follow: with few rows these are
  // bound by the latency of their weights, which is that of the memory-side cache then and not that of HBM.  Nothing is
  // read where no row is computed, or every workgroup has a tile.  (Stacks of 12 768-wide layers whose weights come from
  // HBM, microseconds: one sequence of 128 tokens 1059 -> 1015, prefix keys with 2 of 16 sequences computed 2930 -> 2842;
  // with the second product too, 4 of 37 sequences of 197 tokens 1168 -> 1131, 24 1024-wide layers with 32 of 256 sequences
  // 6370 -> 6251.)  The fp32 products keep their loads in flight long enough: with it 8 x 128 tokens took 1924 for 1897.
  auto read_ahead = [&](std::initializer_list<std::pair<const void*, size_t>> weights) {
    int i = 0;
    for (const auto& w : weights)
      if (e == 2 && w.second * e < (1ull << 28)) { g.ahead[i] = w.first; g.ahead_bytes[i++] = (uint32_t)(w.second * e); }
    for (; i < 3; ++i) { g.ahead[i] = nullptr; g.ahead_bytes[i] = 0; }
  };
  const std::pair<const void*, size_t> wo = {L->d_wo, (size_t)d * d}, w1 = {L->d_w1, (size_t)d * dff}, w2 = {L->d_w2, (size_t)d * dff};
  if (L->arch == 0) {
    read_ahead({wo, w1, w2});
    LLMC_TRY(gemm(h_in, d, rows, L->d_wqkv, L->d_bqkv, 3 * d, d, 0, nullptr, nullptr, qkv, nullptr));
    LLMC_TRY(launch_attention<T>(qkv, ctx, S, d, L->n_heads, false, count, B, st));
    read_ahead({w1, w2});
    LLMC_TRY(gemm(ctx, d, nullptr, L->d_wo, L->d_bo, d, d, 0, h_in, rows, t0, nullptr));
    read_ahead({});
    LLMC_TRY(launch_ln<T>(t0, nullptr, t1, nullptr, L->d_ln1_g, L->d_ln1_b, L->ln_eps, d, S, count, B, st));
    LLMC_TRY(gemm(t1, d, nullptr, L->d_w1, L->d_b1, dff, d, act, nullptr, nullptr, ff, nullptr));
    LLMC_TRY(gemm(ff, dff, nullptr, L->d_w2, L->d_b2, d, dff, 0, t1, nullptr, t0, nullptr));
    if (pool_partial && pooled_flags && ln_pool_fits<T>(d))
      LLMC_TRY(launch_ln_pool<T>(t0, h_out, rows, L->d_ln2_g, L->d_ln2_b, L->ln_eps, d, S, count, B, pool_partial,
                                 pooled_flags, st));
    else
      LLMC_TRY(launch_ln<T>(t0, nullptr, h_out, rows, L->d_ln2_g, L->d_ln2_b, L->ln_eps, d, S, count, B, st));
  } else {
    LLMC_TRY(launch_ln<T>(h_in, rows, t1, nullptr, L->d_ln1_g, L->d_ln1_b, L->ln_eps, d, S, count, B, st));
    read_ahead({wo, w1, w2});
    LLMC_TRY(gemm(t1, d, nullptr, L->d_wqkv, L->d_bqkv, 3 * d, d, 0, nullptr, nullptr, qkv, nullptr));
    LLMC_TRY(launch_attention<T>(qkv, ctx, S, d, L->n_heads, true, count, B, st));
    read_ahead({w1, w2});
    LLMC_TRY(gemm(ctx, d, nullptr, L->d_wo, L->d_bo, d, d, 0, h_in, rows, t0, nullptr));
    read_ahead({});
    LLMC_TRY(launch_ln<T>(t0, nullptr, t1, nullptr, L->d_ln2_g, L->d_ln2_b, L->ln_eps, d, S, count, B, st));
    LLMC_TRY(gemm(t1, d, nullptr, L->d_w1, L->d_b1, dff, d, act, nullptr, nullptr, ff, nullptr));
    LLMC_TRY(gemm(ff, dff, nullptr, L->d_w2, L->d_b2, d, dff, 0, t0, nullptr, h_out, rows));
  }
  return LLMC_OK;
}

// ---- prefix attention statistics (Section IV-B): MHA over the first tokens of every sequence ----------------------
// out[b][t][:] = in[b][t][:] for t < n_prefix; one workgroup per token row, 16-byte vectors
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void prefix_copy_kernel(const u32x4_t* __restrict__ in, u32x4_t* __restrict__ out,
                                                          int S, int n_prefix, int vec_per_row) {
  const int b = blockIdx.x / n_prefix, t = blockIdx.x % n_prefix;
  const u32x4_t* src = in + ((size_t)b * S + t) * vec_per_row;
  u32x4_t* dst = out + (size_t)blockIdx.x * vec_per_row;
  for (int v = threadIdx.x; v < vec_per_row; v += 256) dst[v] = src[v];
}

size_t prefix_attention_ws_bytes(const llmc_layer_desc_t* L, int B, int n_prefix) {
  const size_t T = (size_t)B * n_prefix, e = elem_size(L->dtype);
  return align_up(T * 3 * L->d * e, 256) + 3 * align_up(T * L->d * e, 256);
}

template <typename T>
static llmc_status_t prefix_attention_t(const llmc_layer_desc_t* L, const void* h, int B, int S, int n_p, void* ws,
                                        float* out, int ld_out, hipStream_t st) {
  const int d = L->d;
  const size_t Tn = (size_t)B * n_p, e = sizeof(T);
  char* p = (char*)ws;
  void* qkv = p; p += align_up(Tn * 3 * d * e, 256);
  void* x = p;   p += align_up(Tn * d * e, 256);
  void* ctx = p; p += align_up(Tn * d * e, 256);
  void* ao = p;
  { ProfScope ps_("prefix_copy_kernel", st);
    LLMC_KERNEL_GGL(prefix_copy_kernel, dim3((unsigned)Tn), dim3(256), 0, st, (const u32x4_t*)h, (u32x4_t*)x, S, n_p,
                    (int)((size_t)d * e / 16)); }
  LLMC_LAUNCH_CHECK("prefix_copy_kernel");
  const void* a_in = x;
  if (L->arch == 1) {       // the pre-LayerNorm block attends over LN1(x)
    LLMC_TRY(launch_ln<T>(x, nullptr, ctx, nullptr, L->d_ln1_g, L->d_ln1_b, L->ln_eps, d, n_p, nullptr, B, st));
    a_in = ctx;
  }
  GemmArgs g{};
  g.S = n_p; g.count = nullptr; g.max_seqs = B; g.act = 0; g.resid = nullptr; g.r_rows = nullptr; g.a_rows = nullptr;
  g.o_rows = nullptr;
  GemmArgs a = g;
  a.A = a_in; a.lda = d; a.W = L->d_wqkv; a.bias = L->d_bqkv; a.N = 3 * d; a.K = d; a.ldr = 3 * d; a.out = qkv; a.ldo = 3 * d;
  LLMC_TRY(launch_gemm(a, L->dtype, st));
  void* ctx2 = L->arch == 1 ? x : ctx;        // LN1's output has been consumed by the projection above
  LLMC_TRY(launch_attention<T>(qkv, ctx2, n_p, d, L->n_heads, L->arch == 1, nullptr, B, st));
  a = g;
  a.A = ctx2; a.lda = d; a.W = L->d_wo; a.bias = L->d_bo; a.N = d; a.K = d; a.ldr = d; a.out = ao; a.ldo = d;
  LLMC_TRY(launch_gemm(a, L->dtype, st));
  // the projections have been consumed: their space takes the chunk sums (at most one fp32 row per 64 tokens).  One
  // workgroup per sequence, without chunk sums, took 18.1 us at 16 x 256 tokens of 768; the two launches take 7.7 + 4.1
  return launch_pool_means(ao, B, n_p, d, L->dtype, qkv, out, ld_out, st);
}

llmc_status_t launch_prefix_attention_mean(const llmc_layer_desc_t* L, const void* d_h, int B, int S, int n_prefix,
                                           void* ws, float* d_out, int ld_out, hipStream_t st) {
  if (L->dtype == LLMC_F32) return prefix_attention_t<float>(L, d_h, B, S, n_prefix, ws, d_out, ld_out, st);
  return prefix_attention_t<bf16_t>(L, d_h, B, S, n_prefix, ws, d_out, ld_out, st);
}

llmc_status_t launch_linear(const void* A, int lda, const int32_t* a_rows, const void* W, const void* bias, int N, int K,
                            void* out, int ldo, const int32_t* o_rows, int S, const int32_t* count, int max_seqs,
                            int dtype, hipStream_t st) {
  GemmArgs a{};
  a.A = A; a.lda = lda; a.a_rows = a_rows; a.W = W; a.bias = bias; a.N = N; a.K = K; a.act = 0;
  a.resid = nullptr; a.ldr = N; a.r_rows = nullptr; a.out = out; a.ldo = ldo; a.o_rows = o_rows;
  a.S = S; a.count = count; a.max_seqs = max_seqs;
  return launch_gemm(a, dtype, st);
}

bool layer_pools_outputs(const llmc_layer_desc_t* L) {
  return L->arch == 0 && (L->dtype == LLMC_F32 ? ln_pool_fits<float>(L->d) : ln_pool_fits<bf16_t>(L->d));
}

llmc_status_t launch_layer(const llmc_layer_desc_t* L, const void* d_h_in, void* d_h_out, int B, int S,
                           const int32_t* d_rows, const int32_t* d_count, void* ws, hipStream_t st,
                           float* pool_partial, uint8_t* pooled_flags) {
  if (L->dtype == LLMC_F32)
    return layer_t<float>(L, d_h_in, d_h_out, B, S, d_rows, d_count, ws, st, pool_partial, pooled_flags);
  return layer_t<bf16_t>(L, d_h_in, d_h_out, B, S, d_rows, d_count, ws, st, pool_partial, pooled_flags);
}

}  // namespace llmc
