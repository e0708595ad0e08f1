// Host-side launchers of libdualparal's kernels.  Every launcher only enqueues work on `st`.
#pragma once
#include <atomic>
#include "common.h"

// ---- elementwise.hip -------------------------------------------------------------------------
template <typename T> void launch_to_f32(const T* in, float* out, int64_t n, hipStream_t st);
template <typename T> void launch_from_f32(const float* in, T* out, int64_t n, hipStream_t st);
// out[s,:] = LayerNorm(x[s,:]) * (mul + plus_one) + add ; x fp32 [S,D], mul/add fp32 [D].
// xin != null: the rows are read from xin ([S,D]) instead, and x receives their fp32 copy.
template <typename T>
void launch_ln_modulate(float* x, const T* xin, T* out, int64_t S, int D, float eps, const float* mul,
                        const float* add, int plus_one, hipStream_t st);

// src[S, ld] holds un-normalised projections; job j takes columns [col, col+D) of every row:
// dst[head][row0 + s][d] = out_scale * RoPE(RMSNorm_D(src[s, col:col+D]) * g) ; rope == 0 skips the rotation.
// Up to two jobs (e.g. q and k of the fused QKV output) run in one launch.  D % 8 == 0.
template <typename T> struct NormRopeJob {
  int col; const float* g; float out_scale; T* dst; int64_t head_stride; int64_t row0; int rope;
};
// v, if given, is transposed by the same launch.
// vt[head][c][col0 + s] = src[s, col + head*d + c]; vec_ok is filled in
template <typename T> struct VTransposeJob { int col; T* vt; int64_t row_stride, col0; int vec_ok; };
template <typename T>
void launch_norm_rope(const T* src, int64_t ld, int64_t S, int h, int d, float eps, const NormRopeJob<T>* jobs,
                      int n_jobs, const RopeTables* rope, int frame0, int tok_h, int tok_w, hipStream_t st,
                      const VTransposeJob<T>* v = nullptr);
// cs[s][i] = rotation (cos, sin) of channel pair i < head_dim / 2 at token s < S of a block that starts at frame0
struct RopeTokens { RopeTables rt; int frame0, tok_h, tok_w; int64_t S; float2* cs; };
// k[head][row0 + s][:] = (wide ? wide[s][head * d ..] : k[head][row0 + s][:]) * rsqrt(sum_i ssq[i * stride + s] / (h * d) + eps),
// bf16 rows of d elements; wide: fp32 [S][h * d]
void launch_scale_rows_bf16(bf16_t* k, int64_t head_stride, int64_t row0, int64_t S, int h, int d, const float* wide,
                            const float* ssq, int np, int64_t stride, float eps, hipStream_t st);
template <typename T>
void launch_v_transpose(const T* src, int64_t ld, int64_t S, int h, int d, const VTransposeJob<T>& v, hipStream_t st);
// dst[r][0..len) = src[r][0..len) for r < rows (strides in elements)
template <typename T>
void launch_copy2d(const T* src, int64_t src_stride, T* dst, int64_t dst_stride, int64_t rows,
                   int64_t len, hipStream_t st);
// out[n, k] = in[k, n] for n < N, zero rows for N <= n < Npad     (in [K, N] row-major)
template <typename T>
void launch_transpose_pad(const T* in, int64_t K, int64_t N, T* out, int64_t Npad, hipStream_t st);

// Timestep-MLP product of act(x) with W [K, N].  The input is the K sinusoidal features of timestep t (x == null, no
// activation) or a sliced vector: x[k] = SiLU(sum over `parts` rows of x[parts][K] + xbias[k]).  Without a table y receives
// the product's own slices [returned count <= GEMV_MAX_SLICES][N], without a bias (its consumer adds them up); with one
// the whole result goes to mod[l, n] = mtab[l, n] + (result + bias)[n] for l < L (y, if given, may serve as scratch).  rope != null (with sinusoidal
// input only): the launch builds that rotation table next to it.
constexpr int GEMV_MAX_SLICES = 8;
struct GemvIn { const float* x; int parts; float t; };
template <typename T> struct GemvTable { const T* bias; const float* mtab; float* mod; int L; };
template <typename T>
int launch_gemv(const GemvIn& in, const T* xbias, int K, const T* W, int N, float* y, const GemvTable<T>* table,
                const RopeTokens* rope, hipStream_t st);
// The first two of a chain: y = slices of SiLU(b1 + W1^T features(t)) times W2 [D, D] (returned count); mid: scratch as y
template <typename T>
int launch_gemv_pair(float t, const T* W1, const T* b1, int freq, const T* W2, int D, float* mid, float* y, const RopeTokens* rope, hipStream_t st);
void launch_rope_table(float2* tab, int n_pos, int pairs, float theta, hipStream_t st);
void launch_fill_zero(void* p, size_t bytes, hipStream_t st);
// dst[s, head*d + c] (fp32) = src[head][row0 + s][c]
template <typename T>
void launch_gather_heads(const T* src, int64_t head_stride, int64_t row0, int64_t S, int h, int d,
                         float* dst, hipStream_t st);
// dst[s, head*d + c] (fp32) = vt[head][c][col0 + s]
template <typename T>
void launch_gather_vt(const T* vt, int64_t row_stride, int64_t col0, int64_t S, int h, int d,
                      float* dst, hipStream_t st);

// ---- gemm_f32.hip : C = A[M,K] * W[K,N] (+ epilogue), all row-major, fp32 MFMA ---------------
// One launch multiplies by w.n matrices of equal shape; with EPI_STORE matrix i's result goes to columns [i * N, (i + 1) * N)
// of e.out (the other epilogues take one).  The biases are w.bias (null: none); e.bias is not looked at.
struct GemmF32W { const float* w[3]; const float* bias[3]; int n; };
void launch_gemm_f32(const float* A, int64_t lda, const GemmF32W& w, int64_t ldw, int64_t M, int64_t N,
                     int64_t K, int epi, const EpiArgs& e, hipStream_t st);
// ---- attn_f32.hip ----------------------------------------------------------------------------
// q [h][*][d], k [h][*][d] rows k_row0.. (L rows), vt [h][d][*] cols k_row0.. ; out[s, head*d + c], row stride ldo.
// k rows and vt columns must be readable from k_row0 & ~3 up to (k_row0 & ~3) + roundup(L + 3, 32); vt, its rows and ldo
// in 16-byte steps.  scratch: scratch_floats floats for the partial results of work that is cut into key ranges
// (0: never cut).
void launch_attn_f32(const float* q, int64_t q_head_stride, const float* k, int64_t k_head_stride,
                     int64_t k_row0, const float* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                     int h, int d, float* out, int64_t ldo, float* scratch, size_t scratch_floats, hipStream_t st);

// out[f, :] = pool[index[f], :], frame_bytes % 16 == 0, all pointers 16-byte aligned
void launch_gather_frames(const void* pool, int pool_frames, int64_t frame_bytes, const int32_t* index,
                          int n_frames, void* out, hipStream_t st);
// Raises a kernel's dynamic-LDS limit once per device and process (the attribute belongs to the device's copy
// of the code object).  `done` is one bit per device ordinal; safe to call from several host threads.
inline void allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return;
  (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  done.fetch_or(bit, std::memory_order_release);
}

// ---- gemm_bf16.hip : C = A[M,K] * Wt[N,K]^T (+ epilogue), bf16 MFMA, fp32 accumulate --------
// A must be readable for roundup(M, 256) rows, Wt for roundup(N, 256) rows; K % 64 == 0.
bool launch_gemm_bf16(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M,
                      int64_t N, int64_t K, int epi, const EpiArgs& e, hipStream_t st);
// the kernel launch_gemm_bf16 takes: block tile, LDS stages, and ranges that K is cut into (EPI_RESID; scratch_floats: what
// e.scratch holds, 0 if there is none)
struct GemmRoute { int bm, bn, stages, parts; };
GemmRoute gemm_bf16_route(int64_t M, int64_t N, int64_t K, int epi, size_t scratch_floats);
// EPI_RESID may cut K into ranges whose partial sums go through e.scratch (a second launch adds them up, in range order);
// what a problem of up to M rows can make use of:
size_t gemm_bf16_scratch_bytes(int64_t M, int64_t N);
// whether launch_gemm_bf16(.., EPI_HEADS, ..) can take this problem; if not it launches nothing and returns false
bool gemm_bf16_heads_ok(int64_t M, int64_t N, const HeadsArgs& h);
// whether it can for sections of `dim` columns and any number of rows from M on: false for M, false for all beyond
bool gemm_bf16_heads_ever(int64_t M, int64_t N, int64_t dim);
// whether its plain sections can be had as fp32 rows (HeadSection::wide)
bool gemm_bf16_heads_wide(int64_t M, int64_t N);
// ---- attn_bf16.hip : flash attention on MFMA, head_dim 64 or 128 ------------------------------
// q must already be multiplied by log2(e)/sqrt(d) (attn_bf16_q_scale) and be readable for
// roundup(S, 256) rows per head; k rows / vt columns readable (finite in vt) up to
// k_row0 + roundup(L, 64).
// scratch: attn_bf16_scratch_bytes(d) bytes of device memory for the partial results of work that is
// split over key ranges (contents need not be kept between calls), or nullptr to never split.
inline float attn_bf16_q_scale(int d) { return 1.4426950408889634f / sqrtf((float)d); }
// Deferred RMSNorm of the queries: row s of q (all heads) is multiplied by
// rsqrt(sum_i ssq[i * stride + s] * inv_dim + eps) * scale as it is loaded (ssq == nullptr: q is used as stored).
struct AttnQNorm { const float* ssq; int np; int64_t stride; float inv_dim, eps, scale; };
// test hook: q[head][s][:] of all heads, token-major fp32, scaled and rounded exactly as the attention kernel does
void launch_gather_heads_qnorm(const bf16_t* src, int64_t head_stride, int64_t S, int h, int d, const AttnQNorm& qn,
                               float* dst, hipStream_t st);
// out[i] = a[i] * b[i]
void launch_mul_f32(const float* a, const float* b, float* out, int64_t n, hipStream_t st);
size_t attn_bf16_scratch_bytes(int d);
void launch_attn_bf16(const bf16_t* q, int64_t q_head_stride, const bf16_t* k, int64_t k_head_stride,
                      int64_t k_row0, const bf16_t* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                      int h, int d, bf16_t* out, int64_t ldo, float* scratch, const AttnQNorm* qnorm, hipStream_t st);
