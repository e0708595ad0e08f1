// The two ends of the denoising model and the scheduler update (Sec. 2: latent x_t in R^{F x H x W x C} ->
// p = F x H' x W' tokens of hidden size h -> prediction in latent shape -> x_{t-1} = S(eps_t, x_t, t)).
// The paper leaves these steps to the base model; this is a Wan-shaped reading:
//   patch embedding : token (f, y, x) = the 1x2x2 patch (f, 2y+dy, 2x+dx, c), ordered (dy, dx, c), times
//                     W_pe [4C, h] plus b_pe
//   output head     : (shift, scale) = m_head[2, h] + e, e the timestep embedding (before the 6h projection);
//                     LayerNorm(x) (1 + scale) + shift, times W_head [h, 4C] plus b_head, scattered to pixels
//   scheduler step  : flow-matching Euler, x += (sigma_next - sigma) v
// Latents and velocities are fp32; tokens are in the stage's storage type.  The GEMMs, LayerNorm and timestep
// MLP are the stage's kernels.
#include <cstdint>
#include <mutex>
#include <new>

#include "../../include/dualparal.h"
#include "kernels.h"

int dp_set_error(int code, const char* msg);   // defined next to dp_last_error

static inline int64_t rup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

struct dp_ends {
  dp_ends_config cfg{};
  dp_ends_weights w{};
  int64_t tok, Smax, Spad, P;                  // P = 4 * channels values per token
  void *patches, *h, *w_pe_t, *w_pe_f, *w_head_t;   // storage type; w_pe_f: in the order of k_embed's fragments
  float *x32, *out32, *e1, *e, *mhead, *mod;
};

// token s, value r = (dy*2 + dx)*C + c  <->  latent element ((f*H + 2y+dy)*W + 2x+dx)*C + c
__device__ __forceinline__ int64_t patch_elem(uint32_t s, int r_, int tok_, int tw_, int C_) {   // at most 2^24 tokens
  const uint32_t r = r_, tok = tok_, tw = tw_, C = C_;
  const uint32_t f = s / tok, rem = s % tok, y = rem / tw, x = rem % tw;
  const uint32_t dy = r / (2 * C), dx = (r / C) & 1, c = r % C;
  const int64_t H = 2 * (tok / tw), W = 2 * tw;
  return ((f * H + 2 * y + dy) * W + 2 * x + dx) * C + c;
}
template <typename T>
__global__ void k_patchify(const float* __restrict__ latent, T* __restrict__ out, int64_t n, int P, int tok,
                           int tw, int C) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) Elem<T>::st(out + i, latent[patch_elem(i / P, (int)(i % P), tok, tw, C)]);
}
__global__ void k_unpatchify(const float* __restrict__ in, float* __restrict__ latent, int64_t n, int P, int tok,
                             int tw, int C) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) latent[patch_elem(i / P, (int)(i % P), tok, tw, C)] = in[i];
}
__global__ void k_euler(float* __restrict__ x, const float* __restrict__ v, int64_t n, float ds) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) x[i] = x[i] + ds * v[i];
}

// ------------------------------------------------------------------------------------------ bf16 ends in one kernel each
// Both ends are contractions with one narrow side (4C values per token), so they are bound by one pass over the tokens;
// as patchify + GEMM and as conversion + LayerNorm + GEMM + scatter they made three and six passes of it.
// v_mfma_f32_16x16x32_bf16 with the weights as the A operand: lane l supplies / receives token l % 16, k (8 of them) or
// output quad l / 16.  The weights are packed once in the order of the fragments, so a fragment is 1 KiB read in one piece.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk(float a, float b) {
  f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
constexpr int kEndsMaxP = 256;                       // widest narrow side that stays in registers; beyond it: the GEMMs
// fragment (chunk, tile) lane l, element e <- W[k = 32 chunk + 8 (l / 16) + e][n], W row-major [K, N], with
// n = 16 tile + l % 16 (quad = 0), or (quad = 1) n = 64 (tile / 4) + 16 (l % 16 / 4) + 4 (tile % 4) + l % 4: the four
// tiles of a 64-column group then leave 16 consecutive columns in one lane
__global__ __launch_bounds__(256) void k_pack_frags(const bf16_t* __restrict__ W, int K, int N, int quad, uint4* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)(K / 32) * (N / 16) * 64) return;
  const int l = (int)(i & 63), tile = (int)((i >> 6) % (N / 16)), chunk = (int)((i >> 6) / (N / 16)), r = l & 15;
  const int n = quad ? 64 * (tile >> 2) + 16 * (r >> 2) + 4 * (tile & 3) + (r & 3) : 16 * tile + r;
  const bf16_t* src = W + (int64_t)(32 * chunk + 8 * (l >> 4)) * N + n;
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = (uint32_t)src[(int64_t)(2 * e) * N] | (uint32_t)src[(int64_t)(2 * e + 1) * N] << 16;
  out[i] = make_uint4(w[0], w[1], w[2], w[3]);
}
static void launch_pack_frags(const bf16_t* W, int64_t K, int64_t N, int quad, void* out, hipStream_t st) {
  k_pack_frags<<<(unsigned)((K * N / 8 + 255) / 256), 256, 0, st>>>(W, (int)K, (int)N, quad, (uint4*)out);
}

// Patch embedding.  A wavefront holds 16 tokens' patches (read from the fp32 latent, rounded to bf16) as operands and walks
// 64-column groups of the output; a lane ends up with 16 consecutive columns of its token.  6240 tokens x 64 -> 1536:
// 12.2 us in two launches -> 9.6 us (21 MB, of which a launch alone is 4.6); 14400 x 64 -> 5120: 50 -> 39 us (3.9 TB/s).
// 16-byte stores of 16 different rows an instruction instead of the staged ones: 52 us.
template <int KC>                                    // 32-value chunks of a patch
__global__ __launch_bounds__(256) void k_embed(const float* __restrict__ latent, const uint4* __restrict__ wf,
                                               const bf16_t* __restrict__ bias, bf16_t* __restrict__ out, int64_t S, int D,
                                               int tok, int tw, int C, int aligned) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4;
  const int64_t s = (int64_t)blockIdx.x * 16 + (lane & 15), sc = s < S ? s : S - 1;
  __shared__ uint4 stage[4][16][9];
  const int tiles = D >> 4, step = gridDim.y * 4;
  int g = blockIdx.y * 4 + wave;
  uint4 w[KC][4];
  auto fetch = [&](int grp) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int t = 0; t < 4; ++t) w[c][t] = wf[((int64_t)c * tiles + grp * 4 + t) * 64 + lane];
  };
  if (g * 64 < D) fetch(g);
  bf16x8 x[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const float* p = latent + patch_elem(sc, c * 32 + q * 8, tok, tw, C);      // 8 values of one pixel: C % 16 == 0
    float v[8];
    if (aligned) { *(float4*)v = *(const float4*)p; *(float4*)(v + 4) = *(const float4*)(p + 4); }
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p[e];
    }
    uint32_t u[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) u[e] = cvt_pk(v[2 * e], v[2 * e + 1]);
    x[c] = __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
  }
  for (; g * 64 < D; g += step) {
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint2 b = *(const uint2*)(bias + g * 64 + q * 16 + t * 4);
      acc[t] = f32x4{bf16_to_f32((bf16_t)(b.x & 0xffff)), bf16_to_f32((bf16_t)(b.x >> 16)),
                     bf16_to_f32((bf16_t)(b.y & 0xffff)), bf16_to_f32((bf16_t)(b.y >> 16))};
    }
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[c][t]), x[c], acc[t], 0, 0, 0);
    if ((g + step) * 64 < D) fetch(g + step);
    // through LDS (the wavefront's own 16 x 64 tile: no barrier), so that a store covers whole 128-byte pieces of rows
    uint4* o = &stage[wave][lane & 15][q * 2];
    o[0] = make_uint4(cvt_pk(acc[0][0], acc[0][1]), cvt_pk(acc[0][2], acc[0][3]), cvt_pk(acc[1][0], acc[1][1]), cvt_pk(acc[1][2], acc[1][3]));
    o[1] = make_uint4(cvt_pk(acc[2][0], acc[2][1]), cvt_pk(acc[2][2], acc[2][3]), cvt_pk(acc[3][0], acc[3][1]), cvt_pk(acc[3][2], acc[3][3]));
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int tk = i * 8 + (lane >> 3);
      const uint4 d = stage[wave][tk][lane & 7];
      const int64_t row = (int64_t)blockIdx.x * 16 + tk;
      if (row < S) __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)(out + row * D + g * 64 + (lane & 7) * 8));
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Output head: LayerNorm (two-pass statistics in fp32) -> (1 + scale), shift -> bf16 -> times W_head -> scatter.  A block of 8
// wavefronts owns RT * 16 tokens; wavefront w holds the 64-channel groups w, w + 8, .. of their rows in registers, in operand
// layout, so a row is read once.  The wavefronts' partial products over their channels meet in LDS, summed in wavefront
// order.  blockIdx.y: 64 of the 4C output values.  14400 tokens x 5120: 237 us in six launches -> 57 us (147 MB).
template <int NG, int RT>
__global__ __launch_bounds__(512, 2) void k_head(const bf16_t* __restrict__ x, int64_t S, int D, float eps,
                                                 const float* __restrict__ scale, const float* __restrict__ shift,
                                                 const uint4* __restrict__ wf, const bf16_t* __restrict__ bias, int P,
                                                 float* __restrict__ v_out, int tok, int tw, int C, int x_aligned, int v_aligned) {
  __shared__ float red[2][RT][8][16];
  __shared__ __align__(16) float part[8][RT * 16][68];            // [wavefront][token][64 values, padded]
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, lt = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t s0 = (int64_t)blockIdx.x * (RT * 16);
  const int groups = D >> 6;
  u32x4 xr[NG][RT][2];
  float sum[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int64_t s = s0 + t * 16 + lt;
    const bf16_t* p = x + (s < S ? s : S - 1) * D + wave * 64 + q * 8;
    if (x_aligned) {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          xr[g][t][c] = wave + 8 * g < groups ? *(const u32x4*)(p + g * 512 + c * 32) : u32x4{0, 0, 0, 0};
    } else {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bf16_t* pe = p + g * 512 + c * 32 + 2 * e;
            xr[g][t][c][e] = wave + 8 * g < groups ? pe[0] | (uint32_t)pe[1] << 16 : 0u;
          }
    }
  }
  // keeps the packed values, and nothing unpacked from them, in registers from one pass over the row to the next
  auto repack = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) asm volatile("" : "+v"(xr[g][t][c]));
  };
  auto elem = [&](int g, int t, int c, int e) __attribute__((always_inline)) {
    const uint32_t w = xr[g][t][c][e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  };
  // sum over a token's channels: the lane's own, the other three lanes of the token, the 8 wavefronts in order
  auto token_sum = [&](float (&v)[RT], int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      v[t] += __shfl_xor(v[t], 16, 64);
      v[t] += __shfl_xor(v[t], 32, 64);
      if (q == 0) red[slot][t][wave][lt] = v[t];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      v[t] = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) v[t] += red[slot][t][w][lt];
    }
  };
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    sum[t] = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        float p = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) p += elem(g, t, c, e);
        sum[t] += p;
      }
  }
  token_sum(sum, 0);
  repack();
  float mean[RT], rstd[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    mean[t] = sum[t] / (float)D;
    sum[t] = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      if (wave + 8 * g < groups) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          float p = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) { const float d = elem(g, t, c, e) - mean[t]; p += d * d; }
          sum[t] += p;
        }
      }
  }
  token_sum(sum, 1);
  repack();
#pragma unroll
  for (int t = 0; t < RT; ++t) rstd[t] = rsqrtf(sum[t] / (float)D + eps);

  f32x4 acc[RT][4];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int ptiles = P >> 4;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (wave + 8 * g < groups) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k0 = (wave + 8 * g) * 64 + c * 32, kl = k0 + q * 8;
        uint4 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = wf[((int64_t)(k0 >> 5) * ptiles + blockIdx.y * 4 + j) * 64 + lane];
        float m[8], a[8];
        *(float4*)m = *(const float4*)(scale + kl); *(float4*)(m + 4) = *(const float4*)(scale + kl + 4);
        *(float4*)a = *(const float4*)(shift + kl); *(float4*)(a + 4) = *(const float4*)(shift + kl + 4);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          uint32_t h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            h[e] = cvt_pk((elem(g, t, c, 2 * e) - mean[t]) * rstd[t] * (m[2 * e] + 1.f) + a[2 * e],
                          (elem(g, t, c, 2 * e + 1) - mean[t]) * rstd[t] * (m[2 * e + 1] + 1.f) + a[2 * e + 1]);
          const bf16x8 hv = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j]), hv, acc[t][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);           // without it the loads of all groups move up and spill
      }
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) *(f32x4*)&part[wave][t * 16 + lt][j * 16 + q * 4] = acc[t][j];
  __syncthreads();
  for (int i = tid; i < RT * 16 * 16; i += 512) {    // four values of one token each
    const int tk = i >> 4, r = (i & 15) * 4, p = blockIdx.y * 64 + r;
    if (s0 + tk >= S) continue;
    f32x4 v = *(const f32x4*)&part[0][tk][r];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += *(const f32x4*)&part[w][tk][r];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += bf16_to_f32(bias[p + e]);
    float* o = v_out + patch_elem(s0 + tk, p, tok, tw, C);          // consecutive channels of one pixel: C % 16 == 0
    if (v_aligned) *(f32x4*)o = v;
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = v[e];
    }
  }
}

// The output head where the modulation is not worth a product of its own (see head_streamed): the modulation moves into the
// weights, W' = (1 + scale) W, rounded to bf16 once per call, and the statistics out of the product:
//   out = rstd (x W' - mean sum_k W') + sum_k shift W + b
// so the tokens stream through the MFMAs as they are, unrounded, and a row need not be held until its mean is known.
// k_head_fold: W' in fragment order, and each 64 channels' share of the two sums over k (of W' as rounded, so that the mean
// cancels) to pc[D / 64][2][P].
__global__ __launch_bounds__(256) void k_head_fold(const float* __restrict__ e, int parts, const bf16_t* __restrict__ ebias,
                                                   const float* __restrict__ mhead, int D, const uint4* __restrict__ wf, int P,
                                                   uint4* __restrict__ wm, float* __restrict__ pc) {
  __shared__ float mul[64], add[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k0 = blockIdx.x * 64;
  if (tid < 64) {
    float v = bf16_to_f32(ebias[k0 + tid]);
    for (int i = 0; i < parts; ++i) v += e[(int64_t)i * D + k0 + tid];
    add[tid] = mhead[k0 + tid] + v;
    mul[tid] = 1.f + (mhead[D + k0 + tid] + v);
  }
  __syncthreads();
  const int ptiles = P >> 4;
  for (int tile = wave; tile < ptiles; tile += 4) {
    float c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int64_t at = ((int64_t)(blockIdx.x * 2 + c) * ptiles + tile) * 64 + lane;
      const uint4 w4 = wf[at];
      const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
      uint32_t r[4];
      const int kl = c * 32 + (lane >> 4) * 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = __uint_as_float(w[i] << 16), b = __uint_as_float(w[i] & 0xffff0000u);
        c2 += add[kl + 2 * i] * a; c2 += add[kl + 2 * i + 1] * b;
        r[i] = cvt_pk(mul[kl + 2 * i] * a, mul[kl + 2 * i + 1] * b);
        c1 += __uint_as_float(r[i] << 16); c1 += __uint_as_float(r[i] & 0xffff0000u);
      }
      wm[at] = make_uint4(r[0], r[1], r[2], r[3]);
    }
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) { c1 += __shfl_xor(c1, o, 64); c2 += __shfl_xor(c2, o, 64); }
    if (lane < 16) {
      pc[((int64_t)blockIdx.x * 2 + 0) * P + tile * 16 + lane] = c1;
      pc[((int64_t)blockIdx.x * 2 + 1) * P + tile * 16 + lane] = c2;
    }
  }
}
// A block of 8 wavefronts owns TB = TG * RT * 16 tokens.  The channels are dealt in slots of 32 to eight shares (slot n to share
// n % 8), and KH = 8 / TG wavefronts walk them for the same tokens: wavefront w has RT * 16 tokens and the shares w / TG + KH z, z <
// TG (slot i * KH + w / TG in step i), in a ring of NS stages in LDS: its tokens' values, in operand order, and a TG-th of the
// slot's weights, which TG wavefronts read; NS - 1 steps are in flight, waited for by count.  Every share has its own accumulators
// and statistics, which are joined in one order (k and k + 4 first), so that a token's result does not depend on TG, and so not on how
// many tokens the call has.  (Into registers the compiler waits for all loads in flight at every branch.)  A step's
// operands are read from LDS while the step before is multiplied and added up.  Statistics: a lane sums its values' distances
// from the mean of its first eight, and their squares, so what cancels in the variance is no larger than the token's own
// spread; the lanes of a token meet in LDS by their own means.  blockIdx.y: 64 of the 4C output values.
// What bounds it: one pass over the tokens at 14400 x 5120 (147 MB in 28.6 us, 5.1 TB/s; k_head 57, which holds a block's rows in
// registers and so loads and computes in turn); with fewer tokens the 40 to 160 steps of a block, latency each.  Reading the
// operands of a step behind its own barrier: 54 instead of 53 us for the call; asking for all weights ahead: 56.
template <int TG, int RT, int NS>
__global__ __launch_bounds__(512, 2) void k_head_stream(const bf16_t* __restrict__ x, int64_t S, int D, float eps,
                                                 const uint4* __restrict__ wm, const float* __restrict__ pc,
                                                 const bf16_t* __restrict__ bias, int P4, float* __restrict__ v_out, int tok, int tw,
                                                 int C, int v_aligned) {
  constexpr int KH = 8 / TG, TB = TG * RT * 16, P = NS - 1;        // wavefronts that share tokens, tokens, steps in flight
  constexpr int NW = 4 / TG, NL = NW + RT;             // weight fragments and loads per wavefront and step
  constexpr int STAGE = (KH * 4 + 8 * RT) * 64;        // 16-byte chunks: the slots' weights, the wavefronts' tokens
  static_assert((TG == 1 || TG == 2) && NS * STAGE * 16 >= KH * TB * 68 * 4, "the partial products fit the ring");
  __shared__ __align__(16) uint4 ring[NS * STAGE];     // afterwards the partial products
  __shared__ float2 stat[8 * 4][TB];                   // [share, lane quarter][token]: mean, sum of squares about it
  __shared__ float cs[4][128], tm[TB], tr[TB];
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, lt = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), tg = wave % TG, kh = wave / TG;
  const int64_t s0 = (int64_t)blockIdx.x * TB;
  const int chunks = D >> 5, ptiles = P4 >> 4, steps = (chunks + KH - 1) / KH;
  const bf16_t* const xb = x + s0 * D;
  const int rows = (int)(S - s0 < TB ? S - s0 : TB);
  uint32_t xo[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int r = (tg * RT + t) * 16 + lt;
    xo[t] = (uint32_t)((r < rows ? r : rows - 1) * D + q * 8) * 2;
  }
  uint4* const wst = ring + kh * 256;                  // of stage 0: this slot's weights, this wavefront's tokens
  uint4* const xst = ring + KH * 256 + wave * RT * 64;
  auto load = [&](int i, int st) __attribute__((always_inline)) {
    const int c = i * KH + kh < chunks ? i * KH + kh : chunks - 1;      // past the end the last one is loaded, and not used
#pragma unroll
    for (int f = 0; f < NW; ++f)
      __builtin_amdgcn_global_load_lds((glb_void_t*)(wm + ((int64_t)c * ptiles + blockIdx.y * 4 + tg * NW + f) * 64 + lane), (lds_void_t*)(wst + st * STAGE + (tg * NW + f) * 64), 16, 0, 0);
#pragma unroll
    for (int t = 0; t < RT; ++t)
      __builtin_amdgcn_global_load_lds((glb_void_t*)((const char*)(xb + c * 32) + xo[t]), (lds_void_t*)(xst + st * STAGE + t * 64), 16, 0, 0);
  };
  const uint32_t wl = (uint32_t)(uintptr_t)(lds_void_t*)wst + (uint32_t)lane * 16, xl = (uint32_t)(uintptr_t)(lds_void_t*)xst + (uint32_t)lane * 16;
  f32x4 acc[TG][RT][4];
  float sh[TG][RT], sd[TG][RT], sq[TG][RT];
#pragma unroll
  for (int z = 0; z < TG; ++z)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      sh[z][t] = sd[z][t] = sq[z][t] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[z][t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  u32x4 xr[2][RT], w[2][4];
  auto read = [&](int st, auto b_) __attribute__((always_inline)) {
    constexpr int b = decltype(b_)::value;
    const uint32_t o = (uint32_t)st * STAGE * 16;
    static_for<RT>([&](auto t_) __attribute__((always_inline)) { constexpr int t = decltype(t_)::value; xr[b][t] = lds_read16_raw<t * 1024>(xl + o); });
    static_for<4>([&](auto j_) __attribute__((always_inline)) { constexpr int j = decltype(j_)::value; w[b][j] = lds_read16_raw<j * 1024>(wl + o); });
  };
  auto elem = [&](const u32x4& v, int i) __attribute__((always_inline)) { return __uint_as_float((i & 1) ? (v[i >> 1] & 0xffff0000u) : (v[i >> 1] << 16)); };
  auto add = [&](int i, auto b_) __attribute__((always_inline)) {
    constexpr int b = decltype(b_)::value, z = b % TG;                // b: parity of i
    if (i < TG) {
#pragma unroll
      for (int t = 0; t < RT; ++t) {
#pragma unroll
        for (int k = 0; k < 8; ++k) sh[z][t] += elem(xr[b][t], k);
        sh[z][t] *= 0.125f;
      }
    }
    if (i * KH + kh >= chunks) return;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[z][t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[b][j]), __builtin_bit_cast(bf16x8, xr[b][t]), acc[z][t][j], 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float d = elem(xr[b][t], k) - sh[z][t];
        sd[z][t] += d;
        sq[z][t] += d * d;
      }
    }
  };
#pragma unroll
  for (int z = 0; z < P; ++z) load(z, z);
  int st = 0;
  for (int i0 = 0; i0 < steps + 1; i0 += 2) {
    static_for<2>([&](auto u_) __attribute__((always_inline)) {
      constexpr int u = decltype(u_)::value;
      const int i = i0 + u;
      __builtin_amdgcn_sched_barrier(0);
      if (i < steps) {
        vm_wait<(P - 1) * NL>();                       // this step's loads have landed
        __builtin_amdgcn_s_barrier();                  // everyone's have, and the stage of the step before is free
        __builtin_amdgcn_sched_barrier(0);
        load(i + P, st == 0 ? NS - 1 : st - 1);
        read(st, u_);
        __builtin_amdgcn_sched_barrier(0);
        st = st + 1 == NS ? 0 : st + 1;
      }
      if (i > 0 && i <= steps) add(i - 1, std::integral_constant<int, u ^ 1>{});
      __builtin_amdgcn_sched_barrier(0);
      lds_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  // values of share k that a lane has had
  auto share = [&](int k) __attribute__((always_inline)) { return (float)(8 * ((chunks - k + 7) / 8)); };
  tile_barrier();                                      // nothing is in flight, everyone is done with the ring
  float (*const part)[TB][68] = (float (*)[TB][68])ring;           // [wavefront of the token][token][64 values, padded]
  {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int tk = (tg * RT + t) * 16 + lt;
#pragma unroll
      for (int z = 0; z < TG; ++z) {
        const float m = sd[z][t] / share(z * KH + kh);
        stat[(z * KH + kh) * 4 + q][tk] = make_float2(sh[z][t] + m, sq[z][t] - sd[z][t] * m);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) *(f32x4*)&part[kh][tk][j * 16 + q * 4] = TG == 1 ? acc[0][t][j] : acc[0][t][j] + acc[TG - 1][t][j];
    }
    // this block's 64 columns of both sums over k: four shares of the channels
    float c = 0.f;
    const float* pp = pc + (int64_t)((tid >> 6) & 1) * P4 + blockIdx.y * 64 + (tid & 63);
#pragma unroll 4
    for (int i = tid >> 7; i < D >> 6; i += 4) c += pp[(int64_t)i * 2 * P4];
    cs[tid >> 7][tid & 127] = c;
  }
  __syncthreads();
  if (tid < TB) {
    float m = 0.f, v = 0.f;
    for (int k = 0; k < 8; ++k) {
      const float cnt = share(k);
      for (int i = 0; i < 4; ++i) m += stat[k * 4 + i][tid].x * cnt;
    }
    m /= (float)D;
    for (int k = 0; k < 8; ++k) {
      const float cnt = share(k);
      for (int i = 0; i < 4; ++i) {
        const float2 a = stat[k * 4 + i][tid];
        v += a.y + cnt * (a.x - m) * (a.x - m);
      }
    }
    tm[tid] = m;
    tr[tid] = rsqrtf(v / (float)D + eps);
  }
  __syncthreads();
  for (int i = tid; i < TB * 16; i += 512) {           // four values of one token each
    const int tk = i >> 4, r = (i & 15) * 4, o0 = blockIdx.y * 64 + r;
    if (s0 + tk >= S) continue;
    auto pair = [&](int k) __attribute__((always_inline)) {
      return TG == 1 ? *(const f32x4*)&part[k][tk][r] + *(const f32x4*)&part[KH - 4 + k][tk][r] : *(const f32x4*)&part[k][tk][r];
    };
    f32x4 v = pair(0);
#pragma unroll
    for (int k = 1; k < 4; ++k) v += pair(k);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float c1 = cs[0][r + k] + cs[1][r + k] + cs[2][r + k] + cs[3][r + k];
      const float c2 = cs[0][64 + r + k] + cs[1][64 + r + k] + cs[2][64 + r + k] + cs[3][64 + r + k];
      v[k] = tr[tk] * (v[k] - tm[tk] * c1) + c2 + bf16_to_f32(bias[o0 + k]);
    }
    float* o = v_out + patch_elem(s0 + tk, o0, tok, tw, C);         // consecutive channels of one pixel: C % 16 == 0
    if (v_aligned) *(f32x4*)o = v;
    else {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = v[k];
    }
  }
}

static const char* validate(const dp_ends_config* c) {
  if (!c) return "null config";
  if (c->dim < 1 || c->tok_h < 1 || c->tok_w < 1 || c->channels < 1 || c->max_frames < 1) return "non-positive size";
  if (c->dtype != DP_F32 && c->dtype != DP_BF16) return "dtype must be DP_F32 or DP_BF16";
  if (c->freq_dim < 2 || (c->freq_dim & 1)) return "freq_dim must be even";
  if (!(c->eps >= 0.f)) return "bad eps";
  if (c->dim % 8 || c->dim > 8192) return "dim must be a multiple of 8 and at most 8192";
  // upper limits far beyond any model, so that no size below can overflow
  if (c->channels > (1 << 16) || c->freq_dim > (1 << 16) || (int64_t)c->tok_h * c->tok_w > (1 << 24) ||
      (int64_t)c->tok_h * c->tok_w * c->max_frames > (1 << 24))
    return "channels / freq_dim beyond 2^16 or more than 2^24 tokens";
  if (c->dtype == DP_BF16 && (c->dim % 64 || (4 * c->channels) % 64)) return "bf16 path needs dim and 4*channels % 64 == 0";
  return nullptr;
}

// The one-kernel forms: bf16, at most 256 values per token (they stay in registers; wider ones re-read the tokens once per 64
// values), and for the head rows of at most 5120 channels (10 groups of 64 per wavefront: 160 registers).
// k_embed reads all weights once per 16 tokens, 4C / 16 times the bytes it stores.  With 4C = 64, or weights of at most
// 384 KB (512 KB with 4C = 128), that stays below the separate patchify pass and GEMM; beyond, only while the tokens are
// few.  One kernel / patchify + GEMM in us: 4C = 64: 1560 x 5120 9.0 / 11.0, 14400 x 5120 38.0 / 48.4; 4C = 128: 6240 x 2048
// 16.2 / 15.9 (that and 6240 x 1536 are behind by 2 %, no other), 18720 x 2048 32.2 / 38.3, 1560 x 4096 9.8 / 10.9, 6240 x 5120
// 30.5 / 27.5; 4C = 256: 18720 x 768 28.7 / 34.7, 780 x 5120 10.3 / 11.8, 1560 x 3072 12.6 / 12.3, 14400 x 5120 100.7 / 82.6.
static bool embed_frags(const dp_ends_config& c) { return c.dtype == DP_BF16 && 4 * c.channels <= kEndsMaxP; }
static bool embed_gemm(const dp_ends_config& c) {
  return !embed_frags(c) || (c.channels > 16 && (int64_t)c.dim * 4 * c.channels > ((c.channels == 32 ? 256 : 192) << 10));
}
static bool embed_fused(const dp_ends_config& c, int64_t S) {
  return embed_frags(c) && (!embed_gemm(c) || S * c.dim * 4 * c.channels <= ((int64_t)1 << 30));
}
static bool head_fused(const dp_ends_config& c) { return embed_frags(c) && c.dim <= 5120; }
// k_head_stream: where the timestep product is added up by a launch of its own in any case (launch_gemv: more than 2048 rows),
// whose place k_head_fold takes, and both sets of fragments fit the repacked head matrix, whose rows are padded to 256.
static bool head_streamed(const dp_ends_config& c) { return head_fused(c) && c.dim > 2048 && c.channels <= 32; }

static size_t carve(dp_ends* s, void* base) {
  const dp_ends_config& c = s->cfg;
  const int64_t E = c.dtype == DP_BF16 ? 2 : 4, D = c.dim;
  s->tok = (int64_t)c.tok_h * c.tok_w;
  s->Smax = s->tok * c.max_frames;
  s->Spad = rup(s->Smax, 256);
  s->P = 4 * (int64_t)c.channels;
  char* b = (char*)base; size_t off = 0;
  auto take = [&](size_t bytes) { off = (size_t)rup((int64_t)off, 256); void* p = b ? b + off : nullptr; off += bytes; return p; };
  // the one-kernel forms need none of this but a copy of an input that their output overlaps (head: h, embedding: out32)
  s->patches = embed_gemm(c) ? take(s->Spad * s->P * E) : nullptr;
  s->h = take(s->Spad * D * E);
  s->x32 = head_fused(c) ? nullptr : (float*)take(s->Spad * D * 4);
  s->out32 = (float*)take(s->Spad * s->P * 4);
  s->w_pe_t = embed_gemm(c) ? take(rup(D, 256) * s->P * E) : nullptr;
  s->w_pe_f = embed_frags(c) ? take(D * s->P * E) : nullptr;
  s->w_head_t = take(rup(s->P, 256) * D * E);
  s->e1 = (float*)take(GEMV_MAX_SLICES * D * 4); s->e = (float*)take(GEMV_MAX_SLICES * D * 4);   // sliced vectors
  s->mhead = (float*)take(2 * D * 4); s->mod = (float*)take(2 * D * 4);
  return (size_t)rup((int64_t)off, 256);
}

static void pack_head(dp_ends* s, hipStream_t st) {
  const bf16_t* w = (const bf16_t*)s->w.w_head;
  if (head_fused(s->cfg)) launch_pack_frags(w, s->cfg.dim, s->P, 0, s->w_head_t, st);
  else launch_transpose_pad<bf16_t>(w, s->cfg.dim, s->P, (bf16_t*)s->w_head_t, rup(s->P, 256), st);
}

extern "C" size_t dp_ends_workspace_bytes(const dp_ends_config* cfg) {
  const char* why = validate(cfg);
  if (why) { dp_set_error(DP_EINVAL, why); return 0; }
  dp_ends tmp; tmp.cfg = *cfg;
  return carve(&tmp, nullptr);
}

extern "C" int dp_ends_init(const dp_ends_config* cfg, const dp_ends_weights* w, void* workspace,
                            size_t workspace_bytes, void* hip_stream, dp_ends_t** out) {
  if (!out) return dp_set_error(DP_EINVAL, "dp_ends_init: out is null");
  *out = nullptr;
  const char* why = validate(cfg);
  if (why) return dp_set_error(DP_EINVAL, why);
  if (!w || !workspace) return dp_set_error(DP_EINVAL, "dp_ends_init: null pointer");
  const void* const* p = (const void* const*)w;
  for (size_t i = 0; i < sizeof(dp_ends_weights) / sizeof(void*); ++i)
    if (!p[i]) return dp_set_error(DP_EINVAL, "dp_ends_init: null weight pointer");
  if (((uintptr_t)workspace) % 256) return dp_set_error(DP_EINVAL, "dp_ends_init: workspace must be 256-byte aligned");
  dp_ends* s = new (std::nothrow) dp_ends();
  if (!s) return dp_set_error(DP_ENOMEM, "dp_ends_init: out of host memory");
  s->cfg = *cfg; s->w = *w;
  if (carve(s, nullptr) > workspace_bytes) { delete s; return dp_set_error(DP_ENOMEM, "dp_ends_init: workspace too small"); }
  carve(s, workspace);
  hipStream_t st = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  const int64_t D = cfg->dim;
  // padding rows of the GEMM operands; k_embed and k_head read no such rows
  if (embed_gemm(*cfg)) launch_fill_zero(s->patches, (size_t)(s->Spad * s->P) * (cfg->dtype == DP_BF16 ? 2 : 4), st);
  if (!head_fused(*cfg)) launch_fill_zero(s->h, (size_t)((char*)s->e1 - (char*)s->h), st);
  if (cfg->dtype == DP_BF16) {
    if (embed_frags(*cfg)) launch_pack_frags((const bf16_t*)w->w_pe, s->P, D, 1, s->w_pe_f, st);
    if (embed_gemm(*cfg)) launch_transpose_pad<bf16_t>((const bf16_t*)w->w_pe, s->P, D, (bf16_t*)s->w_pe_t, rup(D, 256), st);
    pack_head(s, st);
    launch_to_f32<bf16_t>((const bf16_t*)w->m_head, s->mhead, 2 * D, st);
  } else {
    launch_to_f32<float>((const float*)w->m_head, s->mhead, 2 * D, st);
  }
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) { delete s; return dp_set_error(DP_EHIP, "dp_ends_init: a launch failed"); }
  *out = s;
  return DP_OK;
}

extern "C" void dp_ends_free(dp_ends_t* ends) { delete ends; }

template <typename T>
static void gemm(dp_ends* s, const void* A, int64_t lda, const void* W, const void* wt, int64_t M, int64_t N, int64_t K,
                 int epi, const EpiArgs& e, hipStream_t st) {
  if constexpr (sizeof(T) == 2) launch_gemm_bf16((const bf16_t*)A, lda, (const bf16_t*)wt, K, M, N, K, epi, e, st);
  else launch_gemm_f32((const float*)A, lda, GemmF32W{{(const float*)W}, {(const float*)e.bias}, 1}, N, M, N, K, epi, e, st);
  (void)s;
}

// Both one-kernel forms store results while other blocks still load their input.  The entry points take an output that shares
// memory with its input, so such a call's input is copied into scratch first (the general paths read all of it before
// they store anything).
static bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
  return pa < pb + b_bytes && pb < pa + a_bytes;
}

static void launch_embed(dp_ends* s, const float* latent, void* x_out, int64_t S, hipStream_t st) {
  const dp_ends_config& c = s->cfg;
  const int64_t rows = (S + 15) / 16;
  const int groups = c.dim / 64, per = (groups + 3) / 4;           // 64-column groups; blocks of 4 that cover them
  // few tokens: the columns are dealt over blocks, many: a block walks all of them.  4C <= 128, five and three blocks to a CU:
  // until there are 512 blocks (by whole rounds of resident blocks, 4C = 64: 4096 x 5120 12.9 instead of 11.9 us, 14400 x 5120
  // 40.0 instead of 38.0, 6240 x 5120 17.9 instead of 19.7; 4C = 128: 14400 x 1024 18.8 instead of 16.3).  Wider ones, two
  // to a CU, so that whole rounds of them take least, a round being the column groups a block walks and about 1.5 more
  // (4C = 256: 6240 x 768 12.6 us, 15.3 the other way; 1560 x 3072 12.6 and 14.7).
  int64_t cols = 1;
  if (s->P <= 128) {
    cols = (512 + rows - 1) / rows;
    cols = cols > per ? per : cols;
  } else {
    double best = 1e30;
    for (int k = 1; k <= per; ++k) {
      const double cost = (double)((rows * k + 511) / 512) * ((double)((groups + 4 * k - 1) / (4 * k)) + 1.5);
      if (cost < best) { best = cost; cols = k; }
    }
  }
  const dim3 grid((unsigned)rows, (unsigned)cols);
  const int al = ((uintptr_t)latent & 15) == 0;
#define EMBED_CASE(KC) k_embed<KC><<<grid, 256, 0, st>>>(latent, (const uint4*)s->w_pe_f, (const bf16_t*)s->w.b_pe, (bf16_t*)x_out, S, c.dim, (int)s->tok, c.tok_w, c.channels, al)
  if (s->P == 64) EMBED_CASE(2);
  else if (s->P == 128) EMBED_CASE(4);
  else if (s->P == 192) EMBED_CASE(6);
  else EMBED_CASE(8);
#undef EMBED_CASE
}

template <typename T>
static void embed_typed(dp_ends* s, const float* latent, void* x_out, int n_frames, hipStream_t st) {
  const dp_ends_config& c = s->cfg;
  const int64_t S = s->tok * n_frames, n = S * s->P;
  if constexpr (sizeof(T) == 2) {
    if (embed_fused(c, S)) {
      if (overlap(latent, (size_t)n * 4, x_out, (size_t)(S * c.dim) * 2)) {
        const int64_t row = (int64_t)2 * c.tok_w * c.channels;        // values per pixel row
        launch_copy2d<float>(latent, row, s->out32, row, n / row, row, st);
        latent = s->out32;
      }
      launch_embed(s, latent, x_out, S, st);
      return;
    }
  }
  k_patchify<T><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(latent, (T*)s->patches, n, (int)s->P, (int)s->tok, c.tok_w, c.channels);
  gemm<T>(s, s->patches, s->P, s->w.w_pe, s->w_pe_t, S, c.dim, s->P, EPI_STORE, EpiArgs{x_out, c.dim, s->w.b_pe, nullptr, 0, nullptr}, st);
}

extern "C" int dp_embed_forward(dp_ends_t* s, const float* latent, void* x_out, int32_t n_frames, void* hip_stream) {
  if (!s || !latent || !x_out) return dp_set_error(DP_EINVAL, "dp_embed_forward: null pointer");
  if (n_frames < 1 || n_frames > s->cfg.max_frames) return dp_set_error(DP_EINVAL, "dp_embed_forward: n_frames outside [1, max_frames]");
  hipStream_t st = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  if (s->cfg.dtype == DP_BF16) embed_typed<bf16_t>(s, latent, x_out, n_frames, st);
  else embed_typed<float>(s, latent, x_out, n_frames, st);
  if (hipGetLastError() != hipSuccess) return dp_set_error(DP_EHIP, "dp_embed_forward: a launch failed");
  return DP_OK;
}

// e: the timestep product's slices, without its bias
static void launch_head_streamed(dp_ends* s, const float* e, int parts, const void* x_in, float* v_out, int64_t S, hipStream_t st) {
  const dp_ends_config& c = s->cfg;
  const int va = ((uintptr_t)v_out & 15) == 0, P = (int)s->P;
  uint4* const wm = (uint4*)s->w_head_t + (size_t)c.dim * P / 8;    // behind the fragments as packed
  float* const pc = s->e1;                                          // the first product's slices have been read: D / 32 * P <= 8 D floats
  k_head_fold<<<(unsigned)(c.dim / 64), 256, 0, st>>>(e, parts, (const bf16_t*)s->w.bt2, s->mhead, c.dim, (const uint4*)s->w_head_t, P, wm, pc);
  // Tokens per block, by whole rounds of blocks (one to a CU) and what a round takes.  16 / 32 / 64 tokens in us (the whole call, of
  // which 24 are the timestep's and k_head_fold): 3600 x 5120 38.4 / 42.0 / 51.2, 7200 x 5120 53.2 / 42.7 / 51.3, 14400 x 5120 80.9 /
  // 60.7 / 53.2, 18720 x 4096 79.0 / 75.0 / 64.2, 6240 x 2112 31.7 / 25.7 / 29.9.
  auto cost = [&](int tokens, int us) { return ((S + tokens - 1) / tokens * (P / 64) + 255) / 256 * us; };
  const int64_t c16 = cost(16, 14), c32 = cost(32, 19), c64 = cost(64, 27);
#define HEAD_CASE(TG, RT, NS) k_head_stream<TG, RT, NS><<<dim3((unsigned)((S + 16 * TG * RT - 1) / (16 * TG * RT)), (unsigned)(P / 64)), 512, 0, st>>>((const bf16_t*)x_in, S, c.dim, c.eps, \
    wm, pc, (const bf16_t*)s->w.b_head, P, v_out, (int)s->tok, c.tok_w, c.channels, va)
  if (c64 <= c32 && c64 <= c16) HEAD_CASE(2, 2, 4); else if (c32 <= c16) HEAD_CASE(2, 1, 5); else HEAD_CASE(1, 1, 3);
#undef HEAD_CASE
}

static void launch_head(dp_ends* s, const void* x_in, float* v_out, int64_t S, hipStream_t st) {
  const dp_ends_config& c = s->cfg;
  const int ng = (c.dim / 64 + 7) / 8, xa = ((uintptr_t)x_in & 15) == 0, va = ((uintptr_t)v_out & 15) == 0;
  // 32 tokens a block halve the reads of the weights, 16 spread few tokens over more CUs: up to 4095, or one round of 16-token
  // blocks.  16 / 32 tokens a block in us (the whole call): 4096 x 1536 23.7 / 25.2, 4590 x 1536 26.0 / 25.2, 4096 x 4096 37.1 / 39.4,
  // 4590 x 4096 43.3 / 39.4, 14400 x 5120 85.6 / 76.7; four times the blocks with 64 latent channels: 4096 x 1536 35.4 / 34.2,
  // 3072 x 1536 30.4 / 33.9.  (9360 tokens are 293 blocks of 32: 34.9 us at 1536, 30.6 with 16.)
  const bool two = S >= 4096 && (S + 15) / 16 * (s->P / 64) > 256;
  const dim3 grid((unsigned)((S + (two ? 31 : 15)) / (two ? 32 : 16)), (unsigned)(s->P / 64));
#define HEAD_CASE(NG, RT) k_head<NG, RT><<<grid, 512, 0, st>>>((const bf16_t*)x_in, S, c.dim, c.eps, s->mod + c.dim, s->mod, \
    (const uint4*)s->w_head_t, (const bf16_t*)s->w.b_head, (int)s->P, v_out, (int)s->tok, c.tok_w, c.channels, xa, va)
#define HEAD_NG(RT) do { if (ng <= 1) HEAD_CASE(1, RT); else if (ng <= 2) HEAD_CASE(2, RT); else if (ng <= 3) HEAD_CASE(3, RT); \
    else if (ng <= 4) HEAD_CASE(4, RT); else if (ng <= 6) HEAD_CASE(6, RT); else if (ng <= 8) HEAD_CASE(8, RT); else HEAD_CASE(10, RT); } while (0)
  if (two) HEAD_NG(2); else HEAD_NG(1);
#undef HEAD_NG
#undef HEAD_CASE
}

template <typename T>
static void head_typed(dp_ends* s, const void* x_in, float t, float* v_out, int n_frames, hipStream_t st) {
  const dp_ends_config& c = s->cfg;
  const int64_t D = c.dim, S = s->tok * n_frames, n = S * s->P;
  // mod rows: shift, scale
  const GemvTable<T> table{(const T*)s->w.bt2, s->mhead, s->mod, 2};
  int parts = launch_gemv<T>(GemvIn{nullptr, 0, t}, (const T*)nullptr, c.freq_dim, (const T*)s->w.wt1, (int)D, s->e1, nullptr, nullptr, st);
  const bool streamed = sizeof(T) == 2 && head_streamed(c);
  parts = launch_gemv<T>(GemvIn{s->e1, parts, 0.f}, (const T*)s->w.bt1, (int)D, (const T*)s->w.wt2, (int)D, s->e, streamed ? nullptr : &table, nullptr, st);
  if constexpr (sizeof(T) == 2) {
    if (head_fused(c)) {
      // k_head_stream loads 16 bytes at once: tokens that start elsewhere are copied too, so that their bits do not depend on where they lie
      if (overlap(x_in, (size_t)(S * D) * 2, v_out, (size_t)n * 4) || (streamed && ((uintptr_t)x_in & 15))) {
        launch_copy2d<bf16_t>((const bf16_t*)x_in, D, (bf16_t*)s->h, D, S, D, st);
        x_in = s->h;
      }
      if (streamed) launch_head_streamed(s, s->e, parts, x_in, v_out, S, st);
      else launch_head(s, x_in, v_out, S, st);
      return;
    }
  }
  launch_to_f32<T>((const T*)x_in, s->x32, S * D, st);
  launch_ln_modulate<T>(s->x32, nullptr, (T*)s->h, S, (int)D, c.eps, s->mod + D, s->mod, 1, st);
  // fp32 output through the residual epilogue (out32 += h W + b) on a cleared buffer
  launch_fill_zero(s->out32, (size_t)n * 4, st);
  gemm<T>(s, s->h, D, s->w.w_head, s->w_head_t, S, s->P, D, EPI_RESID, EpiArgs{nullptr, 0, s->w.b_head, s->out32, s->P, nullptr}, st);
  k_unpatchify<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(s->out32, v_out, n, (int)s->P, (int)s->tok, c.tok_w, c.channels);
}

extern "C" int dp_head_forward(dp_ends_t* s, const void* x_in, float timestep, float* v_out, int32_t n_frames,
                               void* hip_stream) {
  if (!s || !x_in || !v_out) return dp_set_error(DP_EINVAL, "dp_head_forward: null pointer");
  if (n_frames < 1 || n_frames > s->cfg.max_frames) return dp_set_error(DP_EINVAL, "dp_head_forward: n_frames outside [1, max_frames]");
  if (!(timestep == timestep)) return dp_set_error(DP_EINVAL, "dp_head_forward: timestep is NaN");
  hipStream_t st = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  if (s->cfg.dtype == DP_BF16) head_typed<bf16_t>(s, x_in, timestep, v_out, n_frames, st);
  else head_typed<float>(s, x_in, timestep, v_out, n_frames, st);
  if (hipGetLastError() != hipSuccess) return dp_set_error(DP_EHIP, "dp_head_forward: a launch failed");
  return DP_OK;
}

// ------------------------------------------------------------------------------------------ no allocation
// dp_head_forward for callers that cannot allocate (code under HIP graph capture, tight serving loops, harnesses
// that forbid it): no handle and no workspace.  Everything dp_head_forward keeps in the caller's workspace (the
// timestep-MLP vectors, the repacked head matrix; where the head takes the GEMM the fp32 copy of the tokens, the
// normalised tokens and the fp32 result before the scatter) lives in one file-scope device array instead.  Each GPU the
// library runs on holds its own copy of the array at its own address, looked up once per device; host code only ever
// uses that address.
constexpr size_t kHeadScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kHeadScratchBytes];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[64] = {};                 // by device ordinal; filled on a device's first call

static int head_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
    return dp_set_error(DP_EHIP, "dp_head_forward_static: no current device (or an ordinal beyond 63)");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
      return dp_set_error(DP_EHIP, "dp_head_forward_static: hipGetSymbolAddress failed");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return DP_OK;
}

// the head's share of carve(), sized for the frames of this call.  The GEMM's buffers are laid out in either case: they
// are the documented size limit, and h takes the copy of an overlapped input.
static size_t carve_head(dp_ends* s, void* base, int n_frames) {
  const dp_ends_config& c = s->cfg;
  const int64_t E = c.dtype == DP_BF16 ? 2 : 4, D = c.dim;
  s->tok = (int64_t)c.tok_h * c.tok_w;
  s->Smax = s->tok * n_frames;
  s->Spad = rup(s->Smax, 256);
  s->P = 4 * (int64_t)c.channels;
  char* b = (char*)base; size_t off = 0;
  auto take = [&](size_t bytes) { off = (size_t)rup((int64_t)off, 256); void* p = b ? b + off : nullptr; off += bytes; return p; };
  s->patches = nullptr; s->w_pe_t = nullptr; s->w_pe_f = nullptr;
  s->h = take(s->Spad * D * E);
  s->x32 = (float*)take(s->Spad * D * 4);
  s->out32 = (float*)take(s->Spad * s->P * 4);
  s->w_head_t = take(rup(s->P, 256) * D * E);
  s->e1 = (float*)take(GEMV_MAX_SLICES * D * 4); s->e = (float*)take(GEMV_MAX_SLICES * D * 4);   // sliced vectors
  s->mhead = (float*)take(2 * D * 4); s->mod = (float*)take(2 * D * 4);
  return (size_t)rup((int64_t)off, 256);
}

extern "C" int dp_head_forward_static(const dp_ends_config* cfg, const dp_ends_weights* w, const void* x_in,
                                      float timestep, float* v_out, int32_t n_frames, void* hip_stream) {
  const char* why = validate(cfg);
  if (why) return dp_set_error(DP_EINVAL, why);
  if (!w || !x_in || !v_out) return dp_set_error(DP_EINVAL, "dp_head_forward_static: null pointer");
  if (!w->m_head || !w->w_head || !w->b_head || !w->wt1 || !w->bt1 || !w->wt2 || !w->bt2)
    return dp_set_error(DP_EINVAL, "dp_head_forward_static: null weight pointer");
  if (n_frames < 1 || n_frames > cfg->max_frames) return dp_set_error(DP_EINVAL, "dp_head_forward_static: n_frames outside [1, max_frames]");
  if (!(timestep == timestep)) return dp_set_error(DP_EINVAL, "dp_head_forward_static: timestep is NaN");
  dp_ends s;                                            // host struct on the stack: nothing is allocated
  s.cfg = *cfg; s.w = *w;
  if (carve_head(&s, nullptr, n_frames) + (size_t)rup(4 * (int64_t)cfg->freq_dim, 256) > kHeadScratchBytes)   // the documented limit
    return dp_set_error(DP_ENOMEM, "dp_head_forward_static: this many tokens need more than the 64 MiB of static scratch; "
                                   "call it per frame or use dp_head_forward with a workspace");
  void* base = nullptr;
  const int rc = head_scratch(&base);
  if (rc != DP_OK) return rc;
  carve_head(&s, base, n_frames);
  hipStream_t st = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  const int64_t D = cfg->dim, S = s.tok * n_frames;
  const bool bf = cfg->dtype == DP_BF16;
  // the array keeps the last call's contents: rows of the GEMM operand beyond this call's tokens are cleared with
  // a fill kernel (no memset call, so the entry point can be captured), the rest is overwritten below
  if (s.Spad > S && !head_fused(*cfg)) launch_fill_zero((char*)s.h + S * D * (bf ? 2 : 4), (size_t)((s.Spad - S) * D * (bf ? 2 : 4)), st);
  if (bf) {
    pack_head(&s, st);
    launch_to_f32<bf16_t>((const bf16_t*)w->m_head, s.mhead, 2 * D, st);
    head_typed<bf16_t>(&s, x_in, timestep, v_out, n_frames, st);
  } else {
    launch_to_f32<float>((const float*)w->m_head, s.mhead, 2 * D, st);
    head_typed<float>(&s, x_in, timestep, v_out, n_frames, st);
  }
  if (hipGetLastError() != hipSuccess) return dp_set_error(DP_EHIP, "dp_head_forward_static: a launch failed");
  return DP_OK;
}

extern "C" int dp_euler_step(float* x, const float* v, int64_t n, float sigma, float sigma_next, void* hip_stream) {
  if (n < 0) return dp_set_error(DP_EINVAL, "dp_euler_step: negative size");
  if (n == 0) return DP_OK;
  if (!x || !v) return dp_set_error(DP_EINVAL, "dp_euler_step: null pointer");
  if (!(sigma == sigma) || !(sigma_next == sigma_next)) return dp_set_error(DP_EINVAL, "dp_euler_step: sigma is NaN");
  (void)hipGetLastError();
  const int64_t blocks = (n + 255) / 256;                      // grid-stride beyond 2^20 blocks: any n fits
  k_euler<<<(unsigned)(blocks < (1 << 20) ? blocks : (1 << 20)), 256, 0, (hipStream_t)hip_stream>>>(x, v, n, sigma_next - sigma);
  if (hipGetLastError() != hipSuccess) return dp_set_error(DP_EHIP, "dp_euler_step: the launch failed");
  return DP_OK;
}
