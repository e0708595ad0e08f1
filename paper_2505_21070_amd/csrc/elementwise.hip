// Bandwidth-bound kernels of the stage: type conversion, fused LayerNorm+modulate, q/k RMSNorm with
// 3D RoPE, V transposition, cache copies, the timestep-modulation vector and small utilities.
#include "kernels.h"

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------- conversions
// One thread per 8 elements (16 bytes of bf16, two 16-byte accesses of fp32) when pointers and length allow it.
template <typename T>
__global__ void k_to_f32(const T* __restrict__ in, float* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) out[i] = Elem<T>::ld(in + i);
}
template <typename T>
__global__ void k_from_f32(const float* __restrict__ in, T* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) Elem<T>::st(out + i, in[i]);
}
__global__ __launch_bounds__(256) void k_bf16_to_f32_x8(const uint4* __restrict__ in, float4* __restrict__ out, int64_t n8) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  const uint4 v = in[i];
  out[2 * i] = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                           __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
  out[2 * i + 1] = make_float4(__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xffff0000u),
                               __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xffff0000u));
}
__global__ __launch_bounds__(256) void k_f32_to_bf16_x8(const float4* __restrict__ in, uint4* __restrict__ out, int64_t n8) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  const float4 a = in[2 * i], b = in[2 * i + 1];
  out[i] = make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
}
template <typename T> void launch_to_f32(const T* in, float* out, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  if (sizeof(T) == 2 && n % 8 == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)out % 16 == 0) {
    k_bf16_to_f32_x8<<<cdiv(n / 8, 256), 256, 0, st>>>((const uint4*)in, (float4*)out, n / 8);
    return;
  }
  int grid = cdiv(n, 256); if (grid > 8192) grid = 8192;
  k_to_f32<T><<<grid, 256, 0, st>>>(in, out, n);
}
template <typename T> void launch_from_f32(const float* in, T* out, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  if (sizeof(T) == 2 && n % 8 == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)out % 16 == 0) {
    k_f32_to_bf16_x8<<<cdiv(n / 8, 256), 256, 0, st>>>((const float4*)in, (uint4*)out, n / 8);
    return;
  }
  int grid = cdiv(n, 256); if (grid > 8192) grid = 8192;
  k_from_f32<T><<<grid, 256, 0, st>>>(in, out, n);
}
template void launch_to_f32<float>(const float*, float*, int64_t, hipStream_t);
template void launch_to_f32<bf16_t>(const bf16_t*, float*, int64_t, hipStream_t);
template void launch_from_f32<bf16_t>(const float*, bf16_t*, int64_t, hipStream_t);

__global__ void k_mul_f32(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a[i] * b[i];
}
void launch_mul_f32(const float* a, const float* b, float* out, int64_t n, hipStream_t st) {
  if (n > 0) k_mul_f32<<<cdiv(n, 256), 256, 0, st>>>(a, b, out, n);
}

__global__ void k_fill_zero(uint32_t* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}
void launch_fill_zero(void* p, size_t bytes, hipStream_t st) {   // bytes % 4 == 0
  int64_t n = (int64_t)(bytes / 4);
  if (n <= 0) return;
  int grid = cdiv(n, 256); if (grid > 16384) grid = 16384;
  k_fill_zero<<<grid, 256, 0, st>>>((uint32_t*)p, n);
}

// ---------------------------------------------------------------- LayerNorm + modulate
// NW wavefronts per row (1: a wavefront owns a row, 4 rows per block; 4: the block owns one row and the
// statistics meet in LDS); the row lives in registers (NCH float4 per lane), so x is read once.  Two-pass
// statistics (mean, then centred variance) in fp32, partial sums added in a fixed order.
// The row is read and the result written with non-temporal accesses: both are streamed once, and on this part
// a kernel that reads 4 and writes 2 bytes per element runs 1.4-1.7x faster that way (measured on flushed
// caches: 5120-wide rows 152 -> 89 us for 442 MB, 1536-wide rows 24 -> 15 us for 57 MB), faster than a plain
// conversion pass of the same bytes.  Wide rows gain another 25 % from four wavefronts per row (more rows in
// flight per compute unit, 5 instead of 20 outstanding loads per lane).
// xin != null: the row is read from xin (storage type) instead of x, and x receives its fp32 copy (the first
// LayerNorm of a stage, which thereby also fills the fp32 residual stream).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
// All of a row's loads are issued before the first use and the modulation's right behind them, in straight-line code (positions
// beyond the row read its last one and count as zero): with the loads in branches, as a row's length would have it, the
// compiler waited for each before the next.  In a stage (us each, with the launch gap): 1008 x 1024 8.3 -> 6.7, 1560 x 1536 10.5 -> 7.5, 6240 x
// 1536 16.5 -> 15.9, 14400 x 5120 100.4 -> 92.0.
template <typename T, int NCH, int NW, bool XIN>
__global__ __launch_bounds__(256) void k_ln_modulate(float* __restrict__ x, const T* __restrict__ xin,
                                                     T* __restrict__ out, int64_t S, int D, float eps,
                                                     const float* __restrict__ mul, const float* __restrict__ add, float plus) {
  constexpr int RPB = 4 / NW;                        // rows per block of 4 wavefronts
  __shared__ float red[2][4];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row0 = (int64_t)blockIdx.x * RPB + w / NW;
  const int part = (w % NW) * 64 + lane;             // this lane's float4 slot inside a run of NW * 64 slots
  const bool live = row0 < S;                        // rows of a block end together only when NW > 1 shares them
  const int64_t row = live ? row0 : S - 1;
  const int nvec = D >> 2;
  f32x4_t v[NCH], m[NCH], a[NCH];
  auto at = [&](int i) __attribute__((always_inline)) { const int idx = i * (NW * 64) + part; return idx < nvec ? idx : nvec - 1; };
  f32x4_t* const xr = (f32x4_t*)(x + row * D);
  if constexpr (!XIN) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) v[i] = __builtin_nontemporal_load(xr + at(i));
  } else if constexpr (sizeof(T) == 2) {
    u32x2_t r[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) r[i] = __builtin_nontemporal_load((const u32x2_t*)(xin + row * D) + at(i));
#pragma unroll
    for (int i = 0; i < NCH; ++i)
      v[i] = f32x4_t{__uint_as_float(r[i].x << 16), __uint_as_float(r[i].x & 0xffff0000u), __uint_as_float(r[i].y << 16), __uint_as_float(r[i].y & 0xffff0000u)};
  } else {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const T* p = xin + row * D + at(i) * 4;        // the caller's buffer may start anywhere
      v[i] = f32x4_t{p[0], p[1], p[2], p[3]};
    }
  }
#pragma unroll
  for (int i = 0; i < NCH; ++i) m[i] = ((const f32x4_t*)mul)[at(i)];
#pragma unroll
  for (int i = 0; i < NCH; ++i) a[i] = ((const f32x4_t*)add)[at(i)];
  __builtin_amdgcn_sched_barrier(0);
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const bool in = i * (NW * 64) + part < nvec;
    if (XIN && in && live) xr[i * (NW * 64) + part] = v[i];
    sum += in ? (v[i].x + v[i].y) + (v[i].z + v[i].w) : 0.f;
  }
  // sum over the row's NW wavefronts (consecutive wavefronts of the block), in wavefront order
  auto row_sum = [&](float part_sum, int slot) __attribute__((always_inline)) {
    float t = wave_sum(part_sum);
    if constexpr (NW > 1) {
      if (lane == 0) red[slot][w] = t;
      __syncthreads();
      t = 0.f;
#pragma unroll
      for (int i = 0; i < NW; ++i) t += red[slot][(w / NW) * NW + i];
    }
    return t;
  };
  const float mean = row_sum(sum, 0) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const float p = v[i].x - mean, q = v[i].y - mean, r = v[i].z - mean, t = v[i].w - mean;
    sq += i * (NW * 64) + part < nvec ? (p * p + q * q) + (r * r + t * t) : 0.f;
  }
  const float rstd = rsqrtf(row_sum(sq, 1) / (float)D + eps);
  if (!live) return;
  T* orow = out + row * D;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int idx = i * (NW * 64) + part;
    const float r0 = (v[i].x - mean) * rstd * (m[i].x + plus) + a[i].x;
    const float r1 = (v[i].y - mean) * rstd * (m[i].y + plus) + a[i].y;
    const float r2 = (v[i].z - mean) * rstd * (m[i].z + plus) + a[i].z;
    const float r3 = (v[i].w - mean) * rstd * (m[i].w + plus) + a[i].w;
    if (idx < nvec) {
      if constexpr (sizeof(T) == 2) {
        u32x2_t pk; pk.x = pack_bf16x2(r0, r1); pk.y = pack_bf16x2(r2, r3);
        __builtin_nontemporal_store(pk, (u32x2_t*)orow + idx);
      } else {
        __builtin_nontemporal_store(f32x4_t{r0, r1, r2, r3}, (f32x4_t*)orow + idx);
      }
    }
  }
}
template <typename T>
void launch_ln_modulate(float* x, const T* xin, T* out, int64_t S, int D, float eps, const float* mul,
                        const float* add, int plus_one, hipStream_t st) {
  if (S <= 0) return;
  const float plus = plus_one ? 1.f : 0.f;
#define LN_CASE(NCH, NW) do { \
    if (xin) k_ln_modulate<T, NCH, NW, true><<<cdiv(S, 4 / NW), 256, 0, st>>>(x, xin, out, S, D, eps, mul, add, plus); \
    else k_ln_modulate<T, NCH, NW, false><<<cdiv(S, 4 / NW), 256, 0, st>>>(x, xin, out, S, D, eps, mul, add, plus); \
  } while (0)
  // slots beyond the row are loads all the same: a step for every 256 channels of narrow rows (8000 x 512 in a stage: 13.2 us with six, 10.0)
  if (D <= 256) LN_CASE(1, 1);
  else if (D <= 512) LN_CASE(2, 1);
  else if (D <= 768) LN_CASE(3, 1);
  else if (D <= 1024) LN_CASE(4, 1);
  else if (D <= 1536) LN_CASE(6, 1);
  else if (D <= 2048) LN_CASE(8, 1);
  else if (D <= 3072) LN_CASE(3, 4);
  else if (D <= 4096) LN_CASE(4, 4);
  else if (D <= 5120) LN_CASE(5, 4);
  else if (D <= 6144) LN_CASE(6, 4);
  else LN_CASE(8, 4);                                  // D <= 8192
#undef LN_CASE
}
template void launch_ln_modulate<float>(float*, const float*, float*, int64_t, int, float, const float*, const float*, int, hipStream_t);
template void launch_ln_modulate<bf16_t>(float*, const bf16_t*, bf16_t*, int64_t, int, float, const float*, const float*, int, hipStream_t);

// ---------------------------------------------------------------- V -> V^T (per head [d][L])
template <typename T> struct alignas(sizeof(T) * 8) Vec8 { T v[8]; };
// 64 tokens x 64 channels through LDS: 16-byte reads along channels, 16-byte writes along tokens.
template <typename T>
__device__ __forceinline__ void v_transpose_tile(const VTransposeJob<T>& j, const T* __restrict__ src, int64_t ld, int64_t S, int D,
                                                 int64_t s0, int c0, T (&tile)[64][72]) {  // [channel][token], row padded, rows stay vector-aligned
  const int t = threadIdx.x;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = (t >> 3) + pass * 32, cc = (t & 7) * 8;
    const int64_t s = s0 + r;
    Vec8<T> x;
    if (s < S && c0 + cc < D) x = *(const Vec8<T>*)(src + s * ld + j.col + c0 + cc);
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x.v[e] = (T)0;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[cc + e][r] = x.v[e];
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int ch = (t >> 3) + pass * 32, tk = (t & 7) * 8;
    const int c = c0 + ch;
    const int64_t s = s0 + tk;
    if (c < D && s < S) {
      T* o = j.vt + (int64_t)c * j.row_stride + j.col0 + s;     // channel c = head*d + cc: row c of [h*d][row_stride]
      if (j.vec_ok && s + 8 <= S) *(Vec8<T>*)o = *(const Vec8<T>*)&tile[ch][tk];
      else for (int e = 0; e < 8 && s + e < S; ++e) o[e] = tile[ch][tk + e];
    }
  }
}

// ---------------------------------------------------------------- RMSNorm over D + 3D RoPE, head-major output
// One wavefront per token and job (blockIdx.y: e.g. q and k of the same row), four tokens per block.  A lane
// owns VPL groups of 8 consecutive channels (one 16-byte access each for bf16), all loaded before the first
// use so that a wavefront keeps VPL KiB in flight, and kept in registers between the sum-of-squares pass and
// the normalise/rotate/store pass: the row is read once, and nothing but wavefront shuffles synchronises.
// The first tiles_s * cdiv(D, 64) blocks along x, if any, transpose the same rows' values instead, 64 x 64 each: they depend on
// nothing that the others do (two fp32 layers of 128 tokens x 128 channels 143.5 us with a launch of their own, 137.2 this way).
// Loads are straight-line (lanes beyond the row read its last group), and up to 1536 channels the gains and rotations are requested
// with the row: in branches, or behind the sum of squares, the compiler waited for each.  Beyond, their registers would halve
// the wavefronts in flight.  In a stage (us each, with the launch gap): 6240 x 1536 13.0 -> 11.2, 1560 x 1536 7.2 -> 6.6.
template <typename T, int VPL>
__global__ __launch_bounds__(256) void k_norm_rope(const T* __restrict__ src, int64_t ld, int64_t S, int h, int d,
                                                   float eps, NormRopeJob<T> j0, NormRopeJob<T> j1, VTransposeJob<T> jv, int tiles_s, int v_blocks,
                                                   RopeTables rt, int frame0, int tok_h, int tok_w) {
  __shared__ __align__(32) T tile[64][72];
  const int D = h * d, nvec = D >> 3;
  if ((int)blockIdx.x < v_blocks) {
    if (blockIdx.y == 0) v_transpose_tile(jv, src, ld, S, D, (int64_t)((int)blockIdx.x % tiles_s) * 64, (int)blockIdx.x / tiles_s * 64, tile);
    return;
  }
  const NormRopeJob<T> job = blockIdx.y == 0 ? j0 : j1;
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)((int)blockIdx.x - v_blocks) * 4 + (threadIdx.x >> 6);
  if (s >= S) return;
  const Vec8<T>* row = (const Vec8<T>*)(src + s * ld + job.col);
  auto at = [&](int i) __attribute__((always_inline)) { return lane + i * 64 < nvec ? lane + i * 64 : nvec - 1; };
  Vec8<T> raw[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) raw[i] = row[at(i)];
  const int tok = tok_h * tok_w;
  const int f = frame0 + (int)(s / tok), rem = (int)(s % tok);
  const int y = rem / tok_w, x = rem % tok_w;
  // gains and rotations of group i: requested with the row where the registers allow it (a trip to memory each otherwise)
  constexpr int G = VPL <= 3 ? VPL : 1;
  float4 gg[G][2];
  float2 cs[G][4];
  auto request = [&](int i) __attribute__((always_inline)) {
    const int c0 = at(i) * 8, p0 = (c0 % d) >> 1;        // first channel, its pair in the head
    gg[i % G][0] = *(const float4*)(job.g + c0); gg[i % G][1] = *(const float4*)(job.g + c0 + 4);
    if (job.rope) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pi = p0 + e;
        const float2* const t = pi < rt.c_f ? rt.f + (int64_t)f * rt.c_f + pi : pi < rt.c_f + rt.c_h ? rt.y + y * rt.c_h + (pi - rt.c_f) : rt.x + x * rt.c_w + (pi - rt.c_f - rt.c_h);
        cs[i % G][e] = *t;
      }
    }
  };
  if constexpr (G == VPL) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) request(i);
  }
  __builtin_amdgcn_sched_barrier(0);
  float v[VPL][8];
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[i][e] = lane + i * 64 < nvec ? Elem<T>::ld(&raw[i].v[e]) : 0.f;
      sq += v[i][e] * v[i][e];
    }
  }
  const float r = rsqrtf(wave_sum(sq) / (float)D + eps) * job.out_scale;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int vi = lane + i * 64;
    if constexpr (G != VPL) request(i);
    const int c0 = vi * 8, head = c0 / d;
    const float gs[8] = {gg[i % G][0].x, gg[i % G][0].y, gg[i % G][0].z, gg[i % G][0].w, gg[i % G][1].x, gg[i % G][1].y, gg[i % G][1].z, gg[i % G][1].w};
    Vec8<T> o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float a = v[i][2 * e] * r * gs[2 * e], b = v[i][2 * e + 1] * r * gs[2 * e + 1];
      if (job.rope) {
        const float2 c = cs[i % G][e];
        const float a2 = a * c.x - b * c.y, b2 = a * c.y + b * c.x;
        a = a2; b = b2;
      }
      Elem<T>::st(&o.v[2 * e], a);
      Elem<T>::st(&o.v[2 * e + 1], b);
    }
    if (vi < nvec) *(Vec8<T>*)(job.dst + (int64_t)head * job.head_stride + (job.row0 + s) * d + (c0 % d)) = o;
  }
}
// whether whole groups of eight tokens can be stored at once
template <typename T> static VTransposeJob<T> vec_checked(VTransposeJob<T> v) {
  v.vec_ok = (v.col0 % 8 == 0) && (v.row_stride % 8 == 0) && ((uintptr_t)v.vt % (8 * sizeof(T)) == 0);
  return v;
}
template <typename T>
void launch_norm_rope(const T* src, int64_t ld, int64_t S, int h, int d, float eps, const NormRopeJob<T>* jobs,
                      int n_jobs, const RopeTables* rope, int frame0, int tok_h, int tok_w, hipStream_t st, const VTransposeJob<T>* v) {
  if (S <= 0 || n_jobs <= 0) return;
  const int tiles_s = v ? cdiv(S, 64) : 1, v_blocks = v ? tiles_s * cdiv(h * d, 64) : 0;
  const VTransposeJob<T> jv = v ? vec_checked(*v) : VTransposeJob<T>{};
  RopeTables rt = rope ? *rope : RopeTables{nullptr, nullptr, nullptr, 0, 0, 0};
  NormRopeJob<T> j0 = jobs[0], j1 = jobs[n_jobs > 1 ? 1 : 0];
  if (!rope) { j0.rope = 0; j1.rope = 0; }
  const dim3 grid((unsigned)(cdiv(S, 4) + v_blocks), (unsigned)(n_jobs > 1 ? 2 : 1));
  const int th = tok_h > 0 ? tok_h : 1, tw = tok_w > 0 ? tok_w : 1;
  const int vpl = (h * d / 8 + 63) / 64;               // 16-byte groups per lane; dim <= 8192
#define NORM_ROPE_CASE(V) k_norm_rope<T, V><<<grid, 256, 0, st>>>(src, ld, S, h, d, eps, j0, j1, jv, tiles_s, v_blocks, rt, frame0, th, tw)
  if (vpl <= 1) NORM_ROPE_CASE(1);
  else if (vpl <= 3) NORM_ROPE_CASE(3);
  else if (vpl <= 6) NORM_ROPE_CASE(6);
  else if (vpl <= 10) NORM_ROPE_CASE(10);
  else NORM_ROPE_CASE(16);
#undef NORM_ROPE_CASE
}
template void launch_norm_rope<float>(const float*, int64_t, int64_t, int, int, float, const NormRopeJob<float>*, int, const RopeTables*, int, int, int, hipStream_t, const VTransposeJob<float>*);
template void launch_norm_rope<bf16_t>(const bf16_t*, int64_t, int64_t, int, int, float, const NormRopeJob<bf16_t>*, int, const RopeTables*, int, int, int, hipStream_t, const VTransposeJob<bf16_t>*);

// ---------------------------------------------------------------- deferred RMSNorm of head-major bf16 rows
// k[head][row0 + s][:] *= rsqrt(sum_i ssq[i * stride + s] * inv_dim + eps) for every head: the row scale of an
// RMSNorm whose gains and rotation a GEMM epilogue has applied already.  One wavefront per token.  WIDE: the rows come as
// fp32 from `wide`, so that the keys are rounded once; rounded before the rotation and behind it, as by k_norm_rope, their error
// lies across the channel pairs, rounded twice behind it along the large channels, where queries that match a key weigh it most
// (self-attention with 8 times the usual gains, dim 192: 4.43e-3 from 64 bits against 4.30e-3; once 4.06e-3).
template <int VPL, bool WIDE>
__global__ __launch_bounds__(256) void k_scale_rows(bf16_t* __restrict__ k, int64_t head_stride, int64_t row0, int64_t S,
                                                    int h, int d, const float* __restrict__ wide, const float* __restrict__ ssq,
                                                    int np, int64_t stride, float inv_dim, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= S) return;
  const int nvec = (h * d) >> 3;
  uint4 raw[VPL][WIDE ? 2 : 1];
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int c0 = (lane + i * 64) * 8;
    if (lane + i * 64 >= nvec) continue;
    const uint4* const p = WIDE ? (const uint4*)(wide + s * (h * d) + c0) : (const uint4*)(k + (int64_t)(c0 / d) * head_stride + (row0 + s) * d + c0 % d);
    raw[i][0] = p[0];
    if constexpr (WIDE) raw[i][1] = p[1];
  }
  float sum = 0.f;
  for (int i = lane; i < np; i += 64) sum += ssq[i * stride + s];
  const float r = rsqrtf(wave_sum(sum) * inv_dim + eps);
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int c0 = (lane + i * 64) * 8;
    if (lane + i * 64 < nvec) {
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (WIDE) {
          const uint4 v = raw[i][e >> 1];
          o[e] = pack_bf16x2(__uint_as_float(e & 1 ? v.z : v.x) * r, __uint_as_float(e & 1 ? v.w : v.y) * r);
        } else {
          const uint4 v = raw[i][0];
          const uint32_t w = e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
          o[e] = pack_bf16x2(bf16_to_f32((bf16_t)(w & 0xffff)) * r, bf16_to_f32((bf16_t)(w >> 16)) * r);
        }
      }
      *(uint4*)(k + (int64_t)(c0 / d) * head_stride + (row0 + s) * d + c0 % d) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}
void launch_scale_rows_bf16(bf16_t* k, int64_t head_stride, int64_t row0, int64_t S, int h, int d, const float* wide,
                            const float* ssq, int np, int64_t stride, float eps, hipStream_t st) {
  if (S <= 0) return;
  const int vpl = (h * d / 8 + 63) / 64;
  const float inv_dim = 1.f / (float)(h * d);
#define SCALE_ROWS(V, W) k_scale_rows<V, W><<<cdiv(S, 4), 256, 0, st>>>(k, head_stride, row0, S, h, d, wide, ssq, np, stride, inv_dim, eps)
#define SCALE_ROWS_CASE(V) do { if (wide) SCALE_ROWS(V, true); else SCALE_ROWS(V, false); } while (0)
  if (vpl <= 1) SCALE_ROWS_CASE(1);
  else if (vpl <= 3) SCALE_ROWS_CASE(3);
  else if (vpl <= 6) SCALE_ROWS_CASE(6);
  else if (vpl <= 10) SCALE_ROWS_CASE(10);
  else SCALE_ROWS_CASE(16);
#undef SCALE_ROWS_CASE
#undef SCALE_ROWS
}

// ---------------------------------------------------------------- V -> V^T (per head [d][L]) by itself
template <typename T>
__global__ __launch_bounds__(256) void k_v_transpose(VTransposeJob<T> j, const T* __restrict__ src, int64_t ld, int64_t S, int D) {
  __shared__ __align__(32) T tile[64][72];
  v_transpose_tile(j, src, ld, S, D, (int64_t)blockIdx.x * 64, blockIdx.y * 64, tile);
}
template <typename T>
void launch_v_transpose(const T* src, int64_t ld, int64_t S, int h, int d, const VTransposeJob<T>& v, hipStream_t st) {
  if (S <= 0) return;
  k_v_transpose<T><<<dim3(cdiv(S, 64), cdiv(h * d, 64)), 256, 0, st>>>(vec_checked(v), src, ld, S, h * d);
}
template void launch_v_transpose<float>(const float*, int64_t, int64_t, int, int, const VTransposeJob<float>&, hipStream_t);
template void launch_v_transpose<bf16_t>(const bf16_t*, int64_t, int64_t, int, int, const VTransposeJob<bf16_t>&, hipStream_t);

// ---------------------------------------------------------------- strided row copy (feature-cache hand-over)
// Rows are copied in 16-byte pieces when dst, its stride and the length allow it; those of a src that starts anywhere are loads that
// claim an element's alignment (14400 x 5120 bf16 off a 16-byte boundary, the output head's tokens: 154 us by elements, 60 this way).
template <typename T> struct Piece16 { T v[16 / sizeof(T)]; };
template <typename T, typename V>
__global__ void k_copy2d(const T* __restrict__ src, int64_t src_stride, T* __restrict__ dst,
                         int64_t dst_stride, int64_t len_v) {
  typedef std::conditional_t<sizeof(V) == 16, uint4, V> W;
  const V* s = (const V*)(src + (int64_t)blockIdx.y * src_stride);
  W* d = (W*)(dst + (int64_t)blockIdx.y * dst_stride);
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < len_v; i += stride) d[i] = __builtin_bit_cast(W, s[i]);
}
template <typename T>
void launch_copy2d(const T* src, int64_t src_stride, T* dst, int64_t dst_stride, int64_t rows,
                   int64_t len, hipStream_t st) {
  if (rows <= 0 || len <= 0) return;
  if (src_stride == len && dst_stride == len) { len *= rows; src_stride = dst_stride = len; rows = 1; }
  const int per = 16 / (int)sizeof(T), most = rows == 1 ? 8192 : 64;         // blocks to a row
  const bool vec = ((uintptr_t)dst % 16 == 0) && (dst_stride % per == 0) && (len % per == 0);
  const bool src16 = ((uintptr_t)src % 16 == 0) && (src_stride % per == 0);
  // rows can exceed the grid.y limit only for absurd shapes; split defensively
  for (int64_t r0 = 0; r0 < rows; r0 += 32768) {
    const int64_t nr = rows - r0 < 32768 ? rows - r0 : 32768;
    if (vec) {
      const int64_t lv = len / per;
      int gx = cdiv(lv, 256); if (gx > most) gx = most;
      if (src16) k_copy2d<T, uint4><<<dim3(gx, (unsigned)nr), 256, 0, st>>>(src + r0 * src_stride, src_stride, dst + r0 * dst_stride, dst_stride, lv);
      else k_copy2d<T, Piece16<T>><<<dim3(gx, (unsigned)nr), 256, 0, st>>>(src + r0 * src_stride, src_stride, dst + r0 * dst_stride, dst_stride, lv);
    } else {
      int gx = cdiv(len, 256); if (gx > most) gx = most;
      k_copy2d<T, T><<<dim3(gx, (unsigned)nr), 256, 0, st>>>(src + r0 * src_stride, src_stride,
                                                             dst + r0 * dst_stride, dst_stride, len);
    }
  }
}
template void launch_copy2d<float>(const float*, int64_t, float*, int64_t, int64_t, int64_t, hipStream_t);
template void launch_copy2d<bf16_t>(const bf16_t*, int64_t, bf16_t*, int64_t, int64_t, int64_t, hipStream_t);

// ---------------------------------------------------------------- weight repack: [K,N] -> [Npad,K]
template <typename T>
__global__ __launch_bounds__(256) void k_transpose_pad(const T* __restrict__ in, int64_t K, int64_t N,
                                                       T* __restrict__ out, int64_t Npad) {
  __shared__ T tile[64][65];
  const int64_t k0 = (int64_t)blockIdx.x * 64, n0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) {
    const int64_t k = k0 + r, n = n0 + tx;
    tile[r][tx] = (k < K && n < N) ? in[k * N + n] : (T)0;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {
    const int64_t n = n0 + r, k = k0 + tx;
    if (n < Npad && k < K) out[n * K + k] = tile[tx][r];
  }
}
template <typename T>
void launch_transpose_pad(const T* in, int64_t K, int64_t N, T* out, int64_t Npad, hipStream_t st) {
  dim3 grid(cdiv(K, 64), cdiv(Npad, 64));
  k_transpose_pad<T><<<grid, 256, 0, st>>>(in, K, N, out, Npad);
}
template void launch_transpose_pad<float>(const float*, int64_t, int64_t, float*, int64_t, hipStream_t);
template void launch_transpose_pad<bf16_t>(const bf16_t*, int64_t, int64_t, bf16_t*, int64_t, hipStream_t);

// ---------------------------------------------------------------- timestep modulation vector
// Matrix-vector products of the timestep MLP, bound by one read of W.  A block owns 64 * CPL output columns; a wavefront
// instruction reads one row's piece of them (256 bytes at CPL = 2 in bf16), 16 to 32 rows in flight per wavefront, and the
// 16 wavefronts' sums meet in LDS.  (Lanes of a wavefront on different rows, 16 bytes each, took 108 us where this took
// 82: every row is another page.)
// The sum over K: slices of the rows (launch_gemv); in a slice wavefront w takes rows w, w + 16, .. into four chains in turn
// (one chain per wavefront is 1.4 times as far from 64 bits at K = 5120), (0 + 1) + (2 + 3), the wavefronts in order; bias +
// slices in order.  A product is either sliced over blocks, partial results left for the consumer to add up, or whole: a
// block takes all slices of its columns and adds its result to the L rows of a table.
// 5120 x 30720: 315 MB in 78 us = 4.0 TB/s, what a read-only pass reaches here; more rows in flight do not change it.
// The chain (features, three products, table, rotation table) is three launches (k_gemv_pair: two): 128-wide model 28 -> 13 us, 1536-wide
// 39 -> 29 us under the profiler, which counts a launch as 4.6 us; 1 us each otherwise.
template <typename T> struct GemvArgs {
  GemvIn in;
  const T *xbias, *W, *ybias;
  int K, N, slices;
  float* y;                    // [slices][N], or null: whole
  const float* mtab; float* mod; int L;
  int cols;                    // blocks along N; further ones build the rotation table
};
// cs[s][i] = (cos, sin) of channel pair i at token s = (frame0 + s / (tok_h * tok_w), y, x), gathered from the per-axis tables
__device__ __forceinline__ void rope_token(const RopeTokens& r, int64_t i) {
  const uint32_t half = r.rt.c_f + r.rt.c_h + r.rt.c_w, s = (uint32_t)(i / half), pi = (uint32_t)(i % half);
  const uint32_t tok = (uint32_t)r.tok_h * r.tok_w, rem = s % tok, f = r.frame0 + s / tok, y = rem / r.tok_w, x = rem % r.tok_w;
  const uint32_t cf = r.rt.c_f, ch = r.rt.c_h, cw = r.rt.c_w;
  r.cs[i] = pi < cf ? r.rt.f[(int64_t)f * cf + pi] : pi < cf + ch ? r.rt.y[y * ch + (pi - cf)] : r.rt.x[x * cw + (pi - cf - ch)];
}
// SINUS: the input is the sinusoidal features of a.in.t (a kernel of its own: their double-precision code would cost every
// product registers and scratch memory).  CPL == 2: bf16, rows of W in 4-byte steps.  At most 64 registers, so that a CU
// holds two blocks: with 72 it held one, and a grid of a few more blocks than CUs took two rounds (fp32 5120 x 30720, 480
// blocks: the chain 157 -> 148 us; bf16 6144 x 36864, 288 blocks: 161 -> 145; fp32 8192 x 49152, three whole rounds:
// 351 -> 359).
template <typename T, int CPL, bool SINUS>
__global__ __launch_bounds__(1024, SINUS ? 4 : 8) void k_gemv(GemvArgs<T> a, RopeTokens rope) {
  constexpr int KC = 8192, U = SINUS ? 4 : 16, MS = CPL == 1 && !SINUS ? GEMV_MAX_SLICES : 1;   // MS: most slices a block takes
  __shared__ float xs[KC];
  __shared__ float red[MS][16][64 * CPL];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (SINUS && (int)blockIdx.x >= a.cols) {
    const int64_t i = ((int64_t)((int)blockIdx.x - a.cols) * gridDim.y + blockIdx.y) * 1024 + tid;
    if (i < rope.S * (rope.rt.c_f + rope.rt.c_h + rope.rt.c_w)) rope_token(rope, i);
    return;
  }
  const int s0 = a.y ? (int)blockIdx.y : 0, ns = a.y ? 1 : MS < a.slices ? MS : a.slices;     // this block's slices
  auto bound = [&](int s) __attribute__((always_inline)) { return (int)((int64_t)a.K * (s0 + s) / a.slices); };
  const int n0 = (int)blockIdx.x * 64 * CPL, n = n0 + lane * CPL;
  const T* const wn = a.W + (n < a.N ? n : 0);
  float acc[4][CPL];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int v = 0; v < CPL; ++v) acc[c][v] = 0.f;
  auto flush = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < CPL; ++v) {
      red[s][wave][lane * CPL + v] = (acc[0][v] + acc[1][v]) + (acc[2][v] + acc[3][v]);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c][v] = 0.f;
    }
  };
  const int lo = bound(0), hi = bound(ns);
  for (int w0 = lo; w0 < hi; w0 += KC) {               // several windows only in one slice: K <= KC otherwise
    const int w1 = hi - w0 < KC ? hi : w0 + KC;
    if (w0 > lo) __syncthreads();
    // rows k, k + 16, .. of this wavefront, up to row e of the slice: groups of U, the next group requested before this one
    // is used (past the end: the last row again, not added)
    using Piece = std::conditional_t<CPL == 2, uint32_t, T>;
    Piece d[2][U];
    auto fetch = [&](int k, int e, int z) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) d[z][u] = *(const Piece*)(wn + (int64_t)(k + u * 16 < e ? k + u * 16 : e - 1) * a.N);
    };
    auto add = [&](int k, int e, int z) __attribute__((always_inline)) {
      auto one = [&](int u, int c) __attribute__((always_inline)) {
        const float x = xs[k - w0 + u * 16];
        if constexpr (CPL == 2) {
          acc[c][0] += x * __uint_as_float(d[z][u] << 16);
          acc[c][1] += x * __uint_as_float(d[z][u] & 0xffff0000u);
        } else {
          acc[c][0] += x * Elem<T>::ld(&d[z][u]);
        }
      };
      if (k + (U - 1) * 16 < e) {
#pragma unroll
        for (int u = 0; u < U; ++u) one(u, u & 3);
      } else {                                         // rows of an incomplete last four all go to the first chain
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (k + (u | 3) * 16 < e) one(u, u & 3);
          else if (k + u * 16 < e) one(u, 0);
        }
      }
    };
    int s = 0, k = w0 + wave, e = ns > 1 ? bound(1) : w1;
    fetch(k, e, 0);                                    // travels while the activations are made
    for (int i = tid; i < w1 - w0; i += 1024) {
      const int kk = w0 + i;
      if constexpr (SINUS) {
        const int half = a.K >> 1, j = kk < half ? kk : kk - half;
        const double ang = (double)a.in.t * pow(10000.0, -(double)j / (double)half);
        xs[i] = kk < half ? (float)cos(ang) : (float)sin(ang);
      } else {
        float v = Elem<T>::ld(a.xbias + kk);
        const float* const xp = a.in.x + kk;
        for (int p0 = 0; p0 < a.in.parts; p0 += 4) {   // four parts requested together
          float part[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) part[p] = xp[(int64_t)(p0 + p < a.in.parts ? p0 + p : p0) * a.K];
#pragma unroll
          for (int p = 0; p < 4; ++p)
            if (p0 + p < a.in.parts) v += part[p];
        }
        xs[i] = v / (1.0f + expf(-v));                 // SiLU
      }
    }
    __syncthreads();
    // one group, with the next one (of this slice or the next) on its way; false behind the window's last
    auto step = [&](int z) __attribute__((always_inline)) {
      int s2 = s, k2 = k + 16 * U, e2 = e;
      if (k2 >= e) {
        ++s2;
        k2 = e + wave;
        e2 = s2 < ns ? bound(s2 + 1) : e;
      }
      const bool more = s2 < ns;
      if (more) fetch(k2, e2, z ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      add(k, e, z);
      __builtin_amdgcn_sched_barrier(0);
      if (more && s2 != s) flush(s);
      s = s2; k = k2; e = e2;
      return more;
    };
    while (step(0) && step(1)) {}
  }
  flush(ns - 1);
  __syncthreads();
  if (tid < 64 * CPL && n0 + tid < a.N) {
    float y = a.y ? 0.f : Elem<T>::ld(a.ybias + n0 + tid);
    for (int s = 0; s < ns; ++s) {
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += red[s][i][tid];
      y += sum;
    }
    if (a.y) a.y[(int64_t)s0 * a.N + n0 + tid] = y;
    else
      for (int l = 0; l < a.L; ++l) a.mod[(int64_t)l * a.N + n0 + tid] = a.mtab[(int64_t)l * a.N + n0 + tid] + y;
  }
}
// The first two products of a chain in one launch, for 256 features and less than 2048 channels: a block makes the piece of the
// first product that its slice of the second one reads (at most 256 columns; all blocks of a slice make it, from L2), while the
// second one's weights are on their way.  Sums in the order of the two launches, so with their bits.
// What bounds it: latency, four trips to memory instead of six and a launch less; the whole chain of a stage at 256 channels 14.8 ->
// 12.6 us, at 1024 19.0 -> 17.9 (with the launch gaps).
template <typename T> struct GemvPairArgs { float t; const T *W1, *b1, *W2; int D, slices; float* y; int cols; };
template <typename T>
__global__ __launch_bounds__(1024, 4) void k_gemv_pair(GemvPairArgs<T> a, RopeTokens rope) {
  __shared__ float feat[256], xs[256];
  __shared__ float red1[4][4][16][64], red2[16][64];     // [64 columns][64 features][wavefront][column]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x >= a.cols) {
    const int64_t i = ((int64_t)((int)blockIdx.x - a.cols) * gridDim.y + blockIdx.y) * 1024 + tid;
    if (i < rope.S * (rope.rt.c_f + rope.rt.c_h + rope.rt.c_w)) rope_token(rope, i);
    return;
  }
  const int lo = (int)((int64_t)a.D * blockIdx.y / a.slices), hi = (int)((int64_t)a.D * (blockIdx.y + 1) / a.slices), groups = (hi - lo + 63) >> 6;
  const int n = (int)blockIdx.x * 64 + lane;
  const T* const w2 = a.W2 + (n < a.D ? n : 0);
  T d2[16], d1[2][16];
#pragma unroll
  for (int u = 0; u < 16; ++u) d2[u] = w2[(int64_t)(lo + wave + u * 16 < hi ? lo + wave + u * 16 : hi - 1) * a.D];
  auto fetch = [&](int g, auto z_) __attribute__((always_inline)) {      // rows 64 s + 16 c + wave of 64 columns
    constexpr int z = decltype(z_)::value;
    const int c = lo + g * 64 + lane;
    const T* const w1 = a.W1 + (c < hi ? c : hi - 1);
#pragma unroll
    for (int u = 0; u < 16; ++u) d1[z][u] = w1[(int64_t)(u * 16 + wave) * a.D];
  };
  fetch(0, std::integral_constant<int, 0>{});
  if (tid < 256) {
    const int j = tid < 128 ? tid : tid - 128;
    const double ang = (double)a.t * pow(10000.0, -(double)j / 128.0);
    feat[tid] = tid < 128 ? (float)cos(ang) : (float)sin(ang);
  }
  __syncthreads();
  static_for<4>([&](auto g_) __attribute__((always_inline)) {
    constexpr int g = decltype(g_)::value;
    if (g < groups) {
      if (g + 1 < groups) fetch(g + 1, std::integral_constant<int, (g + 1) & 1>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float p[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = fmaf(feat[s * 64 + c * 16 + wave], Elem<T>::ld(&d1[g & 1][s * 4 + c]), 0.f);   // rounded by itself, as in k_gemv
        red1[g][s][wave][lane] = (p[0] + p[1]) + (p[2] + p[3]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  });
  __syncthreads();
  if (tid < hi - lo) {
    float v = Elem<T>::ld(a.b1 + lo + tid);
    for (int s = 0; s < 4; ++s) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < 16; ++w) sum += red1[tid >> 6][s][w][tid & 63];
      v += sum;
    }
    xs[tid] = v / (1.0f + expf(-v));                     // SiLU
  }
  __syncthreads();
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < 16; ++u) {                         // rows of an incomplete last four all go to the first chain
    const int k = wave + u * 16;
    if (lo + wave + (u | 3) * 16 < hi) acc[u & 3] += xs[k] * Elem<T>::ld(&d2[u]);
    else if (lo + k < hi) acc[0] += xs[k] * Elem<T>::ld(&d2[u]);
  }
  red2[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (tid < 64 && n < a.D) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) sum += red2[w][tid];
    a.y[(int64_t)blockIdx.y * a.D + n] = sum;
  }
}
// mod[l, i] = mtab[l, i] + (bias[i] + sum_p e[p][i]): a sliced vector added to every row of a table
template <typename T>
__global__ __launch_bounds__(256) void k_mod_add(const float* __restrict__ e, int parts, GemvTable<T> t, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = Elem<T>::ld(t.bias + i);
  for (int p = 0; p < parts; ++p) v += e[(int64_t)p * n + i];
  for (int l = 0; l < t.L; ++l) t.mod[(int64_t)l * n + i] = t.mtab[(int64_t)l * n + i] + v;
}
// enough blocks of 64 columns for the 256 CUs, at least 64 rows each
static int gemv_slices(int K, int N) {
  int ks = cdiv(256, cdiv(N, 64));
  if (ks > GEMV_MAX_SLICES) ks = GEMV_MAX_SLICES;
  while (ks > 1 && K / ks < 64) --ks;
  return ks;
}
template <typename T>
int launch_gemv(const GemvIn& in, const T* xbias, int K, const T* W, int N, float* y, const GemvTable<T>* table,
                const RopeTokens* rope, hipStream_t st) {
  // A product that ends in a table stays whole unless its columns make less than half a round of blocks that each have many
  // rows to read (5120 x 5120: 38 us whole, 21 sliced with a launch more; 1536 x 1536: 13 and 11 under the
  // profiler, which counts the launch as 4.6 us).  A caller that gives no y wants it whole: the stage's, 6 * dim columns
  // (the whole chain / as six launches, us: dim 512 16.5 / 21.8, 1152 24.9 / 24.9, 1536 23.0 / 26.8, 5120 87 / 100).
  const bool whole = table && (!y || cdiv(N, 64) >= 128 || K <= 2048);
  // short slices cost a whole product a load latency each (chain at dim 512 24.7 us with six of them, 16.5 with one); the
  // kernel's limits for several in one block are K <= 8192 and no features to make
  int slices = gemv_slices(K, N);
  if (whole && (K / slices < 384 || K > 8192 || !in.x)) slices = 1;
  // two columns per lane where one would make more blocks than CUs: stage chains at dim 2816, 264 blocks of 64 columns or
  // 132 of 128: 57.8 and 38.4 us, 44.1 as six launches; head at 1560 x 2560, 280 or 140: 27.0 and 25.8 us.  (The features'
  // product, a few columns and rows, stays at one; a whole product with so many columns has one slice.)
  const bool wide = sizeof(T) == 2 && in.x && N % 2 == 0 && ((uintptr_t)W & 3) == 0 && cdiv(N, 64) * (whole ? 1 : slices) > 256;
  const int cols = cdiv(N, wide ? 128 : 64);
  GemvArgs<T> a{in, xbias, W, table ? table->bias : nullptr, K, N, slices, whole ? nullptr : y, table ? table->mtab : nullptr,
                table ? table->mod : nullptr, table ? table->L : 0, cols};
  const RopeTokens r = rope ? *rope : RopeTokens{};
  const int per = 1024 * (whole ? 1 : slices);
  const int64_t extra = rope ? (rope->S * (rope->rt.c_f + rope->rt.c_h + rope->rt.c_w) + per - 1) / per : 0;
  const dim3 grid((unsigned)(cols + extra), (unsigned)(whole ? 1 : slices));
  if (!in.x) k_gemv<T, 1, true><<<grid, 1024, 0, st>>>(a, r);
  else if (!wide) k_gemv<T, 1, false><<<grid, 1024, 0, st>>>(a, r);
  else if constexpr (sizeof(T) == 2) k_gemv<T, 2, false><<<grid, 1024, 0, st>>>(a, r);
  if (table && !whole) k_mod_add<T><<<cdiv(N, 256), 256, 0, st>>>(y, slices, *table, N);
  return slices;
}
template <typename T>
int launch_gemv_pair(float t, const T* W1, const T* b1, int freq, const T* W2, int D, float* mid, float* y, const RopeTokens* rope, hipStream_t st) {
  // by the two launches where the features are other than 256, or so many channels that each block's share of the first product
  // is more than a latency (the first product's four slices, whose order is kept, are those of up to 5440 columns).  The whole chain
  // in a stage, one launch / two in us: 1536 channels 21.8 / 22.9 (640 tokens), 26.2 / 26.6 (8000), 1984 27.6 / 28.0, 33.4 / 34.1, 2048 28.1 /
  // 27.1, 34.9 / 34.3
  if (freq != 256 || D >= 2048) {
    const int parts = launch_gemv<T>(GemvIn{nullptr, 0, t}, (const T*)nullptr, freq, W1, D, mid, nullptr, rope, st);
    return launch_gemv<T>(GemvIn{mid, parts, 0.f}, b1, D, W2, D, y, nullptr, nullptr, st);
  }
  const int slices = gemv_slices(D, D), cols = cdiv(D, 64), per = 1024 * slices;
  const RopeTokens r = rope ? *rope : RopeTokens{};
  const int64_t extra = rope ? (rope->S * (rope->rt.c_f + rope->rt.c_h + rope->rt.c_w) + per - 1) / per : 0;
  k_gemv_pair<T><<<dim3((unsigned)(cols + extra), (unsigned)slices), 1024, 0, st>>>(GemvPairArgs<T>{t, W1, b1, W2, D, slices, y, cols}, r);
  return slices;
}
template int launch_gemv_pair<float>(float, const float*, const float*, int, const float*, int, float*, float*, const RopeTokens*, hipStream_t);
template int launch_gemv_pair<bf16_t>(float, const bf16_t*, const bf16_t*, int, const bf16_t*, int, float*, float*, const RopeTokens*, hipStream_t);
template int launch_gemv<float>(const GemvIn&, const float*, int, const float*, int, float*, const GemvTable<float>*, const RopeTokens*, hipStream_t);
template int launch_gemv<bf16_t>(const GemvIn&, const bf16_t*, int, const bf16_t*, int, float*, const GemvTable<bf16_t>*, const RopeTokens*, hipStream_t);

// cos/sin of pos * theta^(-i/pairs), angles in double
__global__ void k_rope_table(float2* tab, int n_pos, int pairs, float theta) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_pos * pairs) return;
  const int pos = i / pairs, j = i % pairs;
  const double ang = (double)pos * pow((double)theta, -(double)j / (double)pairs);
  tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}
void launch_rope_table(float2* tab, int n_pos, int pairs, float theta, hipStream_t st) {
  if (n_pos * pairs <= 0) return;
  k_rope_table<<<cdiv((int64_t)n_pos * pairs, 256), 256, 0, st>>>(tab, n_pos, pairs, theta);
}

// ---------------------------------------------------------------- test-hook gathers (head-major -> token-major fp32)
template <typename T>
__global__ void k_gather_heads(const T* __restrict__ src, int64_t head_stride, int64_t row0, int64_t S,
                               int h, int d, float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int D = h * d;
  if (i >= S * D) return;
  const int64_t s = i / D; const int c = (int)(i % D);
  dst[i] = Elem<T>::ld(src + (int64_t)(c / d) * head_stride + (row0 + s) * d + (c % d));
}
template <typename T>
void launch_gather_heads(const T* src, int64_t head_stride, int64_t row0, int64_t S, int h, int d,
                         float* dst, hipStream_t st) {
  if (S <= 0) return;
  k_gather_heads<T><<<cdiv(S * h * d, 256), 256, 0, st>>>(src, head_stride, row0, S, h, d, dst);
}
// the queries as the bf16 attention kernel uses them when their RMSNorm is deferred: same sums, same rounding
__global__ void k_gather_heads_qnorm(const bf16_t* __restrict__ src, int64_t head_stride, int64_t S, int h, int d,
                                     AttnQNorm qn, float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int D = h * d;
  if (i >= S * D) return;
  const int64_t s = i / D; const int c = (int)(i % D);
  float even = 0.f, odd = 0.f;
  for (int j = 0; j < qn.np; j += 2) even += qn.ssq[j * qn.stride + s];
  for (int j = 1; j < qn.np; j += 2) odd += qn.ssq[j * qn.stride + s];
  const float r = rsqrtf((even + odd) * qn.inv_dim + qn.eps) * qn.scale;
  dst[i] = bf16_to_f32(f32_to_bf16(bf16_to_f32(src[(int64_t)(c / d) * head_stride + s * d + (c % d)]) * r));
}
void launch_gather_heads_qnorm(const bf16_t* src, int64_t head_stride, int64_t S, int h, int d, const AttnQNorm& qn,
                               float* dst, hipStream_t st) {
  if (S <= 0) return;
  k_gather_heads_qnorm<<<cdiv(S * h * d, 256), 256, 0, st>>>(src, head_stride, S, h, d, qn, dst);
}
template void launch_gather_heads<float>(const float*, int64_t, int64_t, int64_t, int, int, float*, hipStream_t);
template void launch_gather_heads<bf16_t>(const bf16_t*, int64_t, int64_t, int64_t, int, int, float*, hipStream_t);

template <typename T>
__global__ void k_gather_vt(const T* __restrict__ vt, int64_t row_stride, int64_t col0, int64_t S, int h,
                            int d, float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int D = h * d;
  if (i >= S * D) return;
  const int64_t s = i / D; const int c = (int)(i % D);
  dst[i] = Elem<T>::ld(vt + (int64_t)c * row_stride + col0 + s);
}
template <typename T>
void launch_gather_vt(const T* vt, int64_t row_stride, int64_t col0, int64_t S, int h, int d, float* dst,
                      hipStream_t st) {
  if (S <= 0) return;
  k_gather_vt<T><<<cdiv(S * h * d, 256), 256, 0, st>>>(vt, row_stride, col0, S, h, d, dst);
}
template void launch_gather_vt<float>(const float*, int64_t, int64_t, int64_t, int, int, float*, hipStream_t);
template void launch_gather_vt<bf16_t>(const bf16_t*, int64_t, int64_t, int64_t, int, int, float*, hipStream_t);

// ---------------------------------------------------------------- coordinated noise initialisation: frame gather
// out[f, :] = pool[index[f], :] in 16-byte vectors; a frame whose index is out of range is written as zeros
__global__ __launch_bounds__(256) void k_gather_frames(const uint4* __restrict__ pool, int pool_frames,
                                                       int64_t frame_vecs, const int32_t* __restrict__ index,
                                                       uint4* __restrict__ out) {
  const int f = blockIdx.y;
  const int src = index[f];
  const bool ok = src >= 0 && src < pool_frames;
  const uint4* s = pool + (int64_t)(ok ? src : 0) * frame_vecs;
  uint4* d = out + (int64_t)f * frame_vecs;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < frame_vecs; i += (int64_t)gridDim.x * 256)
    d[i] = ok ? s[i] : make_uint4(0, 0, 0, 0);
}
void launch_gather_frames(const void* pool, int pool_frames, int64_t frame_bytes, const int32_t* index,
                          int n_frames, void* out, hipStream_t st) {
  if (n_frames <= 0 || frame_bytes <= 0) return;
  const int64_t vecs = frame_bytes / 16;
  int64_t bx = cdiv(vecs, 256 * 4);                 // 4 vectors per thread
  if (bx < 1) bx = 1;
  if (bx > 4096) bx = 4096;
  k_gather_frames<<<dim3((unsigned)bx, (unsigned)n_frames), 256, 0, st>>>((const uint4*)pool, pool_frames, vecs, index, (uint4*)out);
}
