// fp32 flash attention for the DP_F32 path on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32: fp32 operands,
// fp32 accumulation, nothing rounded below fp32).
//
// Like the bf16 kernel, scores are computed transposed: S^T = K Q^T (keys are MFMA rows, queries columns), so a lane
// owns one query, the softmax is a reduction over the lane's own registers plus one exchange with lane ^ 32, and the
// exponentiated accumulators are the B operand of O^T = V^T P^T as they stand: accumulator register 4g + t of lane
// group lg is key 8g + 4lg + t, which is also the key that lane group supplies to the t-th of four MFMAs when its V^T
// operand is one 16-byte piece of a channel's row.  The K operand is 16 bytes of a key's row the same way (the order
// in which the head dimension is summed is free).
//
// Bound: the fp32 matrix rate (64 cycles an MFMA; 157 TFLOP/s over the chip).  A 16-byte operand read feeds four MFMAs
// = 256 cycles, so operands come straight from L1/L2 into registers, one group of four reads ahead (1024 cycles of
// MFMAs), and no LDS tile or barrier is needed.  1560 queries x 3120 keys x 12 heads x 128: 4648 us with one wavefront
// per query on the vector unit, 354 + 9 (merge) us here = 82 TFLOP/s; 1560 x 512 keys 984 -> 75 us; 128 x 192 x 2 heads x 64
// 58 -> 10 us.
#include "kernels.h"

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A block of four wavefronts owns QG * 32 queries of one head; the key tiles of its range are dealt to KG groups.
// QG = 4: the wavefronts walk the same keys for four query tiles and meet in L1.  QG = 1: four key groups for one query
// tile, joined through LDS at the end (few queries or few keys: blocks are a quarter as long).
// parts > 1: a block takes one of `parts` key ranges and leaves (m, l, O) unnormalised for k_attn_f32_merge.
template <int HD, int QG, int KG>
__global__ __launch_bounds__(256, 2) void k_attn_f32(const float* __restrict__ q, int64_t q_head_stride,
                                                     const float* __restrict__ k, int64_t k_head_stride,
                                                     int64_t k_row0, const float* __restrict__ vt,
                                                     int64_t vt_row_stride, int64_t S, int64_t L, int lead,
                                                     float* __restrict__ out, int64_t ldo, float scale, int qblocks,
                                                     int blocks, int parts, float* __restrict__ partial) {
  static_assert(QG * KG == 4, "four wavefronts");
  constexpr int GN = HD / 32;                        // operand groups of K per tile, and of V^T
  constexpr int QB = QG * 32;
  __shared__ float xch[KG > 1 ? (KG - 1) * (GN * 16 + 2) * 64 : 1];
  // every XCD (blocks are dealt round-robin) takes a contiguous run of work: one head's blocks share its L2
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= blocks) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int qt = wave % QG, kg = wave / QG;
  const int wid = pid / parts, part = pid % parts;
  const int head = wid / qblocks;
  const int64_t q0 = (int64_t)(wid % qblocks) * QB + qt * 32;
  // The key range starts at a 16-byte boundary of the V^T rows: `lead` keys in front of the first real one and those
  // at or beyond lead + L are masked (and their V taken as 0: what lies there is not this call's).
  const int64_t La = L + lead;
  const int NKT = (int)((La + 31) / 32);
  const int p0 = (int)((int64_t)part * NKT / parts), p1 = (int)((int64_t)(part + 1) * NKT / parts);
  const int t0 = p0 + (int)((int64_t)kg * (p1 - p0) / KG), t1 = p0 + (int)((int64_t)(kg + 1) * (p1 - p0) / KG);

  f32x4 qf[HD / 8];
  {
    const int64_t row = q0 + lr < S ? q0 + lr : S - 1;
    const float* qr = q + (int64_t)head * q_head_stride + row * HD + lg * 4;
#pragma unroll
    for (int j = 0; j < HD / 8; ++j) qf[j] = *(const f32x4*)(qr + j * 8) * scale;
  }
  const float* kp = k + (int64_t)head * k_head_stride + (k_row0 - lead + lr) * HD + lg * 4;
  const float* vp = vt + ((int64_t)head * HD + lr) * vt_row_stride + (k_row0 - lead) + lg * 4;

  f32x16 o[GN];
#pragma unroll
  for (int a = 0; a < GN; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[a][r] = 0.f;
  float m = -INFINITY, l = 0.f;                      // l: this lane's share (its own 16 keys of every tile)

  // operand group i of tile kt: 4 x 16 bytes; i < GN: head-dim columns [32i, 32i + 32) of the tile's keys, else the
  // tile's keys of channels [32(i - GN), ..)
  f32x4 buf[2][4];
  auto fetch = [&](int kt, int i, int to) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      buf[to][c] = i < GN ? *(const f32x4*)(kp + (int64_t)kt * 32 * HD + i * 32 + c * 8)
                          : *(const f32x4*)(vp + (int64_t)(i - GN) * 32 * vt_row_stride + kt * 32 + c * 8);
  };
  if (t0 < t1) fetch(t0, 0, 0);
  for (int kt = t0; kt < t1; ++kt) {
    const int lo = lead - kt * 32;                   // keys [lo, hi) of this tile are real
    const int64_t hi = La - (int64_t)kt * 32;
    const bool ragged = lo > 0 || hi < 32;
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
#pragma unroll
    for (int i = 0; i < GN; ++i) {
      fetch(kt, i + 1, (i + 1) & 1);
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) {                // two chains: an MFMA does not wait for the one before it
          f32x16& s = (c & 1) ? s1 : s0;
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i & 1][c][t], qf[i * 4 + c][t], s, 0, 0, 0);
        }
    }
    s0 += s1;
    if (ragged) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = (r >> 2) * 8 + lg * 4 + (r & 3);
        if (key < lo || key >= hi) s0[r] = -INFINITY;
      }
    }
    float mx = s0[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s0[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx);
    if (__any(mnew > m)) {                           // some query's maximum rose (the first tile: alpha = 0)
      const float alpha = expf(m - mnew);
      l *= alpha;
#pragma unroll
      for (int a = 0; a < GN; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[a][r] *= alpha;
      m = mnew;
    }
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s0[r] = expf(s0[r] - m); ps += s0[r]; }
    l += ps;
    const int nt = kt + 1 < t1 ? kt + 1 : kt;        // past the end: the same tile again, never used
#pragma unroll
    for (int a = 0; a < GN; ++a) {
      if (a + 1 < GN) fetch(kt, GN + a + 1, (GN + a + 1) & 1);
      else fetch(nt, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x4 v = buf[(GN + a) & 1][c];
        if (ragged) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int key = c * 8 + lg * 4 + t;
            if (key < lo || key >= hi) v[t] = 0.f;
          }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) o[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[t], s0[c * 4 + t], o[a], 0, 0, 0);
      }
    }
  }
  l += __shfl_xor(l, 32, 64);

  if constexpr (KG > 1) {                            // the other key groups publish m, l, O^T; group 0 adds them up
    float* mine = xch + (kg - 1) * (GN * 16 + 2) * 64 + lane;
    if (kg > 0) {
      mine[0] = m; mine[64] = l;
#pragma unroll
      for (int a = 0; a < GN; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(2 + a * 16 + r) * 64] = o[a][r];
    }
    __syncthreads();
    if (kg > 0) return;
    float mall = m;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g) mall = fmaxf(mall, xch[g * (GN * 16 + 2) * 64 + lane]);
    // a group without a tile has m = -inf and adds exp(-inf) = 0
    const float w0 = expf(m - mall);
    l *= w0;
#pragma unroll
    for (int a = 0; a < GN; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[a][r] *= w0;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g) {
      const float* other = xch + g * (GN * 16 + 2) * 64 + lane;
      const float w = expf(other[0] - mall);
      l += other[64] * w;
#pragma unroll
      for (int a = 0; a < GN; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[a][r] += other[(2 + a * 16 + r) * 64] * w;
    }
    m = mall;
  }
  // a lane holds channels a*32 + 8g + 4lg + (0..3) of query q0 + lr
  if (parts > 1) {
    float* ps = partial + (size_t)pid * (2 * QB + QB * HD);
    const int ql = qt * 32 + lr;
    if (lg == 0) { ps[ql] = m; ps[QB + ql] = l; }
#pragma unroll
    for (int a = 0; a < GN; ++a)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(f32x4*)(ps + 2 * QB + ((size_t)(a * 8 + g * 2 + lg) * QB + ql) * 4) =
            f32x4{o[a][g * 4], o[a][g * 4 + 1], o[a][g * 4 + 2], o[a][g * 4 + 3]};
    return;
  }
  if (q0 + lr < S) {
    const float inv = 1.f / l;
    float* orow = out + (q0 + lr) * ldo + (int64_t)head * HD + lg * 4;
#pragma unroll
    for (int a = 0; a < GN; ++a)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(f32x4*)(orow + a * 32 + g * 8) = f32x4{o[a][g * 4], o[a][g * 4 + 1], o[a][g * 4 + 2], o[a][g * 4 + 3]} * inv;
  }
}

// O = sum_i e^(m_i - m) O_i / sum_i e^(m_i - m) l_i over the key ranges of a query, m = max_i m_i, in range order.
// One thread per (query, 4 channels); the query index is fastest, so partials are read in whole lines.
template <int HD, int QB>
__global__ __launch_bounds__(256) void k_attn_f32_merge(const float* __restrict__ partial, int blocks, int parts,
                                                        int qblocks, int64_t S, float* __restrict__ out, int64_t ldo) {
  constexpr int C4 = HD / 4, QPB = 256 / C4, SLOT = 2 * QB + QB * HD;
  const int tid = (int)threadIdx.x, gq = (int)blockIdx.x * QPB + tid % QPB, c4 = tid / QPB;
  const int wid = gq / QB, ql = gq % QB;
  if (wid * parts >= blocks) return;
  const int head = wid / qblocks;
  const int64_t qi = (int64_t)(wid % qblocks) * QB + ql;
  if (qi >= S) return;
  const float* ps = partial + (size_t)wid * parts * SLOT;
  float m = -INFINITY, l = 0.f;
  for (int i = 0; i < parts; ++i) m = fmaxf(m, ps[(size_t)i * SLOT + ql]);
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < parts; ++i) {
    const float* pi = ps + (size_t)i * SLOT;
    const float w = expf(pi[ql] - m);
    l += w * pi[QB + ql];
    o += w * *(const f32x4*)(pi + 2 * QB + ((size_t)c4 * QB + ql) * 4);
  }
  *(f32x4*)(out + qi * ldo + (int64_t)head * HD + c4 * 4) = o * (1.f / l);
}

template <int HD, int QG, int KG>
static void launch_cfg(const float* q, int64_t q_head_stride, const float* k, int64_t k_head_stride, int64_t k_row0,
                       const float* vt, int64_t vt_row_stride, int64_t S, int64_t L, int lead, int h, float* out,
                       int64_t ldo, int parts, float* scratch, hipStream_t st) {
  constexpr int QB = QG * 32;
  const int qblocks = (int)((S + QB - 1) / QB), blocks = qblocks * h * parts;
  k_attn_f32<HD, QG, KG><<<(unsigned)((blocks + 7) / 8 * 8), 256, 0, st>>>(
      q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, S, L, lead, out, ldo, 1.0f / sqrtf((float)HD), qblocks, blocks, parts, scratch);
  if (parts > 1) {
    constexpr int QPB = 256 / (HD / 4);
    k_attn_f32_merge<HD, QB><<<(unsigned)(qblocks * h * (QB / QPB)), 256, 0, st>>>(scratch, blocks, parts, qblocks, S, out, ldo);
  }
}

void launch_attn_f32(const float* q, int64_t q_head_stride, const float* k, int64_t k_head_stride,
                     int64_t k_row0, const float* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                     int h, int d, float* out, int64_t ldo, float* scratch, size_t scratch_floats, hipStream_t st) {
  if (S <= 0 || L <= 0) return;
  const int lead = (int)(k_row0 & 3);
  const int64_t nkt = (L + lead + 31) / 32, b4 = (S + 127) / 128 * h;
  // A CU holds two blocks, the chip 512.  Four query tiles a block and whole key ranges if that fills the chip;
  // otherwise either four key groups per block (few keys, or so few queries that even a cut key range would not fill
  // it) or key ranges cut over blocks, as many as make the rounds of 512 blocks shortest.
  int parts = 1;
  const bool groups = b4 < 512 && (nkt < 32 || b4 < 64);
  if (!groups && b4 < 1024) {
    double best = 1e30;
    for (int p = 1; p <= 8 && p * 8 <= nkt; ++p) {
      if (p > 1 && (size_t)(b4 * p) * 128 * (2 + (size_t)d) > scratch_floats) break;
      const double cost = (double)((b4 * p + 511) / 512) / p + 0.01 * p;
      if (cost < best) { best = cost; parts = p; }
    }
  }
#define ATTN_ARGS q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, S, L, lead, h, out, ldo, parts, scratch, st
  if (d == 64) { if (groups) launch_cfg<64, 1, 4>(ATTN_ARGS); else launch_cfg<64, 4, 1>(ATTN_ARGS); }
  else { if (groups) launch_cfg<128, 1, 4>(ATTN_ARGS); else launch_cfg<128, 4, 1>(ATTN_ARGS); }
#undef ATTN_ARGS
}
