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
// Bound: the fp32 matrix rate (64 cycles an MFMA; 157 TFLOP/s over the chip).  Many queries: k_attn_f32_tiles, four query
// tiles that share key tiles in LDS.  Few: k_attn_f32, a query tile and four key groups that read operands straight from
// L1/L2.  1560 queries x 3120 keys x 12 heads x 128: 366 us with every wavefront's operands from L1 -> 313 us with tiles in LDS,
// + 9 (merge), = 96 TFLOP/s; 1560 x 512 keys 77 us; 128 x 192 x 2 heads x 64 10 us.
#include "kernels.h"

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One key tile's scores s (S^T, masked) of a lane's query against the running maximum m and this lane's share l of the sum:
// s becomes the probabilities, o is rescaled where some query's maximum rose (the first tile: alpha = 0).  Scores of -inf weigh 0 also
// where a query has had no others yet (m still -inf).
template <int GN>
__device__ __forceinline__ void softmax_tile(f32x16& s, f32x16 (&o)[GN], float& m, float& l) {
  float mx = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float mnew = fmaxf(m, mx);
  if (__any(mnew > m)) {
    const float alpha = expf(m - (mnew == -INFINITY ? 0.f : mnew));
    l *= alpha;
#pragma unroll
    for (int a = 0; a < GN; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[a][r] *= alpha;
    m = mnew;
  }
  const float ref = m == -INFINITY ? 0.f : m;
  float ps = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) { s[r] = expf(s[r] - ref); ps += s[r]; }
  l += ps;
}
// scores of keys outside [lo, hi) of the tile
__device__ __forceinline__ void mask_scores(f32x16& s, int lg, int lo, int64_t hi) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int key = (r >> 2) * 8 + lg * 4 + (r & 3);
    if (key < lo || key >= hi) s[r] = -INFINITY;
  }
}
// the same for piece c of a channel's values: what lies there is not this call's
__device__ __forceinline__ void mask_values(f32x4& v, int c, int lg, int lo, int64_t hi) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int key = c * 8 + lg * 4 + t;
    if (key < lo || key >= hi) v[t] = 0.f;
  }
}

// Four wavefronts walk the same keys for four query tiles.  A tile of 32 keys (K rows, V^T columns) goes to LDS directly, one
// tile ahead, each byte once per block; straight from L1 an operand read is 32 rows of 32 bytes, 32 such reads a wavefront
// and tile, and no depth of prefetch hid them.  Measured with it: matrix pipes busy 78 % of the time a CU has a block (66 %
// before), no bank conflicts; what is left is the softmax between the two products and 468 blocks on 512 places.
// Two blocks of 64 KB (head_dim 128) fit a CU.  Slot p of the K tile: chunk (p % CK) ^ (row & 15) of row p / CK; of the V^T tile:
// chunk (p & 7) ^ ((row >> 1) & 7) of channel p >> 3: 16 rows read at one chunk cover all banks.
// parts > 1: a block takes one of `parts` key ranges and leaves (m, l, O) unnormalised for k_attn_f32_merge.
template <int HD>
__global__ __launch_bounds__(256, 2) void k_attn_f32_tiles(const float* __restrict__ q, int64_t q_head_stride,
                                                           const float* __restrict__ k, int64_t k_head_stride,
                                                           int64_t k_row0, const float* __restrict__ vt,
                                                           int64_t vt_row_stride, int64_t S, int64_t L, int lead,
                                                           float* __restrict__ out, int64_t ldo, float scale, int qblocks,
                                                           int blocks, int parts, float* __restrict__ partial) {
  constexpr int GN = HD / 32, QB = 128, CK = HD / 4, KCH = 32 * CK, STAGE = 2 * KCH, NI = KCH / 256;   // NI: load instructions of a wavefront, K and V^T each
  __shared__ __align__(256) uint4 smem[2 * STAGE];
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // as in k_attn_f32
  if (pid >= blocks) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int wid = pid / parts, part = pid % parts, head = wid / qblocks;
  const int64_t q0 = (int64_t)(wid % qblocks) * QB + wave * 32;
  const int64_t La = L + lead;                       // `lead` as in k_attn_f32
  const int NKT = (int)((La + 31) / 32);
  const int t0 = (int)((int64_t)part * NKT / parts), t1 = (int)((int64_t)(part + 1) * NKT / parts);

  const float* const kp = k + (int64_t)head * k_head_stride + (k_row0 - lead) * HD;
  const float* const vp = vt + (int64_t)head * HD * vt_row_stride + (k_row0 - lead);
  const uint32_t nv = (uint32_t)(7 * vt_row_stride + 32) * 4;      // eight channels' pieces of one tile: one instruction
  // an instruction is 1 KiB: rows of K from (n * 4 + wave) * (64 / CK) on, 4096 bytes further for every n; row & 15 in the
  // swizzle flips its bit 3 with n at head_dim 128
  const int krow = wave * (64 / CK) + lane / CK;
  const uint32_t vk = (uint32_t)(krow * CK + ((lane % CK) ^ (krow & 15))) * 16;
  // channels from (n * 4 + wave) * 8 on: (channel >> 1) & 7 = 4 * (wave & 1) + (lane >> 4)
  const uint32_t vv = (uint32_t)((lane >> 3) * vt_row_stride + (((lane & 7) ^ ((wave & 1) * 4 + (lane >> 4))) * 4)) * 4;
  auto load_tile = [&](int kt, int st) __attribute__((always_inline)) {
    uint4* const base = smem + st * STAGE;
#pragma unroll
    for (int n = 0; n < NI; ++n) load_lds16(kp + (int64_t)kt * 32 * HD, 32 * HD * 4, HD == 128 && (n & 1) ? vk ^ 128u : vk, n * 4096, base + (n * 4 + wave) * 64);
#pragma unroll
    for (int n = 0; n < NI; ++n)
      load_lds16(vp + (int64_t)(n * 4 + wave) * 8 * vt_row_stride + kt * 32, nv, vv, 0, base + KCH + (n * 4 + wave) * 64);
  };
  if (t0 < t1) load_tile(t0, 0);

  f32x4 qf[HD / 8];
  {
    const int64_t row = q0 + lr < S ? q0 + lr : S - 1;
    const float* qr = q + (int64_t)head * q_head_stride + row * HD + lg * 4;
#pragma unroll
    for (int j = 0; j < HD / 8; ++j) qf[j] = *(const f32x4*)(qr + j * 8) * scale;
  }
  f32x16 o[GN];
#pragma unroll
  for (int a = 0; a < GN; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[a][r] = 0.f;
  float m = -INFINITY, l = 0.f;                      // l: this lane's share (its own 16 keys of every tile)

  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  const uint32_t fk = lds0 + (uint32_t)lr * (HD * 4) + (uint32_t)(lg ^ (lr & 15)) * 16;
  const uint32_t fv = lds0 + KCH * 16 + (uint32_t)lr * 128 + (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  f32x4 buf[2][4];
  // operand group i of the tile at byte offset st: 4 x 16 bytes; i < GN: head-dim columns [32i, 32i + 32) of the tile's keys,
  // else the tile's keys of channels [32(i - GN), ..)
  auto fetch = [&](auto i_, uint32_t st) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    static_for<4>([&](auto c_) __attribute__((always_inline)) {
      constexpr int c = decltype(c_)::value;
      if constexpr (i < GN) buf[i & 1][c] = __builtin_bit_cast(f32x4, lds_read16_raw<(i >> 1) * 256>((fk + st) ^ (uint32_t)((i & 1) * 128 + c * 32)));
      else buf[i & 1][c] = __builtin_bit_cast(f32x4, lds_read16_raw<(i - GN) * 4096>((fv + st) ^ (uint32_t)(c * 32)));
    });
  };
  for (int kt = t0; kt < t1; ++kt) {
    const int stage = (kt - t0) & 1;
    const uint32_t st = (uint32_t)stage * (STAGE * 16);
    __builtin_amdgcn_sched_barrier(0);
    vm_wait<0>();
    __builtin_amdgcn_s_barrier();                    // tile kt is there, and everyone is done with tile kt - 1
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < t1) load_tile(kt + 1, stage ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    fetch(std::integral_constant<int, 0>{}, st);
    const int lo = lead - kt * 32;                   // keys [lo, hi) of this tile are real
    const int64_t hi = La - (int64_t)kt * 32;
    const bool ragged = lo > 0 || hi < 32;
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
    static_for<GN>([&](auto i_) __attribute__((always_inline)) {
      constexpr int i = decltype(i_)::value;
      fetch(std::integral_constant<int, i + 1>{}, st);
      lds_wait<4>();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) {                // two chains: an MFMA does not wait for the one before it
          f32x16& s = (c & 1) ? s1 : s0;
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i & 1][c][t], qf[i * 4 + c][t], s, 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    });
    lds_wait<0>();                                   // the first group of V^T: nothing is in flight over the softmax
    __builtin_amdgcn_sched_barrier(0);
    s0 += s1;
    if (ragged) mask_scores(s0, lg, lo, hi);
    softmax_tile<GN>(s0, o, m, l);
    static_for<GN>([&](auto a_) __attribute__((always_inline)) {
      constexpr int a = decltype(a_)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (a + 1 < GN) { fetch(std::integral_constant<int, GN + a + 1>{}, st); lds_wait<4>(); }
      else lds_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x4 v = buf[(GN + a) & 1][c];
        if (ragged) mask_values(v, c, lg, lo, hi);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[t], s0[c * 4 + t], o[a], 0, 0, 0);
      }
    });
  }
  l += __shfl_xor(l, 32, 64);
  // a lane holds channels a*32 + 8g + 4lg + (0..3) of query q0 + lr
  if (parts > 1) {
    float* ps = partial + (size_t)pid * (2 * QB + QB * HD);
    const int ql = wave * 32 + lr;
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

// Few queries or few keys: a block owns 32 queries of one head, and the key tiles are dealt to its four wavefronts, which
// meet in LDS at the end, so that blocks are a quarter as long.  A 16-byte operand read feeds four MFMAs = 256 cycles, and
// operands come straight from L1/L2, one group of four reads ahead (1024 cycles of MFMAs).
template <int HD>
__global__ __launch_bounds__(256, 2) void k_attn_f32(const float* __restrict__ q, int64_t q_head_stride,
                                                     const float* __restrict__ k, int64_t k_head_stride,
                                                     int64_t k_row0, const float* __restrict__ vt,
                                                     int64_t vt_row_stride, int64_t S, int64_t L, int lead,
                                                     float* __restrict__ out, int64_t ldo, float scale, int qblocks,
                                                     int blocks) {
  constexpr int KG = 4, GN = HD / 32;                // key groups; operand groups of K per tile, and of V^T
  __shared__ float xch[(KG - 1) * (GN * 16 + 2) * 64];
  // every XCD (blocks are dealt round-robin) takes a contiguous run of work: one head's blocks share its L2
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= blocks) return;
  const int lane = threadIdx.x & 63, kg = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int head = pid / qblocks;
  const int64_t q0 = (int64_t)(pid % qblocks) * 32;
  // The key range starts at a 16-byte boundary of the V^T rows: `lead` keys in front of the first real one and those
  // at or beyond lead + L are masked (and their V taken as 0: what lies there is not this call's).
  const int64_t La = L + lead;
  const int NKT = (int)((La + 31) / 32);
  const int t0 = (int)((int64_t)kg * NKT / KG), t1 = (int)((int64_t)(kg + 1) * NKT / KG);

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
    if (ragged) mask_scores(s0, lg, lo, hi);
    softmax_tile<GN>(s0, o, m, l);
    const int nt = kt + 1 < t1 ? kt + 1 : kt;        // past the end: the same tile again, never used
#pragma unroll
    for (int a = 0; a < GN; ++a) {
      if (a + 1 < GN) fetch(kt, GN + a + 1, (GN + a + 1) & 1);
      else fetch(nt, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x4 v = buf[(GN + a) & 1][c];
        if (ragged) mask_values(v, c, lg, lo, hi);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[t], s0[c * 4 + t], o[a], 0, 0, 0);
      }
    }
  }
  l += __shfl_xor(l, 32, 64);

  // the other key groups publish m, l, O^T; group 0 adds them up
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
  // a lane holds channels a*32 + 8g + 4lg + (0..3) of query q0 + lr
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

// Key ranges of k_attn_f32_tiles (more than one: joined by the merge kernel), or 0: k_attn_f32.
// A CU holds two blocks, the chip 512.  Four query tiles a block and whole key ranges if that fills the chip;
// otherwise either four key groups per block (few keys, or so few queries that even a cut key range would not fill
// it) or key ranges cut over blocks, as many as make the rounds of 512 blocks shortest.
static int attn_f32_ranges(int64_t S, int64_t L, int lead, int h, int d, size_t scratch_floats) {
  const int64_t nkt = (L + lead + 31) / 32, b4 = (S + 127) / 128 * h;
  if (b4 < 512 && (nkt < 32 || b4 < 64)) return 0;
  int parts = 1;
  if (b4 < 1024) {
    double best = 1e30;
    for (int p = 1; p <= 8 && p * 8 <= nkt; ++p) {
      if (p > 1 && (size_t)(b4 * p) * 128 * (2 + (size_t)d) > scratch_floats) break;
      const double cost = (double)((b4 * p + 511) / 512) / p + 0.01 * p;
      if (cost < best) { best = cost; parts = p; }
    }
  }
  return parts;
}
// for the tests, which state the kernel that each of their shapes is meant to reach
extern "C" int32_t dp_attn_f32_ranges(int64_t S, int64_t L, int64_t k_row0, int32_t h, int32_t d, int64_t scratch_floats) {
  return attn_f32_ranges(S, L, (int)(k_row0 & 3), h, d, (size_t)scratch_floats);
}

void launch_attn_f32(const float* q, int64_t q_head_stride, const float* k, int64_t k_head_stride,
                     int64_t k_row0, const float* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                     int h, int d, float* out, int64_t ldo, float* scratch, size_t scratch_floats, hipStream_t st) {
  if (S <= 0 || L <= 0) return;
  const int lead = (int)(k_row0 & 3);
  const float scale = 1.0f / sqrtf((float)d);
  const int parts = attn_f32_ranges(S, L, lead, h, d, scratch_floats);
  if (parts == 0) {
    const int qblocks = (int)((S + 31) / 32), blocks = qblocks * h;
#define GROUPS_CASE(HD) k_attn_f32<HD><<<(unsigned)((blocks + 7) / 8 * 8), 256, 0, st>>>(q, q_head_stride, k, k_head_stride, k_row0, vt, \
    vt_row_stride, S, L, lead, out, ldo, scale, qblocks, blocks)
    if (d == 64) GROUPS_CASE(64); else GROUPS_CASE(128);
#undef GROUPS_CASE
    return;
  }
  const int qblocks = (int)((S + 127) / 128), blocks = qblocks * h * parts;
#define TILES_CASE(HD) do { \
    k_attn_f32_tiles<HD><<<(unsigned)((blocks + 7) / 8 * 8), 256, 0, st>>>(q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, \
        S, L, lead, out, ldo, scale, qblocks, blocks, parts, scratch); \
    if (parts > 1) k_attn_f32_merge<HD, 128><<<(unsigned)(qblocks * h * (128 * HD / 1024)), 256, 0, st>>>(scratch, blocks, parts, qblocks, S, out, ldo); \
  } while (0)
  if (d == 64) TILES_CASE(64); else TILES_CASE(128);
#undef TILES_CASE
}
