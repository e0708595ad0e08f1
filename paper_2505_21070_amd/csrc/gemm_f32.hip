// fp32 GEMM for the DP_F32 path: C = A[M,K] * W[K,N] with a fused epilogue, on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation, nothing rounded below fp32).
//
// Bound: the fp32 matrix rate, 64 cycles an MFMA, 157 TFLOP/s over the chip (the vector unit has half of that without
// its packed forms, and lost more of it to LDS reads: 45 TFLOP/s).  An MFMA sums two k; a lane group lg of a wavefront
// takes k = 8j + 4lg + t for the t-th of four MFMAs, so that the A operand of four is one 16-byte LDS read of a row and
// the W operand one 4-byte read each.  k-tiles (32 deep, 64 where the wavefronts share out K) go through registers into one
// of two LDS buffers, the loads of the next two in flight while one is multiplied (k_gemm_f32).  Rows of As are the k-tile + 4 floats
// and rows of Ws BN + 8 apart: 16 rows x 16 bytes and the two lane groups' rows (4 apart) then fall on different banks.
// K in steps of 32 with rows in 16-byte steps, the usual case, goes through k_gemm_f32_ring (figures there) unless so few tiles are
// to be had that the 32 x 32 ones of k_gemm_f32 are the faster ones (f32_rows).
#include "kernels.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// VEC: rows of A and W are read (and start) in 16-byte steps.  WGM x WGN x WGK wavefronts: WGM x WGN of them share the
// tile's outputs, WGK the k of every k-tile.  WGK = 4 (32 x 32 tiles) is for problems of a few tiles, whose time is the
// chain of MFMAs through K: a quarter of it each, joined through LDS in wavefront order, on four times the blocks.
template <int BM, int BN, int WGM, int WGN, int WGK, int EPI, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A, int64_t lda, GemmF32W w, int64_t ldw,
                                                  int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n, int tiles,
                                                  EpiArgs e) {
  static_assert(WGM * WGN * WGK == 4, "four wavefronts");
  constexpr int BK = 32 * (WGK > 1 ? 2 : 1), AS = BK + 4, WS = BN + 8, PF = 2;
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  constexpr int IA = BM * BK / 4 / 256, IW = BK * BN / 4 / 256;    // 16-byte pieces per thread and tile
  __shared__ __align__(16) float As[2][BM * AS];
  __shared__ __align__(16) float Ws[2][BK * WS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int wm = wave / (WGN * WGK), wn = wave / WGK % WGN, wk = wave % WGK;
  // each XCD takes a contiguous run of tiles, walked in bands of 8 tile rows so that the run is near square and its
  // panels of A and W are shared in that XCD's L2
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= tiles) return;
  const int tn_all = tiles_n * w.n;                                // w.n matrices side by side
  const int band = pid / (8 * tn_all), in_band = pid % (8 * tn_all);
  const int band_rows = tiles_m - band * 8 < 8 ? tiles_m - band * 8 : 8;
  const int tn = in_band / band_rows, sec = tn / tiles_n;
  const int64_t m0 = (int64_t)(band * 8 + in_band % band_rows) * BM, n0 = (int64_t)(tn % tiles_n) * BN;
  const float* __restrict__ W = w.w[sec];
  const float* __restrict__ bias = w.bias[sec];

  float4 ra[PF][IA], rw[PF][IW];
  // VEC: rows and columns beyond M and N read the last ones (what they produce is not stored), so only a k-tile that
  // reaches beyond K needs a look at its elements
  const float *pa[IA], *pw[IW];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int idx = tid + i * 256;
    const int64_t m = m0 + idx / (BK / 4);
    pa[i] = A + (m < M ? m : M - 1) * lda + idx % (BK / 4) * 4;
  }
#pragma unroll
  for (int i = 0; i < IW; ++i) {
    const int idx = tid + i * 256;
    const int64_t n = n0 + idx % (BN / 4) * 4;
    pw[i] = W + (int64_t)(idx / (BN / 4)) * ldw + (!VEC || n < N ? n : N - 4);
  }
  auto fetch = [&](int64_t k0, int z) __attribute__((always_inline)) {
    if (VEC && k0 + BK <= K) {
#pragma unroll
      for (int i = 0; i < IA; ++i) ra[z][i] = *(const float4*)(pa[i] + k0);
#pragma unroll
      for (int i = 0; i < IW; ++i) rw[z][i] = *(const float4*)(pw[i] + k0 * ldw);
      return;
    }
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int64_t k = k0 + (tid + i * 256) % (BK / 4) * 4;
      ra[z][i].x = k < K ? pa[i][k0] : 0.f;
      ra[z][i].y = k + 1 < K ? pa[i][k0 + 1] : 0.f;
      ra[z][i].z = k + 2 < K ? pa[i][k0 + 2] : 0.f;
      ra[z][i].w = k + 3 < K ? pa[i][k0 + 3] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < IW; ++i) {
      const int idx = tid + i * 256;
      const bool ok = k0 + idx / (BN / 4) < K;
      const int64_t n = n0 + idx % (BN / 4) * 4;
      const float* p = pw[i] + k0 * ldw;
      rw[z][i].x = ok && (VEC || n < N) ? p[0] : 0.f;
      rw[z][i].y = ok && (VEC || n + 1 < N) ? p[1] : 0.f;
      rw[z][i].z = ok && (VEC || n + 2 < N) ? p[2] : 0.f;
      rw[z][i].w = ok && (VEC || n + 3 < N) ? p[3] : 0.f;
    }
  };
  auto stash = [&](int b, int z) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int idx = tid + i * 256;
      *(float4*)&As[b][idx / (BK / 4) * AS + idx % (BK / 4) * 4] = ra[z][i];
    }
#pragma unroll
    for (int i = 0; i < IW; ++i) {
      const int idx = tid + i * 256;
      *(float4*)&Ws[b][idx / (BN / 4) * WS + idx % (BN / 4) * 4] = rw[z][i];
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // k-tiles travel PF ahead of the one being multiplied: a tile's MFMAs take 1024 cycles of a SIMD, a load from beyond
  // L2 several times that (one ahead: 488 us where two take 462 at 1560 x 1536 x 8960; three: 497)
  const int KT = (int)((K + BK - 1) / BK);
#pragma unroll
  for (int z = 0; z < PF; ++z)
    if (z < KT) fetch((int64_t)z * BK, z);
  stash(0, 0);
  if (PF < KT) fetch((int64_t)PF * BK, 0);
  __syncthreads();
  auto step = [&](int kt, int z) __attribute__((always_inline)) {
    const int b = kt & 1;
    // half a k-tile's operands are requested together, the second half's behind the first half's first MFMAs: left to
    // itself the compiler reads each operand right in front of the MFMA that waits for it
    constexpr int NJ = BK / 8 / WGK;                 // this wavefront's share of the k-tile, in groups of 8
    float4 a[NJ][TM];
    float bw[NJ][TN][4];
    auto read = [&](int j) __attribute__((always_inline)) {
      const int k = (wk * NJ + j) * 8 + lg * 4;
#pragma unroll
      for (int i = 0; i < TM; ++i) a[j][i] = *(const float4*)&As[b][(wm * TM * 32 + i * 32 + lr) * AS + k];
#pragma unroll
      for (int c = 0; c < TN; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) bw[j][c][t] = Ws[b][(k + t) * WS + wn * TN * 32 + c * 32 + lr];
    };
    read(0);
    read(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int c = 0; c < TN; ++c) {
            const float av = t == 0 ? a[j][i].x : t == 1 ? a[j][i].y : t == 2 ? a[j][i].z : a[j][i].w;
            acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bw[j][c][t], acc[i][c], 0, 0, 0);
          }
      if (j + 2 < NJ) read(j + 2);
      if (j == 0 && kt + 1 < KT) {                   // the next tile's registers are set (z + 1) % PF
        stash(b ^ 1, (z + 1) % PF);
        if (kt + 1 + PF < KT) fetch((int64_t)(kt + 1 + PF) * BK, (z + 1) % PF);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  };
  for (int kt = 0; kt < KT; kt += PF) {
#pragma unroll
    for (int z = 0; z < PF; ++z)
      if (kt + z < KT) step(kt + z, z);
  }

  auto put = [&](int64_t m, int64_t n, float v, float bv, float gv) __attribute__((always_inline)) {
    if (m >= M) return;
    v += bv;
    if (EPI == EPI_GELU) v = gelu_tanh_f(v);
    if (EPI == EPI_RESID) {
      float* x = e.resid + m * e.ldr + n;
      v = *x + gv * v;
      *x = v;
      if (e.out) ((float*)e.out)[m * e.ldo + n] = v;
    } else {
      ((float*)e.out)[m * e.ldo + (int64_t)sec * N + n] = v;
    }
  };
  // accumulator register r of lane group lg: row (r / 4) * 8 + lg * 4 + r % 4, column lr: 32 lanes write 128 bytes of a row
  if constexpr (WGK > 1) {
    static_assert(TM == 1 && TN == 1 && BM == 32 && BN == 32 && 2 * BM * AS >= 4 * 64 * 16, "the tile's partial sums fit As");
    float* part = &As[0][0];                         // free behind the last step's barrier: [wavefront][register][lane]
#pragma unroll
    for (int r = 0; r < 16; ++r) part[(wk * 16 + r) * 64 + lane] = acc[0][0][r];
    __syncthreads();
    const int64_t n = n0 + lr;
    if (n >= N) return;
    const float bv = bias ? bias[n] : 0.f, gv = EPI == EPI_RESID && e.gate ? e.gate[n] : 1.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {                    // wavefront w finishes registers 4w .. 4w + 3
      const int r = wk * 4 + i;
      float v = part[r * 64 + lane];
#pragma unroll
      for (int w2 = 1; w2 < WGK; ++w2) v += part[(w2 * 16 + r) * 64 + lane];
      put(m0 + (r >> 2) * 8 + lg * 4 + (r & 3), n, v, bv, gv);
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < TN; ++c) {
    const int64_t n = n0 + wn * TN * 32 + c * 32 + lr;
    if (n >= N) continue;
    const float bv = bias ? bias[n] : 0.f, gv = EPI == EPI_RESID && e.gate ? e.gate[n] : 1.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) put(m0 + wm * TM * 32 + i * 32 + (r >> 2) * 8 + lg * 4 + (r & 3), n, acc[i][c][r], bv, gv);
  }
}

// Tiles of BM x 64 in a ring of ST k-tiles (32 deep) that are loaded to LDS directly, waited for by count: k_gemm_f32 holds its
// tiles in registers in between and the compiler waits for all of them in front of each LDS store.  Four wavefronts of BM x 16,
// v_mfma_f32_16x16x4_f32 (same rate); lane group g of a wavefront takes k = 16j + 4g + t for the t-th of four MFMAs, so that a
// 16-byte LDS read of A serves four.  BM in steps of 16, so that a launch divides into whole rounds of CUs (see f32_rows).
// Needs K % 32 == 0 and 16-byte steps everywhere.
// Measured (us, k_gemm_f32 -> this): 1560 x 1536 x 8960 residual 461 -> 344 (80 rows), 1560 x 1536 x 1536 residual 89 -> 64 (80), q | k | v
// of 1560 x 1536 241 -> 179 (112), 1560 x 8960 x 1536 GELU 438 -> 381 (112), 6240 x 8960 x 1536 1492 -> 1434 (112); with equal tiles
// (64 x 64) 461 -> 406, 438 -> 391; these in one chain over K, 0 to 1 % faster than now.
// The sum over K is taken in four runs of k-tiles that are added up in order, like the four chains of the 32 x 32 tiles: a layer
// of 840 tokens x 1024 (FFN 4608) is 4.7e-7 from 64 bits on those, 7.0e-7 in one chain, 3.7e-7 this way; 1560 tokens x 1536
// 1.3e-6 in one chain, 6.7e-7 this way.  Runs of 8 k-tiles: 2.8e-7 and 3.7e-7, but 5 and 2 % slower.
template <int BM, int ST, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32_ring(const float* __restrict__ A, int64_t lda, GemmF32W w, int64_t ldw,
                                                       int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n, int tiles, EpiArgs e) {
  constexpr int TM = BM / 16, BN = 64, ACH = BM * 8, STAGE = ACH + BN * 8;         // 16-byte chunks of a k-tile
  constexpr int AI = BM / 8, IA = (AI + 3) / 4, IW = 2, NL = IA + IW;              // load instructions: of A; per wavefront
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  // work ids as in k_gemm_f32
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= tiles) return;
  const int tn_all = tiles_n * w.n;
  const int band = pid / (8 * tn_all), in_band = pid % (8 * tn_all);
  const int band_rows = tiles_m - band * 8 < 8 ? tiles_m - band * 8 : 8;
  const int tn = in_band / band_rows, sec = tn / tiles_n;
  const int64_t m0 = (int64_t)(band * 8 + in_band % band_rows) * BM, n0 = (int64_t)(tn % tiles_n) * BN;
  const float* const pa = A + m0 * lda;
  const float* const pw = w.w[sec] + n0;
  const float* const bias = w.bias[sec];
  const int KT = (int)(K / 32);
  const int64_t left = (M - m0) * lda * 4;
  const uint32_t na = (uint32_t)(left < 0x7fffffff ? left : 0x7fffffff), nw = (uint32_t)(((K - 1) * ldw + N - n0) * 4);
  // A slot p: chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3; W slot p: chunk (p & 15) ^ (((k >> 2) & 3) << 2) of k p >> 4.
  // Rows of A beyond M and rows of W beyond the matrix's end read as zeros; columns beyond N read what is there.
  uint32_t va[IA], vw[IW];
#pragma unroll
  for (int q = 0; q < IA; ++q) { const int p = (q * 4 + wave) * 64 + lane, row = p >> 3; va[q] = (uint32_t)(row * lda + ((p & 7) ^ ((row >> 1) & 7)) * 4) * 4; }
#pragma unroll
  for (int q = 0; q < IW; ++q) { const int p = (q * 4 + wave) * 64 + lane, k = p >> 4; vw[q] = (uint32_t)(k * ldw + ((p & 15) ^ (((k >> 2) & 3) << 2)) * 4) * 4; }
  auto load_tile = [&](int s, int st) __attribute__((always_inline)) {
    uint4* const base = smem + st * STAGE;
#pragma unroll
    for (int q = 0; q < IA; ++q)
      if (q * 4 + 3 < AI || q * 4 + wave < AI) load_lds16(pa, na, va[q], s * 128, base + (q * 4 + wave) * 64);
#pragma unroll
    for (int q = 0; q < IW; ++q) load_lds16(pw, nw, vw[q], (int)(s * 32 * ldw * 4), base + ACH + (q * 4 + wave) * 64);
  };
  const bool all_a = (IA - 1) * 4 + wave < AI;           // the last wavefronts may have one A load less
  auto wait_behind = [&](int behind) __attribute__((always_inline)) {    // tiles issued behind the one waited for
    static_for<ST - 1>([&](auto d_) __attribute__((always_inline)) {
      constexpr int d = decltype(d_)::value;
      if (d == ST - 2 ? behind >= d : behind == d) { if (all_a) vm_wait<d * NL>(); else vm_wait<d * (NL - 1)>(); }
    });
  };
  f32x4 acc[TM], sum[TM];                                // of the last run of k-tiles; of the runs before it
#pragma unroll
  for (int i = 0; i < TM; ++i) acc[i] = sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  const uint32_t fa = lds0 + (uint32_t)lr * 128, xa = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  const uint32_t fw = lds0 + (uint32_t)(ACH + lg * 4 * 16 + ((wave * 4 + (lr >> 2)) ^ (lg * 4))) * 16 + (uint32_t)(lr & 3) * 4;
#pragma unroll
  for (int z = 0; z < ST - 1; ++z) if (z < KT) load_tile(z, z);
  int stage = 0;
  // k-tile s; LAST: one of the last ST - 1, behind which fewer or none have been requested
  auto tile = [&](int s, auto last_) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_)::value;
    __builtin_amdgcn_sched_barrier(0);
    wait_behind(LAST && KT - 1 - s < ST - 2 ? KT - 1 - s : ST - 2);
    __builtin_amdgcn_s_barrier();                        // tile s is there, and everyone is done with tile s - 1
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!LAST) load_tile(s + ST - 1, stage == 0 ? ST - 1 : stage - 1);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t base = (uint32_t)stage * STAGE * 16;
    f32x4 a[2][TM];
    float2 b[2][2];
    static_for<2>([&](auto j_) __attribute__((always_inline)) {
      constexpr int j = decltype(j_)::value;
      const uint32_t ow = fw + base + j * 16 * 256;
      asm volatile("ds_read2_b32 %0, %1 offset0:0 offset1:64" : "=&v"(b[j][0]) : "v"(ow));
      asm volatile("ds_read2_b32 %0, %1 offset0:128 offset1:192" : "=&v"(b[j][1]) : "v"(ow));
      const uint32_t oa = fa + base + (xa ^ (uint32_t)(j * 64));
      static_for<TM>([&](auto i_) __attribute__((always_inline)) { constexpr int i = decltype(i_)::value; a[j][i] = __builtin_bit_cast(f32x4, lds_read16_raw<i * 16 * 128>(oa)); });
    });
    static_for<2>([&](auto j_) __attribute__((always_inline)) {
      constexpr int j = decltype(j_)::value;
      lds_wait<(1 - j) * (TM + 2)>();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float bt = t == 0 ? b[j][0].x : t == 1 ? b[j][0].y : t == 2 ? b[j][1].x : b[j][1].y;
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(bt, a[j][i][t], acc[i], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    stage = stage + 1 == ST ? 0 : stage + 1;
  };
  const int run = (KT + 3) >> 2, full = KT - (ST - 1);   // the last run takes the last tiles in
  int s = 0;
  while (s < full) {
    const int end = s + run < full ? s + run : full;
    for (; s < end; ++s) tile(s, std::false_type{});
    if (s < full) {
#pragma unroll
      for (int i = 0; i < TM; ++i) { sum[i] += acc[i]; acc[i] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    }
  }
  for (; s < KT; ++s) tile(s, std::true_type{});
#pragma unroll
  for (int i = 0; i < TM; ++i) sum[i] += acc[i];
  // W was the A operand: a lane holds row lr of an accumulator tile and the four columns lg * 4 .. + 3
  const int64_t n = n0 + wave * 16 + lg * 4;
  if (n >= N) return;
  const float4 bv = bias ? make_float4(bias[n], bias[n + 1], bias[n + 2], bias[n + 3]) : make_float4(0.f, 0.f, 0.f, 0.f);
  const float4 gv = EPI == EPI_RESID && e.gate ? *(const float4*)(e.gate + n) : make_float4(1.f, 1.f, 1.f, 1.f);
  float4 x[EPI == EPI_RESID ? TM : 1];
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int i = 0; i < TM; ++i) { const int64_t m = m0 + i * 16 + lr; if (m < M) x[i] = *(const float4*)(e.resid + m * e.ldr + n); }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t m = m0 + i * 16 + lr;
    if (m >= M) continue;
    float4 v = make_float4(sum[i][0] + bv.x, sum[i][1] + bv.y, sum[i][2] + bv.z, sum[i][3] + bv.w);
    if (EPI == EPI_GELU) v = make_float4(gelu_tanh_f(v.x), gelu_tanh_f(v.y), gelu_tanh_f(v.z), gelu_tanh_f(v.w));
    if constexpr (EPI == EPI_RESID) {
      v = make_float4(x[i].x + gv.x * v.x, x[i].y + gv.y * v.y, x[i].z + gv.z * v.z, x[i].w + gv.w * v.w);
      *(float4*)(e.resid + m * e.ldr + n) = v;
      if (e.out) {
        float* o = (float*)e.out + m * e.ldo + n;        // the caller's buffer: any alignment
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
      }
    } else {
      *(float4*)((float*)e.out + m * e.ldo + (int64_t)sec * N + n) = v;
    }
  }
}

template <int BM, int ST>
static void launch_f32_ring(const float* A, int64_t lda, const GemmF32W& w, int64_t ldw, int64_t M, int64_t N, int64_t K,
                            int epi, const EpiArgs& e, hipStream_t st) {
  constexpr int lds = (BM + 64) * 128 * ST;
  const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + 63) / 64), tiles = tm * tn * w.n;
  const unsigned grid = (unsigned)((tiles + 7) / 8 * 8);
  static std::atomic<uint64_t> done[3];
#define RING_F32(E, D) allow_dynamic_lds((const void*)k_gemm_f32_ring<BM, ST, E>, lds, D); k_gemm_f32_ring<BM, ST, E><<<grid, 256, lds, st>>>(A, lda, w, ldw, M, N, K, tm, tn, tiles, e)
  if (epi == EPI_STORE) { RING_F32(EPI_STORE, done[0]); }
  else if (epi == EPI_GELU) { RING_F32(EPI_GELU, done[1]); }
  else { RING_F32(EPI_RESID, done[2]); }
#undef RING_F32
}

template <int BM, int BN, int WGM, int WGN, int WGK>
static void launch_cfg(const float* A, int64_t lda, const GemmF32W& w, int64_t ldw, int64_t M, int64_t N, int64_t K,
                       int epi, const EpiArgs& e, bool vec, hipStream_t st) {
  const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN), tiles = tm * tn * w.n;
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8));
#define GEMM_F32(E, V) k_gemm_f32<BM, BN, WGM, WGN, WGK, E, V><<<grid, 256, 0, st>>>(A, lda, w, ldw, M, N, K, tm, tn, tiles, e)
  if (epi == EPI_STORE) { if (vec) GEMM_F32(EPI_STORE, true); else GEMM_F32(EPI_STORE, false); }
  else if (epi == EPI_GELU) { if (vec) GEMM_F32(EPI_GELU, true); else GEMM_F32(EPI_GELU, false); }
  else { if (vec) GEMM_F32(EPI_RESID, true); else GEMM_F32(EPI_RESID, false); }
#undef GEMM_F32
}

// Rows of the ring's tiles, or 0: the 32 x 32 tiles of k_gemm_f32, K dealt over the wavefronts.  Time in us of a k-tile of 32:
// 0.0077 per row of the blocks a CU has side by side (up to three of 48 or 64 rows, two of more: what LDS holds), where a block
// by itself on a CU counts 1.43; and 3.5 for the ends.  32 x 32: 0.235 for up to a block per CU, in proportion beyond, and 3.
// Model / measured: 1560 x 1536 x 8960 80 rows 348 / 344, 64 rows 418 / 406, 160 rows (not built) 416; q | k | v of 1560 x 1536 112 rows
// 169 / 179, 80 rows 181 / 189; 750 x 768 x 3072 48 rows 54 / 54, 32 x 32 54 / 55; 300 x 768 x 3072 32 x 32 26 / 29, 48 rows 54 / 54;
// 1000 x 4096 x 1024 128 rows 67 / 71, 64 rows 71 / 75.
static int f32_rows(int64_t M, int64_t N, int64_t K, int n) {
  const double kt = (double)(K / 32);
  const int64_t t32 = (M + 31) / 32 * ((N + 31) / 32) * n;
  double best = 0.235 * kt * (t32 > 256 ? (double)t32 / 256 : 1.0) + 3;
  int rows = 0;
  for (int bm : {128, 112, 96, 80, 64, 48}) {
    const int64_t t = (M + bm - 1) / bm * ((N + 63) / 64) * n, c = bm <= 64 ? 3 : 2, rem = t % (256 * c), last = (rem + 255) / 256;
    const double units = (double)(t / (256 * c) * c) + (last == 1 ? 1.43 : (double)last);
    const double cost = 0.0077 * units * bm * kt + 3.5;
    if (cost < best) { best = cost; rows = bm; }
  }
  return rows;
}
// Tiles of k_gemm_f32 for what the ring does not take: K in other steps than 32, rows that do not start in 16-byte steps.  128 x 128,
// two to a CU and half the operand bytes per flop, where they make at least two full rounds; 64 x 64, up to four to a CU; fewer
// than one of those per CU: 32 x 32 with K dealt over the wavefronts.  The lines were measured at aligned sizes, before those
// went to the ring (us): 1560 x 8960 x 1536 (910 of the large tiles) 64 x 64 391, 128 x 128 413; 1560 x 1536 x 8960 (156) 462 and 639;
// 6240 x 8960 x 1536 (3430) 128 x 128 1432, 8 % less than 64 x 64; a stage of 128 tokens x 128 channels 32 x 32 148, 64 x 64 200, of
// 300 x 768 210 and 301, of 750 x 768 340 and 379.
static int f32_tile(int64_t M, int64_t N, int n) {
  if ((M + 127) / 128 * ((N + 127) / 128) * n >= 1024) return 128;
  return (M + 63) / 64 * ((N + 63) / 64) * n >= 256 ? 64 : 32;
}

void launch_gemm_f32(const float* A, int64_t lda, const GemmF32W& w, int64_t ldw, int64_t M, int64_t N,
                     int64_t K, int epi, const EpiArgs& e, hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  bool vec = K % 4 == 0 && N % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)A & 15) == 0;
  for (int i = 0; i < w.n; ++i) vec = vec && ((uintptr_t)w.w[i] & 15) == 0;
  const bool out_vec = epi == EPI_RESID ? e.ldr % 4 == 0 && ((uintptr_t)e.resid & 15) == 0 && ((uintptr_t)e.gate & 15) == 0
                                        : e.ldo % 4 == 0 && ((uintptr_t)e.out & 15) == 0;
  if (vec && out_vec && K % 32 == 0 && K * ldw * 4 < 0x7fffffff && lda < (1 << 22)) {
    switch (f32_rows(M, N, K, w.n)) {
      case 48: launch_f32_ring<48, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      case 64: launch_f32_ring<64, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      case 80: launch_f32_ring<80, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      case 96: launch_f32_ring<96, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      case 112: launch_f32_ring<112, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      case 128: launch_f32_ring<128, 3>(A, lda, w, ldw, M, N, K, epi, e, st); break;
      default: launch_cfg<32, 32, 1, 1, 4>(A, lda, w, ldw, M, N, K, epi, e, vec, st);
    }
    return;
  }
  switch (f32_tile(M, N, w.n)) {
    case 128: launch_cfg<128, 128, 2, 2, 1>(A, lda, w, ldw, M, N, K, epi, e, vec, st); break;
    case 64: launch_cfg<64, 64, 2, 2, 1>(A, lda, w, ldw, M, N, K, epi, e, vec, st); break;
    default: launch_cfg<32, 32, 1, 1, 4>(A, lda, w, ldw, M, N, K, epi, e, vec, st);
  }
}

// For the tests, which state the kernel that each of their products is meant to reach: rows of the ring's tiles (-1: not the ring's
// K, 0: its 32 x 32 tiles); the other products' tiles; and one product by itself.
extern "C" int32_t dp_gemm_f32_rows(int64_t M, int64_t N, int64_t K, int32_t n) { return K % 32 ? -1 : f32_rows(M, N, K, n); }
extern "C" int32_t dp_gemm_f32_tile(int64_t M, int64_t N, int32_t n) { return f32_tile(M, N, n); }
extern "C" void dp_gemm_f32_run(const float* A, int64_t lda, const float* W, int64_t ldw, const float* bias, int64_t M, int64_t N, int64_t K,
                                int32_t epi, float* out, int64_t ldo, float* resid, int64_t ldr, const float* gate, void* hip_stream) {
  launch_gemm_f32(A, lda, GemmF32W{{W}, {bias}, 1}, ldw, M, N, K, epi, EpiArgs{out, ldo, nullptr, resid, ldr, gate}, (hipStream_t)hip_stream);
}
