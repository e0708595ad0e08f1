// bf16 GEMM on the gfx950 matrix cores: C[M,N] = A[M,K] * Wt[N,K]^T, fp32 accumulate, fused epilogue.
// Both operands are K-contiguous, so every MFMA operand fragment is one 16-byte LDS read.
//
// k-tiles go HBM -> LDS directly (no staging registers, no LDS stores).  Large and mid-size problems run as blocks of eight
// wavefronts, two to a SIMD, that take turns at multiplying and at reading their next operands (k_gemm_turns); problems of few
// tiles take small tiles and a ring of loads (k_gemm_ring, k_gemm_thin).  Which takes what: tile_family, big_tile, cut_tile.
// LDS rows are 128 bytes (64 bf16); LDS serves 16 lanes x 16 bytes per cycle from 64 banks, i.e. two rows per
// bank sweep, so the 16-byte chunk index is XOR-swizzled with (row >> 1) & 7, which spreads a column of
// chunks over all banks.
//
// 16-bit outputs are staged through LDS so that global memory is written in whole rows, 16 bytes per lane; the fp32 residual
// update too in tiles of 128 and 160 rows, in the taller ones it takes 64 bytes of a row per four lanes as the accumulators lie.  EPI_HEADS stores per attention head (q | k | v
// sections: channel gains, 3D rotation, transposed V, row sums of squares for a deferred RMSNorm).
#include "kernels.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// tanh-GELU through the logistic function: 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u))
__device__ __forceinline__ float gelu_tanh_fast(float v) {
  const float u2 = -2.0f * 0.7978845608028654f * 1.4426950408889634f * (v + 0.044715f * v * v * v);   // -2u log2(e)
  return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u2));
}

// A block's epilogue over its BM x BN tile, 16-bit outputs; LB: bytes of LDS (free by now) that it may stage through.
template <int BM, int BN, int WGM, int WGN, int TM, int TN, int EPI, int LB>
__device__ __forceinline__ void finish_tile(f32x4 (&acc)[TM][TN], uint4* smem, int64_t m0, int64_t n0, int64_t M,
                                            int64_t N, int sec, bool swapped, const EpiArgs& e, const HeadsArgs& ha) {
  // The MFMAs ran with the weight rows as the A operand, so a lane holds, per accumulator tile, the output row
  // m = .. + lr and the four consecutive columns n = .. + lg*4 + (0..3).
  // The tile goes through LDS (free now) so that global memory sees whole rows: 16 bytes per lane,
  // consecutive lanes on consecutive addresses.  LDS rows are XOR-swizzled with the row index so that
  // neither the column-wise writes nor the row-wise reads conflict on banks.
  constexpr int NW = WGM * WGN, NT = NW * 64, WM = BM / WGM, WN = BN / WGN;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
  constexpr int XM = BN / 4 < 32 ? BN / 4 - 1 : 31;      // row bits in the XOR: a row of 8-byte units has BN / 4 of them
  const bf16_t* bias = (const bf16_t*)e.bias;
  if constexpr (EPI == EPI_HEADS) {
    // Sections of `dim` columns, each stored per attention head (see HeadsArgs).  A plain section gets, per
    // output row, the sum of squares of (acc + bias) over this tile's columns, taken from the fp32
    // accumulators; its channel gains and 3D rotation are applied on the way out of the staging tile, where
    // a lane holds 8 consecutive channels of one row, so that the table and gain reads are contiguous
    // across lanes.  A transposed section is C^T already.
    constexpr int UPR = BN / 4, CPR = BN / 8;
    // Plain sections of 128-column tiles are staged in fp32, so that only the result is rounded, as by the separate kernels
    // (staged in bf16, 64-column tiles left a layer of dim 1664 2.58e-3 from 64 bits, 2.50e-3 this way and by those, in
    // the same time).  The wider tiles' fp32 rows do not all fit.
    constexpr bool WIDE = BN == 128 && BM * BN * 4 + BM * WGN * 4 <= LB;
    constexpr int SB = WIDE ? 4 : 2;
    static_assert(BM * BN * SB + BM * WGN * 4 <= LB, "EPI_HEADS stages the whole tile at once");
    float* const red = (float*)smem + BM * BN * SB / 4;  // [row][wavefront column]: sums of squares
    const HeadSection sc = ha.sec[sec];
    const int64_t nsec = n0 - (int64_t)sec * ha.dim;     // first column of this tile inside its section
    const int hshift = ha.head_dim == 128 ? 7 : 6, hmask = ha.head_dim - 1;
    uint2* l8 = (uint2*)smem;
    __syncthreads();
    if (swapped) {
      // C^T: a lane holds channel wn * WN + j * 16 + lr and, per quad, four consecutive output rows; staged as BN rows of BM
      constexpr int TU = BM / 4, TX = TU % 32 == 0 ? 31 : 7;           // 8-byte units of a row, row bits in the XOR
      static_assert(TU % 8 == 0, "the XOR stays inside a row");
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * WN + j * 16 + lr;
        const float bvr = bias && n0 + row < N ? bf16_to_f32(bias[n0 + row]) : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const uint2 pk = make_uint2(cvt_pk_bf16(acc[i][j][0] + bvr, acc[i][j][1] + bvr), cvt_pk_bf16(acc[i][j][2] + bvr, acc[i][j][3] + bvr));
          l8[row * TU + (((wm * WM + i * 16) / 4 + lg) ^ (row & TX))] = pk;
        }
      }
      __syncthreads();
      for (int c = tid; c < BN * (BM / 8); c += NT) {
        const int row = c / (BM / 8), p = c % (BM / 8);
        uint4 d = smem[c];
        if (row & 1) d = make_uint4(d.z, d.w, d.x, d.y);
        const int64_t m = m0 + (p ^ ((row & TX) >> 1)) * 8;
        if (n0 + row < N && m < M)
          __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)((bf16_t*)sc.dst + (nsec + row) * sc.ld + sc.row0 + m));
      }
      return;
    }
    float ss[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) ss[i] = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int nl = wn * WN + j * 16 + lg * 4;
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (bias && n0 + nl < N) {
        const uint2 b4 = *(const uint2*)(bias + n0 + nl);
        bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
        bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * 16 + lr;
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[i][j][t] + bv[t];
          ss[i] += v[t] * v[t];
        }
        const int u = row * UPR + ((nl >> 2) ^ (row & XM));
        if constexpr (WIDE) ((float4*)smem)[u] = make_float4(v[0], v[1], v[2], v[3]);
        else l8[u] = make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float tot = ss[i];
      tot += __shfl_xor(tot, 16, 64);
      tot += __shfl_xor(tot, 32, 64);
      if (lg == 0) red[(wm * WM + i * 16 + lr) * WGN + wn] = tot;
    }
    __syncthreads();
    if (sc.ssq) {
      // one value per row and tile, tile-major so that rows are contiguous: ssq[tile in section][m]
      for (int row = tid; row < BM; row += NT) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < WGN; ++w) tot += red[row * WGN + w];
        if (m0 + row < M) sc.ssq[(nsec / BN) * ha.ssq_stride + m0 + row] = tot;
      }
    }
    // A lane always takes the same two logical chunks (8 consecutive columns each), BN / 2 columns apart, of
    // its rows, so its gains and channel-pair indices are fixed, and where BN / 2 is a multiple of the head
    // width both chunks rotate by the same table entries.  The loads of a group of rows (staging tile,
    // rotation table) are issued together.
    constexpr int HC = CPR / 2, RP2 = 64 / HC, IT = BM / NW / RP2, G = 4;
    static_assert(BM / NW % RP2 == 0, "rows per wavefront");
    const int c8 = (lane % HC) * 8;                      // first column of chunk 0; chunk 1 starts at c8 + BN / 2
    const bool rotate = sc.rope, scale = sc.gain || sc.rope;
    const bool share = (BN / 2) % ha.head_dim == 0;      // both chunks use the same channel pairs
    const int half = ha.head_dim >> 1;
    float gg[2][8];
    int nn[2], p0[2];
    bool col_ok[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      nn[k] = (int)nsec + c8 + k * (BN / 2);             // first of the chunk's 8 channels inside the section
      p0[k] = (nn[k] & hmask) >> 1;
      col_ok[k] = n0 + c8 + k * (BN / 2) < N;
#pragma unroll
      for (int t = 0; t < 8; ++t) gg[k][t] = 1.f;
      if (sc.gain && col_ok[k]) {
        const float4 g0 = *(const float4*)(sc.gain + nn[k]), g1 = *(const float4*)(sc.gain + nn[k] + 4);
        gg[k][0] = g0.x; gg[k][1] = g0.y; gg[k][2] = g0.z; gg[k][3] = g0.w;
        gg[k][4] = g1.x; gg[k][5] = g1.y; gg[k][6] = g1.z; gg[k][7] = g1.w;
      }
    }
#pragma unroll
    for (int it0 = 0; it0 < IT; it0 += G) {
      uint4 d[G][2];
      float4 df[WIDE ? G : 1][2][2];
      float4 cs[G][2][2];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (it0 + g < IT) {
          const int row = wave * (BM / NW) + (it0 + g) * RP2 + lane / HC;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            if constexpr (WIDE) {
#pragma unroll
              for (int u = 0; u < 2; ++u) df[WIDE ? g : 0][k][u] = ((const float4*)smem)[row * UPR + (((c8 >> 2) + k * (BN / 8) + u) ^ (row & XM))];
              continue;
            }
            d[g][k] = smem[row * CPR + (((c8 >> 3) + k * HC) ^ ((row & XM) >> 1))];
            if (row & 1) d[g][k] = make_uint4(d[g][k].z, d[g][k].w, d[g][k].x, d[g][k].y);
          }
          if (rotate && m0 + row < M) {
            const float4* t = (const float4*)(ha.cs + (m0 + row) * half + p0[0]);
            cs[g][0][0] = t[0]; cs[g][0][1] = t[1];
            if (!share) {
              const float4* t1 = (const float4*)(ha.cs + (m0 + row) * half + p0[1]);
              cs[g][1][0] = t1[0]; cs[g][1][1] = t1[1];
            }
          }
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (it0 + g < IT) {
          const int row = wave * (BM / NW) + (it0 + g) * RP2 + lane / HC;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            if (m0 + row < M && col_ok[k]) {
              const int64_t m = m0 + row;
              uint4 dv = d[g][k];
              if (scale || WIDE) {
                const uint32_t w[4] = {dv.x, dv.y, dv.z, dv.w};
                const float4 f0 = df[WIDE ? g : 0][k][0], f1 = df[WIDE ? g : 0][k][1];
                const float f[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
                const float4 c0 = cs[g][share ? 0 : k][0], c1 = cs[g][share ? 0 : k][1];
                const float csv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
                float v[8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  float a = (WIDE ? f[2 * u] : bf16_to_f32((bf16_t)(w[u] & 0xffff))) * gg[k][2 * u];
                  float b = (WIDE ? f[2 * u + 1] : bf16_to_f32((bf16_t)(w[u] >> 16))) * gg[k][2 * u + 1];
                  if (rotate) {
                    const float a2 = a * csv[2 * u] - b * csv[2 * u + 1], b2 = a * csv[2 * u + 1] + b * csv[2 * u];
                    a = a2; b = b2;
                  }
                  v[2 * u] = a; v[2 * u + 1] = b;
                }
                if (WIDE && sc.wide) {
                  float4* const o = (float4*)(sc.wide + m * ha.dim + nn[k]);
                  o[0] = make_float4(v[0], v[1], v[2], v[3]); o[1] = make_float4(v[4], v[5], v[6], v[7]);
                  continue;
                }
                dv = make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
              }
              // non-temporal like the other streamed outputs (same-box A/B, 14400 x 15360 x 5120: 1915 -> 1851 us)
              __builtin_nontemporal_store(u32x4{dv.x, dv.y, dv.z, dv.w}, (u32x4*)((bf16_t*)sc.dst + (int64_t)(nn[k] >> hshift) * sc.ld + (sc.row0 + m) * ha.head_dim + (nn[k] & hmask)));
            }
          }
        }
      }
    }
  } else {
    constexpr int UPR = BN / 4;                          // 8-byte units (4 bf16) per LDS row
    constexpr int CPR = BN / 8, RPI = 64 / CPR;          // 16-byte chunks per row, rows per wavefront read
    // the whole tile at once if it fits the two operand buffers, else one wavefront row (WM rows) per pass
    constexpr int SP = BM * BN * 2 <= LB ? 1 : WGM, RP = BM / SP;
    uint2* l8 = (uint2*)smem;
#pragma unroll
    for (int pass = 0; pass < SP; ++pass) {
      __syncthreads();                                   // the operand tiles / the previous pass are done with
      if (SP == 1 || wm == pass) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int nl = wn * WN + j * 16 + lg * 4;
          float bv[4] = {0.f, 0.f, 0.f, 0.f};
          if (bias && n0 + nl < N) {
            const uint2 b4 = *(const uint2*)(bias + n0 + nl);
            bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
            bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
          }
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int row = (SP == 1 ? wm * WM : 0) + i * 16 + lr;      // row inside this pass
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              v[t] = acc[i][j][t] + bv[t];
              if (EPI == EPI_GELU) v[t] = gelu_tanh_fast(v[t]);
            }
            uint2 pk;
            pk.x = cvt_pk_bf16(v[0], v[1]);
            pk.y = cvt_pk_bf16(v[2], v[3]);
            l8[row * UPR + ((nl >> 2) ^ (row & XM))] = pk;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < RP / NW / RPI; ++it) {
        const int row = wave * (RP / NW) + it * RPI + lane / CPR, p = lane % CPR;
        uint4 d = smem[row * CPR + p];
        // the chunk read holds units 2p and 2p+1 of the swizzled row, i.e. the two halves of logical
        // chunk p ^ ((row & XM) >> 1), exchanged when the row index is odd
        if (row & 1) d = make_uint4(d.z, d.w, d.x, d.y);
        const int64_t m = m0 + pass * RP + row, n = n0 + (p ^ ((row & XM) >> 1)) * 8;
        // streamed out once; non-temporal so that the output does not displace the operand panels the other
        // tiles still re-read from the caches (measured at the 14400 x 13824 x 5120 GELU shape: -3 %)
        if (m < M && n < N) __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)((bf16_t*)e.out + m * e.ldo + n));
      }
    }
  }
}

// Small problems: 64 x 64 tiles, 2 x 2 wavefronts of 32 x 32, k-tiles of 64 in a ring of ST LDS stages.  A small tile's k-tile is
// multiplied in a fraction of the time its loads travel, and a small problem has no second block to fill the gap, so ST - 1
// k-tiles are in flight: tile kt is waited for by its place in the queue of vector loads (they arrive in order), not by an empty
// queue.
// What bounds it is latency: the launch, one trip to memory, a barrier, LDS reads and four dependent MFMAs per k-tile, and the
// epilogue's own reads.  Those (bias, gate, residual rows, gains, rotations) are requested before anything else here and are there
// when the sums are; against requesting them behind the main loop (us, back to back): 500 x 1024 x 1024 residual 10.1 -> 7.8, 1560 x
// 512 x 512 residual 8.4 -> 6.2, 1008 x 1536 x 512 per-head stores 9.1 -> 8.4, 1008 x 1024 x 256 GELU 4.9 -> 4.3.  A second group of four
// wavefronts with a ring of its own for every other k-tile changed nothing (20.2 -> 19.0 at K = 4096): a CU's operand path is busy.
template <int ST, int EPI>
__global__ __launch_bounds__(256) void k_gemm_ring(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ Bt,
                                                        int64_t ldb, int64_t M, int64_t N, int64_t K, int tiles_n, int tiles,
                                                        int parts, EpiArgs e, HeadsArgs ha) {
  constexpr int NL = 4, STAGE = 128 * 8;                 // loads per wavefront and k-tile, 16-byte chunks of a k-tile
  extern __shared__ uint4 smem[];                        // ST stages
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  // work ids as in k_gemm_turns: a contiguous run per XCD, tiles in bands of 4 tile rows
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= tiles * parts) return;
  const int part = EPI == EPI_PART ? pid / tiles : 0, tile = EPI == EPI_PART ? pid % tiles : pid;
  const int tiles_m = tiles / tiles_n;
  const int band = tile / (4 * tiles_n), in_band = tile % (4 * tiles_n);
  const int band_rows = tiles_m - band * 4 < 4 ? tiles_m - band * 4 : 4;
  const int64_t m0 = (int64_t)(band * 4 + in_band % band_rows) * 64, n0 = (int64_t)(in_band / band_rows) * 64;
  const int kt0 = EPI == EPI_PART ? (int)((K / 64) * part / parts) : 0;
  const int KT = EPI == EPI_PART ? (int)((K / 64) * (part + 1) / parts) - kt0 : (int)(K / 64);
  int sec = 0;
  bool exch = false;
  if constexpr (EPI == EPI_HEADS) { sec = (int)(n0 / ha.dim); exch = ha.sec[sec].transposed != 0; }

  // the epilogue's operands; a thread's columns and rows are known now
  const bf16_t* const bias = (const bf16_t*)e.bias;
  uint2 b4[4] = {};
  float4 gv[4], xv[4];
  if constexpr (EPI != EPI_PART) {
    if (bias) {
      if (exch) { const int64_t n = n0 + wn * 32 + lr; b4[0].x = n < N ? (uint32_t)bias[n] : 0u; }
      else
#pragma unroll
        for (int q = 0; q < 4; ++q) { const int64_t n = n0 + wn * 32 + q * 8 + lg * 4; if (n < N) b4[q] = *(const uint2*)(bias + n); }
    }
  }
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t n = n0 + wn * 32 + q * 8 + lg * 4;
      gv[q] = e.gate && n < N ? *(const float4*)(e.gate + n) : make_float4(1.f, 1.f, 1.f, 1.f);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = (t * 256 + tid) >> 4, c = (tid & 15) ^ (row & 15);
      if (m0 + row < M && n0 + c * 4 < N) xv[t] = *(const float4*)(e.resid + (m0 + row) * e.ldr + n0 + c * 4);
    }
  }
  // EPI_HEADS: a thread takes columns c8 .. c8 + 7 and 32 more of them at c8 + 32 of row tid / 4
  const int hrow = tid >> 2, c8 = (tid & 3) * 8;
  const int64_t nsec = n0 - (int64_t)sec * ha.dim;       // first column of this tile inside its section
  float4 hg[2][2], hc[2][2];
  bool rotate = false, gains = false;
  if constexpr (EPI == EPI_HEADS) {
    rotate = !exch && ha.sec[sec].rope; gains = !exch && ha.sec[sec].gain;
    const int half = ha.head_dim >> 1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int n = (int)nsec + c8 + k * 32;
      if (gains) { hg[k][0] = *(const float4*)(ha.sec[sec].gain + n); hg[k][1] = *(const float4*)(ha.sec[sec].gain + n + 4); }
      if (rotate && m0 + hrow < M) {
        const float4* t = (const float4*)(ha.cs + (m0 + hrow) * half + ((n & (ha.head_dim - 1)) >> 1));
        hc[k][0] = t[0]; hc[k][1] = t[1];
      }
    }
  }

  // slot p of a tile holds chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3
  const bf16_t *ga[2], *gb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = (wave * 2 + i) * 64 + lane, row = p >> 3, ch = (p & 7) ^ ((row >> 1) & 7);
    ga[i] = A + (m0 + row) * lda + kt0 * 64 + ch * 8;
    gb[i] = Bt + (n0 + row) * ldb + kt0 * 64 + ch * 8;
  }
  auto load_tile = [&](int s, int st) __attribute__((always_inline)) {
    uint4* const base = smem + st * STAGE + wave * 128;
#pragma unroll
    for (int i = 0; i < 2; ++i) __builtin_amdgcn_global_load_lds((glb_void_t*)(ga[i] + s * 64), (lds_void_t*)(base + i * 64), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) __builtin_amdgcn_global_load_lds((glb_void_t*)(gb[i] + s * 64), (lds_void_t*)(base + 512 + i * 64), 16, 0, 0);
  };
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  const uint32_t fa = lds0 + (uint32_t)(wm * 32 + lr) * 128, fb = lds0 + 8192 + (uint32_t)(wn * 32 + lr) * 128;
  const uint32_t sx = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  __builtin_amdgcn_sched_barrier(0);                     // the epilogue's reads go first
#pragma unroll
  for (int z = 0; z < ST - 1; ++z) if (z < KT) load_tile(z, z);
  auto multiply = [&](auto exch_) __attribute__((always_inline)) {
    constexpr bool EXCH = decltype(exch_)::value;
    int stage = 0;
    for (int s = 0; s < KT; ++s) {
      const int behind = KT - 1 - s;                     // tiles behind this one that are (or were) still to come
      __builtin_amdgcn_sched_barrier(0);
      static_for<ST - 1>([&](auto r_) __attribute__((always_inline)) {
        constexpr int r = decltype(r_)::value;           // in flight behind tile s: min(ST - 2, behind)
        if (r == ST - 2 ? behind >= r : behind == r) vm_wait<r * NL>();
      });
      __builtin_amdgcn_s_barrier();                      // tile s is there, and everyone is done with tile s - 1
      __builtin_amdgcn_sched_barrier(0);
      if (s + ST - 1 < KT) load_tile(s + ST - 1, stage == 0 ? ST - 1 : stage - 1);
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t base = (uint32_t)stage * STAGE * 16;
      bf16x8 af[4], bfr[4];
      static_for<4>([&](auto k_) __attribute__((always_inline)) {
        constexpr int k = decltype(k_)::value;
        const uint32_t o = base + (sx ^ (uint32_t)(k * 32));
        af[k] = __builtin_bit_cast(bf16x8, lds_read16_raw<0>(fa + o));
        bfr[k] = __builtin_bit_cast(bf16x8, lds_read16_raw<0>(fb + o));
      });
      static_for<4>([&](auto k_) __attribute__((always_inline)) {
        constexpr int k = decltype(k_)::value;
        lds_wait<(3 - k) * 2>();
        __builtin_amdgcn_sched_barrier(0);
        // the weight rows are the A operand: a lane holds output row lr and four consecutive columns per register quad
        acc = EXCH ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[k], bfr[k], acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[k], af[k], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      stage = stage + 1 == ST ? 0 : stage + 1;
    }
  };
  if constexpr (EPI == EPI_HEADS) { if (exch) multiply(std::true_type{}); else multiply(std::false_type{}); }
  else multiply(std::false_type{});

  __syncthreads();                                       // the ring is free
  auto bias4 = [&](int q, float (&bv)[4]) __attribute__((always_inline)) {
    bv[0] = bf16_to_f32((bf16_t)(b4[q].x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4[q].x >> 16));
    bv[2] = bf16_to_f32((bf16_t)(b4[q].y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4[q].y >> 16));
  };
  const int row_in = wm * 32 + lr;                       // this lane's row of the tile
  if constexpr (EPI == EPI_RESID || EPI == EPI_PART) {
    float4* const l16 = (float4*)smem;                   // 64 x 64 floats, 16-byte chunks XOR-swizzled with the row
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float bv[4];
      bias4(q, bv);
      const float4 g = EPI == EPI_RESID ? gv[q] : make_float4(1.f, 1.f, 1.f, 1.f);
      l16[row_in * 16 + ((wn * 8 + q * 2 + lg) ^ (row_in & 15))] =
          make_float4(g.x * (acc[q * 4] + bv[0]), g.y * (acc[q * 4 + 1] + bv[1]), g.z * (acc[q * 4 + 2] + bv[2]), g.w * (acc[q * 4 + 3] + bv[3]));
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = (t * 256 + tid) >> 4, c = (tid & 15) ^ (row & 15);
      const int64_t m = m0 + row, n = n0 + c * 4;
      if (m >= M || n >= N) continue;
      const float4 v = l16[t * 256 + tid];
      if constexpr (EPI == EPI_PART) {
        *(float4*)(e.resid + ((int64_t)part * M + m) * e.ldr + n) = v;
      } else {
        float4 x = xv[t];
        x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
        *(float4*)(e.resid + m * e.ldr + n) = x;
        if (e.out) *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(x.x, x.y), cvt_pk_bf16(x.z, x.w));
      }
    }
  } else {
    uint2* const l8 = (uint2*)smem;                      // 64 x 64 bf16, 8-byte units XOR-swizzled with the row
    float4* const l16 = (float4*)smem;                   // EPI_HEADS, plain sections: 64 x 64 fp32, so that only the result is rounded
    float* const red = (float*)(smem + 1024);            // EPI_HEADS: [row][wavefront column] sums of squares
    if (EPI == EPI_HEADS && exch) {
      // C^T: row = channel wn * 32 + lr, four consecutive output rows per quad
      const int row = wn * 32 + lr;
      const float bvr = bf16_to_f32((bf16_t)b4[0].x);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        l8[row * 16 + ((wm * 8 + q * 2 + lg) ^ (row & 15))] =
            make_uint2(cvt_pk_bf16(acc[q * 4] + bvr, acc[q * 4 + 1] + bvr), cvt_pk_bf16(acc[q * 4 + 2] + bvr, acc[q * 4 + 3] + bvr));
    } else {
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float bv[4], v[4];
        bias4(q, bv);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[q * 4 + t] + bv[t];
          ss += v[t] * v[t];
          if (EPI == EPI_GELU) v[t] = gelu_tanh_fast(v[t]);
        }
        const int u = row_in * 16 + ((wn * 8 + q * 2 + lg) ^ (row_in & 15));
        if constexpr (EPI == EPI_HEADS) l16[u] = make_float4(v[0], v[1], v[2], v[3]);
        else l8[u] = make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
      }
      if constexpr (EPI == EPI_HEADS) {
        ss += __shfl_xor(ss, 32, 64);
        if (lg == 0) red[row_in * 2 + wn] = ss;
      }
    }
    __syncthreads();
    // 16-byte chunk c of a staged row: units 2c and 2c + 1 lie in chunk c ^ ((row & 15) >> 1), exchanged for odd rows
    auto chunk = [&](int row, int c) __attribute__((always_inline)) {
      const uint4 d = smem[row * 8 + (c ^ ((row & 15) >> 1))];
      return row & 1 ? make_uint4(d.z, d.w, d.x, d.y) : d;
    };
    if constexpr (EPI == EPI_HEADS) {
      const HeadSection& sc = ha.sec[sec];
      if (exch) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const uint4 d = chunk(hrow, (tid & 3) + k * 4);
          const int64_t m = m0 + c8 + k * 32;
          if (m < M) __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)((bf16_t*)sc.dst + (nsec + hrow) * sc.ld + sc.row0 + m));
        }
        return;
      }
      // one value per row and tile, tile-major so that rows are contiguous: ssq[tile in section][m]
      if (sc.ssq && tid < 64 && m0 + tid < M) sc.ssq[(nsec >> 6) * ha.ssq_stride + m0 + tid] = red[tid * 2] + red[tid * 2 + 1];
      const int64_t m = m0 + hrow;
      if (m >= M) return;
      const int hshift = ha.head_dim == 128 ? 7 : 6, hmask = ha.head_dim - 1;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int n = (int)nsec + c8 + k * 32;
        const int unit = (tid & 3) * 2 + k * 8;
        const float4 f0 = l16[hrow * 16 + (unit ^ (hrow & 15))], f1 = l16[hrow * 16 + ((unit + 1) ^ (hrow & 15))];
        const float f[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
        const float gs[8] = {hg[k][0].x, hg[k][0].y, hg[k][0].z, hg[k][0].w, hg[k][1].x, hg[k][1].y, hg[k][1].z, hg[k][1].w};
        const float cs[8] = {hc[k][0].x, hc[k][0].y, hc[k][0].z, hc[k][0].w, hc[k][1].x, hc[k][1].y, hc[k][1].z, hc[k][1].w};
        float v[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float a = f[2 * u], b = f[2 * u + 1];
          if (gains) { a *= gs[2 * u]; b *= gs[2 * u + 1]; }
          if (rotate) {
            const float a2 = a * cs[2 * u] - b * cs[2 * u + 1], b2 = a * cs[2 * u + 1] + b * cs[2 * u];
            a = a2; b = b2;
          }
          v[2 * u] = a; v[2 * u + 1] = b;
        }
        if (sc.wide) {
          float4* const o = (float4*)(sc.wide + m * ha.dim + n);
          o[0] = make_float4(v[0], v[1], v[2], v[3]); o[1] = make_float4(v[4], v[5], v[6], v[7]);
          continue;
        }
        const uint4 d = make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
        __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)((bf16_t*)sc.dst + (int64_t)(n >> hshift) * sc.ld + (sc.row0 + m) * ha.head_dim + (n & hmask)));
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int row = (t * 256 + tid) >> 3, c = tid & 7;
        const uint4 d = chunk(row, c);
        const int64_t m = m0 + row, n = n0 + c * 8;
        if (m < M && n < N) __builtin_nontemporal_store(u32x4{d.x, d.y, d.z, d.w}, (u32x4*)((bf16_t*)e.out + m * e.ldo + n));
      }
    }
  }
}

template <int ST, int EPI>
static void launch_ring(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N, int64_t K,
                        const EpiArgs& e, hipStream_t st, int parts) {
  constexpr int lds = 128 * 128 * ST;
  const int tm = (int)((M + 63) / 64), tn = (int)((N + 63) / 64);
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_gemm_ring<ST, EPI>, lds, done);
  HeadsArgs ha{};
  if (EPI == EPI_HEADS) { e.heads->ssq_np = e.heads->dim / 64; ha = *e.heads; }
  k_gemm_ring<ST, EPI><<<(unsigned)((tm * tn * parts + 7) / 8 * 8), 256, lds, st>>>(A, lda, Wt, ldw, M, N, K, tn, tm * tn, parts, e, ha);
}
template <int ST>
static bool launch_ring_cfg(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N, int64_t K,
                            int epi, const EpiArgs& e, hipStream_t st, int parts) {
  if (epi == EPI_STORE) launch_ring<ST, EPI_STORE>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_GELU) launch_ring<ST, EPI_GELU>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_RESID) launch_ring<ST, EPI_RESID>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_HEADS) launch_ring<ST, EPI_HEADS>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_PART) launch_ring<ST, EPI_PART>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else return false;
  return true;
}

// The smallest problems: 32 x 64 tiles, and the k-tiles of 64 dealt to the eight wavefronts (wavefront w: tiles w, w + 8, ...), each
// through its own piece of LDS, nobody waiting for anybody until the eight partial sums are added up in LDS, in wavefront order.
// A CU reads operands at about 80 GB/s whatever the tile, so a 64 x 64 tile takes 0.2 us per k-tile however many are in flight;
// where even these smaller tiles fill at most one round of CUs, 12 KB instead of 16 per k-tile and more CUs is what helps, and
// up to eight k-tiles arrive together.  The epilogue's operands are requested first of all.  Measured (us, back to back,
// k_gemm_ring -> this): 216 x 256 x 256 residual 4.2 -> 3.4, 500 x 512 x 512 5.5 -> 4.6, 500 x 1024 x 1024 7.8 -> 6.5, 216 x 256 x 1024
// 7.5 -> 5.7, 216 x 1536 x 512 per-head stores 6.3 -> 5.8; beyond one round the ring is faster: 1008 x 1024 x 1024 (512 tiles) 8.6
// against 10.4.
template <int EPI>
__global__ __launch_bounds__(512) void k_gemm_thin(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ Bt,
                                                  int64_t ldb, int64_t M, int64_t N, int64_t K, int tiles_n, int tiles,
                                                  EpiArgs e, HeadsArgs ha) {
  constexpr int SLAB = 96 * 8;                           // 16-byte chunks of a k-tile: 32 rows of A, 64 of the weights
  extern __shared__ uint4 smem[];                        // 8 * SLAB
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // a contiguous run per XCD
  if (pid >= tiles) return;
  const int64_t m0 = (int64_t)(pid / tiles_n) * 32, n0 = (int64_t)(pid % tiles_n) * 64;
  const int KT = (int)(K / 64), parts = KT < 8 ? KT : 8;
  int sec = 0;
  bool exch = false;                                     // operands exchanged: C^T
  if constexpr (EPI == EPI_HEADS) { sec = (int)(n0 / ha.dim); exch = ha.sec[sec].transposed != 0; }
  const int64_t nsec = n0 - (int64_t)sec * ha.dim;       // first column of this tile inside its section

  // This thread's outputs: columns n .. n + 3 of row m, or (C^T) rows m .. m + 3 of channel n; and what they need
  const int row = exch ? tid >> 3 : tid >> 4, c = exch ? tid & 7 : tid & 15;
  const int64_t m = m0 + (exch ? c * 4 : row), n = n0 + (exch ? row : c * 4);
  const bool here = m < M && n < N;
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  float4 x = {}, g = make_float4(1.f, 1.f, 1.f, 1.f), cs = {};
  if (here) {
    const bf16_t* const bias = (const bf16_t*)e.bias;
    if (bias && exch) {
      bv[0] = bv[1] = bv[2] = bv[3] = bf16_to_f32(bias[n]);
    } else if (bias) {
      const uint2 b4 = *(const uint2*)(bias + n);
      bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
      bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
    }
    if constexpr (EPI == EPI_RESID) {
      x = *(const float4*)(e.resid + m * e.ldr + n);
      if (e.gate) g = *(const float4*)(e.gate + n);
    }
    if constexpr (EPI == EPI_HEADS) {
      const HeadSection& sc = ha.sec[sec];
      const int ns = (int)nsec + c * 4;
      if (!exch && sc.gain) g = *(const float4*)(sc.gain + ns);
      if (!exch && sc.rope) cs = *(const float4*)(ha.cs + m * (ha.head_dim >> 1) + ((ns & (ha.head_dim - 1)) >> 1));
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  if (wave < parts) {
    uint4* const mine = smem + wave * SLAB;
    // slot p of a k-tile holds chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3; rows of A first.  Instruction i loads rows
    // i * 8 .. i * 8 + 7, so a lane has two swizzles, for even and odd i.
    const bf16_t *ga[2], *gb[2];
    const int r8 = lane >> 3;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int at = wave * 64 + ((lane & 7) ^ (((o * 8 + r8) >> 1) & 7)) * 8;
      ga[o] = A + (m0 + r8) * lda + at;
      gb[o] = Bt + (n0 + r8) * ldb + at;
    }
    auto load = [&](int t) __attribute__((always_inline)) {             // k-tile wave + 8 t
#pragma unroll
      for (int i = 0; i < 4; ++i) __builtin_amdgcn_global_load_lds((glb_void_t*)(ga[i & 1] + i * 8 * lda + t * 512), (lds_void_t*)(mine + i * 64), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i) __builtin_amdgcn_global_load_lds((glb_void_t*)(gb[i & 1] + i * 8 * ldb + t * 512), (lds_void_t*)(mine + (4 + i) * 64), 16, 0, 0);
    };
    load(0);
    f32x16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
    const uint32_t fa = (uint32_t)(uintptr_t)(lds_void_t*)mine + (uint32_t)lr * 128, sx = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
    const int mt = (KT - wave + 7) / 8;
    auto multiply = [&](auto exch_) __attribute__((always_inline)) {
      constexpr bool EXCH = decltype(exch_)::value;
      for (int t = 0; t < mt; ++t) {
        vm_wait<0>();
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 af[4], bfr[4][2];
        static_for<4>([&](auto k_) __attribute__((always_inline)) {
          constexpr int k = decltype(k_)::value;
          const uint32_t o = fa + (sx ^ (uint32_t)(k * 32));
          af[k] = __builtin_bit_cast(bf16x8, lds_read16_raw<0>(o));
          bfr[k][0] = __builtin_bit_cast(bf16x8, lds_read16_raw<32 * 128>(o));
          bfr[k][1] = __builtin_bit_cast(bf16x8, lds_read16_raw<64 * 128>(o));
        });
        lds_wait<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < mt) load(t + 1);                     // this k-tile is in registers: its LDS is free
        static_for<4>([&](auto k_) __attribute__((always_inline)) {
          constexpr int k = decltype(k_)::value;
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[b] = EXCH ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[k], bfr[k][b], acc[b], 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[k][b], af[k], acc[b], 0, 0, 0);
        });
      }
      // 32 x 64 (C^T: 64 x 32) floats over this wavefront's own k-tile, 16-byte chunks XOR-swizzled with the row
      float4* const l16 = (float4*)mine;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int at = EXCH ? (b * 32 + lr) * 8 + ((q * 2 + lg) ^ (lr & 7)) : lr * 16 + ((b * 8 + q * 2 + lg) ^ (lr & 15));
          l16[at] = make_float4(acc[b][q * 4], acc[b][q * 4 + 1], acc[b][q * 4 + 2], acc[b][q * 4 + 3]);
        }
    };
    if constexpr (EPI == EPI_HEADS) { if (exch) multiply(std::true_type{}); else multiply(std::false_type{}); }
    else multiply(std::false_type{});
  }
  __syncthreads();
  const float4* const l16 = (const float4*)smem + (exch ? row * 8 + (c ^ (row & 7)) : row * 16 + (c ^ (row & 15)));
  float4 s = l16[0];
  auto add = [&](int w) __attribute__((always_inline)) {
    const float4 p = l16[w * SLAB];
    s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
  };
  if (parts == 8) {
#pragma unroll
    for (int w = 1; w < 8; ++w) add(w);
  } else {
    for (int w = 1; w < parts; ++w) add(w);
  }
  float v[4] = {s.x + bv[0], s.y + bv[1], s.z + bv[2], s.w + bv[3]};
  if constexpr (EPI == EPI_RESID) {
    if (!here) return;
    x.x += g.x * v[0]; x.y += g.y * v[1]; x.z += g.z * v[2]; x.w += g.w * v[3];
    *(float4*)(e.resid + m * e.ldr + n) = x;
    if (e.out) *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(x.x, x.y), cvt_pk_bf16(x.z, x.w));
  } else if constexpr (EPI == EPI_HEADS) {
    const HeadSection& sc = ha.sec[sec];
    if (exch) {
      if (here) *(uint2*)((bf16_t*)sc.dst + (nsec + row) * sc.ld + sc.row0 + m) = make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
      return;
    }
    if (sc.ssq) {
      // sum of squares over the tile's 64 columns: the 16 threads of a row
      float ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
      if (c == 0 && m < M) sc.ssq[(nsec >> 6) * ha.ssq_stride + m] = ss;
    }
    if (!here) return;
    v[0] *= g.x; v[1] *= g.y; v[2] *= g.z; v[3] *= g.w;
    if (sc.rope) {
      const float a0 = v[0] * cs.x - v[1] * cs.y, b0 = v[0] * cs.y + v[1] * cs.x;
      const float a1 = v[2] * cs.z - v[3] * cs.w, b1 = v[2] * cs.w + v[3] * cs.z;
      v[0] = a0; v[1] = b0; v[2] = a1; v[3] = b1;
    }
    const int ns = (int)nsec + c * 4, hshift = ha.head_dim == 128 ? 7 : 6;
    if (sc.wide) { *(float4*)(sc.wide + m * ha.dim + ns) = make_float4(v[0], v[1], v[2], v[3]); return; }
    *(uint2*)((bf16_t*)sc.dst + (int64_t)(ns >> hshift) * sc.ld + (sc.row0 + m) * ha.head_dim + (ns & (ha.head_dim - 1))) =
        make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
  } else {
    if (!here) return;
    if (EPI == EPI_GELU) {
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = gelu_tanh_fast(v[t]);
    }
    *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
  }
}

template <int EPI>
static void launch_thin(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N, int64_t K,
                        const EpiArgs& e, hipStream_t st) {
  constexpr int lds = 96 * 128 * 8;
  const int tm = (int)((M + 31) / 32), tn = (int)((N + 63) / 64);
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_gemm_thin<EPI>, lds, done);
  HeadsArgs ha{};
  if (EPI == EPI_HEADS) { e.heads->ssq_np = e.heads->dim / 64; ha = *e.heads; }
  k_gemm_thin<EPI><<<(unsigned)((tm * tn + 7) / 8 * 8), 512, lds, st>>>(A, lda, Wt, ldw, M, N, K, tn, tm * tn, e, ha);
}
static bool launch_thin_cfg(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N, int64_t K,
                            int epi, const EpiArgs& e, hipStream_t st) {
  if (epi == EPI_STORE) launch_thin<EPI_STORE>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_GELU) launch_thin<EPI_GELU>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_RESID) launch_thin<EPI_RESID>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_HEADS) launch_thin<EPI_HEADS>(A, lda, Wt, ldw, M, N, K, e, st);
  else return false;
  return true;
}

// Tiles of 128 rows and more: 2 x 4 wavefronts of (TM * 16) x (TN * 16), v_mfma_f32_16x16x32_bf16, k-slabs of 64.  The two
// wavefronts of a SIMD (one of each block half) take turns: while one multiplies a slab, the other reads its next slab's
// fragments into registers and issues its share of the tile loads, with a barrier at every change of roles.  Nothing is
// interleaved by hand, a wavefront needs no second fragment buffer, and once both halves have read a slab its LDS is free, a
// whole multiplication before the next reader: with 64 KB slabs two stages are enough.  A half alone reads its rows of A and
// loads them itself, so its A stage is free one turn earlier than the weights', which have a third stage where it fits (256
// and 192 rows); every load has two to four turns to land and is waited for by its place in the queue.  Turns of 320 rows are
// cut in two, 32 deep: its accumulators leave registers for half a slab's fragments.
// What bounds it: the matrix pipes under the power limit.  256 x 256 at 14400 x 15360 x 5120 runs at 1.46 PFLOP/s, where
// 16x16x32 MFMAs alone, on such data and without any memory traffic, reach 1.57 to 1.62.  Against the two layouts before
// (pinned order with fragments read ahead, 32x32x16, two stages, for 192 to 320 rows; turns over three stages whose loads were
// waited for before the multiplication, for 128 and 160), plain store or as named, us: 14400 x 15360 x 5120 1750 -> 1552; GELU
// 14400 x 13824 x 5120 1603 -> 1450, 6240 x 8960 x 1536 171 -> 153, 3600 x 13824 x 5120 451 -> 388, 1560 x 8960 x 1536 50 -> 43;
// residual 14400 x 5120 x 13824 1727 -> 1521, 14400 x 5120 x 5120 712 -> 621, 6240 x 1536 x 8960 152 -> 135, 18720 x 1536 x 8960
// 480 -> 399; 6240 x 4608 x 1536 85 -> 75, 7800 x 4608 x 1536 107 -> 92.  32x32x16 MFMAs in the same turns: 1680 instead of 1545 at
// 14400 x 15360 x 5120; slabs of 32 in four stages: 1840.
template <int TM, int TN> struct Turns {
  static constexpr int WGM = 2, WGN = 4, WM = TM * 16, WN = TN * 16, BM = WGM * WM, BN = WGN * WN;
  static constexpr int ACH = BM * 8, BCH = BN * 8;       // 16-byte chunks of a slab: 128 bytes of every row
  static constexpr int MAX = 160 * 1024 / 16, N0 = MAX / (ACH + BCH), SA = N0 < 4 ? N0 : 4;      // LDS stages of A's slabs
  static constexpr int SB = SA < 4 && SA * ACH + (SA + 1) * BCH <= MAX ? SA + 1 : SA;            // and of the weights'
  static constexpr int LDS = (SA * ACH + SB * BCH) * 16;
};
template <int TM, int TN, int EPI>
__global__ __launch_bounds__(512) void k_gemm_turns(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ Bt,
                                                   int64_t ldb, int64_t M, int64_t N, int64_t K, int tiles_n, int tiles,
                                                   int parts, EpiArgs e, HeadsArgs ha) {
  typedef Turns<TM, TN> G;
  constexpr int WGN = G::WGN, WM = G::WM, WN = G::WN, BM = G::BM, BN = G::BN, ACH = G::ACH, BCH = G::BCH, SA = G::SA, SB = G::SB;
  constexpr int DA = SA - 1, DB = SB - 1, D = DB;      // slabs in flight
  constexpr int NA = (ACH / 2 + 255) / 256, NB = BCH / 512;              // loads per wavefront and slab
  constexpr bool RAG = ACH / 2 % 256 != 0;               // the last wavefronts of a half have one A load less
  constexpr int PH = TM * TN * 4 + (TM + TN) * 8 <= 230 ? 2 : 1;         // k-steps of 32 that are multiplied in one turn
  static_assert(BCH % 512 == 0 && ACH / 2 % 64 == 0, "whole wavefront instructions");
  extern __shared__ uint4 smem[];                        // SA slabs of A, SB of the weights
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  // Blocks are dealt round-robin over the 8 XCDs, each with its own L2: give every XCD a contiguous run
  // of work ids (row-major tiles, so neighbours share the A row-panel and walk the B panels together).
  // The grid is padded to a multiple of 8; the padding blocks have nothing to do.
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= tiles * parts) return;
  const int part = EPI == EPI_PART ? pid / tiles : 0, tile = EPI == EPI_PART ? pid % tiles : pid;   // K range, output tile
  // tiles are walked in bands of 4 tile rows, column by column inside a band: the ~32 blocks an XCD runs
  // at a time then cover about 4 x 8 tiles and share 4 A panels and 8 B panels instead of 1 and 32
  const int tiles_m = tiles / tiles_n;
  const int band = tile / (4 * tiles_n), in_band = tile % (4 * tiles_n);
  const int band_rows = tiles_m - band * 4 < 4 ? tiles_m - band * 4 : 4;
  const int64_t m0 = (int64_t)(band * 4 + in_band % band_rows) * BM, n0 = (int64_t)(in_band / band_rows) * BN;
  const int s0 = EPI == EPI_PART ? (int)((K / 64) * part / parts) : 0;
  const int NS = EPI == EPI_PART ? (int)((K / 64) * (part + 1) / parts) - s0 : (int)(K / 64);

  // Slot p of a slab holds chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3.  Rows beyond the matrix read as zeros.
  const bf16_t* const pa = A + m0 * lda + s0 * 64;
  const bf16_t* const pb = Bt + n0 * ldb + s0 * 64;
  const int64_t left_a = ((M - m0) * lda - s0 * 64) * 2, left_b = ((N - n0) * ldb - s0 * 64) * 2;
  const uint32_t na = (uint32_t)(left_a < 0x7fffffff ? left_a : 0x7fffffff), nb = (uint32_t)(left_b < 0x7fffffff ? left_b : 0x7fffffff);
  uint32_t va[NA], vb[NB];
#pragma unroll
  for (int q = 0; q < NA; ++q) { const int p = wm * (ACH / 2) + (q * 4 + wn) * 64 + lane, row = p >> 3; va[q] = (uint32_t)(row * lda + ((p & 7) ^ ((row >> 1) & 7)) * 8) * 2; }
#pragma unroll
  for (int q = 0; q < NB; ++q) { const int p = (q * 8 + wave) * 64 + lane, row = p >> 3; vb[q] = (uint32_t)(row * ldb + ((p & 7) ^ ((row >> 1) & 7)) * 8) * 2; }
  const bool all_a = !RAG || ((NA - 1) * 4 + wn) * 64 < ACH / 2;
  auto load_a = [&](int s, int st) __attribute__((always_inline)) {
    uint4* const base = smem + st * ACH + wm * (ACH / 2);
#pragma unroll
    for (int q = 0; q < NA; ++q) if (q < NA - 1 || all_a) load_lds16(pa, na, va[q], s * 128, base + (q * 4 + wn) * 64);
  };
  auto load_b = [&](int s, int st) __attribute__((always_inline)) {
    uint4* const base = smem + SA * ACH + st * BCH;
#pragma unroll
    for (int q = 0; q < NB; ++q) load_lds16(pb, nb, vb[q], s * 128, base + (q * 8 + wave) * 64);
  };
  // at most `a` slabs' A loads and `b` slabs' weight loads of this wavefront outstanding
  auto wait_loads = [&](auto a_, auto b_) __attribute__((always_inline)) {
    constexpr int a = decltype(a_)::value, b = decltype(b_)::value;
    if (all_a) vm_wait<a * NA + b * NB>(); else vm_wait<a * (NA - 1) + b * NB>();
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  const int lr = lane & 15, lg = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  const uint32_t fa = lds0 + (uint32_t)(wm * WM + lr) * 128, fb = lds0 + (uint32_t)(SA * ACH) * 16 + (uint32_t)(wn * WN + lr) * 128;
  const uint32_t sx = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;             // a lane's rows are 16 apart: one swizzle for all of them

  // EPI_RESID: the fp32 residual values that this lane's accumulators are added to, requested a few tile rows ahead.  A lane
  // holds four consecutive columns of a row, so four lanes take 64 bytes of it and the next column tile the 64 beside them.
  // Rows and columns beyond the matrix lie beyond the buffer: they read as zeros and are not written.
  constexpr bool FP32 = EPI == EPI_RESID || EPI == EPI_PART;
  constexpr int XP = 2 * PH;
  // Tiles of 128 and 160 rows, which run in about one round of blocks, all update the residual stream at the same time:
  // theirs goes through LDS, GI accumulator rows of both block halves a step, so that memory sees whole rows, and the first step's
  // residual rows are requested ahead of the last multiplication (in a stage, as it lies / staged in us: 3648 x 1600 x 1600 36.7 / 34.3,
  // 1760 x 2560 x 2560 50.3 / 47.7, 1400 x 3968 x 3968 66.5 / 63.8, 1560 x 3072 x 3072 51.9 / 49.2; 160 rows
  // 16704 x 256 x 256 20.0 / 17.0, 4288 x 1216 x 5824 97.3 / 91.5; 128 x 128 13568 x 256 x 256 13.4 / 12.5).  The taller ones spread over rounds and update it as it lies.
  constexpr bool STAGED = FP32 && TM <= 5;
  constexpr int CPF = BN / 4, RPW = 64 / CPF;            // 16-byte chunks of a row, rows of a wavefront's read
  constexpr int NG = 2 * TM * 16 * BN * 4 <= G::LDS ? 1 : 2, GI = (TM + NG - 1) / NG, NX = GI * 4 / RPW;   // steps, rows in a step, reads per wavefront
  static_assert(!STAGED || 2 * GI * 16 * BN * 4 <= G::LDS, "a step fits");
  u32x4 xv[STAGED ? NG : XP][STAGED ? NX : TN];
  float* const px = FP32 ? e.resid + ((int64_t)part * M + m0) * e.ldr + n0 : nullptr;
  const int64_t left_x = ((M - m0) * e.ldr - n0) * 4;
  const uint32_t nx = (uint32_t)(left_x < 0x7fffffff ? left_x : 0x7fffffff), xrow = (uint32_t)e.ldr * 64;
  uint32_t vx[TN];
  if constexpr (FP32 && !STAGED) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = wn * WN + j * 16 + lg * 4;
      vx[j] = n0 + n < N ? (uint32_t)((wm * WM + lr) * e.ldr + n) * 4 : 0x7fffffffu;
    }
  }
  auto resid_load = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j) xv[i % XP][j] = buffer_load16(px, nx, vx[j] + i * xrow);
  };
  // STAGED, read t of step g: row of the step, row of the tile; a lane's four columns lie XOR-swizzled with the former
  auto step_row = [&](int g, int t, int& row) __attribute__((always_inline)) {
    const int gi = TM - g * GI < GI ? TM - g * GI : GI, r = (t * 8 + wave) * RPW + lane / CPF;
    row = r / (gi * 16) * WM + g * GI * 16 + r % (gi * 16);
    return r;
  };
  auto step_at = [&](int g, int t, int64_t ld, int size, uint32_t& at) __attribute__((always_inline)) {   // byte of that place in a matrix
    int row;
    const int r = step_row(g, t, row), col = ((lane % CPF) ^ (r & 15)) * 4;
    at = n0 + col < N ? (uint32_t)(row * ld + col) * size : 0x7fffffffu;
  };
  auto step_reads = [](int g) constexpr { return (TM - g * GI < GI ? TM - g * GI : GI) * 4 / RPW; };
  auto step_load = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NX; ++t)
      if (t < step_reads(g)) { uint32_t at; step_at(g, t, e.ldr, 4, at); xv[g][t] = buffer_load16(px, nx, at); }
  };

  // A wavefront's queue of loads: in slab s's turn A(s + DA), B(s + DB), and before slab 0's the turns -D .. -1 with what exists
#pragma unroll
  for (int t = -D; t < 0; ++t) {
    if (t + DA >= 0 && t + DA < NS) load_a(t + DA, t + DA);
    if (t + DB >= 0 && t + DB < NS) load_b(t + DB, t + DB);
  }
  // slab 0 is there once no more than what follows its own loads is outstanding; a short K has less behind it and waits for all
  if (NS > D) wait_loads(std::integral_constant<int, DA - 1>{}, std::integral_constant<int, DB - 1>{});
  else vm_wait<0>();
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  if (wm == 1) __builtin_amdgcn_s_barrier();             // the second half starts half a turn later
  __builtin_amdgcn_sched_barrier(0);
  // EXCH: operands exchanged, the accumulators are those of C^T
  auto multiply = [&](auto exch_) __attribute__((always_inline)) {
    constexpr bool EXCH = decltype(exch_)::value;
    int ca = 0, cb = 0;                                  // stages of slab s
    // R: slabs behind this one, or D for any number from D on
    auto slab = [&](int s, auto r_) __attribute__((always_inline)) {
      constexpr int R = decltype(r_)::value;
      const uint32_t ba = (uint32_t)ca * ACH * 16, bb = (uint32_t)cb * BCH * 16;
      bf16x8 af[PH][TM], bfr[PH][TN];
      static_for<2 / PH>([&](auto h_) __attribute__((always_inline)) {
        constexpr int h = decltype(h_)::value;
        constexpr bool LAST = h == 2 / PH - 1;
        __builtin_amdgcn_sched_barrier(0);
        static_for<PH>([&](auto k_) __attribute__((always_inline)) {
          constexpr int k = decltype(k_)::value;
          const uint32_t o = sx ^ (uint32_t)((h * PH + k) * 64);
          static_for<TN>([&](auto j_) __attribute__((always_inline)) { constexpr int j = decltype(j_)::value; bfr[k][j] = __builtin_bit_cast(bf16x8, lds_read16_raw<j * 2048>(fb + bb + o)); });
          static_for<TM>([&](auto i_) __attribute__((always_inline)) { constexpr int i = decltype(i_)::value; af[k][i] = __builtin_bit_cast(bf16x8, lds_read16_raw<i * 2048>(fa + ba + o)); });
        });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (h == 0) {
          // into the stages of slab s - 1.  Its weights have been read by both halves, its rows of A by this half, which alone reads
          // them, and those reads were waited for before the last barrier.
          if constexpr (R >= DA) load_a(s + DA, ca == 0 ? SA - 1 : ca - 1);
          if constexpr (R >= DB) load_b(s + DB, cb == 0 ? SB - 1 : cb - 1);
          if constexpr (EPI == EPI_RESID && STAGED && R == 0) step_load(0);
        }
        // what was requested behind A(s + 1) and behind B(s + 1); the first half reads the second one's share of B(s + 1) right
        // after this turn of the second half's, so that is waited for before the multiplication, the rest behind it
        auto behind = [](int d, bool own_b) constexpr {  // loads of turns s + 2 - d .. s and, for A, the weights of turn s + 1 - d: (A, B) as 100 A + B
          int a = 0, b = 0;
          for (int u = 0; u <= d - 1; ++u) {             // turn s - u
            if (u < d - 1 && R >= DA - u) ++a;
            if ((u < d - 1 || own_b) && R >= DB - u) ++b;
          }
          return 100 * a + b;
        };
        constexpr int QA = behind(DA, true), QB = behind(DB, false);
        if constexpr (LAST && R > 0) {
          if (wm == 1) wait_loads(std::integral_constant<int, QB / 100>{}, std::integral_constant<int, QB % 100>{});
        }
        lds_wait<0>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        static_for<PH>([&](auto k_) __attribute__((always_inline)) {
          constexpr int k = decltype(k_)::value;
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = EXCH ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[k][i], bfr[k][j], acc[i][j], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[k][j], af[k][i], acc[i][j], 0, 0, 0);
          if constexpr (EPI == EPI_RESID && !STAGED && R == 0 && PH == 2 && k == 0) {
            __builtin_amdgcn_sched_barrier(0);
            resid_load(0); resid_load(1);
            __builtin_amdgcn_sched_barrier(0);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        if constexpr (LAST && R > 0) {
          constexpr int q = (QA / 100 * NA + QA % 100 * NB < QB / 100 * NA + QB % 100 * NB) ? QA : QB;
          wait_loads(std::integral_constant<int, q / 100>{}, std::integral_constant<int, q % 100>{});
        }
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      });
      ca = ca + 1 == SA ? 0 : ca + 1; cb = cb + 1 == SB ? 0 : cb + 1;
    };
    for (int s = 0; s < NS - D; ++s) slab(s, std::integral_constant<int, D>{});
    static_for<D>([&](auto t_) __attribute__((always_inline)) {
      constexpr int r = D - 1 - decltype(t_)::value;
      if (NS > r) slab(NS - 1 - r, std::integral_constant<int, r>{});
    });
  };
  int sec = 0;
  bool exch = false;
  if constexpr (EPI == EPI_HEADS) {
    sec = (int)(n0 / ha.dim);
    exch = ha.sec[sec].transposed != 0;
    if (exch) multiply(std::true_type{}); else multiply(std::false_type{});
  } else {
    multiply(std::false_type{});
  }
  if (wm == 0) __builtin_amdgcn_s_barrier();             // the halves meet again
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (STAGED) {
    const bf16_t* bias = (const bf16_t*)e.bias;
    float4* const l16 = (float4*)smem;
    bf16_t* const po = (bf16_t*)e.out + m0 * e.ldo + n0;
    const int64_t left_o = ((M - m0) * e.ldo - n0) * 2;
    const uint32_t no = (uint32_t)(left_o < 0x7fffffff ? left_o : 0x7fffffff);
    static_for<NG>([&](auto g_) __attribute__((always_inline)) {
      constexpr int g = decltype(g_)::value, gi = TM - g * GI < GI ? TM - g * GI : GI;
      if constexpr (EPI == EPI_RESID && g > 0) step_load(g);
      __syncthreads();                                   // the operand slabs / the previous step are done with
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int nl = wn * WN + j * 16 + lg * 4;
        float b[4] = {0.f, 0.f, 0.f, 0.f};
        float4 gv = make_float4(1.f, 1.f, 1.f, 1.f);
        if (EPI == EPI_RESID && n0 + nl < N) {
          if (bias) {
            const uint2 b4 = *(const uint2*)(bias + n0 + nl);
            b[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); b[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
            b[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); b[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
          }
          if (e.gate) gv = *(const float4*)(e.gate + n0 + nl);
        }
#pragma unroll
        for (int i = 0; i < gi; ++i) {
          const f32x4 a = acc[g * GI + i][j];
          const int r = (wm * gi + i) * 16 + lr;
          l16[r * CPF + ((nl >> 2) ^ (r & 15))] = make_float4(gv.x * (a[0] + b[0]), gv.y * (a[1] + b[1]), gv.z * (a[2] + b[2]), gv.w * (a[3] + b[3]));
        }
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < step_reads(g); ++t) {
        int row;
        const float4 v = l16[step_row(g, t, row) * CPF + lane % CPF];
        f32x4 x = {v.x, v.y, v.z, v.w};
        uint32_t at;
        if constexpr (EPI == EPI_RESID) x += __builtin_bit_cast(f32x4, xv[g][t]);
        step_at(g, t, e.ldr, 4, at);
        buffer_store16(__builtin_bit_cast(u32x4, x), px, nx, at);
        if (EPI == EPI_RESID && e.out) {
          step_at(g, t, e.ldo, 2, at);
          buffer_store8(u32x2{cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3])}, po, no, at);
        }
      }
    });
  } else if constexpr (EPI == EPI_PART) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) buffer_store16(__builtin_bit_cast(u32x4, acc[i][j]), px, nx, vx[j] + i * xrow);
  } else if constexpr (EPI == EPI_RESID) {
    const bf16_t* bias = (const bf16_t*)e.bias;
    float bv[TN][4];
    float4 gv[TN];
#pragma unroll
    for (int i = PH == 2 ? 2 : 0; i < XP; ++i) resid_load(i);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t n = n0 + wn * WN + j * 16 + lg * 4;
      bv[j][0] = bv[j][1] = bv[j][2] = bv[j][3] = 0.f;
      gv[j] = make_float4(1.f, 1.f, 1.f, 1.f);
      if (n < N) {
        if (bias) {
          const uint2 b4 = *(const uint2*)(bias + n);
          bv[j][0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[j][1] = bf16_to_f32((bf16_t)(b4.x >> 16));
          bv[j][2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[j][3] = bf16_to_f32((bf16_t)(b4.y >> 16));
        }
        if (e.gate) gv[j] = *(const float4*)(e.gate + n);
      }
    }
    // the same of the rounded copy, if one is asked for
    bf16_t* const po = (bf16_t*)e.out + m0 * e.ldo + n0;
    const int64_t left_o = ((M - m0) * e.ldo - n0) * 2;
    const uint32_t no = (uint32_t)(left_o < 0x7fffffff ? left_o : 0x7fffffff);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      u32x2 r[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4 a = acc[i][j];
        f32x4 x = __builtin_bit_cast(f32x4, xv[i % XP][j]);
        x[0] += gv[j].x * (a[0] + bv[j][0]); x[1] += gv[j].y * (a[1] + bv[j][1]);
        x[2] += gv[j].z * (a[2] + bv[j][2]); x[3] += gv[j].w * (a[3] + bv[j][3]);
        buffer_store16(__builtin_bit_cast(u32x4, x), px, nx, vx[j] + i * xrow);
        r[j] = u32x2{cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3])};
      }
      if (e.out) {
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          // two column tiles at once: lanes of even lg take eight columns of the first, of odd lg of the second, so that four
          // lanes write 64 bytes of a row and not 32
          const auto lo = __builtin_amdgcn_permlane16_swap(r[j].x, r[j + 1].x, false, false);
          const auto hi = __builtin_amdgcn_permlane16_swap(r[j].y, r[j + 1].y, false, false);
          const int n = wn * WN + (j + (lg & 1)) * 16 + (lg >> 1) * 8;
          const uint32_t o = n0 + n < N ? (uint32_t)((wm * WM + i * 16 + lr) * e.ldo + n) * 2 : 0x7fffffffu;
          buffer_store16(u32x4{lo[0], hi[0], lo[1], hi[1]}, po, no, o);
        }
      }
      if (i + XP < TM) resid_load(i + XP);
    }
  } else {
    finish_tile<BM, BN, G::WGM, WGN, TM, TN, EPI, G::LDS>(acc, smem, m0, n0, M, N, sec, exch, e, ha);
  }
}

template <int TM, int TN, int EPI>
static void launch_turns(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                         int64_t K, const EpiArgs& e, hipStream_t st, int parts) {
  typedef Turns<TM, TN> G;
  const int tm = (int)((M + G::BM - 1) / G::BM), tn = (int)((N + G::BN - 1) / G::BN);
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_gemm_turns<TM, TN, EPI>, G::LDS, done);
  HeadsArgs ha{};
  if (EPI == EPI_HEADS) { e.heads->ssq_np = e.heads->dim / G::BN; ha = *e.heads; }
  dim3 grid((unsigned)((tm * tn * parts + 7) / 8 * 8));
  k_gemm_turns<TM, TN, EPI><<<grid, 512, G::LDS, st>>>(A, lda, Wt, ldw, M, N, K, tn, tm * tn, parts, e, ha);
}
// false: this tile shape has no such epilogue (the rules below never ask for it)
template <int TM, int TN>
static bool launch_turns_cfg(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                             int64_t K, int epi, const EpiArgs& e, hipStream_t st, int parts) {
  constexpr bool HEADS = TM != 10, PART = TM != 6 && TM != 10;
  if (epi == EPI_STORE) launch_turns<TM, TN, EPI_STORE>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_GELU) launch_turns<TM, TN, EPI_GELU>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_RESID) launch_turns<TM, TN, EPI_RESID>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_HEADS && HEADS) { if constexpr (HEADS) launch_turns<TM, TN, EPI_HEADS>(A, lda, Wt, ldw, M, N, K, e, st, parts); }
  else if (epi == EPI_PART && PART) { if constexpr (PART) launch_turns<TM, TN, EPI_PART>(A, lda, Wt, ldw, M, N, K, e, st, parts); }
  else return false;
  return true;
}

// Which tile family a problem takes.  A 256-row tile keeps a CU busy by itself but a small problem has too few of them; 64 x 64
// tiles run as a ring of loads, up to three to a CU, 128 x 128 ones in turns (k_gemm_turns), one to a CU.  Lines, measured (us):
// 1008 x 1024 x 4096 (256 tiles of 64^2): 64^2 24, 128^2 41; 1560 x 1536 x 1536 (600): 24 and 21.5, with per-head stores 20 and
// 21; 1008 x 3072 x 1024 (768), per-head stores: 17.4 and 16.9; 4032 x 1024 x 1024 (1008): 28 and 20.5; 1008 x 4096 x 1024 (256
// of 128^2): 128^2 14.8, 128 x 256 20.5; 1560 x 4608 x 1536 (468): 39 and 29.
enum { TILE_64 = 0, TILE_128 = 1, TILE_BIG = 2 };
static int tile_family(int64_t M, int64_t N, int epi) {
  if (((M + 63) / 64) * ((N + 63) / 64) <= (epi == EPI_HEADS ? 768 : 560)) return TILE_64;
  if (((M + 127) / 128) * ((N + 127) / 128) <= 256) return TILE_128;   // one round
  return TILE_BIG;
}
// Tile shape, LDS stages and K ranges of a problem: what the rules below decide and launch_gemm_bf16 runs
static GemmRoute small_tile(int family, int64_t M, int64_t N) {
  if (family == TILE_128) return {128, 128, 4, 1};
  if ((M + 31) / 32 * ((N + 63) / 64) <= 256) return {32, 64, 1, 1};    // k_gemm_thin: one round
  // 64 KB of LDS (two blocks per CU) where two suffice, 48 KB where a third has to fit
  return {64, 64, ((M + 63) / 64) * ((N + 63) / 64) <= 512 ? 4 : 3, 1};
}

// EPI_HEADS.  Sections must be whole tiles wide, a transposed one needs 8 | M and 8 | row0.
static int heads_columns(int64_t M, int64_t N) {         // columns of the tile; grows with M
  const int family = tile_family(M, N, EPI_HEADS);
  return family == TILE_64 ? 64 : family == TILE_128 ? 128 : 256;
}
bool gemm_bf16_heads_wide(int64_t M, int64_t N) { return heads_columns(M, N) < 256; }
bool gemm_bf16_heads_ever(int64_t M, int64_t N, int64_t dim) { return dim % heads_columns(M, N) == 0; }
bool gemm_bf16_heads_ok(int64_t M, int64_t N, const HeadsArgs& h) {
  if (h.dim <= 0 || (h.head_dim != 64 && h.head_dim != 128) || h.dim % heads_columns(M, N) || h.dim % h.head_dim || N % h.dim || N / h.dim > 3) return false;
  for (int i = 0; i < (int)(N / h.dim); ++i) {
    if (h.sec[i].transposed && (M % 8 || h.sec[i].row0 % 8 || h.sec[i].ld % 8)) return false;
    if (h.sec[i].ssq && h.ssq_stride < M) return false;
    if (h.sec[i].wide && (h.sec[i].transposed || !gemm_bf16_heads_wide(M, N))) return false;
  }
  return true;
}
// x[m, n] += gate[n] * (bias[n] + sum over the K ranges, in range order), and its rounded copy.  P ranges, all requested before
// the first is added: one trip to memory, not one each (product and sum, 1560 x 1536 x 8960 in 4 ranges in a stage, 57.9 -> 56.5 us).
template <int P>
__global__ __launch_bounds__(256) void k_add_parts(const float* __restrict__ part, int64_t M, int64_t N, EpiArgs e) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= M * N) return;
  const int64_t m = i / N, n = i % N;
  f32x4 v[P];
#pragma unroll
  for (int p = 0; p < P; ++p) v[p] = *(const f32x4*)(part + (int64_t)p * M * N + i);
  f32x4 x = *(const f32x4*)(e.resid + m * e.ldr + n);
  const f32x4 g = e.gate ? *(const f32x4*)(e.gate + n) : f32x4{1.f, 1.f, 1.f, 1.f};
  const uint2 b = e.bias ? *(const uint2*)((const bf16_t*)e.bias + n) : make_uint2(0, 0);
#pragma unroll
  for (int p = 1; p < P; ++p) v[0] += v[p];
  v[0] += f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xffff0000u)};
  x += g * v[0];
  *(f32x4*)(e.resid + m * e.ldr + n) = x;
  if (e.out) *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3]));
}
template <int P>
static void launch_add_parts(int parts, int64_t M, int64_t N, const EpiArgs& e, hipStream_t st) {   // P <= parts <= 8
  if constexpr (P < 8) if (parts > P) return launch_add_parts<P + 1>(parts, M, N, e, st);
  k_add_parts<P><<<(unsigned)((M * N / 4 + 255) / 256), 256, 0, st>>>(e.scratch, M, N, e);
}
size_t gemm_bf16_scratch_bytes(int64_t M, int64_t N) {
  const size_t most = (size_t)256 * 256 * 256 * 4, need = (size_t)(8 * M * N * 4);      // one round of 256 x 256 tiles
  return need < most ? need : most;
}
// Cutting K.  A long K over few tiles leaves most CUs idle, and small tiles in the hundreds move several times the bytes of
// large ones through the caches.  Tiles whose K is cut over blocks until about one round of CUs is full do neither, for the
// price of one fp32 partial result per range, written and read once.  Costs in us per launch, from measurement: a k-tile of a
// block 0.5 (128 x 128), 0.75 (128 x 256), 0.86 (160 x 256), 1.0 (192 x 256), 1.25 (256 x 256), 1.55 (320 x 256), 0.27 for each 64 x 64 block on the CU; 7 for both
// launches and a block's ends, partials at 6.5 TB/s; uncut 0.185 per k-tile and 3.3 (32 x 64), 0.24 per k-tile and 64 x 64 block
// on the CU and 5, 9 (128 x 128) or 14 for launch and ends.  Cut / best uncut in us: 500 x 1536 x 8960 27.9 (128 x 128, 5 ranges) / 43, 1560 x 1536 x 8960 52 (160 x 256,
// 4) / 75, 1008 x 2048 x 8192 42 (128 x 256, 4) / 64, 2560 x 2048 x 8192 82 (160 x 256, 2) / 92; left uncut 1288 x 5120 x 13824 164.  Outputs narrower than 768 columns
// are left on the 64-, 160- and 256-row tiles and on figures that were measured before the
// loop in turns (a k-tile 1.25 at 160 rows, 8 for ends and 3 for the second launch, 4 TB/s) and not again.  That line is no property of the tiles: the 128-row ones have not been
// measured below it, and the parity tests of the cut 160- and 256-row tiles are shapes of that side.
static GemmRoute big_tile(int64_t M, int64_t N, int epi);
static GemmRoute cut_tile(int64_t M, int64_t N, int64_t K, size_t scratch_floats) {
  GemmRoute r{0, 0, 0, 1};                             // parts == 1: not cut
  if (N % 4) return r;
  const bool narrow = N < 768;
  auto tiles = [&](int64_t rows, int64_t cols) { return (M + rows - 1) / rows * ((N + cols - 1) / cols); };
  const int64_t t256 = tiles(256, 256), t160 = tiles(160, 256), t64 = tiles(64, 64), KT = K / 64;
  const bool fits160 = !narrow || (M + 159) / 160 * 160 <= (M + 255) / 256 * 256;
  const int family = tile_family(M, N, EPI_RESID);
  double best = family == TILE_64 ? (tiles(32, 64) <= 256 ? 0.185 * (double)KT + 3.3 : 0.24 * (double)(KT * ((t64 + 255) / 256)) + 5)
              : family == TILE_128 ? 0.5 * (double)KT + 9 : 1.3 * (double)(KT * ((t256 + 255) / 256)) + 8;
  if (family == TILE_BIG && !narrow) {
    const GemmRoute u = big_tile(M, N, EPI_RESID);
    const double kt = u.bm == 128 ? 0.75 : u.bm == 160 ? 0.86 : u.bm == 192 ? 1.0 : u.bm == 256 ? 1.25 : 1.55;
    best = kt * (double)(KT * ((tiles(u.bm, u.bn) + 255) / 256)) + 14;
  }
  best *= 0.9;                                         // not for a few per cent
  for (int p = 2; p <= 8; ++p) {
    if ((size_t)(p * M * N) > scratch_floats) break;
    const double moved = (double)(M * N) * 4 * (2 * p + 2.5), kt = (double)((KT + p - 1) / p);
    const double big = narrow ? 8 + 3 + moved / 4e6 : 7 + moved / 6.5e6, small = narrow ? 4 + 3 + moved / 4e6 : big;
    const bool deep = KT / p >= 8;
    struct { double c; GemmRoute t; } opt[5] = {
        {narrow && t256 * p <= 256 && deep ? 1.3 * kt + big : 1e30, {256, 256, 2, p}},
        {fits160 && t160 * p <= 256 && deep ? (narrow ? 1.25 : 0.86) * kt + big : 1e30, {160, 256, 3, p}},
        {!narrow && tiles(128, 256) * p <= 256 && deep ? 0.75 * kt + big : 1e30, {128, 256, 3, p}},
        {!narrow && tiles(128, 128) * p <= 256 && deep ? 0.5 * kt + big : 1e30, {128, 128, 4, p}},
        {t64 * p <= 512 && KT / p >= 4 ? 0.27 * kt * (double)((t64 * p + 255) / 256) + small : 1e30, {64, 64, 4, p}}};
    for (const auto& o : opt)
      if (o.c < best) { best = o.c; r = o.t; }
  }
  return r;
}

// One block per CU at a time, so a launch costs ceil(blocks / 256) rounds of one block's duration.  Durations over that of a
// 256 x 256 block, from launches of 2 to 27 rounds at K = 1536 ... 13824, each tile forced in turn: 320 rows 1.18 ... 1.33, 192 rows
// 0.77 ... 0.86 (per-head stores at the upper end), 160 rows 0.70 ... 0.79, 128 rows 0.58 ... 0.62.  Where they decide (us): 1560 x
// 4608 x 1536 128 rows, one round, 23, 160 rows 25, 256 rows 31; 3600 x 13824 x 5120 160 rows in 4 rounds 388, 320 rows in 3 417;
// 6240 x 8960 x 1536 320 rows in 3 154, 256 rows in 4 161; 18720 x 1536 x 8960 256 rows in 2 399, 160 rows in 3 442; 7800 x 4608 x
// 1536 192 rows in 3 92, 160 rows in 4 104; 14400 x 5120 x 5120 192 rows in 6 620, 256 rows in 5 637, 320 rows in 4 690; 14400 x
// 15360 x 5120 256 rows in 14 1552, 192 rows in 18 1600.
// No tile reads anything beyond M.  Narrow outputs and plain stores take the tiles of other heights than 256 rows only where
// they fit M rounded up to 256 (160, 192 and 320 rows) or nearly fill the round (128 rows).  Those lines are no property of the
// tiles: beyond them they have not been measured, and the parity tests of the 192- and 256-row tiles are such shapes.
static GemmRoute big_tile(int64_t M, int64_t N, int epi) {
  const int64_t tn = (N + 255) / 256, mpad = (M + 255) / 256 * 256;
  const bool heads = epi == EPI_HEADS, any = heads || (epi == EPI_RESID && N >= 1536) || (epi == EPI_GELU && N >= 2048);
  auto tiles = [&](int64_t rows) { return (M + rows - 1) / rows * tn; };
  auto fits = [&](int64_t rows) { return (M + rows - 1) / rows * rows <= mpad; };
  auto cost = [&](int64_t rows, double duration, bool ok) { return ok ? duration * (double)((tiles(rows) + 255) / 256) : 1e30; };
  const GemmRoute tile[5] = {{320, 256, 2, 1}, {256, 256, 2, 1}, {160, 256, 3, 1}, {192, 256, 2, 1}, {128, 256, 3, 1}};
  const double c[5] = {cost(320, 1.31, !heads && (any || fits(320))), cost(256, 1.0, true), cost(160, 0.7, any || fits(160)),
                       cost(192, heads ? 0.84 : 0.8, any || fits(192)), cost(128, 0.6, any || (tiles(128) > 210 && tiles(128) <= 256))};
  int best = 0;                                          // on a tie the earlier one: fewer operand bytes per flop
  for (int i = 1; i < 5; ++i) if (c[i] < c[best]) best = i;
  return tile[best];
}

GemmRoute gemm_bf16_route(int64_t M, int64_t N, int64_t K, int epi, size_t scratch_floats) {
  if (epi == EPI_RESID) {
    const GemmRoute r = cut_tile(M, N, K, scratch_floats);
    if (r.parts > 1) return r;
  }
  const int family = tile_family(M, N, epi);
  return family == TILE_BIG ? big_tile(M, N, epi) : small_tile(family, M, N);
}
// for the parity tests, which state the kernel that each of their products is meant to reach (the fifth argument has no
// meaning any more: a tile of any shape stores transposed sections)
extern "C" void dp_gemm_bf16_route(int64_t M, int64_t N, int64_t K, int32_t epi, int32_t, int64_t scratch_floats, int32_t* bm_bn_stages_parts) {
  const GemmRoute r = gemm_bf16_route(M, N, K, epi, (size_t)scratch_floats);
  const int32_t v[4] = {r.bm, r.bn, r.stages, r.parts};
  for (int i = 0; i < 4; ++i) bm_bn_stages_parts[i] = v[i];
}
// the same: whether a projection of M rows stores its N / dim sections per head, the third of them transposed
extern "C" int32_t dp_gemm_bf16_heads(int64_t M, int64_t N, int32_t dim, int32_t head_dim) {
  HeadsArgs h{};
  h.dim = dim; h.head_dim = head_dim; h.sec[2].transposed = 1;
  return gemm_bf16_heads_ok(M, N, h);
}

bool launch_gemm_bf16(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                      int64_t K, int epi, const EpiArgs& e, hipStream_t st) {
  if (M <= 0 || N <= 0) return true;
  if (K < 64 || K % 64) return false;          // whole k-tiles of 64 (the callers validate their widths)
  if (epi == EPI_HEADS && (!e.heads || !gemm_bf16_heads_ok(M, N, *e.heads))) return false;
  const GemmRoute r = gemm_bf16_route(M, N, K, epi, e.scratch && e.ldr % 4 == 0 ? e.scratch_floats : 0);
  const EpiArgs part{nullptr, 0, nullptr, e.scratch, N, nullptr, nullptr, nullptr, 0};
  const EpiArgs& ea = r.parts > 1 ? part : e;
  const int ep = r.parts > 1 ? (int)EPI_PART : epi;
  bool ok = false;
#define RING_TILE(ST) \
  if (r.bm == 64 && r.stages == ST) ok = launch_ring_cfg<ST>(A, lda, Wt, ldw, M, N, K, ep, ea, st, r.parts)
#define TURNS_TILE(TM, TN) \
  if (r.bm == 32 * TM && r.bn == 64 * TN) ok = launch_turns_cfg<TM, TN>(A, lda, Wt, ldw, M, N, K, ep, ea, st, r.parts)
  if (r.bm == 32) ok = launch_thin_cfg(A, lda, Wt, ldw, M, N, K, ep, ea, st);
  else RING_TILE(4);
  else RING_TILE(3);
  else TURNS_TILE(4, 2);
  else TURNS_TILE(4, 4);
  else TURNS_TILE(5, 4);
  else TURNS_TILE(6, 4);
  else TURNS_TILE(8, 4);
  else TURNS_TILE(10, 4);
#undef RING_TILE
#undef TURNS_TILE
  if (r.parts > 1) launch_add_parts<2>(r.parts, M, N, e, st);
  return ok;
}
